// fp32 matrix-core kernels of the general path: sketches, states, rows of the output, for
// sketch features with d, dv and sketch columns <= 128 (any block size, fp32 or bf16 storage).
// Everything is computed in fp32 as the vector kernels of psf_general.hip do (which keep explicit
// exact features, sizes above 128 and what f32_choose leaves to them).  Layouts and operand conventions: psf_f32_tiles.h.
//
// The in-block rule only says which weight a pair of tokens gets; it does not force a state per
// block.  A state is kept per span of several blocks, and pairs of different blocks inside a span
// take their weight <m(q), m(k)>^2 directly: 2 (r + dv) flops a pair against about 2 r^2 dv a
// token for forming and applying a state, and no state traffic (1 MB per block and unit with r = 64).
// f32_plan() chooses the span.
//
// Measured against the vector kernels (us a call, forward / forward and backward): 36 units of 3000
// tokens, r = 32, b = 200, bf16 storage 8540 -> 361; 24 units of 1950, b = 150, forward and backward
// 26940 -> 772; one unit of 1024, r = 16, fp32 storage 248 -> 33.  Relative error against float64
// (fp32 storage, 2400 tokens, r = 64): forward 1.6e-6 -> 3.9e-7, gradients 3.8e-7 to 4.7e-7 -> 3.0e-7
// to 3.7e-7; over 81 shapes no result is further off than on the vector kernels.
#include "psf_f32_tiles.h"
#include "psf_f32.h"

namespace psf {
namespace {

// ---- Algorithm 1 ------------------------------------------------------------------------
constexpr int kSketchRows = 32;

// m(x) of the rows of X1 and (blockIdx.z = 1) X2, fp32, 32 rows a wave.  LDS: x, then the nodes of the levels
// below the root (p / 4 of the first level, for p = 16 two more); padded to 16 columns with zeros.
__host__ __device__ inline int sketch_nodes(int p) { return p == 4 || p == 2 ? 0 : p == 8 ? 2 : 6; }
template <typename T>
__global__ __launch_bounds__(64) void f32_sketch_kernel(const T *__restrict__ X1, const T *__restrict__ X2,
                                                        const T *__restrict__ G, float *__restrict__ M1,
                                                        float *__restrict__ M2, int n, int d, int r, int p, int heads,
                                                        int per_head, size_t g_len, size_t x_unit, size_t m_unit,
                                                        int vec_x, int vec_m)
{
    // x_unit, m_unit: elements from the rows of one unit to those of the next
    extern __shared__ __attribute__((aligned(16))) float smem[];
    const int lane = threadIdx.x, li = lane & 15, g = lane >> 4, u = blockIdx.y, i0 = blockIdx.x * kSketchRows;
    const int dp = (d + 15) / 16 * 16, rp = (r + 15) / 16 * 16, xp = dp + 4, mp = rp + 4;
    const T *X = (blockIdx.z ? X2 : X1) + u * x_unit + (size_t)i0 * d;
    float *M = (blockIdx.z ? M2 : M1) + u * m_unit + (size_t)i0 * (p == 2 ? d : r);
    const int nv = min(kSketchRows, n - i0);
    const int quads = dp / 4;
    for (int idx = lane; idx < kSketchRows * quads; idx += 64) {
        const int row = idx / quads, c = 4 * (idx % quads);
        f4 v = {0.f, 0.f, 0.f, 0.f};
        if (row < nv) v = row_piece(X + (size_t)row * d, c, d, vec_x);
        if (p == 2) {
            if (row < nv) store_piece(M + (size_t)row * d, c, d, vec_m, v);
        } else {
            *(f4 *)&smem[row * xp + c] = v;
        }
    }
    if (p == 2) return;
    __syncthreads();
    const T *gs = G + (per_head ? (size_t)(u % heads) * g_len : 0), *gi = gs + (size_t)(p / 2) * d * r;
    const float sc = sqrtf(1.0f / (float)r);
    float *nodes = smem + kSketchRows * xp;
    int count = p / 4, from = -1;                            // nodes of this level; first node below (-1: x)
    for (int first = 0;; ) {
        for (int k = 0; k < count; ++k) {
            const int in = from < 0 ? d : r, pitch = from < 0 ? xp : mp;
            const T *ga = from < 0 ? gs + (size_t)(2 * k) * d * r : gi + (size_t)(2 * k) * r * r;
            const float *xa = from < 0 ? smem : nodes + (size_t)(from + 2 * k) * kSketchRows * mp;
            const float *xb = from < 0 ? smem : xa + (size_t)kSketchRows * mp;
            for (int c0 = 0; c0 < rp; c0 += 16) {
                f4 a[2], w[2];
                project<2>(ga, in, r, c0, xa, pitch, a, lane);
                project<2>(ga + (size_t)in * r, in, r, c0, xb, pitch, w, lane);
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    f4 m;
#pragma unroll
                    for (int s = 0; s < 4; ++s) m[s] = sc * (a[h][s] * w[h][s]);
                    const int row = 16 * h + li;
                    if (count > 1)
                        *(f4 *)&nodes[((size_t)(first + k) * kSketchRows + row) * mp + c0 + 4 * g] = m;
                    else if (row < nv)
                        store_piece(M + (size_t)row * r, c0 + 4 * g, r, vec_m, m);
                }
            }
        }
        if (count == 1) break;
        __syncthreads();
        if (from >= 0) gi += (size_t)(2 * count) * r * r;
        from = first;
        first += count;
        count /= 2;
    }
}

// ---- states: sum over the tokens of a span of phi'(x_j) [C_j | w_j] --------------------------
// A wave owns two sketch indices, one of tile row `lo` and one of tile row `hi` = RT - 1 - lo (the
// same row for r = 16), so that every wave has RT + 1 tiles of pairs, and walks the tokens:
// A = m_j[a] m_j[b'] (made in registers, one multiply for the products of four column tiles),
// B = C_j.  The denominator column is a running sum of the A operands.  The four column tiles
// are read once for both indices and each staged token serves eight indices a workgroup: 36
// units x 2800 tokens, r = 32: 175 us with one index a wave, 112 so.  Wide values (VT = 8) are split over two workgroups,
// 64 columns each.  Where RT + 1 tiles in two levels of sums exceed the registers (RT = 8), a
// wave takes one index and RT tiles, of which those below the diagonal are empty.
template <int RT, int VT, typename S>
__global__ __launch_bounds__(kF32Threads, RT <= 2 ? 3 : RT == 4 ? 2 : 1) void f32_state_kernel(
    const float *__restrict__ M, const S *__restrict__ C, const float *__restrict__ wts, float *__restrict__ Z,
    F32Shape sh, int span0)
{
    constexpr int MP = pitch_of<RT>(), VP = pitch_of<4>(), KT = RT > 4 ? 32 : 64;
    constexpr bool TWO = RT <= 4;
    constexpr int SLOTS = TWO ? RT + 1 : RT;
    __shared__ __attribute__((aligned(16))) float ms[KT * MP], vs[KT * VP], ws[KT];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, li = lane & 15, g = lane >> 4;
    const int grp = blockIdx.x / (VT / 4), c0 = 64 * (blockIdx.x % (VT / 4));
    // TWO: groups of four index pairs; r = 16 pairs a with a + 8 of the one tile row
    const int lo = RT == 1 ? 0 : grp / 4, a_lo = RT == 1 ? 4 * grp + wave : 16 * lo + 4 * (grp % 4) + wave;
    const int hi = TWO ? RT - 1 - lo : lo, a_hi = RT == 1 ? a_lo + 8 : 16 * hi + 4 * (grp % 4) + wave;
    const int split = RT - lo;                              // slots of a_lo; the others are a_hi's
    const int span = span0 + blockIdx.y, u = blockIdx.z;
    const auto [j_begin, j_end] = state_tokens(sh.n, sh.span, span, sh.dv, c0);
    f4 acc[SLOTS][4];
    float den[SLOTS];
    int mcol[SLOTS];                                        // first sketch column of the slot's tile
#pragma unroll
    for (int e = 0; e < SLOTS; ++e) {
        den[e] = 0.f;
        mcol[e] = 16 * (e < split ? lo + e : min(hi + e - split, RT - 1));
        clear(acc[e]);
    }
    for (int j0 = j_begin; j0 < j_end; j0 += KT) {
        const size_t row = (size_t)u * sh.n + j0;
        const int nv = j_end - j0;
        const S *cp = C + row * sh.dv + c0;
        Tile<RT, KT, float> mt;
        Tile<4, KT, S> ct;
        if (sh.vec_m) mt.load(M + row * sh.mcols, sh.mcols, nv, sh.mcols);
        if (sh.vec_v) ct.load(cp, sh.dv, nv, sh.dv - c0);
        __syncthreads();
        if (sh.vec_m) mt.store(ms, nv, sh.mcols);
        else stage_scalar<RT, KT>(M + row * sh.mcols, sh.mcols, nv, sh.mcols, ms);
        if (sh.vec_v) ct.store(vs, nv, sh.dv - c0);
        else stage_scalar<4, KT>(cp, sh.dv, nv, sh.dv - c0, vs);
        if (threadIdx.x < KT) ws[threadIdx.x] = wts && (int)threadIdx.x < nv ? wts[row + threadIdx.x] : 1.f;
        __syncthreads();
        f4 part[SLOTS][4];                                  // two levels of summation, as in psf_f32_bwd.hip
#pragma unroll
        for (int e = 0; e < SLOTS; ++e) clear(part[e]);
        for (int t16 = 0; t16 < KT; t16 += 16) {
            if (t16 >= nv) break;
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const int j = t16 + 4 * g + s;
                const float wt = ws[j], ma_lo = ms[j * MP + a_lo], ma_hi = TWO ? ms[j * MP + a_hi] : 0.f;
                float vb[4];
#pragma unroll
                for (int ct = 0; ct < 4; ++ct) vb[ct] = vs[j * VP + 16 * ct + li];
#pragma unroll
                for (int e = 0; e < SLOTS; ++e) {
                    if (!TWO && e >= split) break;
                    // the first tile of an index is on the diagonal, the others stand for their mirror too
                    const float ma = e == 0 ? ma_lo : e < split ? 2.f * ma_lo : e == split ? ma_hi : 2.f * ma_hi;
                    const float av = ms[j * MP + mcol[e] + li] * ma;
                    den[e] += av * wt;
#pragma unroll
                    for (int ct = 0; ct < 4; ++ct) part[e][ct] = mm(av, vb[ct], part[e][ct]);
                }
            }
        }
#pragma unroll
        for (int e = 0; e < SLOTS; ++e) add_to(acc[e], part[e]);
    }
    settle();
    float *rec = Z + ((size_t)u * sh.spans + span) * record_floats(RT, VT);
    float *srec = rec + (size_t)tile_pairs(RT) * 256 * 16 * VT;
#pragma unroll
    for (int e = 0; e < SLOTS; ++e) {
        if (!TWO && e >= split) break;
        const int at = e < split ? lo : hi, a = e < split ? a_lo : a_hi, q = mcol[e] / 16;
        const size_t pa = (size_t)(at * RT - at * (at - 1) / 2 + q - at) * 16 + (a & 15);
        const float dsum = over_groups(den[e]);
        if (g == 0 && c0 == 0) srec[pa * 16 + li] = dsum;
#pragma unroll
        for (int ct = 0; ct < 4; ++ct)
#pragma unroll
            for (int k = 0; k < 4; ++k)
                rec[(pa * 16 + 4 * g + k) * (16 * VT) + c0 + 16 * ct + li] = acc[e][ct][k];
    }
}

// In place over the spans of a unit: exclusive prefix, exclusive suffix, or the total in slot 0.
// The record that an exclusive sum never reads (the last, or the first) need not be there.
enum { kScanPrefix = 0, kScanSuffix = 1, kScanTotal = 2 };
__global__ __launch_bounds__(kF32Threads) void f32_scan_kernel(float *__restrict__ Z, size_t pieces, size_t rec,
                                                               int spans, int mode)
{
    const size_t idx = (size_t)blockIdx.x * kF32Threads + threadIdx.x;
    if (idx >= pieces) return;
    const size_t per = rec / 4;
    float *z = Z + (idx / per) * (size_t)spans * rec + (idx % per) * 4;
    f4 run = {0.f, 0.f, 0.f, 0.f};
    if (mode == kScanTotal) {
        for (int l = 0; l < spans; ++l) run += *(const f4 *)(z + (size_t)l * rec);
        *(f4 *)z = run;
        return;
    }
    for (int k = 0; k < spans; ++k) {
        const int l = mode == kScanSuffix ? spans - 1 - k : k;
        f4 h = {0.f, 0.f, 0.f, 0.f};
        if (k < spans - 1) h = *(const f4 *)(z + (size_t)l * rec);
        *(f4 *)(z + (size_t)l * rec) = run;
        run += h;
    }
}

// ---- rows: pairs of the row's span, then phi'(q_i)^T Z, then the division --------------------
// WR = 4: 64 rows a workgroup, a wave per 16 of them, every staged tile serves all four.
// WR = 1: 16 rows a workgroup, the waves share the work on them (keys, state rows) and add up at
// the end: four times the workgroups, for problems that would not fill the chip otherwise.
// With WR = 4 a wave has the whole row, so the sums of a staged tile and of a state piece are formed
// apart and then added to the total; one running sum over 3000 tokens (r = 64, 15 blocks) was 6.8e-7
// from float64, this is 3.3e-7 (36 units x 3000, r = 32: 210 us then, 215 to 220 now).
// GRAD: instead of the output, G_i = [dO_i / D_i | -<dO_i, o_i> / D_i] for the backward pass.
template <int DT, int RT, int VT, int WR, bool GRAD, typename T>
__global__ __launch_bounds__(kF32Threads, DT == 4 ? (RT <= 2 ? 3 : 2) : 1) void f32_rows_kernel(
    const float *__restrict__ MQ, const float *__restrict__ MK, const T *__restrict__ Q, const T *__restrict__ K,
    const T *__restrict__ V, const float *__restrict__ Z, T *__restrict__ O, const T *__restrict__ dO,
    float *__restrict__ GV, float *__restrict__ gden, F32Shape sh)
{
    constexpr int KT = f32_tile_rows(DT, WR), KP = pitch_of<DT>(), MP = pitch_of<RT>(), VP = pitch_of<VT>();
    constexpr int ROWS = 16 * WR, ZA = KT / 16;             // sketch indices a per staged piece of the state,
    constexpr int ZW = WR == 1 ? 1 : ZA;                    // and how many of them a wave takes
    constexpr int kTileFloats = KT * (KP + VP) + (KT > ROWS ? KT : ROWS) * MP;
    static_assert(WR == 4 || KT == 64, "the waves of a 16-row workgroup take one key group each");
    static_assert(DT == VT, "the state is staged through the buffers of K and V in turn");
    __shared__ __attribute__((aligned(16))) float lds[kTileFloats];
    __shared__ __attribute__((aligned(16))) float sden[2][16 * ZA];   // denominator column of a state piece
    float *ks = lds, *vs = lds + KT * KP, *ms = vs + KT * VP;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, li = lane & 15, g = lane >> 4;
    // the longest rows of all units first: what is dealt last is short, and the workgroups that
    // share a CU are of different lengths
    const int per_span = (min(sh.span, sh.n) + ROWS - 1) / ROWS;
    const unsigned flat = blockIdx.y * gridDim.x + blockIdx.x;
    const int u = flat % sh.units, x = flat / sh.units;
    if (x >= per_span * sh.spans) return;
    const int span = sh.spans - 1 - x % sh.spans, s_begin = span * sh.span, s_end = min(sh.n, s_begin + sh.span);
    const int i0 = s_begin + (per_span - 1 - x / sh.spans) * ROWS;
    if (i0 >= s_end) return;
    const int iw = i0 + (WR == 4 ? 16 * wave : 0), i = iw + li;
    const int i_last = min(i0 + ROWS, s_end) - 1, iw_last = min(iw + 15, s_end - 1);
    const bool there = i < s_end;
    const size_t urow = (size_t)u * sh.n;
    float qf[4 * DT], mf[4 * RT];
    if (sh.local_exact) load_frags<DT>(Q + (urow + i) * sh.d, sh.d, there, sh.vec_x, g, qf);
    load_frags<RT>(MQ + (urow + i) * sh.mcols, sh.mcols, there, sh.vec_m, g, mf);
    f4 acc[VT];
    float den = 0.f;
#pragma unroll
    for (int ct = 0; ct < VT; ++ct) acc[ct] = f4{0.f, 0.f, 0.f, 0.f};

    if (sh.pairs) {
        // exact weights for keys from the start of the row's block on
        const int bs = sh.local_exact ? i / sh.b * sh.b : 0x7fffffff;
        const int bs_wg = sh.local_exact ? i0 / sh.b * sh.b : 0x7fffffff;
        const int bs_wg_last = sh.local_exact ? i_last / sh.b * sh.b : 0x7fffffff;
        const int bs_w = sh.local_exact ? iw / sh.b * sh.b : 0x7fffffff;
        const int bs_w_last = sh.local_exact ? iw_last / sh.b * sh.b : 0x7fffffff;
        const int j_end = sh.noncausal ? sh.n : i_last + 1;
        for (int j0 = sh.noncausal ? 0 : s_begin; j0 < j_end; j0 += KT) {
            const int nv = min(KT, j_end - j0);
            const bool exact_g = j0 + KT > bs_wg, cross_g = j0 < bs_wg_last;
            Tile<DT, KT, T> kt;
            Tile<RT, KT, float> mt;
            Tile<VT, KT, T> vt;
            const T *vp = V + (urow + j0) * sh.dv, *kp = K + (urow + j0) * sh.d;
            const float *mp = MK + (urow + j0) * sh.mcols;
            if (sh.vec_v) vt.load(vp, sh.dv, nv, sh.dv);
            if (exact_g && sh.vec_x) kt.load(kp, sh.d, nv, sh.d);
            if (cross_g && sh.vec_m) mt.load(mp, sh.mcols, nv, sh.mcols);
            __syncthreads();
            if (exact_g) {
                if (sh.vec_x) kt.store(ks, nv, sh.d);
                else stage_scalar<DT, KT>(kp, sh.d, nv, sh.d, ks);
            }
            if (cross_g) {
                if (sh.vec_m) mt.store(ms, nv, sh.mcols);
                else stage_scalar<RT, KT>(mp, sh.mcols, nv, sh.mcols, ms);
            }
            if (sh.vec_v) vt.store(vs, nv, sh.dv);
            else stage_scalar<VT, KT>(vp, sh.dv, nv, sh.dv, vs);
            __syncthreads();
            f4 part[VT];                                    // WR = 4: this tile's sums (two levels of summation)
            float dpart = 0.f;
            if constexpr (WR == 4) clear(part);
            for (int sub = (WR == 4 ? 0 : wave); sub < KT / 16; sub += (WR == 4 ? 1 : 4)) {
                f4 (&to)[VT] = WR == 4 ? part : acc;
                const int js = j0 + 16 * sub;
                if (js >= j_end || (!sh.noncausal && js > iw_last)) break;
                f4 se = {0.f, 0.f, 0.f, 0.f}, ss = se;
                if (js + 15 >= bs_w) se = score_rows<DT>(ks, 16 * sub, qf, lane);
                if (js < bs_w_last) ss = score_rows<RT>(ms, 16 * sub, mf, lane);
                float w[4];
                const int j_max = sh.noncausal ? sh.n - 1 : i;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int j = js + 4 * g + k;
                    float e = se[k];
                    for (int q = 1; q < sh.p; q <<= 1) e *= e;
                    w[k] = j > j_max ? 0.f : j >= bs ? e : ss[k] * ss[k];
                    dpart += w[k];
                }
                if (!sh.noncausal && js + 15 > iw) {
                    const int vis = i - js;                 // tile rows 0 .. vis count
                    add_rows<VT, true>(vs, 16 * sub, w, to, lane, vis < 0 ? 0u : 0xffffu >> max(0, 15 - vis));
                } else {
                    add_rows<VT, false>(vs, 16 * sub, w, to, lane, 0u);
                }
            }
            den += dpart;
            if constexpr (WR == 4) add_to(acc, part);
        }
    }

    if (sh.states && (sh.noncausal || span > 0)) {
        const float *z = Z + ((size_t)u * sh.spans + (sh.noncausal ? 0 : span)) * record_floats(RT, VT);
        const float *zs = z + (size_t)tile_pairs(RT) * 256 * 16 * VT;
        constexpr int PIECE = KT * 16 * VT, NP = PIECE / 4 / kF32Threads;     // floats of a piece; 16-byte loads a thread
        constexpr int CH = 16 / ZA, LAST = tile_pairs(RT) * CH - 1;
        f4 pre[NP], pre_s = {0.f, 0.f, 0.f, 0.f};
        auto fetch = [&](int piece) {
#pragma unroll
            for (int k = 0; k < NP; ++k)
                pre[k] = *(const f4 *)(z + (size_t)piece * PIECE + (k * kF32Threads + threadIdx.x) * 4);
            if (threadIdx.x < 4 * ZA) pre_s = *(const f4 *)(zs + (size_t)piece * ZA * 16 + threadIdx.x * 4);
        };
        auto put = [&](float *dst, int buf) {
            if (threadIdx.x < 4 * ZA) *(f4 *)&sden[buf][threadIdx.x * 4] = pre_s;
#pragma unroll
            for (int k = 0; k < NP; ++k) {
                const int idx = k * kF32Threads + threadIdx.x;
                *(f4 *)&dst[(idx / (4 * VT)) * VP + 4 * (idx % (4 * VT))] = pre[k];
            }
        };
        fetch(0);
        __syncthreads();
        put(ks, 0);
        // the wave's own sketch rows, where they can be indexed (sync: the last pairs have been read)
        float *own = ms + ((WR == 4 ? 16 * wave : 0) + li) * MP;
#pragma unroll
        for (int q = 0; q < RT; ++q)
            *(f4 *)&own[16 * q + 4 * g] = f4{mf[4 * q], mf[4 * q + 1], mf[4 * q + 2], mf[4 * q + 3]};
        int at = 0, q = 0;
        f4 mq = *(const f4 *)&own[4 * g];
        for (int piece = 0; piece <= LAST; ++piece) {
            const int ch = piece % CH;
            if (piece && ch == 0) {                         // the next pair of index tiles
                if (++q == RT) q = ++at;
                mq = *(const f4 *)&own[16 * q + 4 * g];
            }
            __syncthreads();
            const float *zt = piece & 1 ? vs : ks;
            if (piece < LAST) fetch(piece + 1);
            f4 part[VT];
            float dpart = 0.f;
            if constexpr (WR == 4) clear(part);
            f4 (&to)[VT] = WR == 4 ? part : acc;
#pragma unroll
            for (int k = 0; k < ZW; ++k) {
                const int aa = WR == 1 ? wave : k;
                const float ma = own[16 * at + ZA * ch + aa];
                const f4 sd = *(const f4 *)&sden[piece & 1][aa * 16 + 4 * g];
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    const float phi = ma * mq[s];
                    dpart += phi * sd[s];
#pragma unroll
                    for (int ct = 0; ct < VT; ++ct)
                        to[ct] = mm(zt[(aa * 16 + 4 * g + s) * VP + 16 * ct + li], phi, to[ct]);
                }
            }
            den += dpart;
            if constexpr (WR == 4) add_to(acc, part);
            if (piece < LAST) put(piece & 1 ? ks : vs, ~piece & 1);
        }
    }

    settle();
    den = over_groups(den);
    if constexpr (WR == 1) {
        constexpr int PER = 4 * VT + 1;
        static_assert(3 * PER * 64 <= kTileFloats, "sums of three waves");
        __syncthreads();
        if (wave > 0) {
            float *to = lds + (size_t)(wave - 1) * PER * 64 + lane;
#pragma unroll
            for (int ct = 0; ct < VT; ++ct)
#pragma unroll
                for (int k = 0; k < 4; ++k) to[(4 * ct + k) * 64] = acc[ct][k];
            to[4 * VT * 64] = den;
        }
        __syncthreads();
        if (wave > 0) return;
        for (int o = 0; o < 3; ++o) {
            const float *from = lds + (size_t)o * PER * 64 + lane;
#pragma unroll
            for (int ct = 0; ct < VT; ++ct)
#pragma unroll
                for (int k = 0; k < 4; ++k) acc[ct][k] += from[(4 * ct + k) * 64];
            den += from[4 * VT * 64];
        }
    }
    if (!there && !GRAD) return;
    const float D = 1.f + den;
    if constexpr (!GRAD) {
#pragma unroll
        for (int ct = 0; ct < VT; ++ct)
            store_piece(O + (urow + i) * sh.dv, 16 * ct + 4 * g, sh.dv, sh.vec_v,
                        f4{acc[ct][0] / D, acc[ct][1] / D, acc[ct][2] / D, acc[ct][3] / D});
    } else {
        float go[4 * VT], dot = 0.f;
        load_frags<VT>(dO + (urow + i) * sh.dv, sh.dv, there, sh.vec_v, g, go);
#pragma unroll
        for (int ct = 0; ct < VT; ++ct)
#pragma unroll
            for (int k = 0; k < 4; ++k) dot += go[4 * ct + k] * acc[ct][k];
        dot = over_groups(dot);
        if (!there) return;
#pragma unroll
        for (int ct = 0; ct < VT; ++ct)
            store_piece(GV + (urow + i) * sh.dv, 16 * ct + 4 * g, sh.dv, sh.dv % 4 == 0,
                        f4{go[4 * ct] / D, go[4 * ct + 1] / D, go[4 * ct + 2] / D, go[4 * ct + 3] / D});
        if (g == 0) gden[urow + i] = -(dot / D) / D;
    }
}

template <typename T>
psf_status sketch_pair(const Problem &pb, const void *X1, const void *X2, const void *G, float *M1, float *M2,
                       size_t x_unit, size_t m_unit, hipStream_t s)
{
    const dim3 grid((unsigned)((pb.n + kSketchRows - 1) / kSketchRows), (unsigned)pb.units, X2 ? 2 : 1);
    const int vx = x_unit % 4 == 0 && (X2 ? pieces_ok<T>(pb.d, {X1, X2}) : pieces_ok<T>(pb.d, {X1}));
    const int vm = m_unit % 4 == 0 && pieces_ok<float>(pb.mcols, {M1, M2 ? M2 : M1});
    const int dp = tiles16(pb.d) * 16, rp = tiles16(pb.r) * 16;
    const size_t lds = (size_t)kSketchRows * (dp + 4 + sketch_nodes(pb.p) * (rp + 4)) * sizeof(float);
    if (lds > (64u << 10))                               // p = 16 with wide sketches: up to 118 KB
        PSF_HIP_TRY(hipFuncSetAttribute((const void *)f32_sketch_kernel<T>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                        (int)lds));
    hipLaunchKernelGGL(f32_sketch_kernel<T>, grid, dim3(64), lds, s, (const T *)X1, (const T *)X2, (const T *)G, M1, M2,
                       pb.n, pb.d, pb.r, pb.p, pb.heads, pb.per_head ? 1 : 0, pb.g_len, x_unit, m_unit, vx, vm);
    PSF_LAUNCH_CHECK();
    return PSF_OK;
}

template <typename S>
psf_status states(const Problem &pb, const F32Plan &pl, const float *M, const S *C, const float *wts, float *Z,
                  int span0, int count, int mode, hipStream_t s)
{
    F32Shape sh = f32_shape(pb, pl);
    sh.vec_m = pieces_ok<float>(pb.mcols, {M});
    sh.vec_v = pieces_ok<S>(pb.dv, {C});
    return with_tiles(pb, [&](auto dt, auto rt) -> psf_status {
        constexpr int VT = decltype(dt)::value, RT = decltype(rt)::value;
        hipLaunchKernelGGL((f32_state_kernel<RT, VT, S>), dim3((RT <= 4 ? RT * 2 : RT * 4) * (VT / 4), (unsigned)count, (unsigned)pb.units),
                           dim3(kF32Threads), 0, s, M, C, wts, Z, sh, span0);
        PSF_LAUNCH_CHECK();
        const size_t rec = record_floats(RT, VT), pieces = (size_t)pb.units * (rec / 4);
        hipLaunchKernelGGL(f32_scan_kernel, dim3((unsigned)((pieces + kF32Threads - 1) / kF32Threads)),
                           dim3(kF32Threads), 0, s, Z, pieces, rec, pl.spans, mode);
        PSF_LAUNCH_CHECK();
        return PSF_OK;
    });
}

template <typename T, bool GRAD>
psf_status rows_launch(const Problem &pb, const F32Plan &pl, const float *MQ, const float *MK, const void *Q,
                       const void *K, const void *V, const float *Z, void *O, const void *dO, float *GV, float *gden,
                       hipStream_t s)
{
    F32Shape sh = f32_shape(pb, pl);
    sh.vec_x = pieces_ok<T>(pb.d, {Q, K});
    sh.vec_v = GRAD ? pieces_ok<T>(pb.dv, {V, dO}) : pieces_ok<T>(pb.dv, {V, O});
    sh.vec_m = pieces_ok<float>(pb.mcols, {MQ, MK});
    return with_tiles(pb, [&](auto dt, auto rt) -> psf_status {
        constexpr int DT = decltype(dt)::value, RT = decltype(rt)::value;
        auto go = [&](auto kernel, int rows) {
            const int per_span = ((pl.span < pb.n ? pl.span : pb.n) + rows - 1) / rows;
            const FlatGrid grid = flat_grid((unsigned long long)per_span * pl.spans * pb.units);
            hipLaunchKernelGGL(kernel, dim3(grid.x, grid.y), dim3(kF32Threads), 0,
                               s, MQ, MK, (const T *)Q, (const T *)K, (const T *)V, Z, (T *)O, (const T *)dO, GV, gden,
                               sh);
        };
        if constexpr (DT == 4) {
            if (f32_split_rows(pb)) {
                go(f32_rows_kernel<DT, RT, DT, 1, GRAD, T>, 16);
                PSF_LAUNCH_CHECK();
                return PSF_OK;
            }
        }
        go(f32_rows_kernel<DT, RT, DT, 4, GRAD, T>, 64);
        PSF_LAUNCH_CHECK();
        return PSF_OK;
    });
}

}  // namespace

bool f32_supported(const Problem &pb)
{
    return !pb.exact_feat && pb.d <= 128 && pb.dv <= 128 && pb.mcols <= 128;
}

bool f32_split_rows(const Problem &pb)
{
    return (long long)pb.units * ((pb.n + 63) / 64) < 512;
}

F32Shape f32_shape(const Problem &pb, const F32Plan &pl)
{
    F32Shape sh = {};
    sh.n = pb.n; sh.d = pb.d; sh.dv = pb.dv; sh.mcols = pb.mcols; sh.p = pb.p; sh.b = pb.b; sh.units = pb.units;
    sh.span = pl.span; sh.spans = pl.spans;
    sh.local_exact = pb.local_exact && !pl.noncausal;
    sh.noncausal = pl.noncausal; sh.pairs = pl.pairs; sh.states = pl.states;
    return sh;
}

// Where the states lie.  Costs in seconds of the whole chip: states at 90 TFLOP/s, pairs at 65 (72 over
// 3000 tokens, 50 over 1950, where the launch is short), state traffic at 4 TB/s, 5 us for the two
// further launches: forming a record and applying it against the pairs that a longer span takes
// directly.  Measured with every span forced (blocks a span: us of a forward call, of a backward call;
// * the plan's choice; two runs of one span differ by up to 6 %):
//   36 units x 3000, r 32, b 200   1: 410, 1277   2: 393*, 1245*   4: 391, 1293   8: 456, 1570   all 15: 469, 1842
//   24 x 1950, r 32, b 150         1: 214, 619    2: 185, 600*     4: 223, 759    8: 246, 776    all 13: 201*, 686
//   12 x 16384, r 32, b 64         1: 806, 2291   4: 569, 1916*    8: 573*, 2050  16: 666, 2444  all: 3535, 14920
//   24 x 8000, r 64, b 250         1: 1634, 5082  2: 1591, 5146*   4: 1658*, 5592 8: 1949, 6737
//   48 x 8192, r 16, b 256         1: 609*, 2074* 2: 667, 2385     4: 832, 3106
// z_floats: room for state records.
static F32Plan f32_plan(const Problem &pb, size_t z_floats, bool noncausal, bool grad)
{
    const bool wide = pb.d > 64 || pb.dv > 64 || pb.mcols > 64;
    int rt = 0, vt = wide ? 8 : 4;
    with_tiles(pb, [&](auto, auto r) -> psf_status { rt = decltype(r)::value; return PSF_OK; });
    const double tokens = (double)pb.units * pb.n, rate = 90e12, pair_rate = 65e12, bw = 4e12;
    const size_t rec = record_floats(rt, vt);
    const double state_flops = tile_pairs(rt) * 256.0 * 16 * vt * 2 * (grad ? 6 : 2);
    const double pair_flops = 2.0 * 16 * (grad ? 5 * rt + 4 * vt : rt + vt);
    const double passes = grad ? 9 : 4;
    F32Plan best = {};
    if (noncausal) {
        const double direct = tokens * pb.n * pair_flops / pair_rate;
        const double with_state = tokens * state_flops / rate + 10e-6;
        // spans only split the sum over the tokens: enough workgroups to fill the chip
        int spans = (int)((2048 + (long long)pb.units * 4 * rt - 1) / ((long long)pb.units * 4 * rt));
        if (spans > pb.n / 256) spans = pb.n / 256;
        if (spans < 1) spans = 1;
        const size_t most = z_floats / ((size_t)pb.units * rec);
        if ((size_t)spans > most) spans = (int)most;
        best.noncausal = 1;
        best.cost = direct;
        if (spans < 1 || direct <= with_state) {
            best.span = pb.n; best.spans = 1; best.pairs = 1;
            return best;
        }
        best.cost = with_state;
        best.span = (pb.n + spans - 1) / spans;
        best.spans = (pb.n + best.span - 1) / best.span;
        best.states = 1;
        return best;
    }
    for (int s = 1;; s *= 2) {
        if (s > pb.t) s = pb.t;
        const int spans = (pb.t + s - 1) / s;
        const double span = (double)s * pb.b;
        if (spans == 1 || (size_t)spans * pb.units * rec <= z_floats) {
            double cost = tokens * (span < pb.n ? span : pb.n) / 2 * pair_flops / pair_rate;
            if (spans > 1)
                cost += tokens * (1.0 - 1.0 / spans) * state_flops / rate +
                        (double)pb.units * spans * rec * 4 * passes / bw + (grad ? 10e-6 : 5e-6);
            if (best.spans == 0 || cost < best.cost) {
                best.cost = cost;
                best.span = s * pb.b; best.spans = spans; best.pairs = 1; best.states = spans > 1;
            }
        }
        if (s == pb.t) break;
    }
    return best;
}

static size_t plan_floats(const Problem &pb, const F32Plan &pl)
{
    size_t rec = 0;
    with_tiles(pb, [&](auto dt, auto rt) -> psf_status {
        rec = record_floats(decltype(rt)::value, decltype(dt)::value);
        return PSF_OK;
    });
    return pl.states ? (size_t)pb.units * pl.spans * rec : 0;
}

// Records are padded to tiles (16 sketch indices, 64 or 128 value columns), the room of the vector
// kernels, t F (dv + 1) floats a unit, is not: with few or small blocks (t mcols^2 (dv + 1) below the
// record's floats) no record fits, and pairs alone cost time quadratic in n.  Where that room
// makes the plan dearer than the best one by more than a quarter, the workspace grows to the
// best plan's records (at most kMostRoom, and not past the library's static scratch where the
// call fitted it).  If that does not bring the cost within four times the best one, the vector
// kernels take the call, whose time is linear.  Measured, without a mask, r = 8, d = 128, dv = 16, two
// blocks (us; pairs, best plan, vector kernels): 12 units x 4096 1274, 272, 714; 12 x 16384 20429, 1050,
// 2487; 96 x 16384 165250, 7607, 10294.  Below 1.25 nothing is to be gained (96 x 1024: 687, 687, 750).
F32Choice f32_choose(const Problem &pb, size_t fixed_bytes, bool noncausal, bool grad)
{
    constexpr size_t kMostRoom = ((size_t)1 << 30) / sizeof(float);
    F32Choice c = {};
    c.z_floats = (size_t)pb.units * pb.t * (size_t)pb.F * (pb.dv + 1);
    if (!f32_supported(pb)) return c;
    c.use = true;
    c.plan = f32_plan(pb, c.z_floats, noncausal, grad);
    const double best = f32_plan(pb, SIZE_MAX, noncausal, grad).cost;
    if (c.plan.cost <= 1.25 * best) return c;
    size_t room = kMostRoom;
    if (!noncausal && !grad && fixed_bytes + align_up(c.z_floats * 4, 256) <= PSF_STATIC_SCRATCH_BYTES)
        room = (PSF_STATIC_SCRATCH_BYTES - fixed_bytes) / 256 * 256 / sizeof(float);
    if (room > c.z_floats) {
        c.plan = f32_plan(pb, room, noncausal, grad);
        const size_t need = plan_floats(pb, c.plan);
        if (need > c.z_floats) c.z_floats = need;
    }
    if (c.plan.cost > 4.0 * best) {
        c = {};
        c.z_floats = (size_t)pb.units * pb.t * (size_t)pb.F * (pb.dv + 1);
    }
    return c;
}

psf_status f32_sketch_pair(const Problem &pb, const void *X1, const void *X2, const void *G, float *M1, float *M2,
                           hipStream_t s)
{
    const size_t x_unit = (size_t)pb.n * pb.d, m_unit = (size_t)pb.n * pb.mcols;
    return pb.bf16 ? sketch_pair<bf16_t>(pb, X1, X2, G, M1, M2, x_unit, m_unit, s)
                   : sketch_pair<float>(pb, X1, X2, G, M1, M2, x_unit, m_unit, s);
}

psf_status f32_sketch_rows(const Problem &pb, const void *X, size_t x_unit, const void *G, float *M, size_t m_unit,
                           hipStream_t s)
{
    return pb.bf16 ? sketch_pair<bf16_t>(pb, X, nullptr, G, M, nullptr, x_unit, m_unit, s)
                   : sketch_pair<float>(pb, X, nullptr, G, M, nullptr, x_unit, m_unit, s);
}

psf_status f32_key_states(const Problem &pb, const F32Plan &pl, const float *MK, const void *V, float *Z, hipStream_t s)
{
    const int count = pl.noncausal ? pl.spans : pl.spans - 1, mode = pl.noncausal ? kScanTotal : kScanPrefix;
    return pb.bf16 ? states<bf16_t>(pb, pl, MK, (const bf16_t *)V, nullptr, Z, 0, count, mode, s)
                   : states<float>(pb, pl, MK, (const float *)V, nullptr, Z, 0, count, mode, s);
}

psf_status f32_mirror_states(const Problem &pb, const F32Plan &pl, const float *MQ, const float *GV, const float *gden,
                             float *R, hipStream_t s)
{
    return states<float>(pb, pl, MQ, GV, gden, R, 1, pl.spans - 1, kScanSuffix, s);
}

psf_status f32_rows(const Problem &pb, const F32Plan &pl, const float *MQ, const float *MK, const void *Q,
                    const void *K, const void *V, const float *Z, void *O, hipStream_t s)
{
    return pb.bf16 ? rows_launch<bf16_t, false>(pb, pl, MQ, MK, Q, K, V, Z, O, nullptr, nullptr, nullptr, s)
                   : rows_launch<float, false>(pb, pl, MQ, MK, Q, K, V, Z, O, nullptr, nullptr, nullptr, s);
}

psf_status f32_rows_grad(const Problem &pb, const F32Plan &pl, const float *MQ, const float *MK, const void *Q,
                         const void *K, const void *V, const float *Z, const void *dO, float *GV, float *gden,
                         hipStream_t s)
{
    return pb.bf16 ? rows_launch<bf16_t, true>(pb, pl, MQ, MK, Q, K, V, Z, nullptr, dO, GV, gden, s)
                   : rows_launch<float, true>(pb, pl, MQ, MK, Q, K, V, Z, nullptr, dO, GV, gden, s);
}

}  // namespace psf
