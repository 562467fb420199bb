// fp32 matrix-core kernels of the general path: states and rows of the output, for sketch features with
// d, dv and sketch columns <= 128 (any block size, fp32 or bf16 storage); the sketches: psf_f32_sketch.h.
// Everything is fp32 as in the vector kernels of psf_general.hip (which keep explicit exact features,
// sizes above 128 and what f32_choose leaves to them); the products are formed from exact bf16
// parts, see psf_parts.h.  Layouts: psf_f32_tiles.h.
//
// The in-block rule only says which weight a pair of tokens gets; it does not force a state per
// block.  A state is kept per span of several blocks, and pairs of different blocks inside a span
// take their weight <m(q), m(k)>^2 directly: 2 (r + dv) flops a pair against about 2 r^2 dv a
// token for forming and applying a state, and no state traffic (1.5 MB per block and unit with r = 64).
// f32_plan() chooses the span.
//
// Measured (us a call, forward / forward and backward; vector kernels, products by
// v_mfma_f32_16x16x4_f32, now): 36 units of 3000 tokens, r = 32, b = 200, bf16 storage 8540, 361, 190;
// 24 units of 1950, b = 150, forward and backward 26940, 772, 450; one unit of 1024, r = 16, fp32
// storage 248, 33, 32.
#include "psf_parts.h"
#include "psf_f32.h"

namespace psf {
namespace {

// ---- states: sum over the tokens of a span of phi'(x_j) [C_j | w_j] --------------------------
// A wave owns two sketch indices, one of tile row `lo` and one of tile row `hi` = RT - 1 - lo (the
// same row for r = 16), so that every wave has RT + 1 tiles of pairs, and walks the tokens, 32 a
// step: A = m_j[a] m_j[b'] (fp32 in registers, then parts), B = the parts of C_j.  The denominator
// column is a running sum of the fp32 products.  The four column tiles are read once for both
// indices.  The sketches lie in LDS by column, so that a lane reads its tokens as 16-byte pieces.
// Bound by the vector instructions that make the operands: 60 of them a tile and step against 12 products
// with values stored as bf16 and 24 with fp32 ones (240 cycles against 192 and 384).
// Wide values (VT = 8) are split over two workgroups, 64 columns each.  Where RT + 1 tiles in two
// levels of sums exceed the registers (RT = 8), a wave takes one index and RT tiles, of which
// those below the diagonal are empty.
template <int RT, int VT, typename S>
__global__ __launch_bounds__(kF32Threads, RT <= 2 ? 2 : 1) void f32_state_kernel(
    const float *__restrict__ M, const S *__restrict__ C, const float *__restrict__ wts, float *__restrict__ Z,
    F32Shape sh, int span0)
{
    constexpr int KT = RT > 4 ? 32 : 64, MP = KT + 4, VP = tr_pitch<4>(), P = parts_of<S>();
    constexpr bool TWO = RT <= 4;
    constexpr int SLOTS = TWO ? RT + 1 : RT, NM = 4 * RT * KT / kF32Threads;
    __shared__ __attribute__((aligned(16))) float ms[16 * RT * MP], ws[KT];
    __shared__ __attribute__((aligned(16))) uint16_t vs[P * KT * VP];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), li = lane & 15, g = lane >> 4;
    const int grp = blockIdx.x / (VT / 4), c0 = 64 * (blockIdx.x % (VT / 4));
    // TWO: groups of four index pairs; r = 16 pairs a with a + 8 of the one tile row
    const int lo = RT == 1 ? 0 : grp / 4, a_lo = RT == 1 ? 4 * grp + wave : 16 * lo + 4 * (grp % 4) + wave;
    const int hi = TWO ? RT - 1 - lo : lo, a_hi = RT == 1 ? a_lo + 8 : 16 * hi + 4 * (grp % 4) + wave;
    const int split = RT - lo;                              // slots of a_lo; the others are a_hi's
    const int span = span0 + blockIdx.y, u = blockIdx.z;
    const TokenRange tokens_of = state_tokens(sh.n, sh.span, span, sh.dv, c0);
    const int j_begin = tokens_of.begin, j_end = tokens_of.end;
    f4 acc[SLOTS][4], part[SLOTS][4];                       // two levels of summation, as in psf_f32_bwd.hip
    float den[SLOTS];
    int mcol[SLOTS];                                        // first sketch column of the slot's tile
#pragma unroll
    for (int e = 0; e < SLOTS; ++e) {
        den[e] = 0.f;
        mcol[e] = 16 * (e < split ? lo + e : min(hi + e - split, RT - 1));
        clear(acc[e]);
        clear(part[e]);
    }
    PartTile<4, KT, VP, S> ct;
    f4 mt[NM];
    float wt = 1.f;
    // a lane takes a token, so that the stores by column go to different banks
    const int m_tok = threadIdx.x % KT, m_c = 4 * (threadIdx.x / KT);
    constexpr int M_STEP = 4 * (kF32Threads / KT);
    auto fetch = [&](int j0) {
        const size_t row = (size_t)u * sh.n + j0;
        const int nv = j_end - j0;
        if (sh.vec_v) ct.load(C + row * sh.dv + c0, sh.dv, nv, sh.dv - c0);
#pragma unroll
        for (int k = 0; k < NM; ++k) {
            const float *mp = M + row * sh.mcols;
            if (sh.vec_m) mt[k] = *(const f4 *)(mp + tile_piece(m_tok, m_c + k * M_STEP, sh.mcols, nv, sh.mcols));
            else mt[k] = row_piece(mp + (size_t)(m_tok < nv ? m_tok : 0) * sh.mcols, m_c + k * M_STEP, sh.mcols, 0);
        }
        if (wts && threadIdx.x < KT) wt = (int)threadIdx.x < nv ? wts[row + threadIdx.x] : 0.f;
    };
    if (j_begin < j_end) fetch(j_begin);
    for (int j0 = j_begin; j0 < j_end; j0 += KT) {
        const int nv = j_end - j0;
        __syncthreads();
#pragma unroll
        for (int k = 0; k < NM; ++k)
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const int c = m_c + k * M_STEP + s;
                ms[c * MP + m_tok] = m_tok < nv && c < sh.mcols ? mt[k][s] : 0.f;
            }
        if (sh.vec_v) ct.template store<false>(vs, nv, sh.dv - c0);
        else stage_parts_scalar<4, KT, VP, S, false>(C + ((size_t)u * sh.n + j0) * sh.dv + c0, sh.dv, nv, sh.dv - c0, vs);
        if (threadIdx.x < KT) ws[threadIdx.x] = wt;
        __syncthreads();
        if (j0 + KT < j_end) fetch(j0 + KT);
#pragma unroll
        for (int t32 = 0; t32 < KT; t32 += 32) {
            if (t32 >= nv) break;
            // tile order: tokens t32 + 4 g + s and 16 further on
            const float *mrow = ms + t32 + 4 * g;
            auto tokens = [&](const float *at, float (&x)[8]) {
                const f4 lo4 = *(const f4 *)at, hi4 = *(const f4 *)(at + 16);
#pragma unroll
                for (int s = 0; s < 4; ++s) { x[s] = lo4[s]; x[4 + s] = hi4[s]; }
            };
            Parts<P> vb[4];
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int i = 0; i < P; ++i) vb[t].v[i] = read_columns(vs + t32 * VP + i * KT * VP, VP, 16 * t, lane);
            float ma_lo[8], ma_hi[8], wj[8];
            tokens(mrow + a_lo * MP, ma_lo);
            if (TWO) tokens(mrow + a_hi * MP, ma_hi);
            if (wts) tokens(ws + t32 + 4 * g, wj);
#pragma unroll
            for (int e = 0; e < SLOTS; ++e) {
                if (!TWO && e >= split) break;
                float mb[8], av[8];
                tokens(mrow + (mcol[e] + li) * MP, mb);
                // the first tile of an index is on the diagonal, the others stand for their mirror too
                const float twice = e == 0 || e == split ? 1.f : 2.f;
                float sum = 0.f;
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    av[k] = mb[k] * (!TWO || e < split ? ma_lo[k] : ma_hi[k]);
                    sum = wts ? __builtin_fmaf(av[k], wj[k], sum) : sum + av[k];
                }
                den[e] = __builtin_fmaf(sum, twice, den[e]);
                Parts<3> ap;
                split8(av, ap);
                mm_columns(ap, vb, part[e]);
            }
        }
        if (((j0 - j_begin) / KT & 1) || j0 + KT >= j_end) {
            settle_parts();
#pragma unroll
            for (int e = 0; e < SLOTS; ++e) {
                const float twice = e == 0 || e == split ? 1.f : 2.f;
#pragma unroll
                for (int t = 0; t < 4; ++t) acc[e][t] += part[e][t] * twice;
                clear(part[e]);
            }
        }
    }
    // An infinity or NaN among the values: its parts are no sum of them (inf - inf), so the wave forms these
    // sums from fp32 products instead.
    if (any_odd(acc)) {
#pragma unroll
        for (int e = 0; e < SLOTS; ++e) clear(acc[e]);
#pragma unroll 1
        for (int j = j_begin; j < j_end; ++j) {
            const float *mp = M + ((size_t)u * sh.n + j) * sh.mcols;
            const S *cp = C + ((size_t)u * sh.n + j) * sh.dv + c0;
            auto m_of = [&](int c) { return c < sh.mcols ? mp[c] : 0.f; };
            const float ma_lo = m_of(a_lo), ma_hi = TWO ? m_of(a_hi) : 0.f;
            float v[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) v[t] = c0 + 16 * t + li < sh.dv ? load_f(cp, 16 * t + li) : 0.f;
#pragma unroll
            for (int e = 0; e < SLOTS; ++e) {
                if (!TWO && e >= split) break;
                const float ma = (!TWO || e < split ? ma_lo : ma_hi) * (e == 0 || e == split ? 1.f : 2.f);
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const float phi = ma * m_of(mcol[e] + 4 * g + k);
#pragma unroll
                    for (int t = 0; t < 4; ++t) acc[e][t][k] += phi * v[t];
                }
            }
        }
    }
    float *rec = Z + ((size_t)u * sh.spans + span) * record_floats(RT, VT);
    float *srec = rec + record_values(RT, VT) / 2 * 3;
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

// In place over the spans of a unit: exclusive prefix, exclusive suffix, or the total in slot 0; the
// values leave as parts (see tile_pairs).  A thread takes eight columns, or four entries of the
// denominator column, of all spans.  Bound by the latency of a step where units are few and spans many: the next four
// records are loaded before these four are written, so that a thread waits once for four of them, and a workgroup is a
// wave (6 units x 32256, r = 16, 126 spans, fp32: the call 357 -> 337 us; 332 with fp32 records).
// The record that an exclusive sum never reads (the last, or the first) need not be there.
enum { kScanPrefix = 0, kScanSuffix = 1, kScanTotal = 2 };
constexpr int kScanThreads = 64;                            // few units: as many CUs as there are waves
__global__ __launch_bounds__(kScanThreads) void f32_scan_kernel(float *__restrict__ Z, int units, size_t values,
                                                               size_t rec, int spans, int mode)
{
    const size_t idx = (size_t)blockIdx.x * kScanThreads + threadIdx.x, per = values / 8 + (rec - values / 2 * 3) / 4;
    if (idx >= (size_t)units * per) return;
    const size_t in = idx % per;
    const bool vals = in < values / 8;
    float *z = Z + (idx / per) * (size_t)spans * rec + (vals ? in * 8 : values / 2 * 3 + (in - values / 8) * 4);
    float *zl = Z + (idx / per) * (size_t)spans * rec + values + in * 4;
    constexpr int AHEAD = 4;
    f4 run[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}}, next[AHEAD][2];
#pragma unroll
    for (int j = 0; j < AHEAD; ++j) clear(next[j]);
    auto load = [&](int k, f4 (&to)[2]) {
        if (k >= (mode == kScanTotal ? spans : spans - 1)) return;
        const float *at = z + (size_t)(mode == kScanSuffix ? spans - 1 - k : k) * rec;
        to[0] = *(const f4 *)at;
        if (vals) to[1] = *(const f4 *)(at + 4);
    };
    auto store = [&](int k) {
        const size_t at = (size_t)(mode == kScanSuffix ? spans - 1 - k : k) * rec;
        if (!vals) {
            *(f4 *)(z + at) = run[0];
            return;
        }
        const float x[8] = {run[0][0], run[0][1], run[0][2], run[0][3], run[1][0], run[1][1], run[1][2], run[1][3]};
        Parts<3> p;
        split8<true>(x, p);
        *(bf8 *)(z + at) = p.v[0];
        *(bf8 *)(z + at + 4) = p.v[1];
        *(bf8 *)(zl + at) = p.v[2];
    };
#pragma unroll
    for (int j = 0; j < AHEAD; ++j) load(j, next[j]);
    for (int k = 0; k < spans; k += AHEAD) {
        f4 h[AHEAD][2];
#pragma unroll
        for (int j = 0; j < AHEAD; ++j) {
            h[j][0] = next[j][0];
            h[j][1] = next[j][1];
        }
#pragma unroll
        for (int j = 0; j < AHEAD; ++j) load(k + AHEAD + j, next[j]);
#pragma unroll
        for (int j = 0; j < AHEAD; ++j) {
            if (k + j >= spans) break;
            if (mode != kScanTotal) store(k + j);
            run[0] += h[j][0];
            run[1] += h[j][1];
        }
    }
    if (mode == kScanTotal) store(0);
}

// the end of a row: acc^T holds its unnormalised output
template <int VT, bool GRAD, typename T>
__device__ __forceinline__ void finish_row(const f4 (&acc)[VT], float D, bool there, int li, int g, size_t row,
                                           T *__restrict__ O, const T *__restrict__ dO, float *__restrict__ GV,
                                           float *__restrict__ gden, const F32Shape &sh)
{
    if constexpr (!GRAD) {
#pragma unroll
        for (int ct = 0; ct < VT; ++ct)
            store_piece(O + row * sh.dv, 16 * ct + 4 * g, sh.dv, sh.vec_v,
                        f4{acc[ct][0] / D, acc[ct][1] / D, acc[ct][2] / D, acc[ct][3] / D});
    } else {
        float go[4 * VT], dot = 0.f;
        load_frags<VT>(dO + row * sh.dv, sh.dv, there, sh.vec_v, g, go);
#pragma unroll
        for (int ct = 0; ct < VT; ++ct)
#pragma unroll
            for (int k = 0; k < 4; ++k) dot += go[4 * ct + k] * acc[ct][k];
        dot = over_groups(dot);
        if (!there) return;
#pragma unroll
        for (int ct = 0; ct < VT; ++ct)
            store_piece(GV + row * sh.dv, 16 * ct + 4 * g, sh.dv, sh.dv % 4 == 0,
                        f4{go[4 * ct] / D, go[4 * ct + 1] / D, go[4 * ct + 2] / D, go[4 * ct + 3] / D});
        if (g == 0) gden[row] = -(dot / D) / D;
    }
}

// ---- rows: pairs of the row's span, then phi'(q_i)^T Z, then the division --------------------
// WR waves take 16 rows each, and WK such sets share the keys of a tile (32 each) and the indices a of a
// state and add up at the end; every staged tile serves all of them.
//   WR 4, WK 1: two or more workgroups a CU; two groups of 32 keys a tile, one after the other
//   WR 4, WK 2: fewer, but one for most CUs: half the steps each
//   WR 1, WK 4: four times the workgroups
// The sums of a staged tile are formed apart and then added to the total.
// GRAD: instead of the output, G_i = [dO_i / D_i | -<dO_i, o_i> / D_i] for the backward pass.
// SPLIT: up to gridDim.z workgroups share the key tiles of the same rows, `share` each, and leave their sums in slots of
// `part`, in the order of the registers, for f32_rows_sum_kernel (see f32_row_share).
template <int DT, int RT, int WR, int WK, typename T>
struct RowsLds {
    static constexpr int P = parts_of<T>(), MT = RT < 2 ? 2 : RT, OP = pitch_of<RT>(), ROWS = 16 * WR;
    // (fp32 storage, r = 64: four sets only fit with narrower rows of V, which cost bank conflicts.  1024 tokens of a
    // unit 52 us with two sets of 16 rows, 32 so; 64 rows 40.)
    static constexpr bool TIGHT = WR == 1 && DT == 4 && MT == 4 && P == 3;
    static constexpr int KP = row_pitch<DT>(), VP = TIGHT ? 16 * DT + 4 : tr_pitch<DT>(), MP = row_pitch<MT>();
    static constexpr int ZP = tr_pitch<DT>();                         // rows of a state piece
    static constexpr int kRow = P * KP + P * VP + 3 * MP;             // 16-bit places of a key
    static constexpr int kThreads = 64 * WR * WK, KT = WK == 1 ? f32_tile_rows(DT) : 32 * WK;
    static constexpr int kKeys = P * KT * KP, kVals = P * KT * VP;
    static constexpr int kBuffers = WK == 4 ? 1 : 2;
    static constexpr int kPiece = 3 * 32 * ZP, kOwn = ROWS * OP * 2;  // a state piece; sketches of the rows, fp32
    static constexpr int kBack = WK * ROWS * (16 * DT + 4) * 2;       // the states' share of the rows, fp32
    static constexpr int kSums = (WK - 1) * WR * (4 * DT + 1) * 64 * 2;
    static constexpr int most(int a, int b) { return a > b ? a : b; }
    static constexpr int kPlaces = most(most(KT * kRow, kBuffers * WK * kPiece + kOwn), most(kBack, kSums));
};

template <int DT, int RT, int WR, int WK, bool GRAD, bool SPLIT, typename T>
__device__ __forceinline__ void rows_workgroup(
    const float *__restrict__ MQ, const float *__restrict__ MK, const T *__restrict__ Q, const T *__restrict__ K,
    const T *__restrict__ V, const float *__restrict__ Z, T *__restrict__ O, const T *__restrict__ dO,
    float *__restrict__ GV, float *__restrict__ gden, const F32Shape &sh, int share, float *__restrict__ part)
{
    using L = RowsLds<DT, RT, WR, WK, T>;
    constexpr int VT = DT, ROWS = L::ROWS, KT = L::KT, P = L::P, MT = L::MT, KP = L::KP, VP = L::VP, MP = L::MP;
    constexpr int THREADS = L::kThreads;
    __shared__ __attribute__((aligned(16))) uint16_t lds[L::kPlaces];
    __shared__ __attribute__((aligned(16))) float sden[L::kBuffers][32 * WK];        // denominator column of a state piece
    __shared__ int odd_tile[2];                                       // the tile of V holds an infinity or NaN
    uint16_t *ks = lds, *vs = ks + L::kKeys, *ms = vs + L::kVals;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), li = lane & 15, g = lane >> 4;
    RowPlace at_rows;
    const int per_span = (min(sh.span, sh.n) + ROWS - 1) / ROWS;
    if (!row_place(blockIdx.y * gridDim.x + blockIdx.x, sh.units, sh.spans, per_span, at_rows)) return;
    const int u = at_rows.unit, span = sh.spans - 1 - at_rows.span;
    const int s_begin = span * sh.span, s_end = min(sh.n, s_begin + sh.span);
    const int i0 = s_begin + (per_span - 1 - at_rows.k) * ROWS;
    if (i0 >= s_end) return;
    if constexpr (SPLIT) {
        static_assert(WR == 1 && WK == 4 && DT == 4 && !GRAD, "blocks of 16 rows, tiles of 128 keys, slots");
        if ((int)blockIdx.z >= row_slices(i0 / 16, sh.n, share, !sh.noncausal)) return;
    }
    const int wr = wave % WR, wk = wave / WR, iw = i0 + 16 * wr, i = iw + li;
    const int i_last = min(i0 + ROWS, s_end) - 1, iw_last = min(iw + 15, s_end - 1);
    const bool there = i < s_end;
    const size_t urow = (size_t)u * sh.n;
    const size_t i_row = urow + min(i, s_end - 1);          // (rows that are not there hold another's values and are not stored)
    f4 acc[VT];
    float den = 0.f;
    clear(acc);

    // The state's share.  T_a = sum over b' of Z[a][b'] m(q)[b'] is a product with the rows' sketches as fixed
    // operands, and the share is sum over a of m(q)[a] T_a in fp32 vector arithmetic: 16 of them a
    // lane for 24 products, where features phi' as operands cost 8 multiplications and 44 instructions to take
    // them apart.  A wave takes 16 columns (32 of wide values) of all 64 rows, so that an operand read
    // from LDS serves four products of rows.  A piece is one a with 32 b' (two index tiles, the
    // first of which holds zeros where it lies left of the diagonal).
    if (sh.states && (sh.noncausal || span > 0)) {
        constexpr int KS = MT / 2, ZP = L::ZP, C = VT / WR, H = WR, OP = L::OP, CP = 16 * VT, CH = CP / 8;
        const float *z = Z + ((size_t)u * sh.spans + (sh.noncausal ? 0 : span)) * record_floats(RT, VT);
        const float *zs = z + record_values(RT, VT) / 2 * 3;
        constexpr int NP = 32 * CH * WK / THREADS;
        static_assert(32 * CH * WK % THREADS == 0 && 16 % WK == 0, "whole pieces");
        RecordPiece pre[NP];
        float pre_s = 0.f;
        int fa = 0, fk = 0;                                 // the pieces to fetch: first sketch index, pair of tiles
        auto fetch = [&]() {
            const int at = fa >> 4, first = at * RT - at * (at - 1) / 2 - at;
#pragma unroll
            for (int k = 0; k < NP; ++k) {
                const int idx = k * THREADS + threadIdx.x, row = idx / CH % 32, q = 2 * fk + (row >> 4);
                const int a16 = (fa & 15) + idx / (32 * CH);
                if (q >= at && q < RT)
                    pre[k].load(z, record_values(RT, VT), CP, ((first + q) * 16 + a16) * 16 + (row & 15), 8 * (idx % CH));
                else pre[k].zero();
            }
            if (threadIdx.x < 32 * WK) {
                const int q = 2 * fk + (threadIdx.x >> 4 & 1), a16 = (fa & 15) + threadIdx.x / 32;
                pre_s = q >= at && q < RT ? zs[((first + q) * 16 + a16) * 16 + (threadIdx.x & 15)] : 0.f;
            }
            if (++fk == KS) { fa += WK; fk = fa >> 5; }
        };
        auto put = [&](int buf) {
            if (threadIdx.x < 32 * WK) sden[buf][threadIdx.x] = pre_s;
#pragma unroll
            for (int k = 0; k < NP; ++k) {
                const int idx = k * THREADS + threadIdx.x;
                pre[k].store(lds + (buf * WK + idx / (32 * CH)) * L::kPiece + (idx / CH % 32) * ZP + 8 * (idx % CH), 32 * ZP);
            }
        };
        fetch();
        // the rows' sketches, where they can be indexed
        float *own = (float *)(lds + L::kBuffers * WK * L::kPiece);
        Parts<3> mb[H][KS];
        float md[8 * KS];                                   // of the wave's 16 rows, for the denominator
        {
            OwnRow<KS, float> rows[H], mine;
#pragma unroll
            for (int h = 0; h < H; ++h)
                rows[h].load(MQ + (urow + min(i0 + 16 * h + li, s_end - 1)) * sh.mcols, sh.mcols, sh.vec_m, g);
            mine.load(MQ + i_row * sh.mcols, sh.mcols, sh.vec_m, g);
            put(0);
#pragma unroll
            for (int h = 0; h < H; ++h) rows[h].parts(mb[h], sh.mcols, g);
#pragma unroll
            for (int e = 0; e < 2 * KS; ++e) {
                const f4 v = mine.at(e, sh.mcols, g);
                const int c = 32 * (e / 2) + 8 * g + 4 * (e % 2);
#pragma unroll
                for (int s = 0; s < 4; ++s) md[4 * e + s] = v[s];
                if (wk == 0 && c < 16 * RT) *(f4 *)&own[(16 * wr + li) * OP + c] = v;
            }
        }
        f4 sum[H * C];
        clear(sum);
        int buf = 0;
#pragma unroll 1                                            // (r = 16 and two sets: all eight turns at once spill)
        for (int a0 = 0; a0 < 16 * RT; a0 += WK) {
            const int a = a0 + wk;
            f4 ta[H * C];
            clear(ta);
            float sd = 0.f;
#pragma unroll
            for (int k = 0; k < KS; ++k) {
                if (k < (a0 >> 5)) continue;
                __syncthreads();
                const bool more = fa < 16 * RT;
                if (more) fetch();
#pragma unroll
                for (int e = 0; e < 8; e += 4) {
                    const f4 s = *(const f4 *)&sden[buf][32 * wk + 8 * g + e];
                    sd += (s[0] * md[8 * k + e] + s[1] * md[8 * k + e + 1]) + (s[2] * md[8 * k + e + 2] + s[3] * md[8 * k + e + 3]);
                }
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    Parts<3> zp;
#pragma unroll
                    for (int i = 0; i < 3; ++i)
                        zp.v[i] = read_rows_tr(lds + (buf * WK + wk) * L::kPiece + i * 32 * ZP, ZP, 16 * (C * wr + c), lane);
                    mm_rows(zp, mb, k, ta + H * c);
                }
                settle_parts();                             // (the step may be left out)
                if (L::kBuffers == 1) __syncthreads();
                else buf ^= 1;
                if (more) put(buf);
            }
            float ma[H];
#pragma unroll
            for (int h = 0; h < H; ++h) ma[h] = own[(16 * h + li) * OP + a];
            den += own[(16 * wr + li) * OP + a] * sd;
#pragma unroll
            for (int h = 0; h < H; ++h)
#pragma unroll
                for (int c = 0; c < C; ++c) sum[H * c + h] += ta[H * c + h] * ma[h];
        }
        // from columns of all rows to all columns of the wave's rows
        __syncthreads();
        float *back = (float *)lds + wk * ROWS * (CP + 4);
#pragma unroll
        for (int h = 0; h < H; ++h)
#pragma unroll
            for (int c = 0; c < C; ++c) *(f4 *)&back[(16 * h + li) * (CP + 4) + 16 * (C * wr + c) + 4 * g] = sum[H * c + h];
        __syncthreads();
#pragma unroll
        for (int ct = 0; ct < VT; ++ct) acc[ct] = *(const f4 *)&back[(16 * wr + li) * (CP + 4) + 16 * ct + 4 * g];
        // an infinity or NaN in the record, as in the state kernel: the set's share again, from fp32 products
        static_assert(L::kBack <= L::kBuffers * WK * L::kPiece, "the rows' sketches are still there");
        if (any_odd(acc)) {
            clear(acc);
            const float *m_row = own + (16 * wr + li) * OP;
#pragma unroll 1
            for (int a = wk; a < 16 * RT; a += WK) {
                const int at = a >> 4, first = at * RT - at * (at - 1) / 2 - at;
#pragma unroll 1
                for (int b = 16 * at; b < 16 * RT; ++b) {
                    const int row = ((first + (b >> 4)) * 16 + (a & 15)) * 16 + (b & 15);
                    const float phi = m_row[a] * m_row[b];
#pragma unroll
                    for (int ct = 0; ct < VT; ++ct)
                        acc[ct] += record_columns(z, record_values(RT, VT), CP, row, 16 * ct + 4 * g) * phi;
                }
            }
        }
    }

    if (sh.pairs) {
        // exact weights for keys from the start of the row's block on
        const int bs = sh.local_exact ? i / sh.b * sh.b : 0x7fffffff;
        const int bs_wg = sh.local_exact ? i0 / sh.b * sh.b : 0x7fffffff;
        const int bs_wg_last = sh.local_exact ? i_last / sh.b * sh.b : 0x7fffffff;
        const int bs_w = sh.local_exact ? iw / sh.b * sh.b : 0x7fffffff;
        const int bs_w_last = sh.local_exact ? iw_last / sh.b * sh.b : 0x7fffffff;
        const int j_end = sh.noncausal ? sh.n : i_last + 1;
        const int j_max = sh.noncausal ? sh.n - 1 : i, all_see = sh.noncausal ? sh.n - 1 : iw;
        if (threadIdx.x < 2) odd_tile[threadIdx.x] = 0;
        int turn = 0;
        PartTile<DT, KT, KP, T, THREADS> kt;
        PartTile<MT, KT, MP, float, THREADS> mt;
        PartTile<VT, KT, VP, T, THREADS> vt;
        auto fetch = [&](int j0) {
            const int nv = min(KT, j_end - j0);
            if (sh.vec_v) vt.load(V + (urow + j0) * sh.dv, sh.dv, nv, sh.dv);
            if (j0 + KT > bs_wg && sh.vec_x) kt.load(K + (urow + j0) * sh.d, sh.d, nv, sh.d);
            if (j0 < bs_wg_last && sh.vec_m) mt.load(MK + (urow + j0) * sh.mcols, sh.mcols, nv, sh.mcols);
        };
        // this workgroup's share of the key tiles
        const int j_first = sh.noncausal ? 0 : s_begin;
        const int j_begin = SPLIT ? j_first + (int)blockIdx.z * share * KT : j_first;
        const int j_stop = SPLIT ? min(j_end, j_begin + share * KT) : j_end;
        fetch(j_begin);
        Parts<P> qf[DT / 2];
        Parts<3> mf[MT / 2];
        {
            OwnRow<DT / 2, T> q_row;
            OwnRow<MT / 2, float> m_row;
            if (sh.local_exact) q_row.load(Q + i_row * sh.d, sh.d, sh.vec_x, g);
            m_row.load(MQ + i_row * sh.mcols, sh.mcols, sh.vec_m, g);
            if (sh.local_exact) q_row.parts(qf, sh.d, g);
            m_row.parts(mf, sh.mcols, g);
        }
        for (int j0 = j_begin; j0 < j_stop; j0 += KT, turn ^= 1) {
            const int nv = min(KT, j_end - j0);
            const bool exact_g = j0 + KT > bs_wg, cross_g = j0 < bs_wg_last;
            __syncthreads();
            if (exact_g) {
                if (sh.vec_x) kt.template store<false>(ks, nv, sh.d);
                else stage_parts_scalar<DT, KT, KP, T, false, THREADS>(K + (urow + j0) * sh.d, sh.d, nv, sh.d, ks);
            }
            if (cross_g) {
                if (sh.vec_m) mt.template store<false>(ms, nv, sh.mcols);
                else stage_parts_scalar<MT, KT, MP, float, false, THREADS>(MK + (urow + j0) * sh.mcols, sh.mcols, nv, sh.mcols, ms);
            }
            bool odd;
            if (sh.vec_v) odd = vt.template store<true>(vs, nv, sh.dv);
            else odd = stage_parts_scalar<VT, KT, VP, T, true, THREADS>(V + (urow + j0) * sh.dv, sh.dv, nv, sh.dv, vs);
            if (odd) odd_tile[turn] = 1;
            __syncthreads();
            odd = odd_tile[turn] != 0;
            if (threadIdx.x == 0) odd_tile[turn ^ 1] = 0;   // (read for the last time before the barrier above)
            if (j0 + KT < j_stop) fetch(j0 + KT);
            f4 tile[VT];                                    // this tile's sums (two levels of summation)
            float dpart = 0.f;
            clear(tile);
            for (int sub = wk; sub < KT / 32; sub += WK) {
                const int js = j0 + 32 * sub;
                if (js >= j_end || (!sh.noncausal && js > iw_last)) break;
                const bool exact_w = js + 31 >= bs_w, cross_w = js < bs_w_last;
                f4 w[2], ss[2];
                if (exact_w) score_parts<2, DT / 2, P, P>(ks, KT * KP, KP, 32 * sub, qf, lane, w);
                if (cross_w) score_parts<2, MT / 2, 3, 3>(ms, KT * MP, MP, 32 * sub, mf, lane, ss);
                settle_parts();
                if (exact_w)
                    for (int q = 1; q < sh.p; q <<= 1) { w[0] *= w[0]; w[1] *= w[1]; }
                if (cross_w) {
#pragma unroll
                    for (int t = 0; t < 2; ++t) {
                        ss[t] *= ss[t];
                        if (exact_w) {
#pragma unroll
                            for (int k = 0; k < 4; ++k) w[t][k] = js + 16 * t + 4 * g + k >= bs ? w[t][k] : ss[t][k];
                        } else {
                            w[t] = ss[t];
                        }
                    }
                }
                if (js + 31 > all_see) {
#pragma unroll
                    for (int t = 0; t < 2; ++t)
#pragma unroll
                        for (int k = 0; k < 4; ++k) w[t][k] = js + 16 * t + 4 * g + k > j_max ? 0.f : w[t][k];
                }
                dpart += ((w[0][0] + w[0][1]) + (w[0][2] + w[0][3])) + ((w[1][0] + w[1][1]) + (w[1][2] + w[1][3]));
                const float flat_w[8] = {w[0][0], w[0][1], w[0][2], w[0][3], w[1][0], w[1][1], w[1][2], w[1][3]};
                if (odd) {
                    const int vis = j_max - js;             // tile rows 0 .. vis count
                    add_parts_odd<VT, P>(vs + 32 * sub * VP, KT * VP, VP, flat_w, tile, lane,
                                         vis < 0 ? 0u : vis >= 31 ? 0xffffffffu : (2u << vis) - 1u);
                } else {
                    Parts<3> wp;
                    split8(flat_w, wp);
                    add_parts<VT, P>(vs + 32 * sub * VP, KT * VP, VP, wp, tile, lane);
                }
                settle_parts();
            }
            den += dpart;
            add_settled(acc, tile);
        }
    }

    settle_parts();
    den = over_groups(den);
    if constexpr (WK > 1) {
        constexpr int PER = 4 * VT + 1;
        __syncthreads();
        if (wk > 0) {
            float *to = (float *)lds + (size_t)((wk - 1) * WR + wr) * PER * 64 + lane;
#pragma unroll
            for (int ct = 0; ct < VT; ++ct)
#pragma unroll
                for (int k = 0; k < 4; ++k) to[(4 * ct + k) * 64] = acc[ct][k];
            to[4 * VT * 64] = den;
        }
        __syncthreads();
        if (wk > 0) return;
        for (int o = 0; o < WK - 1; ++o) {
            const float *from = (const float *)lds + (size_t)(o * WR + wr) * PER * 64 + lane;
#pragma unroll
            for (int ct = 0; ct < VT; ++ct)
#pragma unroll
                for (int k = 0; k < 4; ++k) acc[ct][k] += from[(4 * ct + k) * 64];
            den += from[4 * VT * 64];
        }
    }
    if constexpr (SPLIT) {
        const int block = i0 / 16, slices = row_slices(block, sh.n, share, !sh.noncausal);
        if (slices > 1) {
            const int before = row_slots_before(block, sh.n, share, !sh.noncausal);
            const int unit_slots = row_slots_before((sh.n + 15) / 16, sh.n, share, !sh.noncausal);
            float *const to = part + ((size_t)u * unit_slots + before + blockIdx.z) * kSlotFloats;
#pragma unroll
            for (int ct = 0; ct < VT; ++ct) *(f4 *)&to[(ct * 64 + lane) * 4] = acc[ct];
            if (g == 0) to[1024 + li] = den;
            return;
        }
    }
    if (!there && !GRAD) return;
    const float D = 1.f + den;
    finish_row<VT, GRAD>(acc, D, there, li, g, urow + i, O, dO, GV, gden, sh);
}

template <int DT, int RT, int WR, int WK, bool GRAD, typename T>
__global__ __launch_bounds__((RowsLds<DT, RT, WR, WK, T>::kThreads), WK == 1 && DT == 4 ? (RT <= 2 ? 3 : 2) : 1) void f32_rows_kernel(
    const float *__restrict__ MQ, const float *__restrict__ MK, const T *__restrict__ Q, const T *__restrict__ K,
    const T *__restrict__ V, const float *__restrict__ Z, T *__restrict__ O, const T *__restrict__ dO,
    float *__restrict__ GV, float *__restrict__ gden, F32Shape sh)
{
    rows_workgroup<DT, RT, WR, WK, GRAD, false, T>(MQ, MK, Q, K, V, Z, O, dO, GV, gden, sh, 0, nullptr);
}

template <int RT, typename T>
__global__ __launch_bounds__((RowsLds<4, RT, 1, 4, T>::kThreads), 1) void f32_shared_rows_kernel(
    const float *__restrict__ MQ, const float *__restrict__ MK, const T *__restrict__ Q, const T *__restrict__ K,
    const T *__restrict__ V, T *__restrict__ O, F32Shape sh, int share, float *__restrict__ part)
{
    rows_workgroup<4, RT, 1, 4, false, true, T>(MQ, MK, Q, K, V, nullptr, O, nullptr, nullptr, nullptr, sh, share, part);
}

// Adds up what the slices of a block of 16 rows left, in their order, and finishes the rows: a wave a block.
template <typename T>
__global__ __launch_bounds__(64) void f32_rows_sum_kernel(const float *__restrict__ part, int share, T *__restrict__ O, F32Shape sh)
{
    constexpr int VT = 4;
    const int lane = threadIdx.x, li = lane & 15, g = lane >> 4, blocks = (sh.n + 15) / 16;
    const int u = blockIdx.x / blocks, block = blockIdx.x % blocks, i = 16 * block + li, causal = !sh.noncausal;
    const int slices = row_slices(block, sh.n, share, causal);
    if (slices < 2) return;
    const float *from = part + ((size_t)u * row_slots_before(blocks, sh.n, share, causal) +
                                row_slots_before(block, sh.n, share, causal)) * kSlotFloats;
    f4 acc[VT];
    float den = 0.f;
    clear(acc);
    for (int sl = 0; sl < slices; ++sl, from += kSlotFloats) {
#pragma unroll
        for (int ct = 0; ct < VT; ++ct) acc[ct] += *(const f4 *)&from[(ct * 64 + lane) * 4];
        den += from[1024 + li];
    }
    if (i < sh.n)
        finish_row<VT, false>(acc, 1.f + den, true, li, g, (size_t)u * sh.n + i, O, (const T *)nullptr, nullptr, nullptr, sh);
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
        const size_t rec = record_floats(RT, VT), values = record_values(RT, VT);
        const size_t pieces = (size_t)pb.units * (values / 8 + tile_pairs(RT) * 64);
        hipLaunchKernelGGL(f32_scan_kernel, dim3((unsigned)((pieces + kScanThreads - 1) / kScanThreads)),
                           dim3(kScanThreads), 0, s, Z, pb.units, values, rec, pl.spans, mode);
        PSF_LAUNCH_CHECK();
        return PSF_OK;
    });
}

// `few` of f32_deal for the rows
constexpr int rows_few(int rt, bool bf16) { return rt == 4 && !bf16 ? 50 : bf16 && rt <= 2 ? 110 : 70; }

template <typename T, bool GRAD>
psf_status rows_launch(const Problem &pb, const F32Plan &pl, const float *MQ, const float *MK, const void *Q,
                       const void *K, const void *V, const float *Z, void *O, const void *dO, float *GV, float *gden,
                       hipStream_t s, int share = 0, float *part = nullptr)
{
    F32Shape sh = f32_shape(pb, pl);
    sh.vec_x = pieces_ok<T>(pb.d, {Q, K});
    sh.vec_v = GRAD ? pieces_ok<T>(pb.dv, {V, dO}) : pieces_ok<T>(pb.dv, {V, O});
    sh.vec_m = pieces_ok<float>(pb.mcols, {MQ, MK});
    return with_tiles(pb, [&](auto dt, auto rt) -> psf_status {
        constexpr int DT = decltype(dt)::value, RT = decltype(rt)::value;
        auto go = [&](auto wr, auto wk) {
            constexpr int WR = decltype(wr)::value, WK = decltype(wk)::value;
            using L = RowsLds<DT, RT, WR, WK, T>;
            const int per_span = ((pl.span < pb.n ? pl.span : pb.n) + L::ROWS - 1) / L::ROWS;
            const FlatGrid grid = flat_grid(row_groups(pb.units, pl.spans, per_span));
            if constexpr (DT == 4 && WR == 1 && WK == 4 && !GRAD) {
                if (share > 0) {
                    const int blocks = (pb.n + 15) / 16;
                    const unsigned slices = (unsigned)row_slices(blocks - 1, pb.n, share, !pl.noncausal);
                    hipLaunchKernelGGL((f32_shared_rows_kernel<RT, T>), dim3(grid.x, grid.y, slices), dim3(L::kThreads), 0, s, MQ,
                                       MK, (const T *)Q, (const T *)K, (const T *)V, (T *)O, sh, share, part);
                    PSF_LAUNCH_CHECK();
                    hipLaunchKernelGGL((f32_rows_sum_kernel<T>), dim3((unsigned)(pb.units * blocks)), dim3(64), 0, s, part, share,
                                       (T *)O, sh);
                    PSF_LAUNCH_CHECK();
                    return PSF_OK;
                }
            }
            hipLaunchKernelGGL((f32_rows_kernel<DT, RT, WR, WK, GRAD, T>), dim3(grid.x, grid.y), dim3(L::kThreads), 0, s,
                               MQ, MK, (const T *)Q, (const T *)K, (const T *)V, Z, (T *)O, (const T *)dO, GV, gden, sh);
            PSF_LAUNCH_CHECK();
            return PSF_OK;
        };
        return f32_deal<DT, true, !(RT == 4 && sizeof(T) == 4)>(pb, pl, RT, rows_few(RT, sizeof(T) == 2), go);
    });
}

}  // namespace

// Rows so few that even 16 of them a workgroup leave CUs idle, in a call that keeps no states: the key tiles of the
// same rows are shared out (row_share); the slots for the sums take the room of the state records, which such a call
// does not use.  us a call: 1 unit of 1024 tokens, fp32 storage, r = 16 32.5 -> 22.4, r = 64 37.9 -> 22.2; no mask, r = 16
// 31.0 -> 23.2; 2 units, r = 32 32.6 -> 23.1.  (Room for one tile fewer a workgroup would take the first to 18.)
int f32_row_share(const Problem &pb, const F32Plan &pl, size_t part_floats)
{
    if (pl.states || pl.spans != 1) return 0;
    bool sixteen = false;
    with_tiles(pb, [&](auto dt, auto rt) -> psf_status {
        constexpr int DT = decltype(dt)::value, RT = decltype(rt)::value;
        return f32_deal<DT, true, true>(pb, pl, RT, rows_few(RT, pb.bf16), [&](auto wr, auto wk) -> psf_status {
            sixteen = DT == 4 && decltype(wr)::value == 1 && decltype(wk)::value == 4;
            return PSF_OK;
        });
    });
    return sixteen ? row_share(pb.units, pb.n, !pl.noncausal, pb.bf16 && pb.mcols <= 32, part_floats / kSlotFloats) : 0;
}

bool f32_supported(const Problem &pb)
{
    return !pb.exact_feat && pb.d <= 128 && pb.dv <= 128 && pb.mcols <= 128;
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

// Where the states lie.  Costs in seconds of the whole chip, relative to each other (wide tiles in brackets):
// forming and applying states at 90 (80) TFLOP/s, pairs at 75 (60), with the rows that a span is padded to 64 with;
// state traffic at 4 TB/s; 7 us for two further launches, 14 for the four of a backward call; and the longest walk of a workgroup, 1 (1.5)
// us a block of 64 keys where r + dv = 128, which is what a call of few rows takes.
// Measured with every span forced (blocks a span: us of a forward call, of a forward and a backward call;
// * the plan's own choice; bf16 storage where nothing is said):
//   36 units x 3000, r 32, b 200   1: 226, 1056    2: 199, 936*    4: 188*, 933   8: 222, 1171   all 15: 185, 1163
//   24 x 1950, r 32, b 150         1: 128, 535     2: 105, 473     4: 113, 524    8: 116, 543    all 13: 82*, 441*
//   12 x 8192, r 32, b 64          1: 435, 1542    2: 232, 994     4: 188*, 861*  8: 188, 872    all 128: 412
//   24 x 8000, r 64, b 250         1: 1334, 4939   2: 1158, 4546   4: 1065*, 4434* 8: 1102, 4885 all 32: 1139, 6352
//   48 x 8192, r 16, b 256, fp32   1: 585*, 2383*  2: 616, 2629    4: 758, 3344   8: 1077, 4868
//   3 x 2048, r 16, b 256, fp32    1: 44*, 179*    2: 59, 229      4: 80, 306     all 8: 57, 258
//   36 x 3000, r 64, b 200         1: 869, 3229    2: 686, 2694    4: 542, 2250   8: 511, 2224   all 15: 272*, 1519*
// Over 230 such calls (r 16 to 128, d 64 and 128, 1 to 48 units, both storage types) the choice is within 2 % of the best
// one in the mean; it misses most where few rows make a call short (1 unit x 1024 to 3 x 2048: up to a third).
// z_floats: room for state records.
static F32Plan f32_plan(const Problem &pb, size_t z_floats, bool noncausal, bool grad)
{
    const bool wide = pb.d > 64 || pb.dv > 64 || pb.mcols > 64;
    int rt = 0, vt = wide ? 8 : 4;
    with_tiles(pb, [&](auto, auto r) -> psf_status { rt = decltype(r)::value; return PSF_OK; });
    const double tokens = (double)pb.units * pb.n, bw = 4e12;
    const double rate = wide ? 80e12 : 90e12, pair_rate = wide ? 60e12 : 75e12;
    const size_t rec = record_floats(rt, vt);
    const double state_flops = tile_pairs(rt) * 256.0 * 16 * vt * 2 * (grad ? 6 : 2);
    const double pair_flops = 2.0 * 16 * (grad ? 5 * rt + 4 * vt : rt + vt);
    const double traffic = (grad ? 9 : 4) * (rt * (rt + 1) / 2) * 256.0 * (16 * vt + 1) * 4;    // bytes a record
    const double step = (wide ? 1.5e-6 : 1e-6) * (rt + vt) / 8 * (grad ? 3 : 1);                // of the longest walk
    F32Plan best = {};
    if (noncausal) {
        const double direct = tokens * pb.n * pair_flops / pair_rate + step * ((pb.n + 63) / 64);
        const double with_state = tokens * state_flops / rate + 12e-6 + step * state_walk(rt);
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
        const int spans = (pb.t + s - 1) / s, span = (long long)s * pb.b < pb.n ? s * pb.b : pb.n;
        if (spans == 1 || (size_t)spans * pb.units * rec <= z_floats) {
            const double blocks = (span + 63) / 64, padded = blocks * 64 / span;
            double cost = padded * tokens * span / 2 * pair_flops / pair_rate + step * blocks;
            if (spans > 1)
                cost += (1 + padded) / 2 * tokens * (1.0 - 1.0 / spans) * state_flops / rate +
                        (double)pb.units * spans * traffic / bw + (grad ? 14e-6 : 7e-6) + step * state_walk(rt);
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

// Records are padded to tiles (16 sketch indices, 64 or 128 value columns) and hold three bf16 parts a value; the
// room of the vector kernels, t F (dv + 1) floats a unit, is neither.  Few or small blocks find no room for any record
// (pairs alone cost time quadratic in n), r = 16 and 32 none for one a block.  Where that room makes the plan
// dearer than the best one the workspace grows to the best plan's records (at most kMostRoom, 1.5 GiB, and not past
// the library's static scratch where the call fitted it).  If that does not bring the cost
// within four times the best one, the vector kernels take the call, whose time is linear.  Measured, without a
// mask, r = 8, d = 128, dv = 16, two blocks (us; pairs, best plan, vector kernels): 12 units x 4096 1274, 272, 714;
// 12 x 16384 20429, 1050, 2487; 96 x 16384 165250, 7607, 10294.  A state for two blocks instead of each, r = 16, b =
// 256, 48 x 8192: 616 against 585 us, with the backward pass 2629 against 2383; below 4 % or 1.5 us of modelled
// loss nothing is to be gained.
F32Choice f32_choose(const Problem &pb, size_t fixed_bytes, bool noncausal, bool grad)
{
    constexpr size_t kMostRoom = ((size_t)3 << 29) / sizeof(float);
    F32Choice c = {};
    c.z_floats = (size_t)pb.units * pb.t * (size_t)pb.F * (pb.dv + 1);
    if (!f32_supported(pb)) return c;
    c.use = true;
    c.plan = f32_plan(pb, c.z_floats, noncausal, grad);
    const F32Plan most = f32_plan(pb, SIZE_MAX, noncausal, grad);
    const double best = most.cost;
    if (c.plan.cost <= 1.04 * best + 1.5e-6 && !(noncausal && most.states && c.plan.spans < most.spans)) return c;
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
                    const void *K, const void *V, const float *Z, void *O, hipStream_t s, int share, float *part)
{
    return pb.bf16 ? rows_launch<bf16_t, false>(pb, pl, MQ, MK, Q, K, V, Z, O, nullptr, nullptr, nullptr, s, share, part)
                   : rows_launch<float, false>(pb, pl, MQ, MK, Q, K, V, Z, O, nullptr, nullptr, nullptr, s, share, part);
}

psf_status f32_rows_grad(const Problem &pb, const F32Plan &pl, const float *MQ, const float *MK, const void *Q,
                         const void *K, const void *V, const float *Z, const void *dO, float *GV, float *gden,
                         hipStream_t s)
{
    return pb.bf16 ? rows_launch<bf16_t, true>(pb, pl, MQ, MK, Q, K, V, Z, nullptr, dO, GV, gden, s)
                   : rows_launch<float, true>(pb, pl, MQ, MK, Q, K, V, Z, nullptr, dO, GV, gden, s);
}

}  // namespace psf
