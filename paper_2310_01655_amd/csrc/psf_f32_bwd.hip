// fp32 matrix-core kernels of the general backward pass (sketch features, d, dv and sketch
// columns <= 128).  The gradient itself is stated at the top of psf_backward.hip; the operand
// conventions in psf_f32_tiles.h; spans, pairs and states as in psf_f32_fwd.hip.
//
// One kernel serves both sides: a wave owns 16 queries and walks the keys of its span up to them
// (dm(Q), dQ), or owns 16 keys and walks the queries from them on (dm(K), dK, dV).  Per group of
// 16 streamed rows: dw = <G_i, C_j>, the scores, then the products of the pair gradients with the
// streamed rows; pair weights and gradients never leave the registers.
#include "psf_f32_tiles.h"
#include "psf_f32.h"

namespace psf {
namespace {

template <int DT, int RT, int VT, int WR, bool KSIDE, typename T>
__global__ __launch_bounds__(kF32Threads, DT == 4 ? 2 : 1) void f32_bwd_kernel(
    const float *__restrict__ Mown, const float *__restrict__ Mstr, const T *__restrict__ Xown,
    const T *__restrict__ Xstr, const T *__restrict__ V, const float *__restrict__ GV, const float *__restrict__ gden,
    const float *__restrict__ Z, float *__restrict__ dM, float *__restrict__ dX, T *__restrict__ dV, F32Shape sh)
{
    constexpr int KT = f32_tile_rows(DT, WR), KP = pitch_of<DT>(), MP = pitch_of<RT>(), VP = pitch_of<VT>();
    constexpr int ROWS = 16 * WR, ZA = KT / 16, ZW = WR == 1 ? 1 : ZA;
    constexpr int kTileFloats = KT * (KP + VP) + (KT > ROWS ? KT : ROWS) * MP;
    static_assert(WR == 4 || KT == 64, "the waves of a 16-row workgroup take one group of streamed rows each");
    static_assert(DT == VT, "the state is staged through the buffers of the streamed rows in turn");
    __shared__ __attribute__((aligned(16))) float lds[kTileFloats + KT];
    __shared__ __attribute__((aligned(16))) float sden[2][16 * ZA];   // denominator column of a state piece
    float *xs = lds, *cs = xs + KT * KP, *ms = cs + KT * VP, *gs = lds + kTileFloats;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, li = lane & 15, g = lane >> 4;
    const int per_span = (min(sh.span, sh.n) + ROWS - 1) / ROWS;
    const unsigned flat = blockIdx.y * gridDim.x + blockIdx.x;
    const int u = flat % sh.units, x = flat / sh.units;     // the longest walks of all units first
    if (x >= per_span * sh.spans) return;
    const int span = KSIDE ? x % sh.spans : sh.spans - 1 - x % sh.spans;
    const int s_begin = span * sh.span, s_end = min(sh.n, s_begin + sh.span);
    const int o0 = s_begin + (KSIDE ? x / sh.spans : per_span - 1 - x / sh.spans) * ROWS;
    if (o0 >= s_end) return;
    const int ow = o0 + (WR == 4 ? 16 * wave : 0), o = ow + li;
    const int o_last = min(o0 + ROWS, s_end) - 1, ow_last = min(ow + 15, s_end - 1);
    const bool there = o < s_end;
    const size_t urow = (size_t)u * sh.n;
    float xf[4 * DT], mf[4 * RT], cf[4 * VT];
    if (sh.local_exact) load_frags<DT>(Xown + (urow + o) * sh.d, sh.d, there, sh.vec_x, g, xf);
    load_frags<RT>(Mown + (urow + o) * sh.mcols, sh.mcols, there, sh.vec_m, g, mf);
    if constexpr (KSIDE) load_frags<VT>(V + (urow + o) * sh.dv, sh.dv, there, sh.vec_v, g, cf);
    else load_frags<VT>(GV + (urow + o) * sh.dv, sh.dv, there, sh.vec_g, g, cf);
    const float own_den = KSIDE ? 1.f : there ? gden[urow + o] : 0.f;
    f4 ax[DT], am[RT], ac[VT];
    clear(ax);
    clear(am);
    clear(ac);

    // streamed rows of the own row's block take the exact weight: query side those from the start
    // of its block on, key side those before its end.  edge: that row, per lane, wave and workgroup.
    const int none = KSIDE ? -1 : 0x7fffffff;
    auto edge_of = [&](int row) { return sh.local_exact ? (row / sh.b + (KSIDE ? 1 : 0)) * sh.b : none; };
    const int edge = edge_of(o), edge_w = edge_of(ow), edge_w_last = edge_of(ow_last), edge_g = edge_of(o0),
              edge_g_last = edge_of(o_last);
    const int x_end = KSIDE ? s_end : o_last + 1;
    for (int x0 = KSIDE ? o0 : s_begin; x0 < x_end; x0 += KT) {
        const int nv = min(KT, x_end - x0);
        const size_t row = urow + x0;
        const bool exact_g = KSIDE ? x0 < edge_g_last : x0 + KT > edge_g;
        const bool cross_g = KSIDE ? x0 + KT > edge_g : x0 < edge_g_last;
        Tile<DT, KT, T> xt;
        Tile<RT, KT, float> mt;
        typedef std::conditional_t<KSIDE, float, T> C;
        Tile<VT, KT, C> ct;
        const T *xp = Xstr + row * sh.d;
        const float *mp = Mstr + row * sh.mcols;
        const C *cp;
        if constexpr (KSIDE) cp = GV + row * sh.dv;
        else cp = V + row * sh.dv;
        const int vec_c = KSIDE ? sh.vec_g : sh.vec_v;
        if (vec_c) ct.load(cp, sh.dv, nv, sh.dv);
        if (exact_g && sh.vec_x) xt.load(xp, sh.d, nv, sh.d);
        if (cross_g && sh.vec_m) mt.load(mp, sh.mcols, nv, sh.mcols);
        __syncthreads();
        if (exact_g) {
            if (sh.vec_x) xt.store(xs, nv, sh.d);
            else stage_scalar<DT, KT>(xp, sh.d, nv, sh.d, xs);
        }
        if (cross_g) {
            if (sh.vec_m) mt.store(ms, nv, sh.mcols);
            else stage_scalar<RT, KT>(mp, sh.mcols, nv, sh.mcols, ms);
        }
        if (vec_c) ct.store(cs, nv, sh.dv);
        else stage_scalar<VT, KT>(cp, sh.dv, nv, sh.dv, cs);
        if (KSIDE && threadIdx.x < KT) gs[threadIdx.x] = (int)threadIdx.x < nv ? gden[row + threadIdx.x] : 0.f;
        __syncthreads();
        f4 px[DT], pm[RT], pc[VT];                          // this tile's sums: two levels of summation,
        clear(px);                                          // as long chains of one sign or both lose digits
        clear(pm);
        clear(pc);
        for (int sub = (WR == 4 ? 0 : wave); sub < KT / 16; sub += (WR == 4 ? 1 : 4)) {
            const int r0 = 16 * sub, xw = x0 + r0;
            if (xw >= x_end || (!KSIDE && xw > ow_last)) break;
            if (KSIDE && xw + 15 < ow) continue;
            const bool exact_w = KSIDE ? xw < edge_w_last : xw + 15 >= edge_w;
            const bool cross_w = KSIDE ? xw + 15 >= edge_w : xw < edge_w_last;
            f4 dw = score_rows<VT>(cs, r0, cf, lane);
            if constexpr (KSIDE) dw += *(const f4 *)&gs[r0 + 4 * g];
            else dw += f4{own_den, own_den, own_den, own_den};
            float we[4], wx[4], wm[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) we[k] = wx[k] = wm[k] = 0.f;
            if (exact_w) {
                const f4 se = score_rows<DT>(xs, r0, xf, lane);
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int at = xw + 4 * g + k;
                    if (KSIDE ? at >= o && at < edge : at <= o && at >= edge) {
                        float pw, pm1;
                        powers(se[k], sh.p, pw, pm1);
                        we[k] = pw;
                        wx[k] = (float)sh.p * pm1 * dw[k];
                    }
                }
            }
            if (cross_w) {
                const f4 ss = score_rows<RT>(ms, r0, mf, lane);
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int at = xw + 4 * g + k;
                    if (KSIDE ? at >= o && at >= edge : at <= o && at < edge) {
                        we[k] = ss[k] * ss[k];
                        wm[k] = 2.f * ss[k] * dw[k];
                    }
                }
            }
            const int rel = o - xw;                         // the own row's place among the streamed ones
            if (KSIDE ? xw < ow + 15 : xw + 15 > ow) {      // some of the 16 x 16 pairs are masked
                const unsigned seen = KSIDE ? (rel > 15 ? 0u : 0xffffu & (0xffffu << max(0, rel)))
                                            : (rel < 0 ? 0u : 0xffffu >> max(0, 15 - rel));
                if (exact_w) add_rows<DT, true>(xs, r0, wx, px, lane, seen);
                if (cross_w) add_rows<RT, true>(ms, r0, wm, pm, lane, seen);
                if (KSIDE) add_rows<VT, true>(cs, r0, we, pc, lane, seen);
            } else {
                if (exact_w) add_rows<DT, false>(xs, r0, wx, px, lane, 0u);
                if (cross_w) add_rows<RT, false>(ms, r0, wm, pm, lane, 0u);
                if (KSIDE) add_rows<VT, false>(cs, r0, we, pc, lane, 0u);
            }
        }
        add_to(ax, px);
        add_to(am, pm);
        if constexpr (KSIDE) add_to(ac, pc);
    }

    // Spans before (query side) or after (key side): with the record R of the state,
    // U[b'] = sum_c R[a][b'][c] C[c] (+ the denominator column), dm[a] += 2 sum_b' U[b'] m[b'],
    // which for the doubled tiles off the diagonal is dm[a] += U m[b'] and, for their mirror,
    // dm[b'] += U m[a]; key side also dV += R^T phi'.
    if (sh.states && (KSIDE ? span < sh.spans - 1 : span > 0)) {
        const float *z = Z + ((size_t)u * sh.spans + span) * record_floats(RT, VT);
        const float *zs = z + (size_t)tile_pairs(RT) * 256 * 16 * VT;
        constexpr int PIECE = KT * 16 * VT, NP = PIECE / 4 / kF32Threads;
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
        put(xs, 0);
        float *own = ms + ((WR == 4 ? 16 * wave : 0) + li) * MP;
#pragma unroll
        for (int q = 0; q < RT; ++q)
            *(f4 *)&own[16 * q + 4 * g] = f4{mf[4 * q], mf[4 * q + 1], mf[4 * q + 2], mf[4 * q + 3]};
        int at = 0, q = 0;
        f4 mq = *(const f4 *)&own[4 * g], ma_sum = {0.f, 0.f, 0.f, 0.f}, mb_sum = ma_sum;
        auto flush = [&](int tile, f4 v) {                  // registers cannot be indexed
#pragma unroll
            for (int k = 0; k < RT; ++k)
                if (k == tile) am[k] += v;
        };
        for (int piece = 0; piece <= LAST; ++piece) {
            const int ch = piece % CH;
            if (piece && ch == 0) {                         // the next pair of index tiles
                flush(at, ma_sum);
                flush(q, mb_sum);
                ma_sum = mb_sum = f4{0.f, 0.f, 0.f, 0.f};
                if (++q == RT) q = ++at;
                mq = *(const f4 *)&own[16 * q + 4 * g];
            }
            __syncthreads();
            const float *zt = piece & 1 ? cs : xs;
            if (piece < LAST) fetch(piece + 1);
            f4 U[ZW], pc[VT];
            clear(pc);
#pragma unroll
            for (int k = 0; k < ZW; ++k)
                U[k] = *(const f4 *)&sden[piece & 1][(WR == 1 ? wave : k) * 16 + 4 * g] * own_den;
#pragma unroll
            for (int qq = 0; qq < VT; ++qq)
#pragma unroll
                for (int k = 0; k < ZW; ++k) {
                    const f4 zr = *(const f4 *)&zt[((WR == 1 ? wave : k) * 16 + li) * VP + 16 * qq + 4 * g];
#pragma unroll
                    for (int s = 0; s < 4; ++s) U[k] = mm(zr[s], cf[4 * qq + s], U[k]);
                }
#pragma unroll
            for (int k = 0; k < ZW; ++k) {
                const int aa = WR == 1 ? wave : k, a16 = ZA * ch + aa;
                const float ma = own[16 * at + a16];
                float t = 0.f;
#pragma unroll
                for (int s = 0; s < 4; ++s) t += U[k][s] * mq[s];
                t = over_groups(t);
                t = at == q ? 2.f * t : t;
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    const float mirror = U[k][s] * ma;
                    mb_sum[s] += at == q ? 0.f : mirror;
                    ma_sum[s] += a16 == 4 * g + s ? t : 0.f;
                }
                if constexpr (KSIDE) {
#pragma unroll
                    for (int s = 0; s < 4; ++s) {
                        const float phi = ma * mq[s];
#pragma unroll
                        for (int ct = 0; ct < VT; ++ct)
                            pc[ct] = mm(zt[(aa * 16 + 4 * g + s) * VP + 16 * ct + li], phi, pc[ct]);
                    }
                }
            }
            if constexpr (KSIDE) add_to(ac, pc);
            if (piece < LAST) put(piece & 1 ? xs : cs, ~piece & 1);
        }
        flush(at, ma_sum);
        flush(q, mb_sum);
    }

    if constexpr (WR == 1) {
        constexpr int PER = 4 * (DT + RT + (KSIDE ? VT : 0));
        static_assert(3 * PER * 64 <= kTileFloats, "sums of three waves");
        __syncthreads();
        if (wave > 0) {
            float *to = lds + (size_t)(wave - 1) * PER * 64 + lane;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
#pragma unroll
                for (int t = 0; t < DT; ++t) to[(4 * t + k) * 64] = ax[t][k];
#pragma unroll
                for (int t = 0; t < RT; ++t) to[(4 * (DT + t) + k) * 64] = am[t][k];
                if constexpr (KSIDE)
#pragma unroll
                    for (int t = 0; t < VT; ++t) to[(4 * (DT + RT + t) + k) * 64] = ac[t][k];
            }
        }
        __syncthreads();
        if (wave > 0) return;
        for (int w = 0; w < 3; ++w) {
            const float *from = lds + (size_t)w * PER * 64 + lane;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
#pragma unroll
                for (int t = 0; t < DT; ++t) ax[t][k] += from[(4 * t + k) * 64];
#pragma unroll
                for (int t = 0; t < RT; ++t) am[t][k] += from[(4 * (DT + t) + k) * 64];
                if constexpr (KSIDE)
#pragma unroll
                    for (int t = 0; t < VT; ++t) ac[t][k] += from[(4 * (DT + RT + t) + k) * 64];
            }
        }
    }
    if (!there) return;
    const int vec_d = sh.d % 4 == 0;                        // dX lies in the workspace
#pragma unroll
    for (int t = 0; t < DT; ++t) store_piece(dX + (urow + o) * sh.d, 16 * t + 4 * g, sh.d, vec_d, ax[t]);
#pragma unroll
    for (int t = 0; t < RT; ++t) store_piece(dM + (urow + o) * sh.mcols, 16 * t + 4 * g, sh.mcols, sh.vec_m, am[t]);
    if constexpr (KSIDE)
#pragma unroll
        for (int t = 0; t < VT; ++t) store_piece(dV + (urow + o) * sh.dv, 16 * t + 4 * g, sh.dv, sh.vec_v, ac[t]);
}

// ---- Algorithm 1's reverse -------------------------------------------------------------------
// A wave takes 16 H rows.  The two projections U, W of every node are formed again level by level
// and kept in LDS; from the root down they become dU = sqrt(1/r) dM * W, dW = sqrt(1/r) dM * U, and
// dM(child 1) = dU G1^T, dM(child 2) = dW G2^T; dX = direct + the same for the first level.
// LDS: x, then U, W of every node, then m of every node but the root.
__host__ __device__ inline int bwd_sketch_nodes(int p) { return p == 4 ? 1 : p == 8 ? 3 : 7; }
size_t bwd_sketch_lds(int d, int r, int p, int h)
{
    const int nodes = bwd_sketch_nodes(p);
    return (size_t)16 * h * ((tiles16(d) * 16 + 4) + (3 * nodes - 1) * (tiles16(r) * 16 + 4)) * sizeof(float);
}

template <int H, typename T>
__global__ __launch_bounds__(64) void f32_bwd_sketch_kernel(const T *__restrict__ X1, const T *__restrict__ X2,
                                                            const T *__restrict__ G, const float *__restrict__ dM1,
                                                            const float *__restrict__ dM2,
                                                            const float *__restrict__ dir1,
                                                            const float *__restrict__ dir2, T *__restrict__ dX1,
                                                            T *__restrict__ dX2, int n, int d, int r, int p, int heads,
                                                            int per_head, size_t g_len, int vec_x, int vec_g)
{
    extern __shared__ __attribute__((aligned(16))) float smem[];
    constexpr int ROWS = 16 * H;
    const int lane = threadIdx.x, li = lane & 15, g = lane >> 4, u = blockIdx.y, i0 = blockIdx.x * ROWS;
    const int dp = (d + 15) / 16 * 16, rp = (r + 15) / 16 * 16, xp = dp + 4, mp = rp + 4;
    const size_t row0 = (size_t)u * n + i0;
    const T *X = (blockIdx.z ? X2 : X1) + row0 * d;
    const float *dM = (blockIdx.z ? dM2 : dM1) + row0 * (p == 2 ? d : r), *dir = (blockIdx.z ? dir2 : dir1) + row0 * d;
    T *dX = (blockIdx.z ? dX2 : dX1) + row0 * d;
    const int nv = min(ROWS, n - i0), quads = dp / 4, vec_m = r % 4 == 0, vec_d = d % 4 == 0;
    for (int idx = lane; idx < ROWS * quads; idx += 64) {
        const int row = idx / quads, c = 4 * (idx % quads);
        if (p == 2) {                                       // m(x) = x
            if (row < nv)
                store_piece(dX + (size_t)row * d, c, d, vec_x,
                            row_piece(dir + (size_t)row * d, c, d, vec_d) + row_piece(dM + (size_t)row * d, c, d, vec_d));
            continue;
        }
        f4 v = {0.f, 0.f, 0.f, 0.f};
        if (row < nv) v = row_piece(X + (size_t)row * d, c, d, vec_x);
        *(f4 *)&smem[row * xp + c] = v;
    }
    if (p == 2) return;
    __syncthreads();
    const T *gs = G + (per_head ? (size_t)(u % heads) * g_len : 0), *gi = gs + (size_t)(p / 2) * d * r;
    const float sc = sqrtf(1.0f / (float)r);
    const int total = bwd_sketch_nodes(p);
    const size_t arr = (size_t)ROWS * mp;                   // floats of an array of row vectors
    float *UW = smem + ROWS * xp, *Mn = UW + 2 * total * arr;
    int count = p / 4, first = 0, from = -1;
    for (;;) {
        for (int k = 0; k < count; ++k) {
            const int in = from < 0 ? d : r, pitch = from < 0 ? xp : mp;
            const T *ga = from < 0 ? gs + (size_t)(2 * k) * d * r : gi + (size_t)(2 * k) * r * r;
            const float *xa = from < 0 ? smem : Mn + (from + 2 * k) * arr, *xb = from < 0 ? smem : xa + arr;
            float *U = UW + 2 * (first + k) * arr, *W = U + arr;
            for (int c0 = 0; c0 < rp; c0 += 16) {
                f4 a[H], w[H];
                project<H>(ga, in, r, c0, xa, pitch, a, lane);
                project<H>(ga + (size_t)in * r, in, r, c0, xb, pitch, w, lane);
#pragma unroll
                for (int h = 0; h < H; ++h) {
                    const int row = 16 * h + li, at = row * mp + c0 + 4 * g;
                    if (count == 1) {                       // the root: its gradient is given
                        f4 dm = {0.f, 0.f, 0.f, 0.f};
                        if (row < nv) dm = row_piece(dM + (size_t)row * r, c0 + 4 * g, r, vec_m) * sc;
                        *(f4 *)&U[at] = dm * w[h];
                        *(f4 *)&W[at] = dm * a[h];
                    } else {
                        *(f4 *)&U[at] = a[h];
                        *(f4 *)&W[at] = w[h];
                        *(f4 *)&Mn[(first + k) * arr + at] = a[h] * w[h] * sc;
                    }
                }
            }
        }
        __syncthreads();
        if (count == 1) break;
        if (from >= 0) gi += (size_t)(2 * count) * r * r;
        from = first;
        first += count;
        count /= 2;
    }
    while (first > 0) {                                     // nodes of a level -> their children
        const int below = first - 2 * count;
        for (int k = 0; k < 2 * count; ++k) {
            const T *ga = gi + (size_t)k * r * r;
            const float *du = UW + (2 * first + k) * arr;   // dU of node k / 2, or its dW
            float *U = UW + 2 * (below + k) * arr, *W = U + arr;
            for (int e0 = 0; e0 < rp; e0 += 16) {
                f4 dm[H];
#pragma unroll
                for (int h = 0; h < H; ++h) dm[h] = f4{0.f, 0.f, 0.f, 0.f};
                back_project<H>(ga, r, r, e0, du, mp, vec_g, dm, lane);
#pragma unroll
                for (int h = 0; h < H; ++h) {
                    const int at = (16 * h + li) * mp + e0 + 4 * g;
                    const f4 a = *(const f4 *)&U[at], w = *(const f4 *)&W[at], gm = dm[h] * sc;
                    *(f4 *)&U[at] = gm * w;
                    *(f4 *)&W[at] = gm * a;
                }
            }
        }
        __syncthreads();
        count *= 2;
        first = below;
        gi -= (size_t)(2 * count) * r * r;                  // (not read at the first level)
    }
    for (int e0 = 0; e0 < dp; e0 += 16) {
        f4 acc[H];
#pragma unroll
        for (int h = 0; h < H; ++h) {
            acc[h] = f4{0.f, 0.f, 0.f, 0.f};
            if (16 * h + li < nv) acc[h] = row_piece(dir + (size_t)(16 * h + li) * d, e0 + 4 * g, d, vec_d);
        }
        for (int k = 0; k < 2 * count; ++k)
            back_project<H>(gs + (size_t)k * d * r, d, r, e0, UW + k * arr, mp, vec_g, acc, lane);
#pragma unroll
        for (int h = 0; h < H; ++h)
            if (16 * h + li < nv) store_piece(dX + (size_t)(16 * h + li) * d, e0 + 4 * g, d, vec_x, acc[h]);
    }
}

template <typename T, bool KSIDE>
psf_status side_launch(const Problem &pb, const F32Plan &pl, const float *MQ, const float *MK, const void *Q,
                       const void *K, const void *V, const float *GV, const float *gden, const float *Z, float *dM,
                       float *dX, void *dV, hipStream_t s)
{
    F32Shape sh = f32_shape(pb, pl);
    sh.vec_x = pieces_ok<T>(pb.d, {Q, K});
    sh.vec_v = KSIDE ? pieces_ok<T>(pb.dv, {V, dV}) : pieces_ok<T>(pb.dv, {V});
    sh.vec_m = pieces_ok<float>(pb.mcols, {MQ, MK, dM});
    sh.vec_g = pieces_ok<float>(pb.dv, {GV});
    return with_tiles(pb, [&](auto dt, auto rt) -> psf_status {
        constexpr int DT = decltype(dt)::value, RT = decltype(rt)::value;
        auto go = [&](auto kernel, int rows) {
            const int per_span = ((pl.span < pb.n ? pl.span : pb.n) + rows - 1) / rows;
            const FlatGrid grid = flat_grid((unsigned long long)per_span * pl.spans * pb.units);
            hipLaunchKernelGGL(kernel, dim3(grid.x, grid.y), dim3(kF32Threads), 0,
                               s, KSIDE ? MK : MQ, KSIDE ? MQ : MK, (const T *)(KSIDE ? K : Q),
                               (const T *)(KSIDE ? Q : K), (const T *)V, GV, gden, Z, dM, dX, (T *)dV, sh);
        };
        if constexpr (DT == 4) {
            if (f32_split_rows(pb)) {
                go(f32_bwd_kernel<DT, RT, DT, 1, KSIDE, T>, 16);
                PSF_LAUNCH_CHECK();
                return PSF_OK;
            }
        }
        go(f32_bwd_kernel<DT, RT, DT, 4, KSIDE, T>, 64);
        PSF_LAUNCH_CHECK();
        return PSF_OK;
    });
}

template <typename T, int H>
psf_status sketch_bwd_launch(const Problem &pb, const void *X1, const void *X2, const void *G, const float *dM1,
                             const float *dM2, const float *dir1, const float *dir2, void *dX1, void *dX2,
                             hipStream_t s)
{
    const size_t lds = pb.p == 2 ? 0 : bwd_sketch_lds(pb.d, pb.r, pb.p, H);
    if (lds > (64u << 10))
        PSF_HIP_TRY(hipFuncSetAttribute((const void *)f32_bwd_sketch_kernel<H, T>,
                                        hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    const int vx = pieces_ok<T>(pb.d, {X1, X2 ? X2 : X1, dX1, dX2 ? dX2 : dX1}), vg = pieces_ok<T>(pb.r, {G}) && pb.d % 4 == 0;
    const dim3 grid((unsigned)((pb.n + 16 * H - 1) / (16 * H)), (unsigned)pb.units, X2 ? 2 : 1);
    hipLaunchKernelGGL((f32_bwd_sketch_kernel<H, T>), grid, dim3(64), lds, s, (const T *)X1, (const T *)X2,
                       (const T *)G, dM1, dM2, dir1, dir2, (T *)dX1, (T *)dX2, pb.n, pb.d, pb.r, pb.p, pb.heads,
                       pb.per_head ? 1 : 0, pb.g_len, vx, vg);
    PSF_LAUNCH_CHECK();
    return PSF_OK;
}

}  // namespace

psf_status f32_bwd_side(const Problem &pb, const F32Plan &pl, bool key_side, const float *MQ, const float *MK,
                        const void *Q, const void *K, const void *V, const float *GV, const float *gden,
                        const float *Z, float *dM, float *dX, void *dV, hipStream_t s)
{
    if (pb.bf16)
        return key_side ? side_launch<bf16_t, true>(pb, pl, MQ, MK, Q, K, V, GV, gden, Z, dM, dX, dV, s)
                        : side_launch<bf16_t, false>(pb, pl, MQ, MK, Q, K, V, GV, gden, Z, dM, dX, dV, s);
    return key_side ? side_launch<float, true>(pb, pl, MQ, MK, Q, K, V, GV, gden, Z, dM, dX, dV, s)
                    : side_launch<float, false>(pb, pl, MQ, MK, Q, K, V, GV, gden, Z, dM, dX, dV, s);
}

// the arrays of all nodes of 16 rows within the 160 KB of a CU (p = 16 stays below r = 120)
bool f32_sketch_bwd_supported(const Problem &pb)
{
    return !pb.learned && !pb.exact_feat && pb.d <= 128 && pb.mcols <= 128 &&
           (pb.p == 2 || bwd_sketch_lds(pb.d, pb.r, pb.p, 1) <= (160u << 10));
}

psf_status f32_sketch_bwd_pair(const Problem &pb, const void *X1, const void *X2, const void *G, const float *dM1,
                               const float *dM2, const float *direct1, const float *direct2, void *dX1, void *dX2,
                               hipStream_t s)
{
    if (pb.p <= 4)
        return pb.bf16 ? sketch_bwd_launch<bf16_t, 2>(pb, X1, X2, G, dM1, dM2, direct1, direct2, dX1, dX2, s)
                       : sketch_bwd_launch<float, 2>(pb, X1, X2, G, dM1, dM2, direct1, direct2, dX1, dX2, s);
    return pb.bf16 ? sketch_bwd_launch<bf16_t, 1>(pb, X1, X2, G, dM1, dM2, direct1, direct2, dX1, dX2, s)
                   : sketch_bwd_launch<float, 1>(pb, X1, X2, G, dM1, dM2, direct1, direct2, dX1, dX2, s);
}

}  // namespace psf
