// fp32 matrix-core kernels of the general backward pass (sketch features, d, dv and sketch
// columns <= 128).  The gradient itself is stated at the top of psf_backward.hip; layouts and
// products in psf_f32_tiles.h and psf_parts.h; spans, pairs and states as in psf_f32_fwd.hip.
//
// One kernel serves both sides: a wave owns 16 queries and walks the keys of its span up to them
// (dm(Q), dQ), or owns 16 keys and walks the queries from them on (dm(K), dK, dV).  Per group of
// 32 streamed rows: dw = <G_i, C_j>, the scores, then the products of the pair gradients with the
// streamed rows; pair weights and gradients never leave the registers.
//
// Bound by vector instructions and LDS reads about equally (a group: 40 to 64 products, about 200 vector
// instructions, 18 to 36 KB of LDS reads a wave).  24 units of 1950 tokens, r = 32, bf16 storage, query and
// key side: 111 and 186 us with v_mfma_f32_16x16x4_f32, 74 and 119 now; 8 units of 2048, r = 64, fp32 storage:
// 116 and 169, 98 and 120 (158 and 134 when both rules' scores and weights were in registers at once).
#include "psf_parts.h"
#include "psf_f32.h"

namespace psf {
namespace {

// to^T += (32 streamed rows)^T w, see add_parts
template <int NT, int P>
__device__ __forceinline__ void add_tile(const uint16_t *tile, int plane, int pitch, const float (&w8)[8], f4 (&to)[NT],
                                         int lane, bool odd, unsigned seen)
{
    f4 part[NT];
    clear(part);
    if (odd) {
        add_parts_odd<NT, P>(tile, plane, pitch, w8, part, lane, seen);
    } else {
        Parts<3> w;
        split8(w8, w);
        add_parts<NT, P>(tile, plane, pitch, w, part, lane);
    }
    settle_parts();
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int k = 0; k < 4; ++k) to[t][k] += part[t][k];
}

// WR, WK as in psf_f32_fwd.hip: the sets of waves share the streamed rows of a tile and the state pieces.
template <int DT, int RT, int WR, int WK, bool KSIDE, typename T>
struct SideLds {
    static constexpr int P = parts_of<T>(), PC = KSIDE ? 3 : P, PO = KSIDE ? P : 3;   // parts of C streamed, own
    static constexpr int MT = RT < 2 ? 2 : RT, OP = pitch_of<RT>(), ROWS = 16 * WR;
    static constexpr int XP = tr_pitch<DT>(), MP = tr_pitch<MT>();
    static constexpr int kRow = (P + PC) * XP + 3 * MP;               // 16-bit places of a streamed row
    static constexpr int kThreads = 64 * WR * WK, KT = 32 * WK, kBuffers = WK == 4 ? 1 : 2;
    static constexpr int kX = P * KT * XP, kM = 3 * KT * MP;
    static constexpr int kPlane = KT * XP, kPiece = 3 * kPlane, kOwn = ROWS * OP * 2;
    static constexpr int kSums = (WK - 1) * WR * 4 * (2 * DT + RT) * 64 * 2;
    static constexpr int most(int a, int b) { return a > b ? a : b; }
    static constexpr int kPlaces = most(most(KT * kRow, kBuffers * kPiece + kOwn), kSums);
};

template <int DT, int RT, int WR, int WK, bool KSIDE, typename T>
__global__ __launch_bounds__((SideLds<DT, RT, WR, WK, KSIDE, T>::kThreads), WK == 1 && DT == 4 ? 2 : 1) void f32_bwd_kernel(
    const float *__restrict__ Mown, const float *__restrict__ Mstr, const T *__restrict__ Xown,
    const T *__restrict__ Xstr, const T *__restrict__ V, const float *__restrict__ GV, const float *__restrict__ gden,
    const float *__restrict__ Z, float *__restrict__ dM, float *__restrict__ dX, T *__restrict__ dV, F32Shape sh)
{
    using L = SideLds<DT, RT, WR, WK, KSIDE, T>;
    constexpr int VT = DT, ROWS = L::ROWS, KT = L::KT, P = L::P, PC = L::PC, PO = L::PO, MT = L::MT, XP = L::XP, MP = L::MP;
    constexpr int THREADS = L::kThreads;
    __shared__ __attribute__((aligned(16))) uint16_t lds[L::kPlaces];
    __shared__ __attribute__((aligned(16))) float gs[KT], sden[2][32 * WK];
    __shared__ int odd_tile[2];                              // the streamed rows hold an infinity or NaN
    uint16_t *xs = lds, *ms = xs + L::kX, *cs = ms + L::kM;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), li = lane & 15, g = lane >> 4;
    const int per_span = (min(sh.span, sh.n) + ROWS - 1) / ROWS;
    RowPlace place;
    if (!row_place(blockIdx.y * gridDim.x + blockIdx.x, sh.units, sh.spans, per_span, place)) return;
    const int u = place.unit, span = KSIDE ? place.span : sh.spans - 1 - place.span;
    const int s_begin = span * sh.span, s_end = min(sh.n, s_begin + sh.span);
    const int o0 = s_begin + (KSIDE ? place.k : per_span - 1 - place.k) * ROWS;
    if (o0 >= s_end) return;
    const int wr = wave % WR, wk = wave / WR, ow = o0 + 16 * wr, o = ow + li;
    const int o_last = min(o0 + ROWS, s_end) - 1, ow_last = min(ow + 15, s_end - 1);
    const bool there = o < s_end;
    const size_t urow = (size_t)u * sh.n;
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
    const int x_end = KSIDE ? s_end : o_last + 1, x_begin = KSIDE ? o0 : s_begin;
    typedef std::conditional_t<KSIDE, float, T> C;
    const C *cp;
    if constexpr (KSIDE) cp = GV + urow * sh.dv;
    else cp = V + urow * sh.dv;
    const int vec_c = KSIDE ? sh.vec_g : sh.vec_v;
    PartTile<DT, KT, XP, T, THREADS> xt;
    PartTile<MT, KT, MP, float, THREADS> mt;
    PartTile<VT, KT, XP, C, THREADS> ct;
    auto exact_in = [&](int x0) { return KSIDE ? x0 < edge_g_last : x0 + KT > edge_g; };
    auto cross_in = [&](int x0) { return KSIDE ? x0 + KT > edge_g : x0 < edge_g_last; };
    auto fetch_rows = [&](int x0) {
        const int nv = min(KT, x_end - x0);
        if (vec_c) ct.load(cp + (size_t)x0 * sh.dv, sh.dv, nv, sh.dv);
        if (exact_in(x0) && sh.vec_x) xt.load(Xstr + (urow + x0) * sh.d, sh.d, nv, sh.d);
        if (cross_in(x0) && sh.vec_m) mt.load(Mstr + (urow + x0) * sh.mcols, sh.mcols, nv, sh.mcols);
    };
    if (threadIdx.x < 2) odd_tile[threadIdx.x] = 0;
    fetch_rows(x_begin);
    const size_t o_row = urow + min(o, s_end - 1);           // (rows that are not there hold another's values and are not stored)
    Parts<P> xf[DT / 2];
    Parts<3> mf[MT / 2];
    Parts<PO> cf[VT / 2];
    float own_den = 1.f;
    {
        typedef std::conditional_t<KSIDE, T, float> CO;
        OwnRow<DT / 2, T> x_row;
        OwnRow<MT / 2, float> m_row;
        OwnRow<VT / 2, CO> c_row;
        if (sh.local_exact) x_row.load(Xown + o_row * sh.d, sh.d, sh.vec_x, g);
        m_row.load(Mown + o_row * sh.mcols, sh.mcols, sh.vec_m, g);
        if constexpr (KSIDE) c_row.load(V + o_row * sh.dv, sh.dv, sh.vec_v, g);
        else c_row.load(GV + o_row * sh.dv, sh.dv, sh.vec_g, g);
        if (!KSIDE) own_den = gden[o_row];
        if (sh.local_exact) x_row.parts(xf, sh.d, g);
        m_row.parts(mf, sh.mcols, g);
        c_row.parts(cf, sh.dv, g);
    }
    int turn = 0;
    for (int x0 = x_begin; x0 < x_end; x0 += KT, turn ^= 1) {
        const int nv = min(KT, x_end - x0);
        __syncthreads();
        bool odd = false;
        if (exact_in(x0)) {
            if (sh.vec_x) odd |= xt.template store<true>(xs, nv, sh.d);
            else odd |= stage_parts_scalar<DT, KT, XP, T, true, THREADS>(Xstr + (urow + x0) * sh.d, sh.d, nv, sh.d, xs);
        }
        if (cross_in(x0)) {
            if (sh.vec_m) odd |= mt.template store<true>(ms, nv, sh.mcols);
            else odd |= stage_parts_scalar<MT, KT, MP, float, true, THREADS>(Mstr + (urow + x0) * sh.mcols, sh.mcols, nv, sh.mcols, ms);
        }
        // (the query side takes C in scores only)
        if (vec_c) odd |= ct.template store<KSIDE>(cs, nv, sh.dv);
        else odd |= stage_parts_scalar<VT, KT, XP, C, KSIDE, THREADS>(cp + (size_t)x0 * sh.dv, sh.dv, nv, sh.dv, cs);
        if (KSIDE && threadIdx.x < KT) gs[threadIdx.x] = (int)threadIdx.x < nv ? gden[urow + x0 + threadIdx.x] : 0.f;
        if (odd) odd_tile[turn] = 1;
        __syncthreads();
        odd = odd_tile[turn] != 0;
        if (threadIdx.x == 0) odd_tile[turn ^ 1] = 0;       // (read for the last time before the barrier above)
        if (x0 + KT < x_end) fetch_rows(x0 + KT);
        const int r0 = 32 * wk, xw = x0 + r0;
        if (xw >= x_end || (KSIDE ? xw + 31 < ow : xw > ow_last)) continue;
        const bool exact_w = KSIDE ? xw < edge_w_last : xw + 31 >= edge_w;
        const bool cross_w = KSIDE ? xw + 31 >= edge_w : xw < edge_w_last;
        const bool masked = KSIDE ? xw < ow + 15 : xw + 31 > ow;      // some of the pairs
        const int rel = o - xw;                             // the own row's place among the streamed ones
        const unsigned seen = KSIDE ? (rel > 31 ? 0u : 0xffffffffu << max(0, rel))
                                    : (rel < 0 ? 0u : 0xffffffffu >> max(0, 31 - rel));
        auto place_of = [&](int k) { return xw + 16 * (k >> 2) + 4 * g + (k & 3); };
        auto mask = [&](float (&w)[8]) {
#pragma unroll
            for (int k = 0; k < 8; ++k) w[k] = (KSIDE ? place_of(k) >= o : place_of(k) <= o) ? w[k] : 0.f;
        };
        // Each rule's weights go into their sums before the other's scores are formed, and each tile's sums
        // are formed apart (two levels of summation, as long chains of one sign or both lose digits): the
        // fewest registers.
        f4 dw[2];
        float we[8];
        score_parts<2, VT / 2, PC, PO>(cs, KT * XP, XP, r0, cf, lane, dw);
        settle_parts();
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            if constexpr (KSIDE) dw[t] += *(const f4 *)&gs[r0 + 16 * t + 4 * g];
            else dw[t] += f4{own_den, own_den, own_den, own_den};
        }
        if (exact_w) {
            f4 se[2];
            float wx[8];
            score_parts<2, DT / 2, P, P>(xs, KT * XP, XP, r0, xf, lane, se);
            settle_parts();
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                float pm1;
                powers(se[k >> 2][k & 3], sh.p, we[k], pm1);
                wx[k] = (float)sh.p * pm1 * dw[k >> 2][k & 3];
                if (cross_w) wx[k] = (KSIDE ? place_of(k) < edge : place_of(k) >= edge) ? wx[k] : 0.f;
            }
            if (masked) mask(wx);
            add_tile<DT, P>(xs + r0 * XP, KT * XP, XP, wx, ax, lane, odd, seen);
        }
        if (cross_w) {
            f4 ss[2];
            float wm[8];
            score_parts<2, MT / 2, 3, 3>(ms, KT * MP, MP, r0, mf, lane, ss);
            settle_parts();
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const float s = ss[k >> 2][k & 3], own = s * s;
                wm[k] = 2.f * s * dw[k >> 2][k & 3];
                if (exact_w) {                              // either rule: the block's edge lies in the group
                    const bool ex = KSIDE ? place_of(k) < edge : place_of(k) >= edge;
                    we[k] = ex ? we[k] : own;
                    wm[k] = ex ? 0.f : wm[k];
                } else {
                    we[k] = own;
                }
            }
            if (masked) mask(wm);
            add_tile<RT, 3>(ms + r0 * MP, KT * MP, MP, wm, am, lane, odd, seen);
        }
        if constexpr (KSIDE) {
            if (masked) mask(we);
            add_tile<VT, PC>(cs + r0 * XP, KT * XP, XP, we, ac, lane, odd, seen);
        }
    }

    // Spans before (query side) or after (key side): with the record R of the state,
    // U[b'] = sum_c R[a][b'][c] C[c] (+ the denominator column), dm[a] += 2 sum_b' U[b'] m[b'],
    // which for the doubled tiles off the diagonal is dm[a] += U m[b'] and, for their mirror,
    // dm[b'] += U m[a]; key side also dV += R^T phi'.  A piece is two a with the 16 b' of a tile;
    // every set of waves has a piece of its own.
    if (sh.states && (KSIDE ? span < sh.spans - 1 : span > 0)) {
        constexpr int CP = 16 * VT, CH = CP / 8, G = WK, NP = 32 * G * CH / THREADS, PER = 8 / G;
        constexpr int LAST = tile_pairs(RT) * PER - 1;      // turns of the workgroup
        static_assert(32 * G * CH % THREADS == 0, "whole pieces");
        const float *z = Z + ((size_t)u * sh.spans + span) * record_floats(RT, VT);
        const float *zs = z + record_values(RT, VT) / 2 * 3;
        RecordPiece pre[NP];
        float pre_s = 0.f;
        auto fetch = [&](int piece) {
#pragma unroll
            for (int k = 0; k < NP; ++k) {
                const int idx = k * THREADS + threadIdx.x;
                pre[k].load(z, record_values(RT, VT), CP, piece * 32 * G + idx / CH, 8 * (idx % CH));
            }
            if (threadIdx.x < 32 * G) pre_s = zs[piece * 32 * G + threadIdx.x];
        };
        auto put = [&](int buf) {
            if (threadIdx.x < 32 * G) sden[buf][threadIdx.x] = pre_s;
#pragma unroll
            for (int k = 0; k < NP; ++k) {
                const int idx = k * THREADS + threadIdx.x;
                pre[k].store(lds + buf * L::kPiece + (idx / CH) * XP + 8 * (idx % CH), L::kPlane);
            }
        };
        fetch(0);
        // key side: an infinity or NaN of a later token's gradient is in its column of every row of the record,
        // the first among them; dV takes it from fp32 products, as within the span
        bool odd_record = false;
        if constexpr (KSIDE) {
            const uint16_t *first = (const uint16_t *)(z + (lane & ~7)) + (lane & 7);
#pragma unroll
            for (int c = 0; c < VT / 4; ++c) odd_record |= (first[128 * c] & 0x7f80u) == 0x7f80u;
            odd_record = __any(odd_record);
        }
        float m_own[4 * RT];
        load_frags<RT>(Mown + o_row * sh.mcols, sh.mcols, true, sh.vec_m, g, m_own);
        __syncthreads();
        put(0);
        float *own = (float *)(lds + L::kBuffers * L::kPiece) + (16 * wr + li) * L::OP;
        if (wk == 0) {
#pragma unroll
            for (int q = 0; q < RT; ++q)
                *(f4 *)&own[16 * q + 4 * g] = f4{m_own[4 * q], m_own[4 * q + 1], m_own[4 * q + 2], m_own[4 * q + 3]};
        }
        __syncthreads();
        int at = 0, q = 0;
        f4 mq = *(const f4 *)&own[4 * g], ma_sum = {0.f, 0.f, 0.f, 0.f}, mb_sum = ma_sum, pc[VT];
        clear(pc);
        auto flush = [&](int tile, f4 v) {                  // registers cannot be indexed
#pragma unroll
            for (int k = 0; k < RT; ++k)
                if (k == tile) am[k] += v;
        };
        for (int piece = 0; piece <= LAST; ++piece) {
            const int ch = piece % PER * G + wk, buf = L::kBuffers == 2 ? piece & 1 : 0;
            if (piece && piece % PER == 0) {                // the next pair of index tiles
                flush(at, ma_sum);
                flush(q, mb_sum);
                ma_sum = mb_sum = f4{0.f, 0.f, 0.f, 0.f};
                if (++q == RT) q = ++at;
                mq = *(const f4 *)&own[16 * q + 4 * g];
            }
            if (piece) __syncthreads();
            if (piece < LAST) fetch(piece + 1);
            const int w0 = 32 * wk;
            const uint16_t *zt = lds + buf * L::kPiece + w0 * XP;
            f4 U[2];
            score_parts<2, VT / 2, 3, PO>(zt, L::kPlane, XP, 0, cf, lane, U);
            settle_parts();
            float phi[8];
            const float diag = at == q ? 2.f : 1.f, off = at == q ? 0.f : 1.f;
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int a16 = 2 * ch + k;
                const float ma = own[16 * at + a16];
                U[k] += *(const f4 *)&sden[buf][w0 + 16 * k + 4 * g] * own_den;
                float t = 0.f;
#pragma unroll
                for (int s = 0; s < 4; ++s) t += U[k][s] * mq[s];
                t = over_groups(t) * diag;
                mb_sum += U[k] * (ma * off);
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    ma_sum[s] += a16 == 4 * g + s ? t : 0.f;
                    phi[4 * k + s] = ma * mq[s];
                }
            }
            if constexpr (KSIDE) {
                if (odd_record) {
                    add_parts_odd<VT, 3>(zt, L::kPlane, XP, phi, pc, lane, 0xffffffffu);
                } else {
                    Parts<3> pp;
                    split8(phi, pp);
                    add_parts<VT, 3>(zt, L::kPlane, XP, pp, pc, lane);
                }
                if (piece & 1) {                            // (an even number of turns)
                    add_settled(ac, pc);
                    clear(pc);
                }
            }
            if (L::kBuffers == 1) __syncthreads();
            if (piece < LAST) put(L::kBuffers == 2 ? buf ^ 1 : 0);
        }
        flush(at, ma_sum);
        flush(q, mb_sum);
    }

    if constexpr (WK > 1) {
        constexpr int PER = 4 * (DT + RT + (KSIDE ? VT : 0));
        __syncthreads();
        if (wk > 0) {
            float *to = (float *)lds + (size_t)((wk - 1) * WR + wr) * PER * 64 + lane;
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
        if (wk > 0) return;
        for (int w = 0; w < WK - 1; ++w) {
            const float *from = (const float *)lds + (size_t)(w * WR + wr) * PER * 64 + lane;
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
        auto go = [&](auto wr, auto wk) {
            constexpr int WR = decltype(wr)::value, WK = decltype(wk)::value;
            using L = SideLds<DT, RT, WR, WK, KSIDE, T>;
            const int per_span = ((pl.span < pb.n ? pl.span : pb.n) + L::ROWS - 1) / L::ROWS;
            const FlatGrid grid = flat_grid(row_groups(pb.units, pl.spans, per_span));
            hipLaunchKernelGGL((f32_bwd_kernel<DT, RT, WR, WK, KSIDE, T>), dim3(grid.x, grid.y), dim3(L::kThreads), 0, s,
                               KSIDE ? MK : MQ, KSIDE ? MQ : MK, (const T *)(KSIDE ? K : Q), (const T *)(KSIDE ? Q : K),
                               (const T *)V, GV, gden, Z, dM, dX, (T *)dV, sh);
            PSF_LAUNCH_CHECK();
            return PSF_OK;
        };
        constexpr bool PARTS4 = RT == 4 && sizeof(T) == 4;
        return f32_deal<DT, !PARTS4, !PARTS4>(pb, pl, RT, 70, go);
    });
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

}  // namespace psf
