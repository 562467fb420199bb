// Algorithm 1 and its reverse for the general path and the decoder's prompt: Gaussian sketches with d and
// sketch columns <= 128, fp32 results, on the bf16 matrix instructions from exact parts (psf_parts.h).
//
// A wave takes 16 H rows and keeps everything of them in registers: x as operand B, and every
// node's results (transposed: rows of the result are sketch columns) as the next level's operand B as
// they stand.  The matrices go through LDS in chunks of 32 rows, both of a node at once, and
// serve the four waves; forward their columns are the operand (read transposed), backward their
// rows.  Nodes are walked depth first and formed again on the way back, so that no level has to be kept.
// Bound by memory: x once in, m once out (72 k rows of 64 columns, r = 32, p = 4, bf16 storage: 13 us
// against 9 at copy rate; 41 with v_mfma_f32_16x16x4_f32 and the matrices read as single values from the caches).
#ifndef PSF_F32_SKETCH_H
#define PSF_F32_SKETCH_H

#include "psf_parts.h"
#include "psf_f32.h"

namespace psf {
namespace {

// levels of the tree of p / 2 first-level projections
constexpr int sketch_level(int p) { return p == 4 ? 1 : p == 8 ? 2 : 3; }

template <int DT, int RT, int H_, typename T>
struct Sketcher {
    static constexpr int H = H_, P = parts_of<T>(), MT = RT < 2 ? 2 : RT, KD = DT / 2, KR = MT / 2, PITCH = tr_pitch<MT>();
    static constexpr int kPlane = 32 * PITCH, kMatrix = P * kPlane;
    typedef f4 Rows[H][RT];                                 // rows 16 t + 4 g + s: sketch columns; column li: a row of x
    typedef Parts<3> Operand[H][KR];                        // the same in tile order
    Parts<P> x[H][KD];                                      // row order
    const T *g_first, *g_inner;
    uint16_t *lds;                                          // a chunk of both matrices of a node
    float sc;
    int d, r, p, vec_g, lane;

    PartTile<MT, 32, PITCH, T> ta, tb;
    __device__ __forceinline__ void fetch(const T *ga, int in, int e0)
    {
        if (!vec_g) return;
        ta.load(ga + (size_t)e0 * r, r, in - e0, r);
        tb.load(ga + (size_t)(in + e0) * r, r, in - e0, r);
    }
    __device__ __forceinline__ void stage(const T *ga, int in, int e0)
    {
        __syncthreads();
        if (vec_g) {
            ta.template store<false>(lds, in - e0, r);
            tb.template store<false>(lds + kMatrix, in - e0, r);
        } else {
            stage_parts_scalar<MT, 32, PITCH, T, false>(ga + (size_t)e0 * r, r, in - e0, r, lds);
            stage_parts_scalar<MT, 32, PITCH, T, false>(ga + (size_t)(in + e0) * r, r, in - e0, r, lds + kMatrix);
        }
        __syncthreads();
    }
    __device__ __forceinline__ const T *matrices(int level, int k) const       // of node k of a level (1: first)
    {
        if (level == 1) return g_first + (size_t)(2 * k) * d * r;
        return g_inner + (size_t)((level == 3 ? p / 4 : 0) + 2 * k) * r * r;
    }

    // U = xa G1, W = xb G2 for the two matrices from ga; every chunk's sum by itself
    template <int KS, int PB, bool TILE_ORDER>
    __device__ __forceinline__ void project(const T *ga, int in, const Parts<PB> (&xa)[H][KS], const Parts<PB> (&xb)[H][KS],
                                            Rows &U, Rows &W)
    {
        fetch(ga, in, 0);
#pragma unroll
        for (int h = 0; h < H; ++h) { clear(U[h]); clear(W[h]); }
#pragma unroll
        for (int k = 0; k < KS; ++k) {
            if (32 * k >= in) break;
            stage(ga, in, 32 * k);
            if (32 * (k + 1) < in) fetch(ga, in, 32 * (k + 1));
#pragma unroll
            for (int t = 0; t < RT; ++t) {
                Parts<P> a, b;
#pragma unroll
                for (int i = 0; i < P; ++i) {
                    const uint16_t *at = lds + i * kPlane;
                    a.v[i] = TILE_ORDER ? read_columns(at, PITCH, 16 * t, lane) : read_rows_tr(at, PITCH, 16 * t, lane);
                    b.v[i] = TILE_ORDER ? read_columns(at + kMatrix, PITCH, 16 * t, lane)
                                        : read_rows_tr(at + kMatrix, PITCH, 16 * t, lane);
                }
                f4 u[H], w[H];
                clear(u);
                clear(w);
                constexpr int LAST = P + PB - 2 < 2 ? P + PB - 2 : 2;
#pragma unroll
                for (int sum = LAST; sum >= 0; --sum)
#pragma unroll
                    for (int i = 0; i < P; ++i)
                        if (sum - i >= 0 && sum - i < PB)
#pragma unroll
                            for (int h = 0; h < H; ++h) {
                                u[h] = mm32(a.v[i], xa[h][k].v[sum - i], u[h]);
                                w[h] = mm32(b.v[i], xb[h][k].v[sum - i], w[h]);
                            }
                settle_parts();
#pragma unroll
                for (int h = 0; h < H; ++h) { U[h][t] += u[h]; W[h][t] += w[h]; }
            }
        }
    }

    __device__ __forceinline__ static void operand(const Rows &m, Operand &o)
    {
#pragma unroll
        for (int h = 0; h < H; ++h)
#pragma unroll
            for (int k = 0; k < KR; ++k) {
                float v[8];
#pragma unroll
                for (int s = 0; s < 8; ++s) v[s] = 2 * k + s / 4 < RT ? m[h][2 * k + s / 4 < RT ? 2 * k + s / 4 : 0][s % 4] : 0.f;
                split8(v, o[h][k]);
            }
    }

    // the two projections of node k of a level
    template <int LEVEL>
    __device__ __forceinline__ void projections(int k, Rows &U, Rows &W)
    {
        if constexpr (LEVEL == 1) {
            project<KD, P, false>(matrices(1, k), d, x, x, U, W);
        } else {
            Operand a, b;
#pragma unroll 1
            for (int child = 0; child < 2; ++child) {       // (one copy of the code of a level)
                Rows m;
                Operand o;
                forward<LEVEL - 1>(2 * k + child, m);
                operand(m, o);
#pragma unroll
                for (int h = 0; h < H; ++h)
#pragma unroll
                    for (int c = 0; c < KR; ++c) {
                        if (child == 0) a[h][c] = o[h][c];
                        b[h][c] = o[h][c];
                    }
            }
            project<KR, 3, true>(matrices(LEVEL, k), r, a, b, U, W);
        }
    }
    template <int LEVEL>
    __device__ __forceinline__ void forward(int k, Rows &m)
    {
        Rows W;
        projections<LEVEL>(k, m, W);
#pragma unroll
        for (int h = 0; h < H; ++h)
#pragma unroll
            for (int t = 0; t < RT; ++t)
#pragma unroll
                for (int s = 0; s < 4; ++s) m[h][t][s] = sc * (m[h][t][s] * W[h][t][s]);
    }

    // out1 += dU G1^T, out2 += dW G2^T (one and the same array: both sums into it)
    template <int OT, typename OUT>
    __device__ __forceinline__ void back_project(const T *ga, int in, const Operand &dU, const Operand &dW, OUT &out1, OUT &out2)
    {
        const int li = lane & 15, g = lane >> 4;
        fetch(ga, in, 0);
#pragma unroll
        for (int k = 0; k < (OT + 1) / 2; ++k) {
            if (32 * k >= in) break;
            stage(ga, in, 32 * k);
            if (32 * (k + 1) < in) fetch(ga, in, 32 * (k + 1));
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                if (2 * k + half >= OT) break;
                f4 u[H], w[H];
                clear(u);
                clear(w);
#pragma unroll
                for (int c = 0; c < KR; ++c) {
                    Parts<P> a, b;
                    const uint16_t *at = lds + (16 * half + li) * PITCH + 32 * c + 4 * g;
                    auto piece = [](const uint16_t *q) {        // tile order along a row
                        const uint2 lo = *(const uint2 *)q, hi = *(const uint2 *)(q + 16);
                        return __builtin_bit_cast(bf8, u4v{lo.x, lo.y, hi.x, hi.y});
                    };
#pragma unroll
                    for (int i = 0; i < P; ++i) { a.v[i] = piece(at + i * kPlane); b.v[i] = piece(at + kMatrix + i * kPlane); }
                    constexpr int LAST = 2;
#pragma unroll
                    for (int sum = LAST; sum >= 0; --sum)
#pragma unroll
                        for (int i = 0; i < P; ++i)
                            if (sum - i >= 0)
#pragma unroll
                                for (int h = 0; h < H; ++h) {
                                    u[h] = mm32(a.v[i], dU[h][c].v[sum - i], u[h]);
                                    w[h] = mm32(b.v[i], dW[h][c].v[sum - i], w[h]);
                                }
                }
                settle_parts();
#pragma unroll
                for (int h = 0; h < H; ++h) { out1[h][2 * k + half] += u[h]; out2[h][2 * k + half] += w[h]; }
            }
        }
    }

    // adds what dm, the gradient of node k's result, gives x: into dx
    template <int LEVEL>
    __device__ __forceinline__ void reverse(int k, const Rows &dm, f4 (&dx)[H][DT])
    {
        Operand dU, dW;
        {
            Rows U, W;
            projections<LEVEL>(k, U, W);
#pragma unroll
            for (int h = 0; h < H; ++h)
#pragma unroll
                for (int t = 0; t < RT; ++t) {
                    const f4 scaled = dm[h][t] * sc, u = U[h][t];
                    U[h][t] = scaled * W[h][t];
                    W[h][t] = scaled * u;
                }
            operand(U, dU);
            operand(W, dW);
        }
        if constexpr (LEVEL == 1) {
            back_project<DT>(matrices(1, k), d, dU, dW, dx, dx);
        } else {
            Rows left, right;
#pragma unroll
            for (int h = 0; h < H; ++h) { clear(left[h]); clear(right[h]); }
            back_project<RT>(matrices(LEVEL, k), r, dU, dW, left, right);
#pragma unroll 1
            for (int child = 0; child < 2; ++child) {
                reverse<LEVEL - 1>(2 * k + child, left, dx);
#pragma unroll
                for (int h = 0; h < H; ++h)
#pragma unroll
                    for (int t = 0; t < RT; ++t) left[h][t] = right[h][t];
            }
        }
    }
};

struct SketchArgs {
    int n, d, r, p, heads, per_head;
    size_t g_len, x_unit, m_unit;                           // elements from the rows of one unit to those of the next
    int vec_x, vec_m, vec_g;
};

template <typename S, typename T>
__device__ __forceinline__ void sketch_begin(S &s, const T *X, const T *G, uint16_t *lds, const SketchArgs &a, int i0)
{
    s.lane = threadIdx.x & 63;
    s.d = a.d; s.r = a.r; s.p = a.p; s.vec_g = a.vec_g;
    s.lds = lds;
    s.sc = sqrtf(1.0f / (float)a.r);
    s.g_first = G + (a.per_head ? (size_t)(blockIdx.y % a.heads) * a.g_len : 0);
    s.g_inner = s.g_first + (size_t)(a.p / 2) * a.d * a.r;
    OwnRow<S::KD, T> rows[S::H];
#pragma unroll
    for (int h = 0; h < S::H; ++h) rows[h].load(X + (size_t)min(i0 + 16 * h + (s.lane & 15), a.n - 1) * a.d, a.d, a.vec_x, s.lane >> 4);
#pragma unroll
    for (int h = 0; h < S::H; ++h) rows[h].parts(s.x[h], a.d, s.lane >> 4);
}

// f(LEVEL) for p = 4, 8, 16
template <typename F>
psf_status with_level(int p, F f)
{
    using std::integral_constant;
    return sketch_level(p) == 1 ? f(integral_constant<int, 1>{})
                                : sketch_level(p) == 2 ? f(integral_constant<int, 2>{}) : f(integral_constant<int, 3>{});
}

SketchArgs sketch_args(const Problem &pb, size_t x_unit, size_t m_unit)
{
    SketchArgs a = {};
    a.n = pb.n; a.d = pb.d; a.r = pb.r; a.p = pb.p; a.heads = pb.heads; a.per_head = pb.per_head ? 1 : 0;
    a.g_len = pb.g_len; a.x_unit = x_unit; a.m_unit = m_unit;
    return a;
}

unsigned plain_grid(size_t len)
{
    const size_t groups = (len + 4 * kF32Threads - 1) / (4 * kF32Threads);
    return (unsigned)(groups < 4096 ? groups : 4096);
}

}  // namespace
}  // namespace psf
#endif
