// Device helpers of the fp32 matrix-core kernels (psf_f32_fwd.hip, psf_f32_bwd.hip).
//
// All products of these kernels are v_mfma_f32_16x16x4_f32: fp32 operands, fp32 accumulation.
// One wave owns 16 rows of the sequence.  With li = lane & 15 and g = lane >> 4 a lane holds
//   operand A (16 x 4): row li, column g;   operand B (4 x 16): row g, column li;
//   result (16 x 16):   column li, rows 4 g + 0 .. 3.
// The sum over k may visit k in any order as long as both operands agree, so step s of a group of
// four steps takes k = 4 g + s.  A lane then reads the four k of a group as one 16-byte piece, and
// a result (rows 4 g + s, column li) is the B operand of the next product as it stands.  Every
// kernel computes its results transposed, with the wave's own rows as columns, so that scores,
// weights, sketches and gradients of row li stay in the lanes li, li + 16, li + 32, li + 48 and no
// intermediate goes through LDS.  A row x of w columns held that way ("fragments") is
// f[4 q + s] = x[16 q + 4 g + s].
#ifndef PSF_F32_TILES_H
#define PSF_F32_TILES_H

#include <type_traits>
#include "psf_f32_index.h"
#include "psf_internal.h"

namespace psf {

typedef float f4 __attribute__((ext_vector_type(4)));

constexpr int kF32Threads = 256;

__device__ __forceinline__ f4 mm(float a, float b, f4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Four columns as stored, and as fp32.
template <typename S> struct Raw4;
template <> struct Raw4<float> { typedef f4 type; };
template <> struct Raw4<bf16_t> { typedef uint2 type; };
__device__ __forceinline__ f4 widen(f4 v) { return v; }
__device__ __forceinline__ f4 widen(uint2 v)
{
    return f4{__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xffff0000u), __uint_as_float(v.y << 16),
              __uint_as_float(v.y & 0xffff0000u)};
}

__device__ __forceinline__ f4 load4(const float *p) { return *(const f4 *)p; }
__device__ __forceinline__ f4 load4(const bf16_t *p)
{
    return widen(*(const uint2 *)p);
}
__device__ __forceinline__ void store4(float *p, f4 v) { *(f4 *)p = v; }
__device__ __forceinline__ void store4(bf16_t *p, f4 v)
{
    *(uint2 *)p = make_uint2((uint32_t)f32_to_bf16(v[0]) | ((uint32_t)f32_to_bf16(v[1]) << 16),
                             (uint32_t)f32_to_bf16(v[2]) | ((uint32_t)f32_to_bf16(v[3]) << 16));
}

template <int N>
__device__ __forceinline__ void clear(f4 (&a)[N])
{
#pragma unroll
    for (int k = 0; k < N; ++k) a[k] = f4{0.f, 0.f, 0.f, 0.f};
}
// Waits until the products issued before it can be read by other instructions.  The compiler
// inserts these waits itself, but it can miss one where a product and its reader lie in different
// basic blocks with a longer and a shorter way between them (seen: the last result of a state
// piece read three instructions after its product); so results that leave a branch or a loop
// are read after this.  tests/test_matrix_waits_host.py follows every way through the machine code.
__device__ __forceinline__ void settle()
{
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_nop 15");
    __builtin_amdgcn_sched_barrier(0);
}

template <int N>
__device__ __forceinline__ void add_to(f4 (&a)[N], const f4 (&x)[N])
{
    settle();
#pragma unroll
    for (int k = 0; k < N; ++k) a[k] += x[k];
}

// Columns c .. c + 3 of a row of `width` columns, zero beyond it.  vec: four columns may be moved
// as one piece (width a multiple of 4 and the tensor's base aligned to the piece).
template <typename S>
__device__ __forceinline__ f4 row_piece(const S *row, int c, int width, int vec)
{
    f4 v = {0.f, 0.f, 0.f, 0.f};
    if (vec) {
        if (c < width) v = load4(row + c);
    } else {
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (c + k < width) v[k] = load_f(row, c + k);
    }
    return v;
}

template <typename S>
__device__ __forceinline__ void store_piece(S *row, int c, int width, int vec, f4 v)
{
    if (vec) {
        if (c < width) store4(row + c, v);
    } else {
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (c + k < width) store_f(row, c + k, v[k]);
    }
}

// fragments of one row (see above); zeros when the row is not there
template <int NT, typename S>
__device__ __forceinline__ void load_frags(const S *row, int width, bool there, int vec, int g, float (&f)[4 * NT])
{
#pragma unroll
    for (int q = 0; q < NT; ++q) {
        f4 v = {0.f, 0.f, 0.f, 0.f};
        if (there) v = row_piece(row, 16 * q + 4 * g, width, vec);
#pragma unroll
        for (int s = 0; s < 4; ++s) f[4 * q + s] = v[s];
    }
}

// LDS rows are padded by four floats: the 16-byte reads of 8 consecutive rows fall into different
// banks, and so do the 4-byte reads of 16 columns of rows 0, 4, 8, 12.
template <int NT>
constexpr int pitch_of() { return 16 * NT + 4; }

// NR rows of 16 * NT columns on their way into LDS; rows >= nvalid and columns >= width (at least
// 1 either) become zero.  All loads are issued before the first result is needed, and none of them
// sits behind a branch: places that are not there load the first piece instead.  A thread
// holds the same columns of kPieces rows, as stored.
template <int NT, int NR, typename S>
struct Tile {
    static constexpr int kPieces = NR * 4 * NT / kF32Threads, kStep = kF32Threads / (4 * NT);
    static_assert(NR * 4 * NT % kF32Threads == 0 && kF32Threads % (4 * NT) == 0, "whole pieces");
    typedef typename Raw4<S>::type raw;
    raw v[kPieces];
    __device__ __forceinline__ void load(const S *src, int ld, int nvalid, int width)
    {
        const int row = threadIdx.x / (4 * NT), c = 4 * (threadIdx.x % (4 * NT));
#pragma unroll
        for (int it = 0; it < kPieces; ++it)
            v[it] = *(const raw *)((const char *)src + tile_piece(row + it * kStep, c, ld, nvalid, width) * (uint32_t)sizeof(S));
    }
    __device__ __forceinline__ void store(float *dst, int nvalid, int width) const
    {
        const int row = threadIdx.x / (4 * NT), c = 4 * (threadIdx.x % (4 * NT));
        const int rows = c < width ? nvalid : 0;
#pragma unroll
        for (int it = 0; it < kPieces; ++it)
            *(f4 *)&dst[(row + it * kStep) * pitch_of<NT>() + c] =
                row + it * kStep < rows ? widen(v[it]) : f4{0.f, 0.f, 0.f, 0.f};
    }
};

// the same for tensors whose rows cannot be moved four columns at a time
template <int NT, int NR, typename S>
__device__ __forceinline__ void stage_scalar(const S *src, int ld, int nvalid, int width, float *dst)
{
    const int c = 4 * (threadIdx.x % (4 * NT));
#pragma unroll 1
    for (int row = threadIdx.x / (4 * NT); row < NR; row += kF32Threads / (4 * NT)) {
        f4 v = {0.f, 0.f, 0.f, 0.f};
        if (row < nvalid) v = row_piece(src + (size_t)row * ld, c, width, 0);
        *(f4 *)&dst[row * pitch_of<NT>() + c] = v;
    }
}

// acc^T += (rows of the LDS tile)^T w for one group of 16 tile rows: acc[ct] has rows
// 16 ct + 4 g + s, column li; w[s] belongs to tile row row0 + 4 g + s.
// GUARD: some of the 16 weights of a lane may be masked zeros whose tile row this lane's own row
// must not see.  0 * inf would carry a later token's inf or NaN to an earlier row, so a group
// that holds one is summed without the masked pairs; seen: bit k set when tile row row0 + k
// counts for this lane's own row.
template <int NT, bool GUARD>
__device__ __forceinline__ void add_rows(const float *tile, int row0, const float (&w)[4], f4 (&acc)[NT], int lane,
                                         unsigned seen)
{
    const int li = lane & 15, g = lane >> 4;
    constexpr int P = pitch_of<NT>();
    const float *at = tile + (row0 + 4 * g) * P + li;
    if (GUARD) {
        float probe = 0.f;
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int ct = 0; ct < NT; ++ct) probe = __builtin_fmaf(at[s * P + 16 * ct], 0.f, probe);
        if (__any(probe != 0.f)) {
            for (int k4 = 0; k4 < 4; ++k4) {
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    const float wk = __shfl(w[s], li + 16 * k4);
                    if ((seen >> (4 * k4 + s)) & 1u) {
#pragma unroll
                        for (int ct = 0; ct < NT; ++ct)
#pragma unroll
                            for (int k = 0; k < 4; ++k)
                                acc[ct][k] += wk * tile[(row0 + 4 * k4 + s) * P + 16 * ct + 4 * g + k];
                    }
                }
            }
            return;
        }
    }
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int ct = 0; ct < NT; ++ct) acc[ct] = mm(at[s * P + 16 * ct], w[s], acc[ct]);
}

// scores of 16 tile rows with the wave's own rows: result rows row0 + 4 g + s, column li
template <int NT>
__device__ __forceinline__ f4 score_rows(const float *tile, int row0, const float (&own)[4 * NT], int lane)
{
    const float *at = tile + (row0 + (lane & 15)) * pitch_of<NT>() + 4 * (lane >> 4);
    // sums of at most 32 columns: p-th powers enlarge what a long sum loses
    constexpr int SUMS = NT >= 4 ? 4 : 2;
    f4 sum[SUMS];
    clear(sum);
#pragma unroll
    for (int q = 0; q < NT; ++q) {
        const f4 a = *(const f4 *)(at + 16 * q);
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int k = SUMS == 4 ? 2 * (2 * q / NT) + s % 2 : s % 2;
            sum[k] = mm(a[s], own[4 * q + s], sum[k]);
        }
    }
    if constexpr (SUMS == 4) return (sum[0] + sum[1]) + (sum[2] + sum[3]);
    else return sum[0] + sum[1];
}

__device__ __forceinline__ float over_groups(float x)       // sum over the four lanes of a row
{
    x += __shfl_xor(x, 16);
    return x + __shfl_xor(x, 32);
}

// x^p and x^(p-1) for p a power of two
__device__ __forceinline__ void powers(float x, int p, float &pw, float &pm1)
{
    pw = x;
    pm1 = 1.f;
    for (int e = 1; e < p; e <<= 1) { pm1 *= pw; pw *= pw; }
}

// ---- projections of Algorithm 1 -----------------------------------------------------------
// A wave takes 16 H rows.  The row vectors live in LDS, [rows][columns + 4], columns padded to 16
// with zeros; result^T = G^T x^T for 16 columns from c0: A = G[e][c] from memory (lane row c,
// k = e; the matrices stay in the caches), each value serving the H groups of 16 rows, B = x
// from LDS in 16-byte pieces.
template <int H, typename T>
__device__ __forceinline__ void project(const T *G, int in, int r, int c0, const float *x, int pitch, f4 (&out)[H],
                                        int lane)
{
    const int li = lane & 15, g = lane >> 4, c = c0 + li;
    const float *xr = x + li * pitch + 4 * g;
    const T *ga = G + (size_t)(4 * g) * r + (c < r ? c : 0);
    clear(out);
    // STEP rows of G: all loads first.  Every 16 rows are a sum of their own: with 32 of them a
    // kernel takes 35 us instead of 42 (72 k rows of 64, r = 32), but gradients were up to 10 %
    // further from float64 than the vector kernels' (r = 32, blocks of 48 tokens).
    auto run = [&](auto step, int e0) {
        constexpr int STEP = decltype(step)::value;
        float a[STEP / 4];
#pragma unroll
        for (int e = 0; e < STEP; e += 16)
#pragma unroll
            for (int s = 0; s < 4; ++s) a[e / 4 + s] = load_f(ga, (size_t)((e0 + e + s) * r));
#pragma unroll
        for (int e = 0; e < STEP; e += 32) {
            f4 even[H], odd[H];
            clear(even);
            clear(odd);
#pragma unroll
            for (int h = 0; h < H; ++h) {
                const float *xh = xr + 16 * h * pitch + e0 + e;
                const f4 xe = *(const f4 *)xh, xo = *(const f4 *)(xh + 16);
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    even[h] = mm(a[e / 4 + s], xe[s], even[h]);
                    odd[h] = mm(a[e / 4 + 4 + s], xo[s], odd[h]);
                }
            }
#pragma unroll
            for (int h = 0; h < H; ++h) out[h] += even[h] + odd[h];
        }
    };
    int e0 = 0;
    if (c0 + 16 <= r) {
        for (; e0 + 64 <= in; e0 += 64) run(std::integral_constant<int, 64>{}, e0);
        if (e0 + 32 <= in) { run(std::integral_constant<int, 32>{}, e0); e0 += 32; }
    }
    for (; e0 < in; e0 += 16) {
        f4 part[H], xv[H];
        clear(part);
#pragma unroll
        for (int h = 0; h < H; ++h) xv[h] = *(const f4 *)(xr + 16 * h * pitch + e0);
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const float a = c < r && e0 + 4 * g + s < in ? load_f(ga, (size_t)(e0 + s) * r) : 0.f;
#pragma unroll
            for (int h = 0; h < H; ++h) part[h] = mm(a, xv[h][s], part[h]);
        }
        add_to(out, part);
    }
}

// the transposed product: acc^T (16 rows e from e0) += G y^T for y [rows][pitch] of r columns
template <int H, typename T>
__device__ __forceinline__ void back_project(const T *G, int in, int r, int e0, const float *y, int pitch, int vec,
                                             f4 (&acc)[H], int lane)
{
    const int li = lane & 15, g = lane >> 4, e = e0 + li;
    const T *ga = G + (size_t)(e < in ? e : 0) * r;
    const float *yr = y + li * pitch + 4 * g;
    f4 part[H];                                             // two levels of summation
    clear(part);
    for (int c0 = 0; c0 < r; c0 += 16) {
        f4 a = {0.f, 0.f, 0.f, 0.f};
        if (e < in) a = row_piece(ga, c0 + 4 * g, r, vec);
#pragma unroll
        for (int h = 0; h < H; ++h) {
            const f4 yv = *(const f4 *)(yr + 16 * h * pitch + c0);
#pragma unroll
            for (int s = 0; s < 4; ++s) part[h] = mm(a[s], yv[s], part[h]);
        }
    }
    add_to(acc, part);
}

// ---- states -----------------------------------------------------------------------------
// phi' = m (x) m is symmetric in its two indices: only tiles of 16 x 16 index pairs (a, b') with
// b' tile >= a tile are formed.  A state record is, for the RT (RT + 1) / 2 tile pairs in the
// order (0,0) (0,1) .. (1,1) .., [a16][b16][16 VT columns] and then, for the same pairs,
// [a16][b16] of the denominator column.  Tiles off the diagonal are stored doubled, for their mirror.
__host__ __device__ constexpr int tile_pairs(int rt) { return rt * (rt + 1) / 2; }
__host__ __device__ constexpr size_t record_floats(int rt, int vt) { return (size_t)tile_pairs(rt) * 256 * (16 * vt + 1); }

// Everything the kernels need to know about the shape and how the sequence is cut.
struct F32Shape {
    int n, d, dv, mcols, p, b, units;
    int span, spans;          // tokens between two states; number of such spans
    int local_exact, noncausal, pairs, states;
    int vec_x, vec_v, vec_m, vec_g;   // 4-column pieces of Q, K (d), V, O (dv), m (mcols), G (r)
};

}  // namespace psf
#endif
