// Device helpers of the fp32 matrix-core kernels (psf_f32_fwd.hip, psf_f32_bwd.hip, psf_f32_sketch.h).
//
// One wave owns 16 rows of the sequence.  With li = lane & 15 and g = lane >> 4 a 16 x 16 result has
// column li, rows 4 g + 0 .. 3 in a lane.  Every kernel computes its results transposed, with the wave's
// own rows as columns, so that scores, weights, sketches and gradients of row li stay in the lanes li,
// li + 16, li + 32, li + 48 and no intermediate goes through LDS.  A row x of w columns held that
// way ("fragments") is f[4 q + s] = x[16 q + 4 g + s].  The products themselves: psf_parts.h.
#ifndef PSF_F32_TILES_H
#define PSF_F32_TILES_H

#include <type_traits>
#include "psf_f32_index.h"
#include "psf_internal.h"

namespace psf {

typedef float f4 __attribute__((ext_vector_type(4)));

constexpr int kF32Threads = 256;

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

// fp32 rows in LDS are padded by four floats: the 16-byte reads of 8 consecutive rows fall into different banks.
template <int NT>
constexpr int pitch_of() { return 16 * NT + 4; }

__device__ __forceinline__ float over_groups(float x)       // sum over the four lanes of a row
{
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// x^p and x^(p-1) for p a power of two
__device__ __forceinline__ void powers(float x, int p, float &pw, float &pm1)
{
    pw = x;
    pm1 = 1.f;
    for (int e = 1; e < p; e <<= 1) { pm1 *= pw; pw *= pw; }
}

// ---- states -----------------------------------------------------------------------------
// phi' = m (x) m is symmetric in its two indices: only tiles of 16 x 16 index pairs (a, b') with
// b' tile >= a tile are formed.  A state record is, for the RT (RT + 1) / 2 tile pairs in the
// order (0,0) (0,1) .. (1,1) .., [a16][b16][16 VT columns] and then, for the same pairs,
// [a16][b16] of the denominator column.  Tiles off the diagonal are stored doubled, for their mirror.
// The scan over the spans leaves the value columns as bf16 parts (psf_parts.h), in place: eight
// columns' 32 bytes hold their h and m, and their l follow behind all value columns, 16 bytes
// for eight columns.  (Reading fp32 records, every workgroup of rows took them apart again: 44 of its 94
// vector instructions a product step.)
__host__ __device__ constexpr int tile_pairs(int rt) { return rt * (rt + 1) / 2; }
__host__ __device__ constexpr size_t record_values(int rt, int vt) { return (size_t)tile_pairs(rt) * 256 * 16 * vt; }
__host__ __device__ constexpr size_t record_floats(int rt, int vt)
{
    return record_values(rt, vt) / 2 * 3 + (size_t)tile_pairs(rt) * 256;
}

// Everything the kernels need to know about the shape and how the sequence is cut.
struct F32Shape {
    int n, d, dv, mcols, p, b, units;
    int span, spans;          // tokens between two states; number of such spans
    int local_exact, noncausal, pairs, states;
    int vec_x, vec_v, vec_m, vec_g;   // 4-column pieces of Q, K (d), V, O (dv), m (mcols), G (r)
};

}  // namespace psf
#endif
