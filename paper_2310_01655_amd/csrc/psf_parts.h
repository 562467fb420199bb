// fp32 products on the bf16 matrix instructions, from exact parts.
//
// An fp32 value is the sum of three bf16 values: h, its upper 16 bits; m, the remainder x - h
// (exact, at most 16 significant bits) rounded to bf16; l, what is left (exact, at most 8 bits).
// (From 2^-110 on.  Below that l, then m, lose bits, as bf16 ends at 2^-133: all of V near 2^-112, 2^-114, 2^-118 and
// 2^-126 gives O a relative error of 2.6e-7, 6.2e-7, 9e-6 and 2.3e-3; 2.2e-7 from 2^-110 on.)
// h truncates, so that no finite value becomes an infinity; m rounds, so that the terms left out
// below have no sign of their own.  A product of two such sums is formed from the six products of
// parts down to 2^-16 of the largest (h h, h m, m h, m m, h l, l h), smallest first; what is left out is
// below 2^-23 of the product.  A value stored as bf16 is its own h: three products, or
// one for two of them, and nothing is left out.  Every product of parts is exact in fp32 and the
// instruction adds 32 of them before it rounds, so that the sums come out closer than those of
// v_mfma_f32_16x16x4_f32: normal operands, relative error of 64 (2048, in tiles of 64) terms
// 1.0e-7 (1.4e-7) against 1.5e-7 (1.9e-7); non-negative ones 7.5e-8 (9.4e-8) against 1.2e-7 (9.1e-8).
//
// Rates a SIMD: 16x16x4 fp32 2048 flops in 32 cycles, 16x16x32 bf16 16384 in 16: six products take
// 3/8 of the time of the fp32 instruction, three 3/16, one 1/16.  Taking a value apart costs 5.5
// vector instructions; staged tiles are taken apart once for all rows of a workgroup.
//
// Operands of v_mfma_f32_16x16x32_bf16, li = lane & 15, g = lane >> 4:
//   A (16 x 32): row li, k = 8 g + j;   B (32 x 16): column li, k = 8 g + j, j < 8 in 4 registers;
//   result (16 x 16): column li, rows 4 g + 0 .. 3.
// The eight k of a lane may stand for any eight places as long as A and B agree:
//   "row order"   places 8 g + j: operands read along a row, 16 bytes a lane;
//   "tile order"  places 4 g + j (j < 4) and 16 + 4 g + j - 4: two results (rows 4 g + s of two tiles) are
//                 such an operand as they stand, and two ds_read_b64_tr_b16 of row-major
//                 LDS rows are the matching one (each: 4 rows x 16 columns a 16-lane group, transposed).
#ifndef PSF_PARTS_H
#define PSF_PARTS_H

#include "psf_f32_tiles.h"

namespace psf {

typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
typedef float fl2 __attribute__((ext_vector_type(2)));
typedef short sh4 __attribute__((ext_vector_type(4)));
typedef uint32_t u4v __attribute__((ext_vector_type(4)));

template <typename T> constexpr int parts_of();             // parts of a stored value
template <> constexpr int parts_of<float>() { return 3; }
template <> constexpr int parts_of<bf16_t>() { return 1; }

// eight values of a lane
template <int P> struct Parts { bf8 v[P]; };

__device__ __forceinline__ f4 mm32(bf8 a, bf8 b, f4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }

__device__ __forceinline__ uint32_t round_pair(float a, float b)
{
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(fl2{a, b}, bf2));
}

// the parts of a and b, packed in pairs (a in the lower half)
struct PairParts { uint32_t h, m, l; };
__device__ __forceinline__ PairParts rest_parts(uint32_t h, float ra, float rb)
{
    const uint32_t m = round_pair(ra, rb);
    const uint32_t l = round_pair(ra - __uint_as_float(m << 16), rb - __uint_as_float(m & 0xffff0000u));
    return {h, m, l};
}
__device__ __forceinline__ PairParts split_pair(float a, float b)
{
    const uint32_t ua = __float_as_uint(a), ub = __float_as_uint(b);
    return rest_parts(__builtin_amdgcn_perm(ub, ua, 0x07060302u), a - __uint_as_float(ua & 0xffff0000u),
                      b - __uint_as_float(ub & 0xffff0000u));
}
// the same for values that may be infinite: an infinity is all h
__device__ __forceinline__ PairParts split_pair_inf(float a, float b)
{
    const uint32_t ua = __float_as_uint(a), ub = __float_as_uint(b);
    const float ra = a - __uint_as_float(ua & 0xffff0000u), rb = b - __uint_as_float(ub & 0xffff0000u);
    return rest_parts(__builtin_amdgcn_perm(ub, ua, 0x07060302u), __builtin_isinf(a) ? 0.f : ra, __builtin_isinf(b) ? 0.f : rb);
}

template <bool INF = false>
__device__ __forceinline__ void split8(const float (&x)[8], Parts<3> &p)
{
    u4v h, m, l;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const PairParts q = INF ? split_pair_inf(x[2 * k], x[2 * k + 1]) : split_pair(x[2 * k], x[2 * k + 1]);
        h[k] = q.h;
        m[k] = q.m;
        l[k] = q.l;
    }
    p.v[0] = __builtin_bit_cast(bf8, h);
    p.v[1] = __builtin_bit_cast(bf8, m);
    p.v[2] = __builtin_bit_cast(bf8, l);
}
// values that are bf16 already
__device__ __forceinline__ void split8(const float (&x)[8], Parts<1> &p)
{
    u4v h;
#pragma unroll
    for (int k = 0; k < 4; ++k)
        h[k] = __builtin_amdgcn_perm(__float_as_uint(x[2 * k + 1]), __float_as_uint(x[2 * k]), 0x07060302u);
    p.v[0] = __builtin_bit_cast(bf8, h);
}

// acc[t] += A[t] B over the parts, smallest products first, the N results in turn
template <int PA, int PB, int N>
__device__ __forceinline__ void mm_parts(const Parts<PA> (&a)[N], const Parts<PB> &b, f4 (&acc)[N])
{
    constexpr int LAST = PA + PB - 2 < 2 ? PA + PB - 2 : 2;
#pragma unroll
    for (int sum = LAST; sum >= 0; --sum)
#pragma unroll
        for (int i = 0; i < PA; ++i)
            if (sum - i >= 0 && sum - i < PB)
#pragma unroll
                for (int t = 0; t < N; ++t) acc[t] = mm32(a[t].v[i], b.v[sum - i], acc[t]);
}

// acc[t] += A B[t]: one operand A, the N operands B in turn
template <int PA, int PB, int N>
__device__ __forceinline__ void mm_columns(const Parts<PA> &a, const Parts<PB> (&b)[N], f4 (&acc)[N])
{
    constexpr int LAST = PA + PB - 2 < 2 ? PA + PB - 2 : 2;
#pragma unroll
    for (int sum = LAST; sum >= 0; --sum)
#pragma unroll
        for (int i = 0; i < PA; ++i)
            if (sum - i >= 0 && sum - i < PB)
#pragma unroll
                for (int t = 0; t < N; ++t) acc[t] = mm32(a.v[i], b[t].v[sum - i], acc[t]);
}

// ---- tiles in LDS: the parts of NR rows of 16 NT columns, part by part, rows PITCH apart -----------
// 8 columns of padding spread the 16-byte reads along rows over the banks, 16 the transposed ones.
template <int NT> constexpr int row_pitch() { return 16 * NT + 8; }
template <int NT> constexpr int tr_pitch() { return 16 * NT + 16; }

template <bool INF>
__device__ __forceinline__ void put4(uint16_t *dst, int plane, uint2 raw, bool there, Parts<1> *)
{
    *(uint2 *)dst = there ? raw : make_uint2(0u, 0u);
}
template <bool INF>
__device__ __forceinline__ void put4(uint16_t *dst, int plane, f4 v, bool there, Parts<3> *)
{
    if (!there) v = f4{0.f, 0.f, 0.f, 0.f};
    const PairParts a = INF ? split_pair_inf(v[0], v[1]) : split_pair(v[0], v[1]);
    const PairParts b = INF ? split_pair_inf(v[2], v[3]) : split_pair(v[2], v[3]);
    *(uint2 *)dst = make_uint2(a.h, b.h);
    *(uint2 *)(dst + plane) = make_uint2(a.m, b.m);
    *(uint2 *)(dst + 2 * plane) = make_uint2(a.l, b.l);
}
// an infinity or NaN among four values
__device__ __forceinline__ bool odd_values(f4 v)
{
    const float probe = __builtin_fmaf(v[0], 0.f, __builtin_fmaf(v[1], 0.f, __builtin_fmaf(v[2], 0.f, v[3] * 0.f)));
    return probe != 0.f;
}
__device__ __forceinline__ bool odd_values(uint2 v)
{
    return ((((v.x & 0x7fff7fffu) + 0x00800080u) | ((v.y & 0x7fff7fffu) + 0x00800080u)) & 0x80008000u) != 0u;
}

// NR rows of 16 * NT columns on their way into LDS; rows >= nvalid and columns >= width (at least
// 1 either) become zero.  All loads are issued before the first result is needed, and none of them
// sits behind a branch: places that are not there load the first piece instead.  store() returns
// whether the thread saw an infinity or NaN (LOOK).
template <int NT, int NR, int PITCH, typename S, int THREADS = kF32Threads>
struct PartTile {
    static constexpr int kPieces = NR * 4 * NT / THREADS, kStep = THREADS / (4 * NT), kPlane = NR * PITCH;
    static_assert(NR * 4 * NT % THREADS == 0 && THREADS % (4 * NT) == 0, "whole pieces");
    typedef typename Raw4<S>::type raw;
    raw v[kPieces];
    // whole tiles take neither bounds nor selects (a third of the vector instructions of the 64-row kernels)
    static __device__ __forceinline__ bool whole(int nvalid, int width) { return nvalid >= NR && width >= 16 * NT; }
    __device__ __forceinline__ void load(const S *src, int ld, int nvalid, int width)
    {
        const int row = threadIdx.x / (4 * NT), c = 4 * (threadIdx.x % (4 * NT));
        if (whole(nvalid, width)) {
            const uint32_t at = (uint32_t)(row * ld + c) * (uint32_t)sizeof(S);
#pragma unroll
            for (int it = 0; it < kPieces; ++it)
                v[it] = *(const raw *)((const char *)(src + it * kStep * ld) + at);
        } else {
#pragma unroll
            for (int it = 0; it < kPieces; ++it)
                v[it] = *(const raw *)((const char *)src +
                                       tile_piece(row + it * kStep, c, ld, nvalid, width) * (uint32_t)sizeof(S));
        }
    }
    template <bool LOOK>
    __device__ __forceinline__ bool store(uint16_t *dst, int nvalid, int width) const
    {
        const int row = threadIdx.x / (4 * NT), c = 4 * (threadIdx.x % (4 * NT));
        bool odd = false;
        if (whole(nvalid, width)) {
#pragma unroll
            for (int it = 0; it < kPieces; ++it) {
                put4<LOOK>(dst + (row + it * kStep) * PITCH + c, kPlane, v[it], true, (Parts<parts_of<S>()> *)nullptr);
                if (LOOK) odd |= odd_values(v[it]);
            }
            return odd;
        }
        const int rows = c < width ? nvalid : 0;
#pragma unroll
        for (int it = 0; it < kPieces; ++it) {
            const bool there = row + it * kStep < rows;
            put4<LOOK>(dst + (row + it * kStep) * PITCH + c, kPlane, v[it], there, (Parts<parts_of<S>()> *)nullptr);
            if (LOOK) odd |= there && odd_values(v[it]);
        }
        return odd;
    }
};

// the same for tensors whose rows cannot be moved four columns at a time
template <int NT, int NR, int PITCH, typename S, bool LOOK, int THREADS = kF32Threads>
__device__ __forceinline__ bool stage_parts_scalar(const S *src, int ld, int nvalid, int width, uint16_t *dst)
{
    const int c = 4 * (threadIdx.x % (4 * NT));
    bool odd = false;
#pragma unroll 1
    for (int row = threadIdx.x / (4 * NT); row < NR; row += THREADS / (4 * NT)) {
        f4 v = {0.f, 0.f, 0.f, 0.f};
        if (row < nvalid) v = row_piece(src + (size_t)row * ld, c, width, 0);
        if (LOOK) odd |= odd_values(v);
        if constexpr (parts_of<S>() == 1)
            *(uint2 *)&dst[row * PITCH + c] = make_uint2(
                __builtin_amdgcn_perm(__float_as_uint(v[1]), __float_as_uint(v[0]), 0x07060302u),
                __builtin_amdgcn_perm(__float_as_uint(v[3]), __float_as_uint(v[2]), 0x07060302u));
        else put4<LOOK>(&dst[row * PITCH + c], NR * PITCH, v, true, (Parts<3> *)nullptr);
    }
    return odd;
}

// A row on its way to operand B in row order: step k holds columns 32 k + 8 g + j.  load() issues every
// load and waits for none, so that several rows and the first tile are in flight together; the
// row has to exist.  at(): four columns, zero from `width` on.
template <int KS, typename S>
struct OwnRow {
    typedef typename Raw4<S>::type raw;
    raw v[2 * KS];
    __device__ __forceinline__ void load(const S *row, int width, int vec, int g)
    {
        if (vec) {
#pragma unroll
            for (int e = 0; e < 2 * KS; ++e) {
                const int c = 32 * (e / 2) + 8 * g + 4 * (e % 2);
                v[e] = *(const raw *)(row + (c < width ? c : 0));
            }
        } else {
#pragma unroll
            for (int e = 0; e < 2 * KS; ++e) {
                const f4 x = row_piece(row, 32 * (e / 2) + 8 * g + 4 * (e % 2), width, 0);
                if constexpr (parts_of<S>() == 1)
                    v[e] = make_uint2(__builtin_amdgcn_perm(__float_as_uint(x[1]), __float_as_uint(x[0]), 0x07060302u),
                                      __builtin_amdgcn_perm(__float_as_uint(x[3]), __float_as_uint(x[2]), 0x07060302u));
                else v[e] = x;
            }
        }
    }
    __device__ __forceinline__ f4 at(int e, int width, int g) const
    {
        return 32 * (e / 2) + 8 * g + 4 * (e % 2) < width ? widen(v[e]) : f4{0.f, 0.f, 0.f, 0.f};
    }
    template <int P>
    __device__ __forceinline__ void parts(Parts<P> (&f)[KS], int width, int g) const
    {
#pragma unroll
        for (int k = 0; k < KS; ++k) {
            const f4 a = at(2 * k, width, g), b = at(2 * k + 1, width, g);
            const float x[8] = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
            split8(x, f[k]);
        }
    }
};

// Waits until the products issued before it can be read by other instructions (4 passes: 8 states).
// The compiler inserts these waits itself, but it can miss one where a product and its reader lie in
// different basic blocks with a longer and a shorter way between them; so results that leave a
// branch or a loop are read after this.  tests/test_matrix_waits_host.py follows every way
// through the machine code.
__device__ __forceinline__ void settle_parts()
{
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_nop 7");
    __builtin_amdgcn_sched_barrier(0);
}
template <int N>
__device__ __forceinline__ void add_settled(f4 (&a)[N], const f4 (&x)[N])
{
    settle_parts();
#pragma unroll
    for (int k = 0; k < N; ++k) a[k] += x[k];
}

// scores of 16 NT tile rows with the wave's own rows: s[t] has rows row0 + 16 t + 4 g + s, column li; one
// sum per 32 columns.  The NT results are formed in turn: each is a chain of dependent products.
// (Read them after settle_parts() if they leave a branch.)
template <int NT, int KS, int PA, int PB>
__device__ __forceinline__ void score_parts(const uint16_t *tile, int plane, int pitch, int row0, const Parts<PB> (&own)[KS],
                                            int lane, f4 (&s)[NT])
{
    const uint16_t *at = tile + (row0 + (lane & 15)) * pitch + 8 * (lane >> 4);
    constexpr int LAST = PA + PB - 2 < 2 ? PA + PB - 2 : 2;
#pragma unroll
    for (int k = 0; k < KS; ++k) {
        Parts<PA> a[NT];
        f4 sum[NT];
        clear(sum);
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int i = 0; i < PA; ++i) a[t].v[i] = *(const bf8 *)(at + 16 * t * pitch + i * plane + 32 * k);
#pragma unroll
        for (int q = LAST; q >= 0; --q)
#pragma unroll
            for (int i = 0; i < PA; ++i)
                if (q - i >= 0 && q - i < PB)
#pragma unroll
                    for (int t = 0; t < NT; ++t) sum[t] = mm32(a[t].v[i], own[k].v[q - i], sum[t]);
#pragma unroll
        for (int t = 0; t < NT; ++t) s[t] = k == 0 ? sum[t] : s[t] + sum[t];
    }
}

// four rows x 16 columns for every 16 lanes, transposed: lane li gets column li of rows 0 .. 3
__device__ __forceinline__ sh4 read_tr(const uint16_t *p)
{
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) sh4 *)p);
}

// operand A in tile order from 32 LDS rows: row of A = tile column c0 + li, k = tile rows
__device__ __forceinline__ bf8 read_columns(const uint16_t *tile, int pitch, int c0, int lane)
{
    const int li = lane & 15, g = lane >> 4;
    const uint16_t *at = tile + (4 * g + (li >> 2)) * pitch + c0 + 4 * (li & 3);
    const sh4 lo = read_tr(at), hi = read_tr(at + 16 * pitch);
    return __builtin_bit_cast(bf8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

// the same with k in row order (places 8 g + j)
__device__ __forceinline__ bf8 read_rows_tr(const uint16_t *tile, int pitch, int c0, int lane)
{
    const int li = lane & 15, g = lane >> 4;
    const uint16_t *at = tile + (8 * g + (li >> 2)) * pitch + c0 + 4 * (li & 3);
    const sh4 lo = read_tr(at), hi = read_tr(at + 4 * pitch);
    return __builtin_bit_cast(bf8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

// acc[h] += A B[h][k]: one operand A for H groups of rows
template <int H, int KS>
__device__ __forceinline__ void mm_rows(const Parts<3> &a, const Parts<3> (&b)[H][KS], int k, f4 *acc)
{
#pragma unroll
    for (int sum = 2; sum >= 0; --sum)
#pragma unroll
        for (int i = 0; i <= sum; ++i)
#pragma unroll
            for (int h = 0; h < H; ++h) acc[h] = mm32(a.v[i], b[h][k].v[sum - i], acc[h]);
}

// acc^T += (32 rows of the LDS tile)^T w: acc[ct] has rows 16 ct + 4 g + s, column li; w in tile order
template <int NT, int P>
__device__ __forceinline__ void add_parts(const uint16_t *tile, int plane, int pitch, const Parts<3> &w, f4 (&acc)[NT],
                                          int lane)
{
    constexpr int N = NT == 1 ? 1 : P == 3 ? 2 : 4;         // results at a time: the operands of N tiles in registers
    static_assert(NT % N == 0, "whole groups of tiles");
#pragma unroll
    for (int c = 0; c < NT; c += N) {
        Parts<P> a[N];
        f4 part[N];
#pragma unroll
        for (int t = 0; t < N; ++t) {
            part[t] = acc[c + t];
#pragma unroll
            for (int i = 0; i < P; ++i) a[t].v[i] = read_columns(tile + i * plane, pitch, 16 * (c + t), lane);
        }
        mm_parts(a, w, part);
#pragma unroll
        for (int t = 0; t < N; ++t) acc[c + t] = part[t];
    }
}

// The same where the tile holds an infinity or NaN: in fp32, without the pairs that are masked
// (0 * inf would carry a later token's value to an earlier row) and without parts (m * inf has either
// sign).  seen: bit k set when tile row k counts for this lane's own row.
template <int NT, int P>
__device__ __forceinline__ void add_parts_odd(const uint16_t *tile, int plane, int pitch, const float (&w8)[8],
                                              f4 (&acc)[NT], int lane, unsigned seen)
{
    const int li = lane & 15, g = lane >> 4;
#pragma unroll 1
    for (int row = 0; row < 32; ++row) {
        float own = w8[0];
#pragma unroll
        for (int k = 1; k < 8; ++k) own = (row & 3) + 4 * (row >> 4) == k ? w8[k] : own;
        const float wk = __shfl(own, li + 16 * ((row & 15) >> 2));
        if ((seen >> row) & 1u) {
#pragma unroll
            for (int ct = 0; ct < NT; ++ct)
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const uint16_t *at = tile + row * pitch + 16 * ct + 4 * g + k;
                    float v = bf16_to_f32(at[0]);
                    if (P == 3) v += bf16_to_f32(at[plane]) + bf16_to_f32(at[2 * plane]);   // (exact)
                    acc[ct][k] += wk * v;
                }
        }
    }
}

// ---- records after the scan ------------------------------------------------------------------
// Eight columns of a record's row on their way into LDS
struct RecordPiece {
    u4v h, m, l;
    // z: the record; row: of its rows (a pair of indices); c: first column; values: record_values
    __device__ __forceinline__ void load(const float *z, size_t values, int cp, int row, int c)
    {
        const float *at = z + (size_t)row * cp + c;
        h = *(const u4v *)at;
        m = *(const u4v *)(at + 4);
        l = *(const u4v *)(z + values + ((size_t)row * cp + c) / 2);
    }
    __device__ __forceinline__ void store(uint16_t *dst, int plane) const
    {
        *(u4v *)dst = h;
        *(u4v *)(dst + plane) = m;
        *(u4v *)(dst + 2 * plane) = l;
    }
    __device__ __forceinline__ void zero() { h = m = l = u4v{0u, 0u, 0u, 0u}; }
};

// four columns of a record's row in fp32
__device__ __forceinline__ f4 record_columns(const float *z, size_t values, int cp, int row, int c)
{
    const uint16_t *at = (const uint16_t *)(z + (size_t)row * cp + (c & ~7)) + (c & 7);
    const uint16_t *low = (const uint16_t *)(z + values) + (size_t)row * cp + c;
    return widen(*(const uint2 *)at) + (widen(*(const uint2 *)(at + 8)) + widen(*(const uint2 *)low));
}

// Whether a lane of the wave holds an infinity or NaN among its sums.  Values that are one show up here, as their
// parts multiply to NaN.
template <int N>
__device__ __forceinline__ float odd_probe(const f4 (&a)[N])
{
    float probe = 0.f;
#pragma unroll
    for (int k = 0; k < N; ++k)
#pragma unroll
        for (int s = 0; s < 4; ++s) probe = __builtin_fmaf(a[k][s], 0.f, probe);
    return probe;
}
template <int N>
__device__ __forceinline__ bool any_odd(const f4 (&a)[N]) { return __any(odd_probe(a) != 0.f); }
template <int M, int N>
__device__ __forceinline__ bool any_odd(const f4 (&a)[M][N])
{
    float probe = 0.f;
#pragma unroll
    for (int k = 0; k < M; ++k) probe += odd_probe(a[k]);
    return __any(probe != 0.f);
}

}  // namespace psf
#endif
