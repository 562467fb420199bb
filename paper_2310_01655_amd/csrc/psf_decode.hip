// Token-by-token evaluation of causal Polysketch attention (PolySketchFormer, arXiv 2310.01655):
// the recurrent form the paper points to when it notes that the state kept for generation does
// not grow with the context (Section 5).  One step consumes the (q, k, v) of position `pos` and
// returns row `pos` of the attention of Section 3, identical to what the block algorithm of
// Sections 3.1 / 3.2 with block size b returns for the sequence so far:
//   o = (phi'(q)^T Z + sum_{j in current block, j <= pos} w_j [v_j | 1]) -> N / (1 + S)
// where Z = sum over the *completed* blocks of phi'(k_j) [v_j | 1]^T is the prefix state Z_l of
// Section 3.1 and w_j = <q, k_j>^p (Section 3.2) or <m(q), m(k_j)>^2 (Section 3.1) inside the
// current block.  When a block completes, its keys are folded into Z.
//
// phi'(x) = m(x) (x) m(x) is symmetric in its two indices, so Z[a][b'] = Z[b'][a] and only the
// pairs a <= b' are kept, the off-diagonal ones doubled: S[a, b'] = Z[a][b'] + Z[b'][a] (b' > a),
// S[a, a] = Z[a][a]; then phi'(q)^T Z = sum_{a <= b'} m(q)[a] m(q)[b'] S[a, b'] -- the same
// numbers from Fs = mcols (mcols + 1) / 2 rows instead of mcols^2.  Pair (a, b') is row
// tri_row(a) + b' - a.
//
// State per (batch, head) unit, caller-owned:
//   ZV [Fs][dv] and ZD [Fs] in fp32: the value columns and the "ones" column of S, kept apart
//   so that rows of ZV are aligned and a step streams them with full-width loads;
//   for bf16 storage also ZH [Fs][dv], ZV rounded to bf16 at every fold: the steps read ZH;
//   then the current block's cache: CK [b][d] keys and CV [b][dv] values in the storage type
//   of the call (fp32 or bf16), CM [b][mcols] sketches m(k) in fp32.
// After the units come the scratch areas: m(q), m(k) of the new token [units][mcols] each and
// the partial sums of the state product [units][kSlices][dv + 1] (used when a unit's product is
// split over several workgroups).
// A step is bound by reading the state once (Fs * (dv * s + 4) bytes per unit, s = 2 with the
// bf16 copy, 4 without) and the cached keys and values of the current block.
#include <algorithm>
#include <type_traits>

#include "psf_internal.h"
#include "psf_f32.h"
#include "psf_lds.h"

namespace psf {
namespace {

constexpr int kThreads = 256;
constexpr int kSlices = 16;        // workgroups per unit in the state product (at most)
constexpr int kMaxPairsPerSlice = 4096;
static_assert((size_t)PSF_MAX_DIM * (PSF_MAX_DIM + 1) / 2 <= (size_t)kSlices * kMaxPairsPerSlice,
              "the largest state fits kSlices slices");

struct DecodeLayout {
    size_t zv, zd, zh, ck, cv, cm, per_unit; // float offsets inside one unit, floats per unit
    size_t mq, mk, part, total;              // float offsets of the scratch areas, total floats
    int shadow;                              // ZH present (see has_shadow)
    int slices;                              // workgroups per unit in the state product
};

// bf16 storage: the steps read a bf16 copy ZH of ZV (rounded once per fold from the fp32 master,
// as the forward kernels round their prefix states), half the bytes of a step.
bool has_shadow(const Problem &pb) { return pb.bf16 && pb.dv % 8 == 0 && pb.dv / 8 <= kThreads; }

// first row of the pairs (a, b' >= a) in the packed upper triangle of an m x m grid
__host__ __device__ inline long long tri_row(int a, int m) { return (long long)a * m - (long long)a * (a - 1) / 2; }
__host__ __device__ inline long long tri_count(int m) { return (long long)m * (m + 1) / 2; }

// the pair of packed row t: a = the largest row index with tri_row(a) <= t (closed form in
// fp32, then corrected by steps of one)
__device__ __forceinline__ void tri_pair(long long t, int m, int &a, int &bp)
{
    const float s = 2.f * m + 1.f;
    int aa = (int)((s - sqrtf(fmaxf(s * s - 8.f * (float)t, 0.f))) * 0.5f);
    aa = max(0, min(aa, m - 1));
    while (aa > 0 && tri_row(aa, m) > t) --aa;
    while (aa + 1 < m && tri_row(aa + 1, m) <= t) ++aa;
    a = aa;
    bp = aa + (int)(t - tri_row(aa, m));
}

DecodeLayout decode_layout(const Problem &pb)
{
    DecodeLayout L;
    auto up = [](size_t v) { return (v + 63) / 64 * 64; };            // 256-byte pieces
    const size_t Fs = (size_t)tri_count(pb.mcols);
    L.shadow = has_shadow(pb) ? 1 : 0;
    // rows per slice: enough for every thread to keep eight 16-byte loads in flight
    // A workgroup costs about a microsecond to start and wind up, as much as streaming a few
    // hundred kilobytes: as few slices as still give every CU about three workgroups, each
    // with at least 256 rows (eight 16-byte loads in flight per thread).
    // A slice's products m(q)[a] m(q)[b'] sit in LDS: at most kMaxPairsPerSlice of them.
    const size_t want = (768 + (size_t)pb.units - 1) / (size_t)pb.units, most = Fs / 256 > 0 ? Fs / 256 : 1;
    const size_t least = (Fs + kMaxPairsPerSlice - 1) / kMaxPairsPerSlice;
    L.slices = (int)(want < most ? want : most);
    if (L.slices < (int)least) L.slices = (int)least;
    if (L.slices > kSlices) L.slices = kSlices;
    L.zv = 0;
    L.zd = up(Fs * pb.dv);
    L.zh = L.zd + up(Fs);
    const size_t per_float = pb.bf16 ? 2 : 1;                         // cached keys / values keep the storage type
    L.ck = L.zh + up(L.shadow ? (Fs * pb.dv + 1) / 2 : 0);
    L.cv = L.ck + up(((size_t)pb.b * pb.d + per_float - 1) / per_float);
    L.cm = L.cv + up(((size_t)pb.b * pb.dv + per_float - 1) / per_float);
    L.per_unit = L.cm + up((size_t)pb.b * pb.mcols);
    L.mq = L.per_unit * pb.units;
    L.mk = L.mq + up((size_t)pb.units * pb.mcols);
    L.part = L.mk + up((size_t)pb.units * pb.mcols);
    L.total = L.part + up((size_t)pb.units * kSlices * (pb.dv + 1));
    return L;
}

__device__ __forceinline__ int pow2_at_least(int v, int lo, int hi)
{
    int p = lo;
    while (p < v && p < hi) p *= 2;
    return p;
}

__device__ __forceinline__ float4 load4_f(const float *p) { return *(const float4 *)p; }
__device__ __forceinline__ float4 load4_f(const bf16_t *p)
{
    const uint2 w = *(const uint2 *)p;
    return make_float4(__uint_as_float(w.x << 16), __uint_as_float(w.x & 0xffff0000u), __uint_as_float(w.y << 16),
                       __uint_as_float(w.y & 0xffff0000u));
}

// sixteen bytes of a state row as floats: four fp32 or eight bf16 columns
template <typename ZT> struct ZRow;
template <> struct ZRow<float> {
    static constexpr int NV = 4;
    float4 raw;
    __device__ __forceinline__ void load(const float *p) { raw = *(const float4 *)p; }
    __device__ __forceinline__ void zero() { raw = make_float4(0.f, 0.f, 0.f, 0.f); }
    __device__ __forceinline__ void fma(float ph, float *acc) const
    {
        acc[0] += ph * raw.x; acc[1] += ph * raw.y; acc[2] += ph * raw.z; acc[3] += ph * raw.w;
    }
    __device__ __forceinline__ float dot(const float *q) const
    {
        return q[0] * raw.x + q[1] * raw.y + q[2] * raw.z + q[3] * raw.w;
    }
};
template <> struct ZRow<bf16_t> {
    static constexpr int NV = 8;
    uint4 raw;
    __device__ __forceinline__ void load(const bf16_t *p) { raw = *(const uint4 *)p; }
    __device__ __forceinline__ void zero() { raw = make_uint4(0u, 0u, 0u, 0u); }
    __device__ __forceinline__ void fma(float ph, float *acc) const
    {
        const uint32_t w[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            acc[2 * i] += ph * __uint_as_float(w[i] << 16);
            acc[2 * i + 1] += ph * __uint_as_float(w[i] & 0xffff0000u);
        }
    }
    __device__ __forceinline__ float dot(const float *q) const
    {
        const uint32_t w[4] = {raw.x, raw.y, raw.z, raw.w};
        float sacc = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            sacc += q[2 * i] * __uint_as_float(w[i] << 16) + q[2 * i + 1] * __uint_as_float(w[i] & 0xffff0000u);
        return sacc;
    }
};

// sum of 256 floats in LDS by the first wave (call with every thread; result valid for tid 0)
__device__ __forceinline__ float sum256(const float *red)
{
    const int tid = threadIdx.x;
    float v = 0.f;
    if (tid < 64) {
        v = (red[tid] + red[tid + 64]) + (red[tid + 128] + red[tid + 192]);
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off);
    }
    return v;
}

// Sum over the nf rows of z [nf][dv] of phi[row] * z[row][.] into rowp[0 .. dv): NV columns per
// thread (16-byte loads), consecutive lane groups on consecutive rows so that a wave reads
// contiguous kilobytes, eight rows in flight per thread.  issue() starts the loads of the
// first eight rows of every thread -- they do not depend on the query, so the kernel calls it
// before anything else -- and finish() multiplies and goes on with the remaining rows.
// `scratch` (NV * kThreads floats) may alias phi: it is written only after every thread has
// finished reading phi.
template <typename ZT>
struct StateRows {
    static constexpr int NV = ZRow<ZT>::NV;
    const ZT *zc;
    int nf, dv, cp, grp, g;
    bool active, lane_on;
    ZRow<ZT> first[8];

    __device__ __forceinline__ void issue(const ZT *z, int nf_, int dv_)
    {
        const int tid = threadIdx.x, cn = dv_ / NV;
        nf = nf_;
        dv = dv_;
        cp = 1;
        while (cp < cn) cp *= 2;
        grp = kThreads / cp;
        g = tid / cp;
        lane_on = tid % cp < cn;
        zc = z + (tid % cp) * NV;
        active = true;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            first[i].zero();
            if (lane_on && g + i * grp < nf) first[i].load(zc + (size_t)(g + i * grp) * dv);
        }
    }

    __device__ __forceinline__ void finish(const float *phi, float *scratch, float *rowp)
    {
        const int tid = threadIdx.x;
        float s0[NV], s1[NV];
#pragma unroll
        for (int j = 0; j < NV; ++j) s0[j] = s1[j] = 0.f;
        if (lane_on) {
#pragma unroll
            for (int i = 0; i < 8; ++i)
                if (g + i * grp < nf) first[i].fma(phi[g + i * grp], (i & 1) ? s1 : s0);
            int ff = g + 8 * grp;
            for (; ff + 7 * grp < nf; ff += 8 * grp) {
                ZRow<ZT> zr[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) zr[i].load(zc + (size_t)(ff + i * grp) * dv);
#pragma unroll
                for (int i = 0; i < 8; ++i) zr[i].fma(phi[ff + i * grp], (i & 1) ? s1 : s0);
            }
            for (; ff < nf; ff += grp) {
                ZRow<ZT> zr;
                zr.load(zc + (size_t)ff * dv);
                zr.fma(phi[ff], s0);
            }
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < NV; ++j) scratch[NV * tid + j] = s0[j] + s1[j];
        __syncthreads();
        if (tid < dv) {
            const int cc = tid / NV, j = tid % NV;
            float sacc = 0.f;
            for (int q2 = 0; q2 < grp; ++q2) sacc += scratch[NV * (q2 * cp + cc) + j];
            rowp[tid] = sacc;
        }
    }
};

// In-block share of a slice: rowp[0 .. dv) += sum_j w_j v_j and rowp[dv] += sum_j w_j over the
// cached tokens j_beg .. j_end - 1, w_j = <qs, key_j>^pw.  A group of `lg` neighbouring lanes
// owns a cached row: lane li reads sixteen bytes of the key row, the group adds up the dot
// product with shuffles, and the same lane then weighs sixteen bytes of the value row -- no
// LDS between the two; four rows in flight per thread, the first four started by issue()
// before the query is known.  Needs wa % NK == 0, dv % NV == 0 and lg <= 64 (see
// cache_rows_group).
template <typename KT, typename VT>
struct CacheRows {
    static constexpr int NK = ZRow<KT>::NV, NV = ZRow<VT>::NV, U = 4;
    const KT *keys;
    const VT *vals;
    int wa, dv, j_beg, j_end, lg, li, g, rows_per_pass;
    ZRow<KT> k_first[U];
    ZRow<VT> v_first[U];

    __device__ __forceinline__ void load_rows(int j0, ZRow<KT> *kr, ZRow<VT> *vr) const
    {
#pragma unroll
        for (int i = 0; i < U; ++i) {
            const int row = j0 + i * rows_per_pass + g;
            kr[i].zero();
            vr[i].zero();
            if (row < j_end && li < wa / NK) kr[i].load(keys + (size_t)row * wa + li * NK);
            if (row < j_end && li < dv / NV) vr[i].load(vals + (size_t)row * dv + li * NV);
        }
    }

    __device__ __forceinline__ void issue(const KT *keys_, int wa_, const VT *vals_, int dv_, int j_beg_,
                                          int j_end_, int lg_)
    {
        const int tid = threadIdx.x;
        keys = keys_; vals = vals_; wa = wa_; dv = dv_; j_beg = j_beg_; j_end = j_end_; lg = lg_;
        li = tid % lg;
        g = tid / lg;
        rows_per_pass = kThreads / lg;
        load_rows(j_beg, k_first, v_first);
    }

    __device__ __forceinline__ void finish(const float *qs, int pw, float *scratch, float *red, float *rowp)
    {
        const int tid = threadIdx.x;
        float qreg[NK];
#pragma unroll
        for (int j = 0; j < NK; ++j) qreg[j] = li < wa / NK ? qs[li * NK + j] : 0.f;
        float acc[NV], wsum = 0.f;
#pragma unroll
        for (int j = 0; j < NV; ++j) acc[j] = 0.f;
        auto weigh = [&](int j0, const ZRow<KT> *kr, const ZRow<VT> *vr) {
#pragma unroll
            for (int i = 0; i < U; ++i) {
                float sdot = kr[i].dot(qreg);
                for (int off = 1; off < lg; off *= 2) sdot += __shfl_xor(sdot, off);
                float wv = 1.f;
                for (int e = 0; e < pw; ++e) wv *= sdot;
                if (j0 + i * rows_per_pass + g >= j_end) wv = 0.f;
                vr[i].fma(wv, acc);
                if (li == 0) wsum += wv;
            }
        };
        weigh(j_beg, k_first, v_first);
        // uniform bounds: every lane takes part in the shuffles
        for (int j0 = j_beg + U * rows_per_pass; j0 < j_end; j0 += U * rows_per_pass) {
            ZRow<KT> kr[U];
            ZRow<VT> vr[U];
            load_rows(j0, kr, vr);
            weigh(j0, kr, vr);
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < NV; ++j) scratch[NV * tid + j] = acc[j];
        red[tid] = wsum;
        __syncthreads();
        if (tid < dv) {
            const int cc = tid / NV, j = tid % NV;
            float sacc = 0.f;
            for (int q2 = 0; q2 < rows_per_pass; ++q2) sacc += scratch[NV * (q2 * lg + cc) + j];
            rowp[tid] += sacc;
        }
        const float tot = sum256(red);
        if (tid == 0) rowp[dv] += tot;
    }
};

// lane-group size for CacheRows, or 0 when the shapes do not fit it
__device__ __forceinline__ int cache_rows_group(int wa, int nk, int dv, int nv)
{
    if (wa % nk != 0 || dv % nv != 0) return 0;
    int lg = 1;
    while (lg < wa / nk || lg < dv / nv) lg *= 2;
    return lg <= 64 ? lg : 0;
}

// Zeroes `count` floats from p + first on, of every unit (blockIdx.y; units `stride` floats apart), and `rest_count`
// from p + rest on.  All offsets of the layout are multiples of 64 floats, and the state is 16-byte aligned at least.
__global__ __launch_bounds__(kThreads) void dec_zero_kernel(float *__restrict__ p, size_t first, size_t count,
                                                            size_t stride, size_t rest, size_t rest_count)
{
    float4 *const to = (float4 *)(p + first + blockIdx.y * stride), *const to2 = (float4 *)(p + rest);
    const size_t step = (size_t)gridDim.x * kThreads, i0 = (size_t)blockIdx.x * kThreads + threadIdx.x;
    for (size_t i = i0; i < count / 4; i += step) to[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    for (size_t i = blockIdx.y * step + i0; i < rest_count / 4; i += gridDim.y * step)
        to2[i] = make_float4(0.f, 0.f, 0.f, 0.f);
}

// part[u][s][c] = the share of slice s in row [N | S] of the new token:
//   cross-block: sum over the packed pairs f = (a, b') of the slice of m(q)[a] m(q)[b'] ZV[f][c]
//   (c < dv; read from the bf16 copy when SHADOW) and, at c = dv, of the same times ZD[f] (only
//   once a block is complete: have_state; F = the number of pairs); the products of the slice
//   sit in LDS;
//   in-block: the slice's share of the `slot` tokens cached since the last block boundary,
//   sum_j w_j [v_j | 1] with the weights of Section 3.2 (LE: keys in the storage type) or 3.1
//   (their fp32 sketches).  The new token itself is not in the cache yet: its own pair is added
//   by dec_finish_kernel.
// The first loads of both parts are issued before the query is read, so that a workgroup waits
// for memory once and not four times in a row.
// MODE 0: slices; dec_finish_kernel adds them up.  MODE 1 (one slice per unit): the workgroup
// has the whole row, so it also does what dec_finish_kernel does -- the new token's own pair,
// the division, the cache append.  MODE 2: it also computes m(q) and m(k) of the new token
// itself (Algorithm 1 with the matrices of the unit's head), and the step is one launch.
// MODE 3: slices as in MODE 0, but every slice sketches the token itself (slice 0 leaves the
// sketches in mq_out / mk_out for dec_finish_kernel): two launches instead of three.
// MODE 4: as MODE 3, but the slice that arrives last at its unit's counter adds the slices up, in
// their order, and does the rest as MODE 2: one launch.  The counter is the first word of the
// partial sums of slice kSlices - 1, which such a call does not have; psf_decode_reset clears
// it, and the last slice sets it back.  Measured against MODE 3 (us a step in the second block, bf16
// storage; r = 64: 1 unit, 8 slices, 16.6 and 20.1; 96 units, 8: 23.0 and 27.1; 192, 4: 28.7 and 31.8;
// 384, 2: 38.3 and 41.2; 700, 2: 68.8 and 69.2.  r = 128: 52 units, 15 slices, 48.9 and 55.8; 64, 12: 50.8 and
// 56.9; 128, 6: 76.5 and 81.0; 500, 3: 254.9 and 257.5; 384, 3 is the one point behind: 219.5 and 217.2).
// With 16 slices there is no room for a counter, and MODE 3 stays.
struct DecSketchArgs {
    const void *G;           // sketch matrices, storage type
    size_t g_len;            // entries per set
    int heads, per_head, r;
};

template <typename T, bool SHADOW, bool LE, int MODE>
__global__ __launch_bounds__(kThreads) void dec_state_kernel(const T *__restrict__ q, const T *__restrict__ k,
                                                             const T *__restrict__ v, float *__restrict__ state,
                                                             const float *__restrict__ mq_new,
                                                             const float *__restrict__ mk_new,
                                                             float *__restrict__ mq_out, float *__restrict__ mk_out,
                                                             float *__restrict__ part, T *__restrict__ o,
                                                             DecodeLayout L, int d, int dv, int p, int mcols,
                                                             long long F, int slot, int have_state,
                                                             DecSketchArgs sk)
{
    constexpr bool FUSE = MODE == 1 || MODE == 2 || MODE == 4, SK = MODE >= 2;
    static_assert(kThreads == kSketchThreads, "sketch_row_lds assumes this workgroup size");
    using ZT = std::conditional_t<SHADOW, bf16_t, float>;
    using KT = std::conditional_t<LE, T, float>;
    constexpr int kMaxPer = kMaxPairsPerSlice;             // decode_layout keeps a slice within this
    __shared__ float mq[PSF_MAX_DIM], qs[PSF_MAX_DIM], red[kThreads], w[kThreads], rowp[PSF_MAX_DIM + 1];
    __shared__ float xk[SK ? PSF_MAX_DIM : 1], mk_s[SK ? PSF_MAX_DIM : 1], xq[SK && !LE ? PSF_MAX_DIM : 1];
    __shared__ union {
        float phi[kMaxPer];          // products of the slice; later the scratch of the reductions
        SketchScratchN<2> sketch;    // before that (MODE 2): intermediates of Algorithm 1 for q and k
    } big;
    float *const phi = big.phi;
    const int u = blockIdx.y, sl = blockIdx.x, tid = threadIdx.x, kc = dv + 1;
    float *su = state + (size_t)u * L.per_unit;
    const int wa = LE ? d : mcols, slices = L.slices;
    // this slice's pairs and cached tokens
    const long long per = (F + slices - 1) / slices;
    const long long f_beg = sl * per;
    const int nf = have_state ? (int)max(0LL, min(F, f_beg + per) - f_beg) : 0;
    const int per_j = (slot + slices - 1) / slices;
    const int j_beg = min(slot, sl * per_j), j_end = min(slot, j_beg + per_j);
    const float *zv = su + L.zv + (size_t)f_beg * dv;
    const float *zd = su + L.zd + f_beg;
    const ZT *zrows = SHADOW ? (const ZT *)((const bf16_t *)(su + L.zh) + (size_t)f_beg * dv) : (const ZT *)zv;
    const KT *keys = LE ? (const KT *)(su + L.ck) : (const KT *)(su + L.cm);
    const T *cvals = (const T *)(su + L.cv);
    const bool zfast = dv % ZRow<ZT>::NV == 0 && dv / ZRow<ZT>::NV <= kThreads;
    const int lg = cache_rows_group(wa, ZRow<KT>::NV, dv, ZRow<T>::NV);

    // every load that does not depend on another one, oldest first (loads complete in order):
    // the query (mcols, wa <= 256: one element per thread), the ones column, the first state
    // rows, the first cached rows
    static_assert(PSF_MAX_DIM <= kThreads, "one query element per thread");
    float mq_reg = 0.f, qs_reg = 0.f, xq_reg = 0.f, xk_reg = 0.f;
    if constexpr (SK) {
        if (tid < d) {
            xq_reg = load_f(q, (size_t)u * d + tid);
            xk_reg = load_f(k, (size_t)u * d + tid);
        }
    } else {
        if (tid < mcols) mq_reg = mq_new[(size_t)u * mcols + tid];
        if (tid < wa) qs_reg = LE ? load_f(q, (size_t)u * d + tid) : mq_new[(size_t)u * mcols + tid];
    }
    const float zd0 = tid < nf ? zd[tid] : 0.f, zd1 = tid + kThreads < nf ? zd[tid + kThreads] : 0.f;
    StateRows<ZT> sr;
    CacheRows<KT, T> cr;
    if (zfast && nf > 0) sr.issue(zrows, nf, dv);
    if (lg > 0 && j_end > j_beg) cr.issue(keys, wa, cvals, dv, j_beg, j_end, lg);

    for (int c = tid; c < kc; c += kThreads) rowp[c] = 0.f;
    if constexpr (SK) {
        // raw rows into LDS (q in qs when the in-block weights use it, else in xq), then
        // Algorithm 1 for q and k together; the results leave the scratch before it is reused
        float *const xq_s = LE ? qs : xq;
        if (tid < d) {
            xq_s[tid] = xq_reg;
            xk[tid] = xk_reg;
        }
        __syncthreads();
        const T *g_set = (const T *)sk.G + (sk.per_head ? (size_t)(u % sk.heads) * sk.g_len : 0);
        const float *const rows[2] = {xq_s, xk};
        const float *fin[2];
        sketch_rows_lds<T, 2>(rows, g_set, d, sk.r, p, big.sketch, fin);
        if (tid < mcols) {
            mq[tid] = fin[0][tid];
            if (!LE) qs[tid] = fin[0][tid];
            mk_s[tid] = fin[1][tid];
            if constexpr (MODE == 3) {
                if (sl == 0) {                             // for dec_finish_kernel
                    mq_out[(size_t)u * mcols + tid] = fin[0][tid];
                    mk_out[(size_t)u * mcols + tid] = fin[1][tid];
                }
            }
        }
    } else {
        if (tid < mcols) mq[tid] = mq_reg;
        if (tid < wa) qs[tid] = qs_reg;
    }
    __syncthreads();
    const int dvp = pow2_at_least(dv, 32, kThreads), groups = kThreads / dvp;
    float *out = part + ((size_t)u * kSlices + sl) * kc;

    if (nf > 0) {
        for (int ff = tid; ff < nf; ff += kThreads) {
            int a, bp;
            tri_pair(f_beg + ff, mcols, a, bp);
            phi[ff] = mq[a] * mq[bp];
        }
        __syncthreads();
        // the ones column first: it reads phi, which StateRows::finish then reuses as scratch
        float a1c = 0.f;
        if (tid < nf) a1c = phi[tid] * zd0;
        if (tid + kThreads < nf) a1c += phi[tid + kThreads] * zd1;
        for (int ff = tid + 2 * kThreads; ff < nf; ff += kThreads) a1c += phi[ff] * zd[ff];
        red[tid] = a1c;
        if (zfast) {
            sr.finish(phi, phi, rowp);
        } else {
            for (int c0 = 0; c0 < dv; c0 += dvp) {
                const int c = c0 + tid % dvp, g = tid / dvp;
                float a0 = 0.f;
                if (c < dv)
                    for (int ff = g; ff < nf; ff += groups) a0 += phi[ff] * zv[(size_t)ff * dv + c];
                __syncthreads();
                w[tid] = a0;
                __syncthreads();
                if (tid < dvp && c0 + tid < dv) {
                    float sacc = 0.f;
                    for (int q2 = 0; q2 < groups; ++q2) sacc += w[q2 * dvp + tid];
                    rowp[c0 + tid] = sacc;
                }
            }
        }
        __syncthreads();                                    // red complete in either branch
        const float tot = sum256(red);
        if (tid == 0) rowp[dv] = tot;
    }

    // in-block: cached tokens j_beg .. j_end - 1 of this slice
    if (lg > 0) {
        if (j_end > j_beg) {
            __syncthreads();                               // phi (the scratch below) and red are free
            cr.finish(qs, LE ? p : 2, phi, red, rowp);
        }
    } else {
        for (int j0 = j_beg; j0 < j_end; j0 += kThreads) {
            const int nj = min(kThreads, j_end - j0);
            __syncthreads();
            // weights of the pass: four threads per key, 64 keys at a time
            for (int kk = 0; kk < nj; kk += kThreads / 4) {
                const int kj = kk + (tid >> 2), part4 = tid & 3;
                float sdot = 0.f;
                if (kj < nj) {
                    const size_t roff = (size_t)(j0 + kj) * wa;
                    for (int e = part4; e < wa; e += 4) sdot += qs[e] * load_f(keys, roff + e);
                }
                sdot += __shfl_xor(sdot, 1);
                sdot += __shfl_xor(sdot, 2);
                if (part4 == 0 && kj < nj) {
                    float wv = sdot * sdot;
                    if (LE) {
                        wv = 1.f;
                        for (int e = 0; e < p; ++e) wv *= sdot;
                    }
                    w[kj] = wv;
                }
            }
            __syncthreads();
            for (int c0 = 0; c0 < dv; c0 += dvp) {            // values: thread (c, g) takes slots g, g + groups, ...
                const int c = c0 + tid % dvp, g = tid / dvp;
                float a = 0.f;
                if (c < dv)
                    for (int jj = g; jj < nj; jj += groups) a += w[jj] * load_f(cvals, (size_t)(j0 + jj) * dv + c);
                __syncthreads();
                red[tid] = a;
                __syncthreads();
                if (tid < dvp && c0 + tid < dv) {
                    float sacc = 0.f;
                    for (int q2 = 0; q2 < groups; ++q2) sacc += red[q2 * dvp + tid];
                    rowp[c0 + tid] += sacc;
                }
            }
            if (tid == 0) {                                   // the "ones" column: sum of the weights
                float sacc = 0.f;
                for (int jj = 0; jj < nj; ++jj) sacc += w[jj];
                rowp[dv] += sacc;
            }
        }
    }
    __syncthreads();
    if constexpr (MODE == 4) {
        // The slices of a unit run on different dies, whose caches do not see each other's plain
        // writes: device-scope stores and loads, which go past those caches.  Every thread waits
        // until its stores have arrived before the workgroup counts itself in (a release fence
        // here would write back the whole cache of the die: 20 us a step instead of 17).  This
        // rests on the hardware and not on the language's memory model, whose way would be that
        // fence: a device-scope store is acknowledged (vmcnt) once it is where every die sees it, the
        // barrier puts all of the workgroup's acknowledgements before the count, and the loads of
        // the last slice are issued after the count has come back.
        for (int c = tid; c < kc; c += kThreads)
            __hip_atomic_store(out + c, rowp[c], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        int *const arrived = (int *)(part + ((size_t)u * kSlices + kSlices - 1) * kc);
        __shared__ int last;
        if (tid == 0)
            last = __hip_atomic_fetch_add(arrived, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == slices - 1;
        __syncthreads();
        if (!last) return;
        if (tid == 0) __hip_atomic_store(arrived, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        for (int c = tid; c < kc; c += kThreads) {
            const float *from = part + (size_t)u * kSlices * kc + c;
            float sum = 0.f;
            for (int q2 = 0; q2 < slices; ++q2)
                sum += __hip_atomic_load(from + (size_t)q2 * kc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            rowp[c] = sum;
        }
        __syncthreads();
    }
    if constexpr (!FUSE) {
        for (int c = tid; c < kc; c += kThreads) out[c] = rowp[c];
    } else {
        // own pair <q, k>^p (or <m(q), m(k)>^2), then N / (1 + S) and the cache append
        float k_own = 0.f;
        if constexpr (SK) {
            if (tid < wa) k_own = LE ? xk[tid] : mk_s[tid];
        } else {
            if (tid < wa) k_own = LE ? load_f(k, (size_t)u * d + tid) : mk_new[(size_t)u * mcols + tid];
        }
        red[tid] = tid < wa ? qs[tid] * k_own : 0.f;
        __syncthreads();
        const float sdot = sum256(red);
        if (tid == 0) {
            float wv = 1.f;
            for (int e = 0; e < (LE ? p : 2); ++e) wv *= sdot;
            w[0] = wv;
        }
        __syncthreads();
        const float w_self = w[0], den = 1.f + rowp[dv] + w_self;
        T *ckeys = (T *)(su + L.ck), *cv_out = (T *)(su + L.cv);
        for (int c = tid; c < dv; c += kThreads) {
            const T vraw = v[(size_t)u * dv + c];
            store_f(o, (size_t)u * dv + c, (rowp[c] + w_self * load_f(&vraw, 0)) / den);
            cv_out[(size_t)slot * dv + c] = vraw;
        }
        for (int e = tid; e < d; e += kThreads) ckeys[(size_t)slot * d + e] = k[(size_t)u * d + e];
        for (int e = tid; e < mcols; e += kThreads)
            su[L.cm + (size_t)slot * mcols + e] = SK ? mk_s[e] : mk_new[(size_t)u * mcols + e];
    }
}

// ---- the step of the common shapes --------------------------------------------------------------
// bf16 storage, degree 4 with Gaussian sketches, exact in-block weights, d = dv = D in {64, 128}, r = R in {32, 64}:
// what dec_state_kernel<bf16_t, true, true, 2 or 4> computes, from the same state, with the shape known.
// A step of few units is bound by its chain of waits, so the chain is short: every first load is issued at the
// start (matrices, rows, state, cache), the sketches are one 16 x 16 product per 16 columns with the rows
// q and k as rows of A (bf16 operands, exact products, fp32 sums), pairs (a, b') are found under the loads,
// state and cached rows add into the same registers, one sum over the lanes and one over the waves serve both,
// and one wave hands the slice over.
// A lane group of D / 8 lanes owns a state row or a cached row, 16 bytes a lane; the lane li of a group also holds
// the pair and the ones-column entry of the group's row li of a batch of eight.
template <int CTRL>
__device__ __forceinline__ float dpp(float v)
{
    return __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(v), CTRL, 0xf, 0xf, true));
}
// the sum over the lane's group of 8 or 16 lanes, the same in all of them
template <int LANES>
__device__ __forceinline__ float group_sum(float v)
{
    v += dpp<0xB1>(v);                                     // quad_perm 1 0 3 2
    v += dpp<0x4E>(v);                                     // quad_perm 2 3 0 1
    v += dpp<0x141>(v);                                    // row_half_mirror
    if constexpr (LANES == 16) v += dpp<0x140>(v);         // row_mirror
    return v;
}
// lane I of the lane's group of 8 or 16
template <int LANES, int I>
__device__ __forceinline__ float group_bcast(float v)
{
    const int w = (int)__float_as_uint(v);
    if constexpr (LANES == 16) return __uint_as_float(__builtin_amdgcn_update_dpp(0, w, 0x150 + I, 0xf, 0xf, true));
    const int lo = __builtin_amdgcn_update_dpp(0, w, 0x150 + I, 0xf, 0x3, true);
    return __uint_as_float(__builtin_amdgcn_update_dpp(lo, w, 0x158 + I, 0xf, 0xc, false));
}

template <int D, int R, bool ALONE>
__global__ __launch_bounds__(kThreads) void dec_step_kernel(const bf16_t *__restrict__ q, const bf16_t *__restrict__ k,
                                                            const bf16_t *__restrict__ v, float *__restrict__ state,
                                                            float *__restrict__ part, bf16_t *__restrict__ o,
                                                            DecodeLayout L, int slot, int have_state, DecSketchArgs sk)
{
    constexpr int CL = D / 8, NG = kThreads / CL, U = 8, UC = 4, F = R * (R + 1) / 2, NV = D / 64;
    constexpr int PITCH = R / 8;                           // 16-byte pieces of a matrix row
    constexpr int GP = D * PITCH / kThreads;               // pieces of one matrix per thread
    static_assert(D * PITCH % kThreads == 0, "whole pieces");
    typedef float f32x4v __attribute__((ext_vector_type(4)));
    __shared__ __attribute__((aligned(16))) bf16_t gl[2][D * R];
    __shared__ float mq[R], mk[R], sums[4][D], den_s[4];
    const int u = blockIdx.y, sl = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int li = tid % CL, grp = tid / CL, s16 = lane & 15, kc = D + 1;
    float *const su = state + (size_t)u * L.per_unit;
    const int slices = ALONE ? 1 : L.slices;
    const int per = ALONE ? F : (int)((unsigned)(F + slices - 1) / (unsigned)slices), f_beg = ALONE ? 0 : sl * per;
    const int nf = have_state ? max(0, min(F, f_beg + per) - f_beg) : 0;
    const int per_j = ALONE ? slot : (int)((unsigned)(slot + slices - 1) / (unsigned)slices);
    const int j_beg = ALONE ? 0 : min(slot, sl * per_j), j_end = ALONE ? slot : min(slot, j_beg + per_j);
    const bf16_t *const zh = (const bf16_t *)(su + L.zh) + (size_t)f_beg * D + 8 * li;
    const float *const zd = su + L.zd + f_beg;
    const bf16_t *const keys = (const bf16_t *)(su + L.ck) + 8 * li, *const vals = (const bf16_t *)(su + L.cv) + 8 * li;

    // loads, in the order in which they are needed
    const uint4 *const g = (const uint4 *)((const bf16_t *)sk.G + (sk.per_head ? (size_t)(u % sk.heads) * sk.g_len : 0));
    uint4 gv[2][GP];
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int i = 0; i < GP; ++i) gv[m][i] = g[m * (D * PITCH) + i * kThreads + tid];
    uint4 xf[D / 32];                                      // A operand: row 0 = q, row 1 = k, the others zero
#pragma unroll
    for (int s = 0; s < D / 32; ++s) {
        xf[s] = make_uint4(0u, 0u, 0u, 0u);
        if (s16 < 2) xf[s] = *(const uint4 *)&(s16 ? k : q)[(size_t)u * D + 32 * s + 8 * (lane >> 4)];
    }
    ZRow<bf16_t> qr, kr0;                                  // this lane's columns of q and k
    qr.load(q + (size_t)u * D + 8 * li);
    kr0.load(k + (size_t)u * D + 8 * li);
    struct Batch {
        ZRow<bf16_t> z[U];
        float zd;
        int pair;
    };
    auto load_batch = [&](int row0) {                      // rows row0 + grp + i NG
        Batch b;
#pragma unroll
        for (int i = 0; i < U; ++i) {
            const int row = row0 + grp + i * NG;
            b.z[i].zero();
            if (row < nf) b.z[i].load(zh + (size_t)row * D);
        }
        const int mine = row0 + grp + li * NG;             // (li < U where there is one: CL = 16 has twice the lanes)
        const bool on = li < U && mine < nf;
        b.zd = on ? zd[mine] : 0.f;
        // the pair (a, b') of the row: a in closed form, off by one at most
        const int t = on ? f_beg + mine : 0;
        const float sf = 2.f * R + 1.f;
        int a = (int)((sf - sqrtf(fmaxf(sf * sf - 8.f * (float)t, 0.f))) * 0.5f);
        a = max(0, min(a, R - 1));
        const int first = a * R - a * (a - 1) / 2;
        a += (first + R - a <= t) - (first > t);
        b.pair = on ? a | (a + t - (a * R - a * (a - 1) / 2)) << 8 : -1;
        return b;
    };
    Batch cur = load_batch(0);
    struct Cached {
        ZRow<bf16_t> key[UC], val[UC];
    };
    auto load_cached = [&](int j0) {
        Cached c;
#pragma unroll
        for (int i = 0; i < UC; ++i) {
            const int row = j0 + grp + i * NG;
            c.key[i].zero();
            c.val[i].zero();
            if (row < j_end) {
                c.key[i].load(keys + (size_t)row * D);
                c.val[i].load(vals + (size_t)row * D);
            }
        }
        return c;
    };
    Cached cc = load_cached(j_beg);

    // Algorithm 1.  Matrices into LDS as they lie, the pieces of a row swapped so that the transposed reads (4 rows,
    // two neighbouring pieces) meet different banks.
    auto swz = [](int e) { return R == 64 ? (e & 3) << 1 : e & 2; };
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int i = 0; i < GP; ++i) {
            const int idx = i * kThreads + tid, e = idx / PITCH;
            *(uint4 *)&gl[m][(e * PITCH + (idx % PITCH ^ swz(e))) * 8] = gv[m][i];
        }
    __syncthreads();
    if (16 * wave < R) {
        f32x4v acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
        for (int s = 0; s < D / 32; ++s)
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                const int e = 32 * s + 8 * (lane >> 4) + s16 / 4, c8 = 2 * wave + (s16 % 4) / 2;
                const bf16_t *const at = &gl[m][(e * PITCH + (c8 ^ swz(e))) * 8 + 4 * (s16 & 1)];
                acc[m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, xf[s]),
                                                                 read_turned(at, at + 4 * PITCH * 8), acc[m], 0, 0, 0);
            }
        if (lane < 16) {
            const float sc = sqrtf(1.0f / (float)R);
            mq[16 * wave + lane] = sc * (acc[0][0] * acc[1][0]);
            mk[16 * wave + lane] = sc * (acc[0][1] * acc[1][1]);
        }
    }
    // the cached rows need no sketch: they go between the sketches and the barrier
    float qreg[8], acc[8], den = 0.f;
#pragma unroll
    for (int j = 0; j < 8; ++j) qreg[j] = acc[j] = 0.f;
    qr.fma(1.f, qreg);
    float wsum = 0.f;
    auto weigh = [&](const Cached &c) {
#pragma unroll
        for (int i = 0; i < UC; ++i) {
            float w = group_sum<CL>(c.key[i].dot(qreg));   // rows past the end are zero, and so is their weight
            w *= w;
            w *= w;
            c.val[i].fma(w, acc);
            wsum += w;
        }
    };
    for (int j0 = j_beg; j0 < j_end; j0 += UC * NG) {
        const Cached now = cc;
        if (j0 + UC * NG < j_end) cc = load_cached(j0 + UC * NG);
        weigh(now);
    }
    if (li == 0) den = wsum;
    float w_self = group_sum<CL>(kr0.dot(qreg));
    w_self *= w_self;
    w_self *= w_self;
    __syncthreads();
    for (int row0 = 0; row0 < nf; row0 += U * NG) {
        const Batch now = cur;
        if (row0 + U * NG < nf) cur = load_batch(row0 + U * NG);
        const float phi = now.pair >= 0 ? mq[now.pair & 0xff] * mq[now.pair >> 8] : 0.f;
        den = fmaf(phi, now.zd, den);
        now.z[0].fma(group_bcast<CL, 0>(phi), acc);
        now.z[1].fma(group_bcast<CL, 1>(phi), acc);
        now.z[2].fma(group_bcast<CL, 2>(phi), acc);
        now.z[3].fma(group_bcast<CL, 3>(phi), acc);
        now.z[4].fma(group_bcast<CL, 4>(phi), acc);
        now.z[5].fma(group_bcast<CL, 5>(phi), acc);
        now.z[6].fma(group_bcast<CL, 6>(phi), acc);
        now.z[7].fma(group_bcast<CL, 7>(phi), acc);
    }

    // sum over the lane groups of the wave, halving the columns a lane holds; column 8 li + 4 h + 2 (odd 16) [+ lane / 8 % 2]
    auto halves = [&](float a, float b) {
        const auto r2 = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
        return __uint_as_float(r2[0]) + __uint_as_float(r2[1]);
    };
    auto quarters = [&](float a, float b) {
        const auto r2 = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
        return __uint_as_float(r2[0]) + __uint_as_float(r2[1]);
    };
    float c4[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) c4[j] = halves(acc[j], acc[j + 4]);
    const float c0 = quarters(c4[0], c4[2]), c1 = quarters(c4[1], c4[3]);
    const int col = 8 * li + 4 * (lane >> 5) + 2 * ((lane >> 4) & 1);
    if constexpr (CL == 8) {
        const bool up = lane & 8;
        sums[wave][col + (up ? 1 : 0)] = (up ? c1 : c0) + dpp<0x128>(up ? c0 : c1);      // row_ror 8
    } else {
        sums[wave][col] = c0;
        sums[wave][col + 1] = c1;
    }
    den = group_sum<16>(den);
    den += __shfl_xor(den, 16);
    den += __shfl_xor(den, 32);
    if (lane == 0) den_s[wave] = den;
    __syncthreads();
    if (wave > 0) {
        if (ALONE) {                                       // the cache takes the new token's sketch: see below
            if (wave == 1 && lane < R) su[L.cm + (size_t)slot * R + lane] = mk[lane];
        }
        return;
    }
    float row[NV], s = (den_s[0] + den_s[1]) + (den_s[2] + den_s[3]);
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int c = 64 * i + lane;
        row[i] = (sums[0][c] + sums[1][c]) + (sums[2][c] + sums[3][c]);
    }
    if constexpr (!ALONE) {
        // as in dec_state_kernel's MODE 4, by one wave: its stores are acknowledged before its first lane counts
        // the slice in, and the last slice's loads are issued after the count has come back
        float *const out = part + ((size_t)u * kSlices + sl) * kc;
#pragma unroll
        for (int i = 0; i < NV; ++i)
            __hip_atomic_store(out + 64 * i + lane, row[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (lane == 0) __hip_atomic_store(out + D, s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        int *const arrived = (int *)(part + ((size_t)u * kSlices + kSlices - 1) * kc);
        int before = 0;
        if (lane == 0) before = __hip_atomic_fetch_add(arrived, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        before = __builtin_amdgcn_readfirstlane(before);
        if (before != slices - 1) return;
        asm volatile("" ::: "memory");
        if (lane == 0) __hip_atomic_store(arrived, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const float *const from = part + (size_t)u * kSlices * kc;
        // all loads before the sums, which keep the order of the slices
        float got[kSlices - 1][NV], got_s[kSlices - 1];
#pragma unroll
        for (int q2 = 0; q2 < kSlices - 1; ++q2) {
            const float *const at = from + (size_t)min(q2, slices - 1) * kc;
            if (q2 < slices) {                             // (the same for the whole launch)
#pragma unroll
                for (int i = 0; i < NV; ++i)
                    got[q2][i] = __hip_atomic_load(at + 64 * i + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                got_s[q2] = __hip_atomic_load(at + D, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            } else {
#pragma unroll
                for (int i = 0; i < NV; ++i) got[q2][i] = 0.f;
                got_s[q2] = 0.f;
            }
        }
        s = 0.f;
#pragma unroll
        for (int i = 0; i < NV; ++i) row[i] = 0.f;
#pragma unroll
        for (int q2 = 0; q2 < kSlices - 1; ++q2) {
#pragma unroll
            for (int i = 0; i < NV; ++i) row[i] += got[q2][i];
            s += got_s[q2];
        }
    }
    // the new token's own pair, the division, and the token into the cache
    const float total = 1.f + s + w_self;
    bf16_t *const ckeys = (bf16_t *)(su + L.ck), *const cvals = (bf16_t *)(su + L.cv);
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int c = 64 * i + lane;
        const bf16_t vraw = v[(size_t)u * D + c];
        o[(size_t)u * D + c] = f32_to_bf16((row[i] + w_self * bf16_to_f32(vraw)) / total);
        cvals[(size_t)slot * D + c] = vraw;
        ckeys[(size_t)slot * D + c] = k[(size_t)u * D + c];
    }
    if (!ALONE && lane < R) su[L.cm + (size_t)slot * R + lane] = mk[lane];
}

// The new token's key, value and m(k) go into cache slot `slot`; row = sum of the slices + the
// new token's own pair; then N / (1 + S).
template <typename T>
__global__ __launch_bounds__(kThreads) void dec_finish_kernel(const T *__restrict__ q, const T *__restrict__ k,
                                                              const T *__restrict__ v,
                                                              float *__restrict__ state,
                                                              const float *__restrict__ mq_new,
                                                              const float *__restrict__ mk_new,
                                                              const float *__restrict__ part,
                                                              T *__restrict__ o, DecodeLayout L, int d,
                                                              int dv, int p, int mcols, int slot,
                                                              int local_exact)
{
    __shared__ float red[kThreads];
    __shared__ float w_self;
    const int u = blockIdx.x, tid = threadIdx.x, kc = dv + 1;
    float *su = state + (size_t)u * L.per_unit;
    T *ckeys = (T *)(su + L.ck), *cvals = (T *)(su + L.cv);
    for (int e = tid; e < d; e += kThreads) ckeys[(size_t)slot * d + e] = k[(size_t)u * d + e];
    for (int c = tid; c < dv; c += kThreads) cvals[(size_t)slot * dv + c] = v[(size_t)u * dv + c];
    for (int e = tid; e < mcols; e += kThreads) su[L.cm + (size_t)slot * mcols + e] = mk_new[(size_t)u * mcols + e];
    // own pair: <q, k>^p, or <m(q), m(k)>^2 with the sketched in-block rule
    const int wa = local_exact ? d : mcols;
    float a = 0.f;
    for (int e = tid; e < wa; e += kThreads)
        a += local_exact ? load_f(q, (size_t)u * d + e) * load_f(k, (size_t)u * d + e)
                         : mq_new[(size_t)u * mcols + e] * mk_new[(size_t)u * mcols + e];
    red[tid] = a;
    __syncthreads();
    const float sdot = sum256(red);
    if (tid == 0) {
        float wv = sdot * sdot;
        if (local_exact) {
            wv = 1.f;
            for (int e = 0; e < p; ++e) wv *= sdot;
        }
        w_self = wv;
    }
    __syncthreads();
    float den = 1.f + w_self;
    for (int sidx = 0; sidx < L.slices; ++sidx) den += part[((size_t)u * kSlices + sidx) * kc + dv];
    for (int c = tid; c < dv; c += kThreads) {
        float acc = w_self * load_f(v, (size_t)u * dv + c);
        for (int sidx = 0; sidx < L.slices; ++sidx) acc += part[((size_t)u * kSlices + sidx) * kc + c];
        store_f(o, (size_t)u * dv + c, acc / den);
    }
}

// ZV[f][c] += sum over the b cached tokens of w_f m_j[a] m_j[b'] v_j[c] for the packed pair
// f = (a, b'), w_f = 2 off the diagonal and 1 on it; ZD[f] += the same without v.
// Workgroup = kFoldFeat pairs; thread (c, g) owns the PER = kFoldFeat / groups pairs
// g * PER .. of column c (groups = 256 / columns per pass).
constexpr int kFoldFeat = 64, kFoldTok = 32;
template <typename T, int PER>
__global__ __launch_bounds__(kThreads) void dec_fold_kernel(float *__restrict__ state, DecodeLayout L,
                                                            int dv, int b, int mcols, long long F)
{
    __shared__ float phi[kFoldTok][kFoldFeat + 1], vt[kFoldTok][PSF_MAX_DIM], pair_w[kFoldFeat];
    __shared__ int pair_a[kFoldFeat], pair_b[kFoldFeat];
    constexpr int groups = kFoldFeat / PER, dvp = kThreads / groups;
    const int tid = threadIdx.x, u = blockIdx.y;
    const long long f0 = (long long)blockIdx.x * kFoldFeat;
    float *su = state + (size_t)u * L.per_unit;
    if (tid < kFoldFeat) {
        int a = 0, bp = 0;
        if (f0 + tid < F) tri_pair(f0 + tid, mcols, a, bp);
        pair_a[tid] = a;
        pair_b[tid] = bp;
        pair_w[tid] = f0 + tid < F ? (bp > a ? 2.f : 1.f) : 0.f;
    }
    for (int c0 = 0; c0 < dv; c0 += dvp) {
        const int c = c0 + tid % dvp, g = tid / dvp;
        float acc[PER];
#pragma unroll
        for (int ff = 0; ff < PER; ++ff) acc[ff] = 0.f;
        float dacc = 0.f;                                 // ZD: thread tid < kFoldFeat owns feature tid
        for (int j0 = 0; j0 < b; j0 += kFoldTok) {
            const int lim = min(kFoldTok, b - j0);
            __syncthreads();
            for (int idx = tid; idx < kFoldTok * kFoldFeat; idx += kThreads) {
                const int jj = idx / kFoldFeat, ff = idx % kFoldFeat;
                float v = 0.f;
                if (jj < lim) {
                    const float *m = su + L.cm + (size_t)(j0 + jj) * mcols;
                    v = pair_w[ff] * m[pair_a[ff]] * m[pair_b[ff]];
                }
                phi[jj][ff] = v;
            }
            for (int idx = tid; idx < kFoldTok * dv; idx += kThreads) {
                const int jj = idx / dv, cc = idx % dv;
                vt[jj][cc] = jj < lim ? load_f((const T *)(su + L.cv), (size_t)(j0 + jj) * dv + cc) : 0.f;
            }
            __syncthreads();
            if (c < dv)
                for (int jj = 0; jj < kFoldTok; ++jj) {
                    const float vv = vt[jj][c];
#pragma unroll
                    for (int ff = 0; ff < PER; ++ff) acc[ff] += phi[jj][g * PER + ff] * vv;
                }
            if (c0 == 0 && tid < kFoldFeat)
                for (int jj = 0; jj < kFoldTok; ++jj) dacc += phi[jj][tid];
        }
        if (c < dv) {
#pragma unroll
            for (int ff = 0; ff < PER; ++ff)
                if (f0 + g * PER + ff < F) {
                    const size_t at = (size_t)(f0 + g * PER + ff) * dv + c;
                    const float znew = su[L.zv + at] + acc[ff];
                    su[L.zv + at] = znew;
                    if (L.shadow) ((bf16_t *)(su + L.zh))[at] = f32_to_bf16(znew);
                }
        }
        if (c0 == 0 && tid < kFoldFeat && f0 + tid < F) su[L.zd + f0 + tid] += dacc;
    }
}

// The same fold on MFMA for bf16 storage (phi'(k) and v as bf16 operands, fp32 accumulation, as
// the forward state kernel does): S[a, b'][c] += w sum_j (m_j[a] m_j[b']) v_j[c] for b' >= a.
// Workgroup = (NA consecutive sketch rows a, unit).  An item is (row a, 32-wide range of b'):
// the fragment m_j[a] m_j[b'] generated for it feeds one MFMA per 32-wide tile of value columns.
// Ranges whose columns b' all lie below the group's first row are skipped; the remaining items
// are dealt evenly to the four waves, a wave's items sharing one range (and with it the
// fragments of m_j[b'] and of v).  64 tokens at a time are staged transposed ([column][token])
// so that a lane's eight tokens of one column are neighbours.
//
// Bound by LDS reads, the vector work of the fragments and, with few tokens, the state's own traffic (us, 768
// units of r = d = 64, 1024 tokens: 812 -> 618, 256: 383 -> 367; 96 of d = 128, 512 tokens: 423 -> 101; 768 of r = 32,
// 1024, 256 and 48 tokens: 204 -> 197, 86.5 -> 87.5, 61 -> 64: a chunk alone takes no advantage of the second buffer
// and waits a little longer for its rows): single values stored column by column met 4-way bank conflicts, and branches on
// a wave's number of rows and on the end of the tokens kept loads and products in order.
// `count` tokens of unit u come from msrc + u m_unit (fp32 sketches) and vsrc + u v_unit (values): the
// unit's block cache, or a prompt's sketches and its values in place.  slices > 1: each slice of the
// tokens leaves its sums in part [unit][slice][pairs (dv + 1)] and dec_fold_sum_kernel adds them to the
// state; slices = 1: they are added here.
typedef __bf16 dec_bf16x8 __attribute__((ext_vector_type(8)));
typedef float dec_f32x16 __attribute__((ext_vector_type(16)));
constexpr int kFoldMfmaTok = 64, kFoldMfmaMaxM = 64, kFoldMfmaMaxDv = 128;

template <int MC, int DV>
struct FoldShape {
    static constexpr int NB = MC / 32, TC = DV / 32;
    static constexpr int IPW = 8 / TC < 4 ? 8 / TC : 4;      // items per wave, at most (accumulators: IPW * TC tiles)
    static constexpr int NA = 4 * IPW / NB;                  // sketch rows per workgroup
};

template <int MC, int DV>
__global__ __launch_bounds__(kThreads, 2) void dec_fold_mfma_kernel(float *state, DecodeLayout L, int count,
                                                                    const float *msrc, size_t m_unit,
                                                                    const bf16_t *vsrc, size_t v_unit,
                                                                    float *part, int slices)
{
    constexpr int mcols = MC, dv = DV;
    constexpr int NB = FoldShape<MC, DV>::NB, TC = FoldShape<MC, DV>::TC, IPW = FoldShape<MC, DV>::IPW;
    constexpr int NA = FoldShape<MC, DV>::NA;
    // rows of 64 tokens: pitches of 68 floats / 72 bf16 keep every 16-byte read aligned and spread
    // the 16 lanes of a read phase over all banks
    constexpr int TOK = kFoldMfmaTok, PITCH = TOK + 4, PITCHV = TOK + 8;
    __shared__ __attribute__((aligned(16))) float mts2[2][MC][PITCH];
    __shared__ __attribute__((aligned(16))) bf16_t vts2[2][DV][PITCHV];
    // The MC / NA workgroups of a unit's slice all stream the same tokens.  Consecutive workgroup
    // ids go to different XCDs, so give each XCD a contiguous range of (unit, row group) pairs:
    // the groups of a unit then share one L2 and run at about the same time.
    constexpr int GROUPS = MC / NA;
    int wg = blockIdx.x;
    if ((gridDim.x & 7) == 0) wg = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
    int u = wg / GROUPS, slice = 0;
    const int a0 = (wg % GROUPS) * NA;
    if (slices > 1) {
        slice = u % slices;
        u /= slices;
    }
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int x = lane & 31, h = lane >> 5;
    float *su = state + (size_t)u * L.per_unit;
    int first = 0, last = count;
    if (slices > 1) {                                       // chunks * slices < 2^30
        const unsigned chunks = (count + TOK - 1) / TOK;
        first = (int)(chunks * slice / slices) * TOK;
        last = min(count, (int)(chunks * (slice + 1) / slices) * TOK);
    }
    // this wave's items: rows a0 + row0 .. + rpw - 1 of range bt
    const int bt_min = a0 / 32, nb_act = NB - bt_min;
    const int rpw = NA * nb_act / 4;                         // 1 .. IPW
    const int bt = bt_min + (wave * rpw) / NA, row0 = (wave * rpw) % NA;
    dec_f32x16 acc[IPW][TC];
    float drow[IPW];
#pragma unroll
    for (int k = 0; k < IPW; ++k) {
        drow[k] = 0.f;
#pragma unroll
        for (int ct = 0; ct < TC; ++ct)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[k][ct][v] = 0.f;
    }
    // A chunk of 64 tokens goes global -> registers -> LDS, transposed on the way: a thread takes four
    // columns of four tokens (neighbouring threads neighbouring columns: whole rows) and stores four tokens
    // of a column at once.  Token quads (m) and octets (v) of column c lie at their number ^ (c / 16) % 4, which
    // keeps the stores' lanes, 16 columns apart in their banks' pattern, off each other.  The loads of the
    // next chunk are in flight while this one is multiplied; two buffers, one barrier a chunk.
    constexpr int MBLK = TOK / 4 * (MC / 4), VBLK = TOK / 4 * (DV / 4);
    constexpr int MP = (MBLK + kThreads - 1) / kThreads, VP = (VBLK + kThreads - 1) / kThreads;
    float4 m_pre[MP][4];
    uint2 v_pre[VP][4];
    const float *cm = msrc + (size_t)u * m_unit;
    const bf16_t *cvv = vsrc + (size_t)u * v_unit;
    // Past the end the last token is loaded again and put() writes zeros over it: loads behind a branch, or
    // registers changed behind one, made the compiler wait for them before the products.
    auto fetch = [&](int j0) {
#pragma unroll
        for (int i = 0; i < MP; ++i) {
            const int idx = min(tid + i * kThreads, MBLK - 1), tb = idx / (MC / 4), c4 = idx % (MC / 4);
#pragma unroll
            for (int t = 0; t < 4; ++t)
                m_pre[i][t] = *(const float4 *)(cm + (size_t)(unsigned)min(j0 + 4 * tb + t, last - 1) * MC + 4 * c4);
        }
#pragma unroll
        for (int i = 0; i < VP; ++i) {
            const int idx = min(tid + i * kThreads, VBLK - 1), tb = idx / (DV / 4), c4 = idx % (DV / 4);
#pragma unroll
            for (int t = 0; t < 4; ++t)
                v_pre[i][t] = *(const uint2 *)(cvv + (size_t)(unsigned)min(j0 + 4 * tb + t, last - 1) * DV + 4 * c4);
        }
    };
    auto put = [&](int buf, int j0) {
#pragma unroll
        for (int i = 0; i < MP; ++i) {
            const int idx = tid + i * kThreads, tb = idx / (MC / 4), c4 = idx % (MC / 4);
            if (MBLK % kThreads == 0 || idx < MBLK) {
                const float4 *m4 = m_pre[i];
                float(*to)[PITCH] = &mts2[buf][4 * c4];
                const int at = 4 * (tb ^ (c4 / 4 % 4));
                *(float4 *)&to[0][at] = make_float4(m4[0].x, m4[1].x, m4[2].x, m4[3].x);
                *(float4 *)&to[1][at] = make_float4(m4[0].y, m4[1].y, m4[2].y, m4[3].y);
                *(float4 *)&to[2][at] = make_float4(m4[0].z, m4[1].z, m4[2].z, m4[3].z);
                *(float4 *)&to[3][at] = make_float4(m4[0].w, m4[1].w, m4[2].w, m4[3].w);
                if (j0 + TOK > last)                        // the same for the workgroup
                    for (int t = max(0, last - j0 - 4 * tb); t < 4; ++t)
                        to[0][at + t] = to[1][at + t] = to[2][at + t] = to[3][at + t] = 0.f;
            }
        }
#pragma unroll
        for (int i = 0; i < VP; ++i) {
            const int idx = tid + i * kThreads, tb = idx / (DV / 4), c4 = idx % (DV / 4);
            if (VBLK % kThreads == 0 || idx < VBLK) {
                const uint2 *v4 = v_pre[i];
                bf16_t(*to)[PITCHV] = &vts2[buf][4 * c4];
                const int at = 8 * (tb / 2 ^ (c4 / 4 % 4)) + 4 * (tb % 2);
                auto low = [](uint32_t p, uint32_t q) { return (p & 0xffffu) | (q << 16); };
                auto high = [](uint32_t p, uint32_t q) { return (p >> 16) | (q & 0xffff0000u); };
                *(uint2 *)&to[0][at] = make_uint2(low(v4[0].x, v4[1].x), low(v4[2].x, v4[3].x));
                *(uint2 *)&to[1][at] = make_uint2(high(v4[0].x, v4[1].x), high(v4[2].x, v4[3].x));
                *(uint2 *)&to[2][at] = make_uint2(low(v4[0].y, v4[1].y), low(v4[2].y, v4[3].y));
                *(uint2 *)&to[3][at] = make_uint2(high(v4[0].y, v4[1].y), high(v4[2].y, v4[3].y));
                if (j0 + TOK > last)
                    for (int t = max(0, last - j0 - 4 * tb); t < 4; ++t)
                        to[0][at + t] = to[1][at + t] = to[2][at + t] = to[3][at + t] = 0;
            }
        }
    };
    const int quad_b = 4 * ((2 * bt + x / 16) % 4);
    // items: the wave's rows, a constant so that no branch lies between an item's products and the next
    // item's operands
    auto multiply = [&](auto items, int buf) {
        constexpr int ITEMS = decltype(items)::value;
        const auto &mts = mts2[buf];
        const auto &vts = vts2[buf];
        float dchunk[ITEMS];                                // the ones column, a chunk at a time: shorter sums
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) dchunk[k] = 0.f;
#pragma unroll 2                                            // (all four: spills)
        for (int sstep = 0; sstep < TOK / 16; ++sstep) {
            const int tok = 16 * sstep + 8 * h;
            const float *mcol = mts[32 * bt + x];
            const float4 mb0 = *(const float4 *)&mcol[tok ^ quad_b], mb1 = *(const float4 *)&mcol[(tok + 4) ^ quad_b];
            const float mb[8] = {mb0.x, mb0.y, mb0.z, mb0.w, mb1.x, mb1.y, mb1.z, mb1.w};
            dec_bf16x8 fb[TC];
#pragma unroll
            for (int ct = 0; ct < TC; ++ct) fb[ct] = *(const dec_bf16x8 *)&vts[32 * ct + x][tok ^ (8 * ((2 * ct + x / 16) % 4))];
#pragma unroll
            for (int k = 0; k < ITEMS; ++k) {
                const int a = a0 + row0 + k;
                const int quad_a = 4 * (a / 16 % 4);
                const float4 ma0 = *(const float4 *)&mts[a][tok ^ quad_a], ma1 = *(const float4 *)&mts[a][(tok + 4) ^ quad_a];
                const float ma[8] = {ma0.x, ma0.y, ma0.z, ma0.w, ma1.x, ma1.y, ma1.z, ma1.w};
                dec_bf16x8 fa;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float pr = ma[e] * mb[e];
                    fa[e] = (__bf16)pr;
                    dchunk[k] += pr;
                }
#pragma unroll
                for (int ct = 0; ct < TC; ++ct)
                    acc[k][ct] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa, fb[ct], acc[k][ct], 0, 0, 0);
            }
        }
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) drow[k] += dchunk[k];
    };
    auto walk = [&](auto items) {
        fetch(first);
        for (int j0 = first, buf = 0; j0 < last; j0 += TOK, buf ^= 1) {
            put(buf, j0);
            __syncthreads();
            fetch(j0 + TOK);
            multiply(items, buf);
        }
    };
    if (rpw == IPW)
        walk(std::integral_constant<int, IPW>{});
    else if constexpr (NB > 1)
        walk(std::integral_constant<int, IPW / 2>{});
#pragma unroll
    for (int k = 0; k < IPW; ++k) {
        if (k >= rpw) break;
        const int a = a0 + row0 + k;
        const size_t rowbase = (size_t)tri_row(a, mcols);
        if (slices > 1) {
            float *const pu = part + ((size_t)u * slices + slice) * tri_count(mcols) * (dv + 1);
#pragma unroll
            for (int ct = 0; ct < TC; ++ct)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int bp = 32 * bt + 8 * (v / 4) + 4 * h + (v % 4);
                    if (bp >= a) pu[(rowbase + bp - a) * dv + 32 * ct + x] = (bp > a ? 2.f : 1.f) * acc[k][ct][v];
                }
            const float tot = drow[k] + __shfl_xor(drow[k], 32);
            const int bp = 32 * bt + x;
            if (h == 0 && bp >= a) pu[(size_t)tri_count(mcols) * dv + rowbase + bp - a] = (bp > a ? 2.f : 1.f) * tot;
            continue;
        }
        // accumulator: lane x = column c, register v = row b' = 8 (v / 4) + 4 h + v % 4.  All rows
        // are read before the first is written: the reads and writes go to one array, so that in
        // one loop every read would wait for the write before it (768 units of r = d = 64:
        // 1240 -> 840 to 885 us).
        float old[TC][16];
#pragma unroll
        for (int ct = 0; ct < TC; ++ct)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int bp = max(a, 32 * bt + 8 * (v / 4) + 4 * h + (v % 4));
                old[ct][v] = su[L.zv + (rowbase + bp - a) * dv + 32 * ct + x];
            }
#pragma unroll
        for (int ct = 0; ct < TC; ++ct) {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int bp = 32 * bt + 8 * (v / 4) + 4 * h + (v % 4);
                if (bp >= a) {
                    const size_t at = (rowbase + bp - a) * dv + 32 * ct + x;
                    const float znew = old[ct][v] + (bp > a ? 2.f : 1.f) * acc[k][ct][v];
                    su[L.zv + at] = znew;
                    if (L.shadow) ((bf16_t *)(su + L.zh))[at] = f32_to_bf16(znew);
                }
            }
        }
        // the "ones" column: lanes x = row b', both halves
        const float tot = drow[k] + __shfl_xor(drow[k], 32);
        const int bp = 32 * bt + x;
        if (h == 0 && bp >= a) su[L.zd + rowbase + bp - a] += (bp > a ? 2.f : 1.f) * tot;
    }
}

// The slices' sums of dec_fold_mfma_kernel are added to the state, in their order: ZV (and its bf16 copy),
// then ZD, one value a thread.
__global__ __launch_bounds__(kThreads) void dec_fold_sum_kernel(float *__restrict__ state, DecodeLayout L,
                                                                const float *__restrict__ part, int slices,
                                                                int pairs, int dv)
{
    const int i = blockIdx.x * kThreads + threadIdx.x, total = pairs * (dv + 1);
    if (i >= total) return;
    const int u = blockIdx.y;
    float *su = state + (size_t)u * L.per_unit;
    const float *from = part + (size_t)u * slices * total + i;
    const bool value = i < pairs * dv;
    const size_t at = value ? L.zv + i : L.zd + (i - pairs * dv);
    float sum = su[at];
    for (int q = 0; q < slices; ++q) sum += from[(size_t)q * total];
    su[at] = sum;
    if (value && L.shadow) ((bf16_t *)(su + L.zh))[i] = f32_to_bf16(sum);
}

// Prompt tokens pos0 + j (j < count) of every unit go into cache slots j: keys and values as
// they are, m(k) from Algorithm 1 (two tokens at a time share the matrices) or, HAVE_M, from
// the rows M_all [units][n_prompt][mcols] computed beforehand (learned sketches).
constexpr int kPrefillTokens = 8;
template <typename T, bool HAVE_M>
__global__ __launch_bounds__(kThreads) void dec_prefill_kernel(const T *__restrict__ K, const T *__restrict__ V,
                                                               const float *__restrict__ M_all,
                                                               float *__restrict__ state, DecodeLayout L, int d,
                                                               int dv, int p, int mcols, int n_prompt, int pos0,
                                                               int count, int m_first, int m_rows, DecSketchArgs sk)
{
    // M_all: [units][m_rows][mcols], the sketches of prompt rows m_first .. m_first + m_rows - 1
    static_assert(kThreads == kSketchThreads, "sketch_rows_lds assumes this workgroup size");
    __shared__ float xs[2][PSF_MAX_DIM];
    __shared__ SketchScratchN<HAVE_M ? 1 : 2> scratch;
    const int u = blockIdx.y, tid = threadIdx.x;
    float *su = state + (size_t)u * L.per_unit;
    T *ckeys = (T *)(su + L.ck), *cvals = (T *)(su + L.cv);
    const T *g_set = (const T *)sk.G + (sk.per_head ? (size_t)(u % sk.heads) * sk.g_len : 0);
    // kPrefillTokens tokens per workgroup, two at a time (a workgroup per pair would spend most
    // of its time starting up)
    for (int j0 = kPrefillTokens * blockIdx.x; j0 < min(count, kPrefillTokens * ((int)blockIdx.x + 1)); j0 += 2) {
        const int nrow = min(2, count - j0);
        for (int i = 0; i < nrow; ++i) {
            const size_t row = (size_t)u * n_prompt + pos0 + j0 + i;
            for (int e = tid; e < d; e += kThreads) ckeys[(size_t)(j0 + i) * d + e] = K[row * d + e];
            for (int c = tid; c < dv; c += kThreads) cvals[(size_t)(j0 + i) * dv + c] = V[row * dv + c];
            if (HAVE_M)
                for (int e = tid; e < mcols; e += kThreads)
                    su[L.cm + (size_t)(j0 + i) * mcols + e] =
                        M_all[((size_t)u * m_rows + (pos0 + j0 + i - m_first)) * mcols + e];
        }
        if constexpr (!HAVE_M) {
            __syncthreads();                               // the previous pair's results have been read
#pragma unroll
            for (int i = 0; i < 2; ++i)
                if (tid < d) xs[i][tid] = i < nrow ? load_f(K, ((size_t)u * n_prompt + pos0 + j0 + i) * d + tid) : 0.f;
            __syncthreads();
            const float *const rows[2] = {xs[0], xs[1]};
            const float *fin[2];
            sketch_rows_lds<T, 2>(rows, g_set, d, sk.r, p, scratch, fin);
            for (int i = 0; i < nrow; ++i)
                if (tid < mcols) su[L.cm + (size_t)(j0 + i) * mcols + tid] = fin[i][tid];
        }
    }
}

// Keys and values of prompt tokens pos0 .. pos0 + count - 1 into cache slots 0 .. count - 1, where
// m(k) comes from elsewhere.  Rows of a unit are contiguous on both sides; PIECE elements at a
// time (16 bytes where sizes and alignment allow it).
template <typename T, int PIECE>
__global__ __launch_bounds__(kThreads) void dec_cache_rows_kernel(const T *__restrict__ K, const T *__restrict__ V,
                                                                  float *__restrict__ state, DecodeLayout L, int d,
                                                                  int dv, int n_prompt, int pos0, int count)
{
    struct __attribute__((aligned(sizeof(T) * PIECE))) Piece { T v[PIECE]; };
    const int u = blockIdx.y;
    float *su = state + (size_t)u * L.per_unit;
    const size_t i = ((size_t)blockIdx.x * kThreads + threadIdx.x) * PIECE, row0 = (size_t)u * n_prompt + pos0;
    if (i < (size_t)count * d) *(Piece *)((T *)(su + L.ck) + i) = *(const Piece *)(K + row0 * d + i);
    if (i < (size_t)count * dv) *(Piece *)((T *)(su + L.cv) + i) = *(const Piece *)(V + row0 * dv + i);
}

// The state after the complete blocks of a prompt, taken from the forward path's state kernel:
// Zg [units][a][b'/8][c][8] bf16 holds sum_j phi'(k_j) v_j^T with this file's convention already
// applied (b' > a doubled, b' < a zero); Spart [units][parts][r][r] fp32 the partial m^T m.
// ZV (and its bf16 copy) take the pairs a <= b' of Zg, ZD the weighted sums of the partials: the first
// zd_groups workgroups of a unit, the longest chains of loads.  Bound by memory.
__global__ __launch_bounds__(kThreads) void dec_import_state_kernel(const bf16_t *__restrict__ Zg,
                                                                    const float *__restrict__ Spart,
                                                                    float *__restrict__ state, DecodeLayout L,
                                                                    int dv, int mcols, int pairs, int parts,
                                                                    int zd_groups)
{
    const int u = blockIdx.y;
    float *su = state + (size_t)u * L.per_unit;
    if ((int)blockIdx.x < zd_groups) {
        const int idx = blockIdx.x * kThreads + threadIdx.x;
        if (idx >= pairs) return;
        int a, bp;
        tri_pair(idx, mcols, a, bp);
        const float *sp = Spart + (size_t)u * parts * mcols * mcols + (size_t)a * mcols + bp;
        float sacc = 0.f;
#pragma unroll 8
        for (int q2 = 0; q2 < parts; ++q2) sacc += sp[(size_t)q2 * mcols * mcols];
        su[L.zd + idx] = (bp > a ? 2.f : 1.f) * sacc;
        return;
    }
    // Four 16-byte pieces of Zg per thread: row a, eight columns b' = 8 o .., value columns 4 c4 .. (consecutive
    // threads: consecutive c4, so reads and the stores of a row are contiguous).  dv is 64 or 128 here.
    const int idx = (blockIdx.x - zd_groups) * kThreads + threadIdx.x, cq = dv / 4;
    const int c4 = idx % cq, o = idx / cq % (mcols / 8), a = idx / cq / (mcols / 8);
    if (a >= mcols || 8 * o + 7 < a) return;
    const uint4 *from = (const uint4 *)(Zg + (size_t)u * mcols * mcols * dv) + (size_t)idx * 4;
    uint4 raw[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) raw[c] = from[c];
    const size_t row0 = (size_t)tri_row(a, mcols);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int bp = 8 * o + e;
        if (bp < a) continue;
        uint32_t bits[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const uint32_t wds[4] = {raw[c].x, raw[c].y, raw[c].z, raw[c].w};
            bits[c] = (e & 1) ? wds[e / 2] >> 16 : wds[e / 2] & 0xffffu;
        }
        const size_t at = (row0 + bp - a) * dv + 4 * c4;
        *(float4 *)&su[L.zv + at] = make_float4(bf16_to_f32((bf16_t)bits[0]), bf16_to_f32((bf16_t)bits[1]),
                                                bf16_to_f32((bf16_t)bits[2]), bf16_to_f32((bf16_t)bits[3]));
        if (L.shadow) *(uint2 *)&((bf16_t *)(su + L.zh))[at] = make_uint2(bits[0] | bits[1] << 16, bits[2] | bits[3] << 16);
    }
}

// 16-byte copies of rows first .. first + rows - 1 of every unit out of [units][n_prompt][w] (bf16)
// into [units][rows][w]
__global__ __launch_bounds__(kThreads) void dec_gather_rows_kernel(const bf16_t *__restrict__ src,
                                                                   bf16_t *__restrict__ dst, int w, int n_prompt,
                                                                   int first, int rows, size_t pieces)
{
    const size_t i = (size_t)blockIdx.x * kThreads + threadIdx.x;       // piece of 8 elements
    if (i >= pieces) return;
    const size_t per_unit = (size_t)rows * w / 8;
    const size_t u = i / per_unit, r8 = i % per_unit;
    *(uint4 *)(dst + i * 8) = *(const uint4 *)(src + (u * n_prompt + first) * w + r8 * 8);
}

// Shapes of dec_fold_mfma_kernel.
bool fold_on_mfma(const Problem &pb)
{
    return pb.bf16 && pb.mcols % 32 == 0 && pb.mcols <= kFoldMfmaMaxM && pb.dv % 32 == 0 && pb.dv <= kFoldMfmaMaxDv;
}

// Sketch rows a per workgroup of that kernel.
int fold_rows(const Problem &pb)
{
    const int tc = pb.dv / 32, nb = pb.mcols / 32, ipw = 8 / tc < 4 ? 8 / tc : 4;
    return 4 * ipw / nb;
}

psf_status launch_fold_mfma(const Problem &pb, const DecodeLayout &L, float *state, int count, const float *m,
                            size_t m_unit, const bf16_t *v, size_t v_unit, float *part, int slices, hipStream_t s)
{
    const dim3 grid((unsigned)(pb.mcols / fold_rows(pb) * pb.units * slices));
#define PSF_FOLD(MC_, DV_)                                                                                       \
    if (pb.mcols == MC_ && pb.dv == DV_) {                                                                        \
        static_assert(FoldShape<MC_, DV_>::NA * FoldShape<MC_, DV_>::NB == 4 * FoldShape<MC_, DV_>::IPW, "");     \
        hipLaunchKernelGGL((dec_fold_mfma_kernel<MC_, DV_>), grid, dim3(kThreads), 0, s, state, L, count, m,      \
                           m_unit, v, v_unit, part, slices);                                                      \
    }
    PSF_FOLD(32, 32) PSF_FOLD(32, 64) PSF_FOLD(32, 96) PSF_FOLD(32, 128)
    PSF_FOLD(64, 32) PSF_FOLD(64, 64) PSF_FOLD(64, 96) PSF_FOLD(64, 128)
#undef PSF_FOLD
    PSF_LAUNCH_CHECK();
    if (slices > 1) {
        const int pairs = (int)tri_count(pb.mcols), total = pairs * (pb.dv + 1);
        hipLaunchKernelGGL(dec_fold_sum_kernel, dim3((unsigned)((total + kThreads - 1) / kThreads), (unsigned)pb.units),
                           dim3(kThreads), 0, s, state, L, part, slices, pairs, pb.dv);
        PSF_LAUNCH_CHECK();
    }
    return PSF_OK;
}

// Folds the b tokens in the block cache into the state (the block is complete).
template <typename T>
psf_status launch_fold(const Problem &pb, const DecodeLayout &L, float *state, hipStream_t s)
{
    if (fold_on_mfma(pb))
        return launch_fold_mfma(pb, L, state, pb.b, state + L.cm, L.per_unit, (const bf16_t *)(state + L.cv),
                                2 * L.per_unit, nullptr, 1, s);
    const long long Fs = tri_count(pb.mcols);
    const dim3 fgrid((unsigned)((Fs + kFoldFeat - 1) / kFoldFeat), (unsigned)pb.units);
    if (pb.dv <= 32)
        hipLaunchKernelGGL((dec_fold_kernel<T, 8>), fgrid, dim3(kThreads), 0, s, state, L, pb.dv, pb.b, pb.mcols, Fs);
    else if (pb.dv <= 64)
        hipLaunchKernelGGL((dec_fold_kernel<T, 16>), fgrid, dim3(kThreads), 0, s, state, L, pb.dv, pb.b, pb.mcols, Fs);
    else if (pb.dv <= 128)
        hipLaunchKernelGGL((dec_fold_kernel<T, 32>), fgrid, dim3(kThreads), 0, s, state, L, pb.dv, pb.b, pb.mcols, Fs);
    else
        hipLaunchKernelGGL((dec_fold_kernel<T, 64>), fgrid, dim3(kThreads), 0, s, state, L, pb.dv, pb.b, pb.mcols, Fs);
    PSF_LAUNCH_CHECK();
    return PSF_OK;
}

template <typename T>
psf_status step_launch(const Problem &pb, const void *q, const void *k, const void *v, const void *G, int pos,
                       float *state, void *o, hipStream_t s)
{
    const DecodeLayout L = decode_layout(pb);
    const int slot = pos % pb.b, le = pb.local_exact ? 1 : 0;
    // one workgroup per unit: it finishes the row itself, and with the sketch of Algorithm 1
    // (no networks) it also sketches the new token
    const bool fuse = L.slices == 1;
    // learned sketches come from the general sketch kernel (modes 0, 1); those of Algorithm 1 are
    // computed inside the step kernel (modes 2 to 4)
    const int mode = pb.learned ? (fuse ? 1 : 0) : fuse ? 2 : L.slices == kSlices ? 3 : 4;
    if (mode < 2) {
        // sketches of the new token: the general sketch kernel on [units, 1, d]
        Problem one = pb;
        one.n = 1;
        psf_status st = general_sketch_pair_f32(one, q, k, G, state + L.mq, state + L.mk, s);   // one launch for both
        if (st != PSF_OK) return st;
    }
    const int have_state = pos >= pb.b ? 1 : 0;          // Z is zero during the first block
    const long long Fs = tri_count(pb.mcols);
    const dim3 sgrid((unsigned)L.slices, (unsigned)pb.units);
    const DecSketchArgs ska{G, pb.g_len, pb.heads, pb.per_head ? 1 : 0, pb.r};
    // the shapes dec_step_kernel knows; it reads rows and matrices 16 bytes at a time
    bool known = false;
    if constexpr (std::is_same_v<T, bf16_t>) {
        const bool aligned = (((uintptr_t)q | (uintptr_t)k | (uintptr_t)G) & 15) == 0;
        auto launch = [&](auto d_tag, auto r_tag) {
            constexpr int D = decltype(d_tag)::value, R = decltype(r_tag)::value;
            if (mode == 2)
                hipLaunchKernelGGL((dec_step_kernel<D, R, true>), sgrid, dim3(kThreads), 0, s, (const T *)q, (const T *)k,
                                   (const T *)v, state, state + L.part, (T *)o, L, slot, have_state, ska);
            else
                hipLaunchKernelGGL((dec_step_kernel<D, R, false>), sgrid, dim3(kThreads), 0, s, (const T *)q, (const T *)k,
                                   (const T *)v, state, state + L.part, (T *)o, L, slot, have_state, ska);
        };
        known = (mode == 2 || mode == 4) && pb.p == 4 && le && aligned && pb.d == pb.dv && (pb.d == 64 || pb.d == 128) &&
                (pb.r == 32 || pb.r == 64);
        using std::integral_constant;
        if (known && pb.d == 64 && pb.r == 64) launch(integral_constant<int, 64>{}, integral_constant<int, 64>{});
        else if (known && pb.d == 64) launch(integral_constant<int, 64>{}, integral_constant<int, 32>{});
        else if (known && pb.r == 64) launch(integral_constant<int, 128>{}, integral_constant<int, 64>{});
        else if (known) launch(integral_constant<int, 128>{}, integral_constant<int, 32>{});
    }
#define PSF_DEC_STATE(SH, LE_, MO)                                                                             \
    hipLaunchKernelGGL((dec_state_kernel<T, SH, LE_, MO>), sgrid, dim3(kThreads), 0, s, (const T *)q,             \
                       (const T *)k, (const T *)v, state, state + L.mq, state + L.mk, state + L.mq, state + L.mk, \
                       state + L.part, (T *)o, L, pb.d, pb.dv, pb.p, pb.mcols, Fs, slot, have_state, ska)
#define PSF_DEC_STATE_MODE(SH, LE_)      \
    do {                                 \
        if (mode == 0)                   \
            PSF_DEC_STATE(SH, LE_, 0);   \
        else if (mode == 1)              \
            PSF_DEC_STATE(SH, LE_, 1);   \
        else if (mode == 2)              \
            PSF_DEC_STATE(SH, LE_, 2);   \
        else if (mode == 3)              \
            PSF_DEC_STATE(SH, LE_, 3);   \
        else                             \
            PSF_DEC_STATE(SH, LE_, 4);   \
    } while (0)
    if (known) {
    } else if (L.shadow) {
        if constexpr (std::is_same_v<T, bf16_t>) {
            if (le) PSF_DEC_STATE_MODE(true, true); else PSF_DEC_STATE_MODE(true, false);
        }
    } else {
        if (le) PSF_DEC_STATE_MODE(false, true); else PSF_DEC_STATE_MODE(false, false);
    }
#undef PSF_DEC_STATE_MODE
#undef PSF_DEC_STATE
    PSF_LAUNCH_CHECK();
    if (mode == 0 || mode == 3) {                         // the slices are added up here
        hipLaunchKernelGGL(dec_finish_kernel<T>, dim3((unsigned)pb.units), dim3(kThreads), 0, s, (const T *)q,
                           (const T *)k, (const T *)v, state, state + L.mq, state + L.mk, state + L.part, (T *)o, L,
                           pb.d, pb.dv, pb.p, pb.mcols, slot, le);
        PSF_LAUNCH_CHECK();
    }
    if (slot == pb.b - 1) return launch_fold<T>(pb, L, state, s);   // the block is complete: fold it into Z
    return PSF_OK;
}

}  // namespace

bool decode_supported(const Problem &pb) { return !pb.exact_feat; }

size_t decode_state_bytes(const Problem &pb) { return decode_layout(pb).total * sizeof(float); }

// Zeroes the state; prefix = false: all but ZV, ZD and ZH, which dec_import_state_kernel writes whole (768
// units of r = d = 64, b = 1024: 0.39 of 1.02 GB).
static psf_status zero_state(const Problem &pb, float *state, bool prefix, hipStream_t s)
{
    const DecodeLayout L = decode_layout(pb);
    if (prefix) {
        hipLaunchKernelGGL(dec_zero_kernel, dim3(2048), dim3(kThreads), 0, s, state, (size_t)0, L.total, (size_t)0,
                           (size_t)0, (size_t)0);
        PSF_LAUNCH_CHECK();
        return PSF_OK;
    }
    const size_t cache = L.per_unit - L.ck;
    const unsigned grid = (unsigned)std::max<size_t>(1, std::min<size_t>(2048 / (size_t)pb.units, cache / 4 / kThreads));
    hipLaunchKernelGGL(dec_zero_kernel, dim3(grid, (unsigned)pb.units), dim3(kThreads), 0, s, state, L.ck, cache,
                       L.per_unit, L.mq, L.total - L.mq);
    PSF_LAUNCH_CHECK();
    return PSF_OK;
}

psf_status decode_reset(const Problem &pb, void *state, hipStream_t s)
{
    return zero_state(pb, (float *)state, true, s);
}

// The complete blocks of a prompt go through the forward path's kernels where those exist
// (bf16, the MFMA shapes, sketches of Algorithm 1): their total state is imported, and only the
// tokens after the last block boundary are written into the cache one block at a time.
static int prefill_fast_tokens(const Problem &pb, int n_prompt)
{
    const int n_full = n_prompt / pb.b * pb.b;
    return n_full > 0 && pb.mcols % 8 == 0 && mfma_total_state_supported(pb, n_full) ? n_full : 0;
}

// Complete blocks that the forward kernels do not take (blocks whose tokens are no multiple of 256, p = 2)
// go into the state together where the fold runs on MFMA: a state does not depend on where the blocks
// ended, and a fold reads and writes the whole state, 0.8 MB a unit, for what may be 48 tokens.  Sketches
// of up to kFoldRoom bytes at a time, their values in place.  A chunk holds at least one block, or the
// prompt goes block by block as before; so does one whose caller has no workspace, or values at odd addresses.
// Few units: the tokens are cut into slices (of 256 and more, until every CU has two workgroups) with sums
// of their own.  (Prompt and twelve steps, us, block by block and together: 288 units of r = 64, 5000
// tokens in blocks of 200: 4801, 1457; 12 of r = 32, 3000 in blocks of 48: 2105, 214; 36 of d = 128 and degree 8, 2000
// in blocks of 300: 1985, 611; 48 with p = 2, 3000 in blocks of 512: 516, 339.)
constexpr size_t kFoldRoom = (size_t)1 << 30;
constexpr int kFoldSlices = 16, kFoldWorkgroups = 512, kFoldSliceTokens = 256;

// Workspace of a hand-over, in this order: the fp32 sketches of the prompt keys that go through
// the cache (learned sketches only: all of them, or those after the last block boundary when
// the forward kernels take the complete blocks), a contiguous copy of those keys (same case),
// room for contiguous copies of the complete blocks of K and V (when a tail follows them; only
// learned sketches still make these copies, the size the query returns is the same for both), the
// forward kernels' own buffers; or, where those take nothing, the sketches of a chunk and the slices' sums.
struct PrefillPlan {
    int n_full, m_rows;                   // tokens through the forward kernels; sketched rows per unit
    int fold_tokens, fold_slices;         // tokens of a chunk that is folded at once (0: block by block)
    size_t m_bytes, ktail_bytes, copy_bytes, fold_m_bytes;
    size_t least, total;                  // what the call cannot do without; what it asks for
};

static PrefillPlan prefill_plan(const Problem &pb, int n_prompt)
{
    PrefillPlan pl = {};
    const bool learned = pb.learned && pb.p > 2;
    pl.n_full = prefill_fast_tokens(pb, n_prompt);
    const int tail = n_prompt - pl.n_full;
    pl.m_rows = learned ? tail : 0;
    pl.m_bytes = align_up((size_t)pb.units * pl.m_rows * pb.mcols * sizeof(float), 256);
    pl.ktail_bytes = learned && pl.n_full > 0 ? align_up((size_t)pb.units * tail * pb.d * 2, 256) : 0;
    pl.copy_bytes = pl.n_full > 0 && tail > 0 ? align_up((size_t)pb.units * pl.n_full * pb.d * 2, 256) : 0;
    pl.least = pl.total = pl.m_bytes + pl.ktail_bytes + 2 * pl.copy_bytes +
                          (pl.n_full > 0 ? mfma_total_state_workspace_bytes(pb, pl.n_full) : 0);
    const int blocks = n_prompt / pb.b * pb.b;
    if (pl.n_full > 0 || blocks == 0 || !fold_on_mfma(pb) || !(learned || f32_supported(pb))) return pl;
    const size_t row = (size_t)pb.units * pb.mcols * sizeof(float);
    size_t tokens = (size_t)blocks;
    if (!learned && tokens * row > kFoldRoom) tokens = kFoldRoom / row / kFoldMfmaTok * kFoldMfmaTok;
    if (tokens < (size_t)pb.b) return pl;
    pl.fold_tokens = (int)tokens;
    const int groups = pb.mcols / fold_rows(pb);
    const long long fill = kFoldWorkgroups / ((long long)pb.units * groups);
    pl.fold_slices = (int)std::max<long long>(1, std::min<long long>({fill, kFoldSlices, pl.fold_tokens / kFoldSliceTokens}));
    pl.fold_m_bytes = learned ? 0 : align_up(tokens * row, 256);
    pl.total += pl.fold_m_bytes;
    if (pl.fold_slices > 1)
        pl.total += align_up((size_t)pb.units * pl.fold_slices * tri_count(pb.mcols) * (pb.dv + 1) * sizeof(float), 256);
    return pl;
}

size_t decode_prefill_workspace_bytes(const Problem &pb, int n_prompt) { return prefill_plan(pb, n_prompt).total; }

size_t decode_prefill_least_bytes(const Problem &pb, int n_prompt) { return prefill_plan(pb, n_prompt).least; }

bool decode_prefill_uses_mfma(const Problem &pb, int n_prompt) { return prefill_fast_tokens(pb, n_prompt) > 0; }

template <typename T>
static psf_status prefill_launch(const Problem &pb, const void *K, const void *V, const void *G, int n_prompt,
                                 float *state, void *ws, size_t ws_bytes, hipStream_t s)
{
    const DecodeLayout L = decode_layout(pb);
    const PrefillPlan pl = prefill_plan(pb, n_prompt);
    psf_status st = zero_state(pb, state, pl.n_full == 0, s);
    if (st != PSF_OK) return st;
    const int first = pl.n_full, tail = n_prompt - first;  // prompt tokens before `first` go through the forward kernels
    float *m_tail = (float *)ws;
    char *ktail = (char *)ws + pl.m_bytes, *wsp = ktail + pl.ktail_bytes;
    if constexpr (std::is_same_v<T, bf16_t>) {
        if (first > 0) {
            const bf16_t *kc = (const bf16_t *)K, *vc = (const bf16_t *)V;
            int src_n = n_prompt;
            if (tail > 0 && pb.learned) {                  // the learned sketch kernel takes contiguous rows
                const size_t pieces = (size_t)pb.units * first * pb.d / 8;
                const unsigned grid = (unsigned)((pieces + kThreads - 1) / kThreads);
                hipLaunchKernelGGL(dec_gather_rows_kernel, dim3(grid), dim3(kThreads), 0, s, (const bf16_t *)K,
                                   (bf16_t *)wsp, pb.d, n_prompt, 0, first, pieces);
                PSF_LAUNCH_CHECK();
                hipLaunchKernelGGL(dec_gather_rows_kernel, dim3(grid), dim3(kThreads), 0, s, (const bf16_t *)V,
                                   (bf16_t *)(wsp + pl.copy_bytes), pb.dv, n_prompt, 0, first, pieces);
                PSF_LAUNCH_CHECK();
                kc = (const bf16_t *)wsp;
                vc = (const bf16_t *)(wsp + pl.copy_bytes);
                src_n = first;
            }
            const void *zg = nullptr;
            const float *spart = nullptr;
            int parts = 0;
            st = mfma_total_state(pb, first, src_n, kc, vc, G, wsp + 2 * pl.copy_bytes, s, &zg, &spart, &parts);
            if (st != PSF_OK) return st;
            const int pairs = (int)tri_count(pb.mcols), threads = pb.mcols * (pb.mcols / 8) * (pb.dv / 4);
            const int zd_groups = (pairs + kThreads - 1) / kThreads;
            const dim3 grid((unsigned)(zd_groups + (threads + kThreads - 1) / kThreads), (unsigned)pb.units);
            hipLaunchKernelGGL(dec_import_state_kernel, grid, dim3(kThreads), 0, s, (const bf16_t *)zg, spart, state, L,
                               pb.dv, pb.mcols, pairs, parts, zd_groups);
            PSF_LAUNCH_CHECK();
        }
    }
    const bool have_m = pl.m_rows > 0;
    if (have_m) {
        // learned sketches of the rows that go through the cache: rows first .. n_prompt - 1 of every unit
        const void *krows = K;
        if constexpr (std::is_same_v<T, bf16_t>) {
            if (first > 0) {
                const size_t pieces = (size_t)pb.units * tail * pb.d / 8;
                hipLaunchKernelGGL(dec_gather_rows_kernel, dim3((unsigned)((pieces + kThreads - 1) / kThreads)),
                                   dim3(kThreads), 0, s, (const bf16_t *)K, (bf16_t *)ktail, pb.d, n_prompt, first, tail,
                                   pieces);
                PSF_LAUNCH_CHECK();
                krows = ktail;
            }
        }
        Problem part = pb;
        part.n = tail;
        st = general_sketch_f32(part, krows, G, m_tail, s);
        if (st != PSF_OK) return st;
    }
    const DecSketchArgs ska{G, pb.g_len, pb.heads, pb.per_head ? 1 : 0, pb.r};
    int cached = first;                                    // tokens before this one are in the state
    if constexpr (std::is_same_v<T, bf16_t>) {
        if (pl.fold_tokens > 0 && ws_bytes >= pl.total && (pl.total == 0 || (ws && ((uintptr_t)ws & 255u) == 0)) &&
            ((uintptr_t)V & 7u) == 0) {
            const int blocks = n_prompt / pb.b * pb.b;
            float *const m = (float *)wsp, *const part = (float *)(wsp + pl.fold_m_bytes);
            for (int c0 = 0; c0 < blocks; c0 += pl.fold_tokens) {
                const int count = std::min(pl.fold_tokens, blocks - c0);
                if (!have_m) {
                    Problem chunk = pb;
                    chunk.n = count;
                    st = f32_sketch_rows(chunk, (const T *)K + (size_t)c0 * pb.d, (size_t)n_prompt * pb.d, G, m,
                                         (size_t)pl.fold_tokens * pb.mcols, s);
                    if (st != PSF_OK) return st;
                }
                const int slices = std::min(pl.fold_slices, (count + kFoldMfmaTok - 1) / kFoldMfmaTok);
                st = launch_fold_mfma(pb, L, state, count, have_m ? m_tail + (size_t)c0 * pb.mcols : m,
                                      (size_t)(have_m ? pl.m_rows : pl.fold_tokens) * pb.mcols,
                                      (const bf16_t *)V + (size_t)c0 * pb.dv, (size_t)n_prompt * pb.dv, part, slices, s);
                if (st != PSF_OK) return st;
            }
            cached = blocks;
        }
    }
    for (int pos0 = cached; pos0 < n_prompt; pos0 += pb.b) {
        const int count = n_prompt - pos0 < pb.b ? n_prompt - pos0 : pb.b;
        const dim3 grid((unsigned)((count + kPrefillTokens - 1) / kPrefillTokens), (unsigned)pb.units);
        if (!have_m && f32_supported(pb)) {
            // sketches on the fp32 matrix cores, straight into the cache (768 units x 1012 tokens of
            // d = r = 64: 310 us and 78 for the rows, against 1690 by two rows a workgroup)
            Problem part = pb;
            part.n = count;
            st = f32_sketch_rows(part, (const T *)K + (size_t)pos0 * pb.d, (size_t)n_prompt * pb.d, G, state + L.cm,
                                 L.per_unit, s);
            if (st != PSF_OK) return st;
            constexpr int kWide = 16 / sizeof(T);
            const bool wide = pb.d % kWide == 0 && pb.dv % kWide == 0 && (((uintptr_t)K | (uintptr_t)V) & 15u) == 0;
            const size_t pieces = (size_t)count * (pb.d > pb.dv ? pb.d : pb.dv) / (wide ? kWide : 1);
            const dim3 cgrid((unsigned)((pieces + kThreads - 1) / kThreads), (unsigned)pb.units);
            if (wide)
                hipLaunchKernelGGL((dec_cache_rows_kernel<T, kWide>), cgrid, dim3(kThreads), 0, s, (const T *)K,
                                   (const T *)V, state, L, pb.d, pb.dv, n_prompt, pos0, count);
            else
                hipLaunchKernelGGL((dec_cache_rows_kernel<T, 1>), cgrid, dim3(kThreads), 0, s, (const T *)K,
                                   (const T *)V, state, L, pb.d, pb.dv, n_prompt, pos0, count);
        } else if (have_m)
            hipLaunchKernelGGL((dec_prefill_kernel<T, true>), grid, dim3(kThreads), 0, s, (const T *)K, (const T *)V,
                               (const float *)m_tail, state, L, pb.d, pb.dv, pb.p, pb.mcols, n_prompt, pos0, count,
                               first, tail, ska);
        else
            hipLaunchKernelGGL((dec_prefill_kernel<T, false>), grid, dim3(kThreads), 0, s, (const T *)K, (const T *)V,
                               (const float *)nullptr, state, L, pb.d, pb.dv, pb.p, pb.mcols, n_prompt, pos0, count,
                               first, tail, ska);
        PSF_LAUNCH_CHECK();
        if (count == pb.b) {
            st = launch_fold<T>(pb, L, state, s);
            if (st != PSF_OK) return st;
        }
    }
    return PSF_OK;
}

psf_status decode_prefill(const Problem &pb, const void *K, const void *V, const void *G, int n_prompt, void *state,
                          void *ws, size_t ws_bytes, hipStream_t s)
{
    return pb.bf16 ? prefill_launch<bf16_t>(pb, K, V, G, n_prompt, (float *)state, ws, ws_bytes, s)
                   : prefill_launch<float>(pb, K, V, G, n_prompt, (float *)state, ws, ws_bytes, s);
}

psf_status decode_step(const Problem &pb, const void *q, const void *k, const void *v, const void *G, int pos,
                       void *state, void *o, hipStream_t s)
{
    return pb.bf16 ? step_launch<bf16_t>(pb, q, k, v, G, pos, (float *)state, o, s)
                   : step_launch<float>(pb, q, k, v, G, pos, (float *)state, o, s);
}

}  // namespace psf
