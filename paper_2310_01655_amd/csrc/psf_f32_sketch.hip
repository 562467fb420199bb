// m(x) of all rows, see psf_f32_sketch.h.
#include "psf_f32_sketch.h"

namespace psf {
namespace {

// m(x) of the rows of X1 and (blockIdx.z = 1) X2
template <int DT, int RT, int LEVEL, int H, typename T>
__global__ __launch_bounds__(kF32Threads) void f32_sketch_kernel(const T *__restrict__ X1, const T *__restrict__ X2,
                                                                 const T *__restrict__ G, float *__restrict__ M1,
                                                                 float *__restrict__ M2, SketchArgs a)
{
    typedef Sketcher<DT, RT, H, T> S;
    __shared__ __attribute__((aligned(16))) uint16_t lds[2 * S::kMatrix];
    const int i0 = (blockIdx.x * 4 + (threadIdx.x >> 6)) * 16 * H;
    S s;
    sketch_begin(s, (blockIdx.z ? X2 : X1) + blockIdx.y * a.x_unit, G, lds, a, i0);
    typename S::Rows m;
    s.template forward<LEVEL>(0, m);
    float *M = (blockIdx.z ? M2 : M1) + blockIdx.y * a.m_unit;
#pragma unroll
    for (int h = 0; h < H; ++h) {
        const int row = i0 + 16 * h + (s.lane & 15);
        if (row < a.n)
#pragma unroll
            for (int t = 0; t < RT; ++t) store_piece(M + (size_t)row * a.r, 16 * t + 4 * (s.lane >> 4), a.r, a.vec_m, m[h][t]);
    }
}

// p = 2: m(x) = x
template <typename T>
__global__ __launch_bounds__(kF32Threads) void f32_plain_kernel(const T *__restrict__ X1, const T *__restrict__ X2,
                                                                float *__restrict__ M1, float *__restrict__ M2,
                                                                size_t unit_len, size_t x_unit, size_t m_unit)
{
    const T *X = (blockIdx.z ? X2 : X1) + blockIdx.y * x_unit;
    float *M = (blockIdx.z ? M2 : M1) + blockIdx.y * m_unit;
    for (size_t i = (size_t)blockIdx.x * kF32Threads + threadIdx.x; i < unit_len; i += (size_t)gridDim.x * kF32Threads)
        M[i] = load_f(X, i);
}
template <typename T>
psf_status sketch_pair(const Problem &pb, const void *X1, const void *X2, const void *G, float *M1, float *M2,
                       size_t x_unit, size_t m_unit, hipStream_t s)
{
    const unsigned z = X2 ? 2 : 1;
    if (pb.p == 2) {
        const size_t len = (size_t)pb.n * pb.d;
        hipLaunchKernelGGL(f32_plain_kernel<T>, dim3(plain_grid(len), (unsigned)pb.units, z), dim3(kF32Threads), 0, s,
                           (const T *)X1, (const T *)X2, M1, M2, len, x_unit, m_unit);
        PSF_LAUNCH_CHECK();
        return PSF_OK;
    }
    SketchArgs a = sketch_args(pb, x_unit, m_unit);
    a.vec_x = x_unit % 4 == 0 && (X2 ? pieces_ok<T>(pb.d, {X1, X2}) : pieces_ok<T>(pb.d, {X1}));
    a.vec_m = m_unit % 4 == 0 && pieces_ok<float>(pb.r, {M1, M2 ? M2 : M1});
    a.vec_g = pieces_ok<T>(pb.r, {G});
    return with_tiles(pb, [&](auto dt, auto rt) -> psf_status {
        return with_level(pb.p, [&](auto level) -> psf_status {
            constexpr int DT = decltype(dt)::value, RT = decltype(rt)::value, LEVEL = decltype(level)::value;
            constexpr int H = parts_of<T>() == 1 && RT * LEVEL <= 4 ? 2 : 1;
            hipLaunchKernelGGL((f32_sketch_kernel<DT, RT, LEVEL, H, T>), dim3((unsigned)((pb.n + 64 * H - 1) / (64 * H)), (unsigned)pb.units, z),
                               dim3(kF32Threads), 0, s, (const T *)X1, (const T *)X2, (const T *)G, M1, M2, a);
            PSF_LAUNCH_CHECK();
            return PSF_OK;
        });
    });
}

}  // namespace

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

}  // namespace psf
