// The gradient of x through m(x), see psf_f32_sketch.h.
#include "psf_f32_sketch.h"

namespace psf {
namespace {

// dX = direct + the gradient through m(x), whose own gradient is dM
template <int DT, int RT, int LEVEL, int H, typename T>
__global__ __launch_bounds__(kF32Threads) void f32_bwd_sketch_kernel(
    const T *__restrict__ X1, const T *__restrict__ X2, const T *__restrict__ G, const float *__restrict__ dM1,
    const float *__restrict__ dM2, const float *__restrict__ dir1, const float *__restrict__ dir2, T *__restrict__ dX1,
    T *__restrict__ dX2, SketchArgs a)
{
    typedef Sketcher<DT, RT, H, T> S;
    __shared__ __attribute__((aligned(16))) uint16_t lds[2 * S::kMatrix];
    const int i0 = (blockIdx.x * 4 + (threadIdx.x >> 6)) * 16 * H;
    const size_t unit_row = (size_t)blockIdx.y * a.n;
    S s;
    sketch_begin(s, (blockIdx.z ? X2 : X1) + unit_row * a.d, G, lds, a, i0);
    const int li = s.lane & 15, g = s.lane >> 4, vec_r = a.r % 4 == 0, vec_d = a.d % 4 == 0;   // (workspace)
    const float *dM = (blockIdx.z ? dM2 : dM1) + unit_row * a.r, *dir = (blockIdx.z ? dir2 : dir1) + unit_row * a.d;
    typename S::Rows dm;
    f4 dx[H][DT];
#pragma unroll
    for (int h = 0; h < H; ++h) {
        const size_t row = min(i0 + 16 * h + li, a.n - 1);
#pragma unroll
        for (int t = 0; t < RT; ++t) dm[h][t] = row_piece(dM + row * a.r, 16 * t + 4 * g, a.r, vec_r);
#pragma unroll
        for (int t = 0; t < DT; ++t) dx[h][t] = row_piece(dir + row * a.d, 16 * t + 4 * g, a.d, vec_d);
    }
    s.template reverse<LEVEL>(0, dm, dx);
    T *dX = (blockIdx.z ? dX2 : dX1) + unit_row * a.d;
#pragma unroll
    for (int h = 0; h < H; ++h) {
        const int row = i0 + 16 * h + li;
        if (row < a.n)
#pragma unroll
            for (int t = 0; t < DT; ++t) store_piece(dX + (size_t)row * a.d, 16 * t + 4 * g, a.d, a.vec_x, dx[h][t]);
    }
}

// p = 2: m(x) = x
template <typename T>
__global__ __launch_bounds__(kF32Threads) void f32_plain_bwd_kernel(const float *__restrict__ dM1, const float *__restrict__ dM2,
                                                                    const float *__restrict__ dir1,
                                                                    const float *__restrict__ dir2, T *__restrict__ dX1,
                                                                    T *__restrict__ dX2, size_t len)
{
    const float *dM = blockIdx.z ? dM2 : dM1, *dir = blockIdx.z ? dir2 : dir1;
    T *dX = blockIdx.z ? dX2 : dX1;
    for (size_t i = (size_t)blockIdx.x * kF32Threads + threadIdx.x; i < len; i += (size_t)gridDim.x * kF32Threads)
        store_f(dX, i, dir[i] + dM[i]);
}

template <typename T>
psf_status sketch_bwd_pair(const Problem &pb, const void *X1, const void *X2, const void *G, const float *dM1,
                           const float *dM2, const float *dir1, const float *dir2, void *dX1, void *dX2, hipStream_t s)
{
    const unsigned z = X2 ? 2 : 1;
    if (pb.p == 2) {
        const size_t len = (size_t)pb.units * pb.n * pb.d;
        hipLaunchKernelGGL(f32_plain_bwd_kernel<T>, dim3(plain_grid(len), 1, z), dim3(kF32Threads), 0, s, dM1, dM2, dir1,
                           dir2, (T *)dX1, (T *)dX2, len);
        PSF_LAUNCH_CHECK();
        return PSF_OK;
    }
    SketchArgs a = sketch_args(pb, 0, 0);
    a.vec_x = X2 ? pieces_ok<T>(pb.d, {X1, X2, dX1, dX2}) : pieces_ok<T>(pb.d, {X1, dX1});
    a.vec_g = pieces_ok<T>(pb.r, {G});
    return with_tiles(pb, [&](auto dt, auto rt) -> psf_status {
        return with_level(pb.p, [&](auto level) -> psf_status {
            constexpr int DT = decltype(dt)::value, RT = decltype(rt)::value, LEVEL = decltype(level)::value;
            constexpr int H = parts_of<T>() == 1 && RT * LEVEL <= 2 && DT == 4 ? 2 : 1;
            hipLaunchKernelGGL((f32_bwd_sketch_kernel<DT, RT, LEVEL, H, T>), dim3((unsigned)((pb.n + 64 * H - 1) / (64 * H)), (unsigned)pb.units, z),
                               dim3(kF32Threads), 0, s, (const T *)X1, (const T *)X2, (const T *)G, dM1, dM2, dir1, dir2,
                               (T *)dX1, (T *)dX2, a);
            PSF_LAUNCH_CHECK();
            return PSF_OK;
        });
    });
}

}  // namespace

bool f32_sketch_bwd_supported(const Problem &pb)
{
    return !pb.learned && !pb.exact_feat && pb.d <= 128 && pb.mcols <= 128;
}

psf_status f32_sketch_bwd_pair(const Problem &pb, const void *X1, const void *X2, const void *G, const float *dM1,
                               const float *dM2, const float *direct1, const float *direct2, void *dX1, void *dX2,
                               hipStream_t s)
{
    return pb.bf16 ? sketch_bwd_pair<bf16_t>(pb, X1, X2, G, dM1, dM2, direct1, direct2, dX1, dX2, s)
                   : sketch_bwd_pair<float>(pb, X1, X2, G, dM1, dM2, direct1, direct2, dX1, dX2, s);
}

}  // namespace psf
