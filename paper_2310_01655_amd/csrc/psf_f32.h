// Host interface of the fp32 matrix-core kernels (psf_f32_fwd.hip, psf_f32_bwd.hip, psf_f32_sketch.h).
#ifndef PSF_F32_H
#define PSF_F32_H

#include <initializer_list>
#include <type_traits>
#include "psf_f32_index.h"
#include "psf_internal.h"

namespace psf {

struct F32Shape;

// How a call cuts the sequence: a state per `span` tokens (whole blocks of a causal call).
struct F32Plan {
    int span, spans;
    int pairs, states;       // weights of pairs inside a span taken directly; states across spans
    int noncausal;
    double cost;             // seconds of the whole chip, see f32_plan
};

// Whether a call runs on these kernels, its plan, and the floats its state records take in the
// workspace (each of the two sets of a backward pass).
struct F32Choice {
    bool use;
    F32Plan plan;
    size_t z_floats;
};

// rows of a staged tile: 64, or 32 where three tiles of 128 columns would leave a CU one workgroup
constexpr int f32_tile_rows(int dt) { return dt == 8 ? 32 : 64; }

bool f32_supported(const Problem &pb);
// fixed_bytes: the rest of the call's workspace; grad: the backward pass
F32Choice f32_choose(const Problem &pb, size_t fixed_bytes, bool noncausal, bool grad);
F32Shape f32_shape(const Problem &pb, const F32Plan &pl);

// m(x) of all rows (X2, M2 may be null); Gaussian sketches only
psf_status f32_sketch_pair(const Problem &pb, const void *X1, const void *X2, const void *G, float *M1, float *M2,
                           hipStream_t s);
// the same for the n rows of every unit that start x_unit elements apart, results m_unit apart
psf_status f32_sketch_rows(const Problem &pb, const void *X, size_t x_unit, const void *G, float *M, size_t m_unit,
                           hipStream_t s);
psf_status f32_key_states(const Problem &pb, const F32Plan &pl, const float *MK, const void *V, float *Z, hipStream_t s);
// share, part: key tiles a workgroup takes where the rows' keys are shared out (0: they are not), and room for the sums
psf_status f32_rows(const Problem &pb, const F32Plan &pl, const float *MQ, const float *MK, const void *Q,
                    const void *K, const void *V, const float *Z, void *O, hipStream_t s, int share, float *part);
constexpr int kSlotFloats = 16 * 65;         // sums of a slice: 16 rows of 64 columns and a denominator
int f32_row_share(const Problem &pb, const F32Plan &pl, size_t part_floats);

// backward pass: G_i as GV [rows][dv] and gden [rows]
psf_status f32_rows_grad(const Problem &pb, const F32Plan &pl, const float *MQ, const float *MK, const void *Q,
                         const void *K, const void *V, const float *Z, const void *dO, float *GV, float *gden,
                         hipStream_t s);
psf_status f32_mirror_states(const Problem &pb, const F32Plan &pl, const float *MQ, const float *GV, const float *gden,
                             float *R, hipStream_t s);

// dM, direct gradients of Q or K and dV of a side; then Algorithm 1's reverse
psf_status f32_bwd_side(const Problem &pb, const F32Plan &pl, bool key_side, const float *MQ, const float *MK,
                        const void *Q, const void *K, const void *V, const float *GV, const float *gden,
                        const float *Z, float *dM, float *dX, void *dV, hipStream_t s);
bool f32_sketch_bwd_supported(const Problem &pb);
psf_status f32_sketch_bwd_pair(const Problem &pb, const void *X1, const void *X2, const void *G, const float *dM1,
                               const float *dM2, const float *direct1, const float *direct2, void *dX1, void *dX2,
                               hipStream_t s);

// rows of `width` columns may be moved four columns at a time
template <typename T>
static inline bool pieces_ok(int width, std::initializer_list<const void *> tensors)
{
    if (width % 4 != 0) return false;
    for (const void *p : tensors)
        if (((uintptr_t)p & (4 * sizeof(T) - 1)) != 0) return false;
    return true;
}

static inline int tiles16(int w) { return (w + 15) / 16; }

// calls f with <DT, RT> as integral constants; the sketch tiles of a 128-wide head are 32, 64 or 128 columns
template <typename F>
static inline psf_status with_tiles(const Problem &pb, F f)
{
    const bool wide = pb.d > 64 || pb.dv > 64 || pb.mcols > 64;
    if (!wide) {
        if (pb.mcols <= 16) return f(std::integral_constant<int, 4>{}, std::integral_constant<int, 1>{});
        if (pb.mcols <= 32) return f(std::integral_constant<int, 4>{}, std::integral_constant<int, 2>{});
        return f(std::integral_constant<int, 4>{}, std::integral_constant<int, 4>{});
    }
    if (pb.mcols <= 32) return f(std::integral_constant<int, 8>{}, std::integral_constant<int, 2>{});
    if (pb.mcols <= 64) return f(std::integral_constant<int, 8>{}, std::integral_constant<int, 4>{});
    return f(std::integral_constant<int, 8>{}, std::integral_constant<int, 8>{});
}

// Blocks of 64 keys that applying a state of rt tiles to 64 rows is worth, by its products.
static inline double state_walk(int rt) { return rt == 1 ? 4 : rt == 2 ? 8 : rt == 4 ? 24 : 88; }

// How the kernels of rows share out the work: f(WR, WK), see psf_f32_fwd.hip.  By row_walks(), W: what counts is for
// how long how many CUs are busy.  Four sets of waves have a chain half as long as two, and two half as long as
// one.  But the former take 16 rows a workgroup instead of 64 and stage every key four times as often:
// below `few`, where that fills CUs that would be idle.  And two sets fill a CU that would else hold two
// workgroups of one: up to 256 of them.
// Measured (us a call; WR 1 WK 4, WR 4 WK 2, WR 4 WK 1; forward, bf16 storage):
//   r = 16, 12 x 500  W 54: 19, 23, 26    16 x 750 W 104: 29, 28, 34    12 x 2000 W 305: 74, 63, 56    14 x 2300 W 401: 86, 86, 61
//   r = 32, 4 x 2000  W 66: 44, 58, 78    32 x 500 W 144: 31, 25, 29    12 x 2000 W 198: 81, 64, 81    96 x 300 W 288: 46, 33, 28
//   r = 64, 2 x 2000  W 33: 53, 68, 93    12 x 700 W 72: 42, 34, 42     7 x 4000 W 224: 341, 142, 182  40 x 1000 W 340: 175, 77, 61
// Without a mask, r = 32, 32 x 500, W 256: 35, 24, 28.  few: 70, and 110 for rows in bf16 storage with r up to 32, where two
// workgroups of four sets fit a CU (12 x 700, r = 16, W 72: 23, 28, 33).
// fp32 storage with r = 64 never has one set, which needs more registers than two waves a SIMD leave it (40 x 1000, W
// 340: 217, 88, 110), and its backward kernels never four, which do not fit the LDS; few is 50 for its rows
// (2 x 2000, W 33: 67, 80, 115; 12 x 500, W 54: 33, 31, 39).
template <int DT, bool FOUR, bool ONE, typename F>
static inline psf_status f32_deal(const Problem &pb, const F32Plan &pl, int rt, int few, F f)
{
    using std::integral_constant;
    if constexpr (DT == 4) {
        const int per_span = ((pl.span < pb.n ? pl.span : pb.n) + 63) / 64;
        const double walks = row_walks(pb.units, pl.spans, per_span, !pl.noncausal, pl.states ? state_walk(rt) : 0);
        if constexpr (FOUR)
            if (walks < few) return f(integral_constant<int, 1>{}, integral_constant<int, 4>{});
        if constexpr (ONE)
            if (walks > 256) return f(integral_constant<int, 4>{}, integral_constant<int, 1>{});
        return f(integral_constant<int, 4>{}, integral_constant<int, 2>{});
    } else {
        return f(integral_constant<int, 4>{}, integral_constant<int, 1>{});
    }
}

}  // namespace psf
#endif
