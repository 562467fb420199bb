// Reads of MFMA operands from LDS (gfx950).
#ifndef PSF_LDS_H
#define PSF_LDS_H

#include <hip/hip_runtime.h>

namespace psf {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// An operand fragment whose contraction index runs across rows in LDS: every group of 16 lanes reads 4 rows x 16
// columns of 16-bit values (lane s: row s / 4, columns 4 (s % 4) ..+3 at its address) and lane i gets column i, rows
// 0..3 in order.  `a` gives entries 0..3 of the fragment, `b` entries 4..7.
__device__ __forceinline__ bf16x8 read_turned(const void *a, const void *b)
{
    typedef short s16x4 __attribute__((ext_vector_type(4)));
    typedef short s16x8 __attribute__((ext_vector_type(8)));
    typedef __attribute__((address_space(3))) s16x4 *at;
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((at)(__attribute__((address_space(3))) const void *)a);
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((at)(__attribute__((address_space(3))) const void *)b);
    return __builtin_bit_cast(bf16x8, (s16x8)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

}  // namespace psf
#endif
