// How the rows are cut into slices for the parameter sums of learned sketches: a plain integer rule, host only.
#ifndef PSF_LEARNED_SLICES_H
#define PSF_LEARNED_SLICES_H

#include <stddef.h>

namespace psf {

struct LearnedSlices { int units, n, per_unit; };

// us of the parameter kernels and of the reduction with `slices` slices of `tiles` times 256 rows: 512 workgroups at a
// time, 31 us for 256 rows in both halves together; each slice writes a blob that the reduction reads.
inline double learned_slices_us(long long slices, long long tiles, int r, size_t g_len)
{
    const long long jobs = 2 * (r / 4 / 4), rounds = (slices * jobs + 511) / 512;
    return 31.0 * (double)(rounds * tiles) + (double)slices * (double)g_len * 8 / 5e6;
}

// One parameter set: the rows of all units are one run; a set per head: the slices stay inside their unit.  A slice is a
// multiple of 256 rows, and at least 512 or a whole unit.
// More slices fill the last round of workgroups better and cost more to add up: the count with the smallest sum of both.
// (48 units of 8192 rows, r = 32: 768 slices a side, by filling alone, 967 us in the three kernels; 128 take 827.)
// One slice a unit is always among the counts: 47 units of 256 rows have no other divisor of 512 rows and more, and as one
// slice a side took a call from 387 us to 1982 (324 with them).
inline LearnedSlices learned_slices(int units, int n, bool shared, int r, size_t g_len)
{
    const bool one_run = shared && (long long)units * n < (1LL << 31);
    LearnedSlices ls{one_run ? 1 : units, one_run ? units * n : n, one_run ? units : 1};
    const int tiles = ls.n / 256, least = n < 512 ? 1 : 2;
    double best = learned_slices_us((long long)ls.units * ls.per_unit, tiles / ls.per_unit, r, g_len);
    for (int k = 1; k <= 2048 && tiles / k >= least; ++k) {
        if (tiles % k) continue;
        const double us = learned_slices_us((long long)ls.units * k, tiles / k, r, g_len);
        if (us < best) {
            best = us;
            ls.per_unit = k;
        }
    }
    return ls;
}

}  // namespace psf
#endif
