"""How the rows are cut for the parameter sums of learned sketches (csrc/psf_learned_slices.h), on the host: whole
multiples of 256 rows that cover every row once, and never a longer chain than one slice a unit would be."""
from test_f32_index_host import run_host

PROGRAM = r"""
#include <cstdio>
#include <initializer_list>
#include "psf_learned_slices.h"
using namespace psf;
int main()
{
    int bad = 0;
    for (int r : {32, 64})
        for (int n = 256; n <= 8192; n += n < 2048 ? 256 : 1280)
            for (int units = 1; units <= 2100; units += units < 140 ? 1 : 53)
                for (int shared = 0; shared < 2; ++shared) {
                    const size_t g_len = 2 * (128 + 64 * 8 * r + 16 * r + 24 * r * r);
                    const LearnedSlices ls = learned_slices(units, n, shared, r, g_len);
                    const long long slices = (long long)ls.units * ls.per_unit, tiles = ls.n / 256 / ls.per_unit;
                    const bool whole = (long long)ls.units * ls.n == (long long)units * n && ls.n % (256 * ls.per_unit) == 0;
                    const double us = learned_slices_us(slices, tiles, r, g_len);
                    if ((!whole || us > learned_slices_us(units, n / 256, r, g_len)) && bad++ < 8)
                        printf("r %d n %d units %d shared %d: %lld slices of %lld\n", r, n, units, shared, slices, tiles);
                }
    return bad != 0;
}
"""


def test_slices_cover_the_rows_in_short_chains(tmp_path):
    run_host(tmp_path, PROGRAM)
