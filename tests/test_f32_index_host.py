"""The addresses of the fp32 matrix-core kernels' staged loads, from the rules the kernels use
(csrc/psf_f32_index.h), on the host: every load of the state kernel stays inside the value tensor,
for value widths on either side of the 64 columns a workgroup takes and last chunks of few rows."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <initializer_list>
#include "psf_f32_index.h"
using namespace psf;
int main()
{
    long long bad = 0, loads = 0;
    for (int rows_staged : {32, 64})                       // tokens of a chunk: RT = 8, smaller RT
        for (int dv = 4; dv <= 128; dv += 4)
            for (int n : {1, 2, 3, 5, 17, 31, 32, 33, 63, 64, 65, 130, 205, 1025})
                for (int span_tokens : {1, 41, 64, 205, n})
                    for (int c0 : {0, 64}) {               // the two workgroups of a wide problem
                        const int spans = (n + span_tokens - 1) / span_tokens;
                        const long long end = (long long)n * dv;          // of the last unit
                        for (int span = 0; span < spans; ++span) {
                            const TokenRange t = state_tokens(n, span_tokens, span, dv, c0);
                            for (int j0 = t.begin; j0 < t.end; j0 += rows_staged)
                                for (int row = 0; row < rows_staged; ++row)
                                    for (int c = 0; c < 64; c += 4) {
                                        const long long at = (long long)j0 * dv + c0 +
                                                             tile_piece(row, c, dv, t.end - j0, dv - c0);
                                        ++loads;
                                        if (at < 0 || at + 4 > end) {
                                            if (bad++ < 4)
                                                printf("dv %d n %d span %d c0 %d: %lld of %lld\n", dv, n, span, c0, at, end);
                                        }
                                    }
                        }
                    }
    printf("loads %lld outside %lld\n", loads, bad);
    return bad ? 1 : 0;
}
"""

GRIDS = r"""
#include <cstdio>
#include <initializer_list>
#include "psf_f32_index.h"
using namespace psf;
int main()
{
    int bad = 0;
    for (unsigned long long groups : {1ull, 7ull, (1ull << 23) - 1, 1ull << 23, (1ull << 23) + 1, 1ull << 24,
                                      (1ull << 24) + 12345, 65535ull * 257, 1ull << 28}) {
        const FlatGrid g = flat_grid(groups);
        const unsigned long long all = (unsigned long long)g.x * g.y;
        if (all < groups || all >= groups + g.x || g.x * 256ull >= 1ull << 32 || g.y > 65535 || all >> 32) {
            printf("%llu workgroups: %u x %u\n", groups, g.x, g.y);
            ++bad;
        }
    }
    return bad;
}
"""


def test_large_launches_stay_within_a_grid_dimension(tmp_path):
    """2^24 workgroups of 256 threads (2^30 rows) are too many for one dimension."""
    run_host(tmp_path, GRIDS)


def run_host(tmp_path, program):
    src, exe = tmp_path / "index.cpp", tmp_path / "index"
    src.write_text(program)
    subprocess.run(["g++", "-std=c++17", "-O2", "-I", os.path.join(ROOT, "paper_2310_01655_amd", "csrc"), str(src),
                    "-o", str(exe)], check=True)
    run = subprocess.run([str(exe)], stdout=subprocess.PIPE, text=True)
    assert run.returncode == 0, run.stdout


def test_state_kernel_loads_stay_inside_the_values(tmp_path):
    run_host(tmp_path, PROGRAM)


SLOTS = r"""
#include <cstdio>
#include "psf_f32_index.h"
using namespace psf;
int main()
{
    int bad = 0;
    for (int causal = 0; causal < 2; ++causal)
        for (int n = 1; n <= 2100; n += n < 300 ? 1 : 37)
            for (int share = 1; share <= 17; ++share) {
                int slots = 0, blocks = (n + 15) / 16;
                for (int block = 0; block <= blocks; ++block) {
                    if (row_slots_before(block, n, share, causal) != slots && bad++ < 4)
                        printf("causal %d n %d share %d block %d: %d, not %d\n", causal, n, share, block,
                               row_slots_before(block, n, share, causal), slots);
                    const int last = 16 * block + 15 < n ? 16 * block + 15 : n - 1;
                    const int tiles = causal ? last / 128 + 1 : (n + 127) / 128, s = (tiles + share - 1) / share;
                    if (block < blocks && row_slices(block, n, share, causal) != s && bad++ < 4)
                        printf("causal %d n %d share %d block %d: %d slices, not %d\n", causal, n, share, block,
                               row_slices(block, n, share, causal), s);
                    slots += s > 1 ? s : 0;
                }
            }
    return bad;
}
"""


def test_slots_of_shared_rows_are_counted_through(tmp_path):
    """Where the workgroups that share a block's keys leave their sums, against counting them."""
    run_host(tmp_path, SLOTS)


SHARES = r"""
#include <cstdio>
#include <initializer_list>
#include "psf_f32_index.h"
using namespace psf;
int main()
{
    int bad = 0;
    for (int causal = 0; causal < 2; ++causal)
        for (int n = 1; n <= 4200; n += n < 300 ? 1 : 37)
            for (int units = 1; units <= 20; ++units)
                for (unsigned long long room : {0ull, 16ull, 200ull, 100000ull})
                    for (int light = 0; light < 2; ++light) {
                        const int share = row_share(units, n, causal, light, room);
                        if (!share) continue;
                        int workgroups = 0, longest = 0, slots = 0;
                        for (int block = 0; block < (n + 15) / 16; ++block) {
                            const int s = row_slices(block, n, share, causal);
                            workgroups += units * s;
                            slots += s > 1 ? units * s : 0;
                            longest = s > 1 ? share : longest;
                        }
                        // one a CU, but for the short ones under a mask; two tiles shorter and more; sums where there is room
                        const int most = !causal ? 256 : share == 1 ? 224 : share == 2 ? 256 : 288;
                        const bool ok = workgroups <= most && longest + (light ? 3 : 2) <= (n + 127) / 128 &&
                                        (unsigned long long)slots <= room;
                        if (!ok && bad++ < 4)
                            printf("causal %d n %d units %d: %d tiles, %d workgroups, %d slots\n", causal, n, units, share,
                                   workgroups, slots);
                    }
    return bad != 0;
}
"""


def test_shared_rows_fill_the_chip_once(tmp_path):
    """More workgroups than CUs wait for each other: a call then takes longer than with its keys not shared out."""
    run_host(tmp_path, SHARES)
