"""Which rows the workgroups of the fp32 matrix-core kernels take (csrc/psf_f32_index.h), on the host:
every block of rows of every span of every unit exactly once, on either side of the number of spans
from which a span's workgroups stay on one die."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <initializer_list>
#include <vector>
#include "psf_f32_index.h"
using namespace psf;
int main()
{
    int bad = 0;
    for (int units : {1, 3, 8, 12, 36, 63, 64, 65, 200})
        for (int spans : {1, 2, 5, 8, 64})
            for (int per_span : {1, 2, 7, 33}) {
                std::vector<int> seen((size_t)units * spans * per_span);
                const FlatGrid g = flat_grid(row_groups(units, spans, per_span));
                for (unsigned flat = 0; flat < g.x * g.y; ++flat) {
                    RowPlace at;
                    if (!row_place(flat, units, spans, per_span, at)) continue;
                    if (at.unit < 0 || at.unit >= units || at.span < 0 || at.span >= spans || at.k < 0 || at.k >= per_span) ++bad;
                    else ++seen[((size_t)at.unit * spans + at.span) * per_span + at.k];
                }
                for (int s : seen) bad += s != 1;
                // how far the blocks of rows walk, over the longest of them
                for (double state : {0.0, 4.0, 24.0}) {
                    double sum = 0;
                    for (int k = 1; k <= per_span; ++k) sum += units * spans * (k + state) / (per_span + state);
                    const double walks = row_walks(units, spans, per_span, 1, state);
                    bad += !(walks > 0.999 * sum && walks < 1.001 * sum);
                }
                bad += row_walks(units, spans, per_span, 0, 4.0) != (double)units * spans * per_span;
            }
    printf("%d\n", bad);
    return bad != 0;
}
"""


def test_every_block_of_rows_is_taken_once(tmp_path):
    src = tmp_path / "places.cpp"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "paper_2310_01655_amd", "csrc"), str(src), "-o",
                    str(tmp_path / "places")], check=True)
    assert subprocess.run([str(tmp_path / "places")]).returncode == 0
