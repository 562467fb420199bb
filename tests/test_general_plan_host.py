"""How the general path cuts the sequence (psf_general_spans), on the host: the work per token must
not grow with the sequence where a state can bound it, however few and however large the blocks are
and however far the padded records exceed the sketch; workspaces hold the records and nothing
that fitted the library's static scratch outgrows it."""
import itertools

import pytest

from paper_2310_01655_amd import binding as psf

WIDTHS = [(16, 16, 16), (32, 8, 8), (64, 64, 24), (64, 1, 16), (64, 64, 64), (128, 128, 16), (128, 16, 8), (64, 64, 40),
          (100, 20, 33), (128, 128, 128)]
STATIC = psf.STATIC_SCRATCH_BYTES


def record_bytes(d, dv, m):
    if max(d, dv, m) <= 64:
        rt, vt = (1 if m <= 16 else 2 if m <= 32 else 4), 4
    else:
        rt, vt = (2 if m <= 32 else 4 if m <= 64 else 8), 8
    return rt * (rt + 1) // 2 * 256 * (16 * vt + 1) * 4


def unpadded(units, n, d, dv, r, b):
    """Bytes of m(Q) and m(K), and of the states of the vector kernels."""
    up = lambda v: (v + 255) // 256 * 256
    return 2 * up(units * n * r * 4), up(units * (n // b) * r * r * (dv + 1) * 4)


@pytest.mark.parametrize("d,dv,r", WIDTHS)
def test_long_sequences_keep_states(d, dv, r):
    n = 65536
    for units, blocks in itertools.product((1, 12, 96), (1, 2, 16, 64, 512)):
        desc = psf.make_desc(1, units, n, d, 4, r, n // blocks, "f32", dv=dv)
        assert psf.kernel_path(desc) == 0
        m, z = unpadded(units, n, d, dv, r, n // blocks)
        spans = psf.general_spans(desc, 1)
        assert spans >= 1, (units, blocks)
        assert psf.noncausal_workspace_bytes(desc) >= m + units * spans * record_bytes(d, dv, r)
        for which, size in ((0, psf.workspace_bytes), (2, psf.bwd_workspace_bytes)):
            spans = psf.general_spans(desc, which)
            assert spans >= (min(blocks, 8) if blocks > 1 else 0), (units, blocks, which)
            assert size(desc) >= m + units * spans * record_bytes(d, dv, r) * (2 if which else 1) * (spans > 1)
        if m + z <= STATIC:
            assert psf.workspace_bytes(desc) <= STATIC


def test_short_sequences_and_fitting_records_take_no_more_room():
    # shapes whose records fit the vector kernels' room: the workspace is what it was
    for units, n, d, dv, r, b in ((36, 3000, 64, 64, 32, 200), (24, 1950, 64, 64, 32, 150), (1, 1024, 64, 64, 16, 128),
                                  (96, 256, 16, 16, 16, 256), (12, 256, 128, 16, 8, 256)):
        desc = psf.make_desc(1, units, n, d, 4, r, b, "f32", dv=dv)
        want = sum(unpadded(units, n, d, dv, r, b))
        assert psf.workspace_bytes(desc) == want
        assert psf.noncausal_workspace_bytes(desc) == want
    assert psf.general_spans(psf.make_desc(1, 1, 65536, 64, 4, 64, 1024, "bf16"), 0) == -1       # bf16 kernels
    assert psf.general_spans(psf.make_desc(1, 1, 1024, 256, 4, 64, 128, "f32"), 0) == -1         # vector kernels


def test_where_the_static_scratch_leaves_no_room_the_vector_kernels_stay():
    # records of 396 KB a unit and span against 2 KB: within the 32 MB neither states nor cheap pairs
    desc = psf.make_desc(1, 40, 16384, 128, 4, 4, 16, "f32", dv=1)
    m, z = unpadded(40, 16384, 128, 1, 4, 16)
    assert m + z <= STATIC
    assert psf.workspace_bytes(desc) <= STATIC
    assert psf.general_spans(desc, 0) == -1 and psf.general_spans(desc, 2) >= 4


@pytest.mark.parametrize("units,n,r,b", [(48, 8192, 16, 256), (24, 8192, 32, 512), (24, 8000, 16, 250)])
def test_narrow_sketches_keep_a_state_for_every_block(units, n, r, b):
    # a record is half as large again as the vector kernels' state (its values are three bf16 parts); two
    # blocks a span cost a tenth of the forward call and a sixth of the backward call more
    desc = psf.make_desc(1, units, n, 64, 4, r, b, "f32")
    for which in (0, 2):
        assert psf.general_spans(desc, which) == n // b, which
