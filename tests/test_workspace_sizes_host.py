"""A buffer made for the longest sequence serves the shorter ones: the sizes the library asks for do not fall as the
sequence grows, for blocks of whole 1024s, which the sketches cut alike at every length.  (At d = r = 64 only for prompts: past a
length the other calls leave their half-precision and fused forms, and with those goes the room for what they hand over.)
Host only."""
import ctypes

import pytest

from paper_2310_01655_amd import binding as psf


@pytest.mark.parametrize("d,p,r", [(64, 4, 32), (64, 8, 32), (64, 4, 64), (128, 4, 32), (128, 4, 64), (128, 8, 64)])
@pytest.mark.parametrize("units,b", [(1, 1024), (12, 1024), (13, 2048), (48, 1024)])
def test_sizes_do_not_fall(d, p, r, units, b):
    last = []
    for blocks in range(1, 161):
        n = blocks * b
        desc = psf.make_desc(1, units, n, d, p, r, b, "bf16", per_head=False)
        longest = psf.make_desc(1, units, 160 * b, d, p, r, b, "bf16", per_head=False)
        now = [psf.lib().psf_decode_prefill_workspace_bytes(ctypes.byref(longest), n)]
        if (d, r) != (64, 64):
            now += [psf.workspace_bytes(desc), psf.noncausal_workspace_bytes(desc), psf.bwd_workspace_bytes(desc),
                    psf.fwd_save_bytes(desc)]
        assert all(x >= y for x, y in zip(now, last)), (n, now, last)
        last = now
