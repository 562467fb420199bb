"""Every way in which the fp32 matrix-core kernels of narrow heads share out their rows (four sets of
waves for 16 rows, two or one for 64), with states, in either storage type: forward, without a mask
and backward.  The way is worked out here from the plan, so that a case that stops reaching it
is noticed.  Reference and bounds as in test_gpu_f32_states.py."""
import pytest
import torch

from paper_2310_01655_amd import binding as psf
from test_gpu_f32_states import REL, make, reference

pytestmark = pytest.mark.gpu


def sets_of_waves(desc, which, r, dtype, rows):
    """How many sets the kernels of a pass take; which: 0 forward, 1 without a mask, 2 backward."""
    units, n, b = desc.batch * desc.heads, desc.n, desc.b
    spans = psf.general_spans(desc, which)
    span, state = n, {16: 4, 32: 8, 64: 24}[r]
    if spans > 1 and which != 1:
        blocks = 1
        while -(-(n // b) // blocks) > spans:
            blocks *= 2
        span = blocks * b
    elif which != 1:
        state = 0
    k = (span + 63) // 64
    if which == 1:
        walks = units * max(spans, 1) * ((-(-n // max(spans, 1)) + 63) // 64)
    else:
        walks = units * max(spans, 1) * k * ((k + 1) / 2 + state) / (k + state)
    fp32_wide = r == 64 and dtype == "f32"
    few = 0 if fp32_wide and not rows else 50 if fp32_wide else 110 if rows and dtype == "bf16" and r <= 32 else 70
    return 4 if walks < few else 2 if walks <= 256 or fp32_wide else 1


CASES = [
    # heads, n, r, b; sets of the row kernels forward, without a mask, and of the backward kernels
    (1, 2961, 16, 47, (4, 4, 4)), (3, 4650, 16, 150, (2, 1, 2)), (12, 1827, 16, 29, (1, 1, 1)),
    (1, 3131, 32, 101, (4, 4, 4)), (5, 3131, 32, 101, (2, 1, 2)), (12, 2250, 32, 150, (1, 1, 1)),
    (1, 2525, 64, 101, (4, 4, 4)), (2, 4650, 64, 150, (2, 2, 2)), (9, 4545, 64, 101, (1, 1, 1)),
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("heads,n,r,b,sets", CASES)
def test_every_way_of_sharing_out_the_rows(heads, n, r, b, sets, dtype):
    desc, (q, k, v, G, dO) = make(heads, n, 64, 64, r, 4, b, dtype)
    assert psf.kernel_path(desc) == 0
    fp32_wide = r == 64 and dtype == "f32"
    for which, want in enumerate(sets):
        want = max(want, 2) if fp32_wide else want
        assert sets_of_waves(desc, which, r, dtype, which != 2) == (2 if fp32_wide and which == 2 else want), which
        if r < 64 or heads > 1:                             # (few rows' pairs are cheaper than wide states)
            assert psf.general_spans(desc, which) >= (1 if which == 1 else 2)
    got = [psf.psf_causal_attn_fwd(desc, q, k, v, G), psf.psf_noncausal_attn_fwd(desc, q, k, v, G),
           *psf.psf_causal_attn_bwd(desc, q, k, v, G, dO)]
    u = heads - 1
    want = reference(q[0, u], k[0, u], v[0, u], G[u], dO[0, u], 4, r, b)
    for name, x, w in zip(("O", "O without a mask", "dQ", "dK", "dV"), got, want):
        x = x[0, u].double()
        assert torch.isfinite(x).all(), name
        rel = float((x - w).norm() / w.norm())
        assert rel <= REL[dtype], "%s: %.3e" % (name, rel)
