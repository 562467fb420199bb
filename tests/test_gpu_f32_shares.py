"""Few rows without states: the key tiles of a block of 16 rows are shared out over workgroups (f32_row_share).
Lengths at the edges of rows, of tiles of 128 keys and of the shares, both storage types, masked and not.
Reference and bounds as in test_gpu_f32_states.py: the slices only change the order of a sum of fp32 tiles."""
import pytest
import torch

from paper_2310_01655_amd import binding as psf
from test_gpu_f32_states import REL, make, reference

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("heads,n,d,dv,r,b", [
    (1, 1024, 64, 64, 16, 128), (1, 1023, 64, 64, 16, 93), (1, 1025, 64, 64, 32, 205), (2, 513, 40, 24, 16, 171),
    (1, 384, 64, 64, 64, 384), (1, 385, 64, 20, 64, 77), (3, 645, 64, 64, 16, 129), (1, 1537, 33, 64, 24, 53),
])
def test_shared_keys(heads, n, d, dv, r, b, dtype):
    desc, (q, k, v, G, dO) = make(heads, n, d, dv, r, 4, b, dtype)
    assert psf.kernel_path(desc) == 0
    got = [psf.psf_causal_attn_fwd(desc, q, k, v, G), psf.psf_noncausal_attn_fwd(desc, q, k, v, G)]
    for u in range(heads):
        want = reference(q[0, u], k[0, u], v[0, u], G[u], dO[0, u], 4, r, b)
        for name, x, w in zip(("O", "O without a mask"), got, want):
            x = x[0, u].double()
            assert torch.isfinite(x).all(), name
            rel = float((x - w).norm() / w.norm())
            assert rel <= REL[dtype], "%s: %.3e" % (name, rel)


def test_an_infinity_in_one_slice_reaches_its_rows_only():
    desc, (q, k, v, G, _) = make(1, 1024, 64, 64, 16, 4, 128, "f32")
    plain = psf.psf_causal_attn_fwd(desc, q, k, v, G)
    v = v.clone()
    v[0, 0, 700, 3] = float("inf")
    odd = psf.psf_causal_attn_fwd(desc, q, k, v, G)
    # (a tile that holds one is summed in another order: both sums err by REL at most, not bit for bit equal)
    assert (odd[0, 0, 700:, 3] == float("inf")).all()
    for x, y in ((odd[0, 0, :700], plain[0, 0, :700]), (odd[0, 0, :, 4:], plain[0, 0, :, 4:])):
        assert torch.isfinite(x).all()
        assert (x - y).norm() <= 2 * REL["f32"] * y.norm()
