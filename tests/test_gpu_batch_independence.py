"""A sequence's rows have the same bits whatever other sequences share its call: the forms of the kernels that go by the
number of units deal tiles or rows, and every sum keeps its order.  (d = r = 64 is left out: its states are summed in
half precision, or by two waves, where there are few units.)"""
import pytest
import torch

from paper_2310_01655_amd import binding as psf
from paper_2310_01655_amd import inputs

pytestmark = pytest.mark.gpu


def rows_by_units(call, n, d, p, r, b, counts):
    """The rows of unit 0 in a call of each number of units."""
    g = torch.Generator(device="cuda")
    g.manual_seed(n + p + r + b)
    Q, K, V = (torch.randn(1, max(counts), n, d, generator=g, device="cuda") for _ in range(3))
    Q, K, V = (Q / Q.norm(dim=-1, keepdim=True)).bfloat16(), (K / K.norm(dim=-1, keepdim=True)).bfloat16(), V.bfloat16()
    G = inputs.make_sketch_matrices(1, d, r, p, per_head=False, seed=0, dtype="bf16").cuda()
    out = []
    for count in counts:
        desc = psf.make_desc(1, count, n, d, p, r, b, "bf16", per_head=False)
        assert psf.kernel_path(desc) == 1
        out.append(call(desc, *(x[:, :count].contiguous() for x in (Q, K, V)), G)[0, 0])
    torch.cuda.synchronize()
    assert torch.isfinite(out[0]).all()
    return out


# r = 32, d = 64: one tile a wave to 42 units, two to 85, full tiles to 128, two from then on
@pytest.mark.parametrize("d,p,r,counts", [
    (64, 4, 32, (1, 42, 43, 60, 85, 86, 129, 171)), (64, 8, 32, (1, 43, 85, 128)),
    (128, 4, 32, (1, 42, 43)), (128, 4, 64, (1, 12, 13)),
])
def test_no_mask(d, p, r, counts):
    first, *others = rows_by_units(psf.psf_noncausal_attn_fwd, 512, d, p, r, 256, counts)
    for count, x in zip(counts[1:], others):
        assert torch.equal(first, x), "%d units" % count


# blocks of whole 1024s: few and many workgroups of the sketches, whose sums over a tile of keys make the denominators
@pytest.mark.parametrize("d,p,r", [(64, 4, 32), (64, 8, 32), (128, 4, 64), (128, 8, 32)])
@pytest.mark.parametrize("call", [psf.psf_causal_attn_fwd, psf.psf_noncausal_attn_fwd], ids=["causal", "no_mask"])
def test_denominators_of_long_blocks(call, d, p, r):
    counts = (1, 20, 70, 140)
    first, *others = rows_by_units(call, 2048, d, p, r, 1024, counts)
    for count, x in zip(counts[1:], others):
        assert torch.equal(first, x), "%d units" % count
