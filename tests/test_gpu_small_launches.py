"""The output kernel takes 128 tokens a workgroup where 256 would leave the chip idle: the rows of one
sequence come out the same, bit for bit, alone and among enough others for the wide form."""
import pytest
import torch

from paper_2310_01655_amd import autograd
from paper_2310_01655_amd import binding as psf
from paper_2310_01655_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("call", ["forward", "noncausal", "train"])
@pytest.mark.parametrize("n,p,r,b", [(512, 4, 32, 256), (768, 8, 32, 768), (256, 4, 32, 256), (512, 8, 64, 256)])
def test_rows_alone_and_among_others(call, n, p, r, b):
    heads, batch, d = 12, 24, 64
    g = torch.Generator(device="cuda")
    g.manual_seed(n + p)
    K, Q, V = (torch.randn(batch, heads, n, d, generator=g, device="cuda") for _ in range(3))
    Q, K, V = (Q / Q.norm(dim=-1, keepdim=True)).bfloat16(), (K / K.norm(dim=-1, keepdim=True)).bfloat16(), V.bfloat16()
    G = inputs.make_sketch_matrices(heads, d, r, p, per_head=True, seed=0, dtype="bf16").cuda()

    def run(count):
        q, k, v = (x[:count].contiguous() for x in (Q, K, V))
        if call == "train":
            q.requires_grad_(True)
            out = autograd.causal_polysketch_attention(q, k, v, G, p, r, b, per_head=True)
            return [out.detach(), torch.autograd.grad(out, q, torch.ones_like(out))[0]]
        desc = psf.make_desc(count, heads, n, d, p, r, b, "bf16", per_head=True)
        return [(psf.psf_noncausal_attn_fwd if call == "noncausal" else psf.psf_causal_attn_fwd)(desc, q, k, v, G)]

    alone, among = run(1), run(batch)
    torch.cuda.synchronize()
    for x, y in zip(alone, among):
        assert torch.isfinite(x).all()
        if r == 64:      # its state kernels go by the number of units: states and rows rounded to bf16 twice
            assert (x[0].float() - y[0].float()).norm() <= 2 * 2.0 ** -8 * y[0].float().norm()
        else:
            assert torch.equal(x[0], y[0])
