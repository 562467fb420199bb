"""Every instance of the fp32 matrix-core kernels that forms and applies states: sketch widths of 1, 2, 4
and 8 tiles, narrow and wide heads, forward, without a mask and backward (the ways of sharing out the
rows: test_gpu_f32_deals.py), with an odd number of blocks so that the last span is shorter.  The plan is asserted, so that a case
that stops reaching the states is noticed.  Reference: plain torch in float64, the last unit.
Bounds: fp32 sums err by 3e-7 to 1e-6 here, a rounding to bf16 by 1.7e-3."""
import pytest
import torch

from paper_2310_01655_amd import binding as psf
from paper_2310_01655_amd import inputs

pytestmark = pytest.mark.gpu

CASES = [
    # heads, n, d, dv, r, p, b, dtype
    (2, 3024, 64, 64, 16, 4, 48, "f32"),         # 1 tile
    (40, 1189, 64, 64, 16, 4, 29, "f32"),        # 1 tile, many units
    (40, 1350, 64, 64, 16, 4, 150, "bf16"),
    (6, 3150, 64, 60, 30, 4, 150, "f32"),        # 2 tiles
    (40, 2987, 64, 64, 32, 4, 29, "f32"),        # 2 tiles, many units
    (1, 5555, 64, 40, 50, 4, 101, "f32"),        # 4 tiles, few units
    (9, 4545, 64, 64, 64, 4, 101, "f32"),        # 4 tiles
    (2, 2929, 128, 64, 32, 8, 101, "f32"),       # wide, no value columns for the second workgroup
    (1, 3219, 66, 127, 17, 4, 29, "f32"),        # wide in the values, widths that four does not divide
    (1, 5959, 128, 32, 60, 4, 101, "f32"),       # wide, 4 tiles
    (1, 14529, 70, 128, 100, 4, 29, "f32"),      # 8 tiles
]
REL = {"f32": 3e-6, "bf16": 4e-3}


def sketch(x, G, d, r, p):
    at, level = 0, []
    mats = []
    for k in range(p // 2):
        mats.append(G[at:at + d * r].view(d, r))
        at += d * r
    level = [(x @ mats[2 * k]) * (x @ mats[2 * k + 1]) * r ** -0.5 for k in range(p // 4)]
    while len(level) > 1:
        up = []
        for k in range(len(level) // 2):
            a, b = G[at:at + r * r].view(r, r), G[at + r * r:at + 2 * r * r].view(r, r)
            at += 2 * r * r
            up.append((level[2 * k] @ a) * (level[2 * k + 1] @ b) * r ** -0.5)
        level = up
    return level[0]


def reference(q, k, v, G, dO, p, r, b):
    """O, O without a mask, dQ, dK, dV of one unit in float64."""
    q, k, v = (x.double().requires_grad_(True) for x in (q, k, v))
    n, d = q.shape
    mq, mk = sketch(q, G.double(), d, r, p), sketch(k, G.double(), d, r, p)
    far = (mq @ mk.t().contiguous()) ** 2
    with torch.no_grad():
        N = (far @ v) / (1 + far.sum(-1, keepdim=True))
    i = torch.arange(n, device=q.device)
    w = torch.where((i[:, None] // b) == (i[None] // b), (q @ k.t().contiguous()) ** p, far) * (i[:, None] >= i[None])
    O = (w @ v) / (1 + w.sum(-1, keepdim=True))
    return [O.detach(), N, *torch.autograd.grad(O, (q, k, v), dO.double())]


def make(heads, n, d, dv, r, p, b, dtype):
    q, k, v = inputs.make_qkv(1, heads, n, d, dv=dv, seed=5, dtype=dtype)
    G = inputs.make_sketch_matrices(heads, d, r, p, per_head=True, seed=2, dtype=dtype)
    dO = inputs.make_dout(1, heads, n, dv, seed=5, dtype=dtype)
    return psf.make_desc(1, heads, n, d, p, r, b, dtype, dv=dv, per_head=True), [x.cuda() for x in (q, k, v, G, dO)]


@pytest.mark.parametrize("heads,n,d,dv,r,p,b,dtype", CASES)
def test_states_of_every_shape(heads, n, d, dv, r, p, b, dtype):
    desc, (q, k, v, G, dO) = make(heads, n, d, dv, r, p, b, dtype)
    assert psf.kernel_path(desc) == 0 and (n // b) % 2 == 1
    assert psf.general_spans(desc, 0) > 1 and psf.general_spans(desc, 1) >= 1 and psf.general_spans(desc, 2) > 1
    got = [psf.psf_causal_attn_fwd(desc, q, k, v, G), psf.psf_noncausal_attn_fwd(desc, q, k, v, G),
           *psf.psf_causal_attn_bwd(desc, q, k, v, G, dO)]
    u = heads - 1
    want = reference(q[0, u], k[0, u], v[0, u], G[u], dO[0, u], p, r, b)
    for name, x, w in zip(("O", "O without a mask", "dQ", "dK", "dV"), got, want):
        x = x[0, u].double()
        assert torch.isfinite(x).all(), name
        rel = float((x - w).norm() / w.norm())
        assert rel <= REL[dtype], "%s: %.3e" % (name, rel)


@pytest.mark.parametrize("heads,n,b,at", [(2, 96, 24, 37), (1, 1300, 325, 901), (2, 3024, 48, 1501), (40, 1189, 29, 600)])
@pytest.mark.parametrize("where", ["Q", "K", "V", "dO"])
def test_an_infinity_stays_within_its_reach_in_the_backward_pass(heads, n, b, at, where):
    """A token's query and dO reach its own dQ and the dK, dV of the tokens up to it; its key and
    value reach every row from it on, and so not the dQ before it."""
    desc, clean = make(heads, n, 64, 64, 16, 4, b, "f32")
    want = psf.psf_causal_attn_bwd(desc, *clean)
    for bad in (float("inf"), float("nan")):
        args = [x.clone() for x in clean]
        args[{"Q": 0, "K": 1, "V": 2, "dO": 4}[where]][:, :, at, 5] = bad
        dQ, dK, dV = psf.psf_causal_attn_bwd(desc, *args)
        if where in ("Q", "dO"):
            others = torch.arange(n, device=dQ.device) != at
            pairs = [(dQ[:, :, others], want[0][:, :, others]), (dK[:, :, at + 1:], want[1][:, :, at + 1:]),
                     (dV[:, :, at + 1:], want[2][:, :, at + 1:])]
        else:
            pairs = [(dQ[:, :, :at], want[0][:, :, :at])]
        for got, ref in pairs:
            assert torch.isfinite(got).all()
            scale = float(ref.abs().max())
            torch.testing.assert_close(got, ref, rtol=1e-5, atol=1e-6 * max(1.0, scale))   # fp32 sums in another order


@pytest.mark.parametrize("d,r,p", [(128, 32, 8), (64, 32, 4), (128, 128, 4)])
def test_gradients_repeat_bit_for_bit(d, r, p):
    """Results read from the matrix pipe too early would differ from run to run."""
    desc, args = make(12, 1500, d, d, r, p, 300, "f32")
    first = psf.psf_causal_attn_bwd(desc, *args)
    for _ in range(3):
        for a, b in zip(first, psf.psf_causal_attn_bwd(desc, *args)):
            assert torch.equal(a, b)
