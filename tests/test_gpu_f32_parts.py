"""The kernels that form fp32 products from bf16 parts, at every way of sharing out the rows and either
storage type: a token's infinity or NaN stays out of the rows before it and arrives in its own, forward
and backward, and is finite everywhere else; and every part of every operand counts.  References: the
same call without the odd token (rows before it), plain torch in float64."""
import pytest
import torch

from paper_2310_01655_amd import binding as psf
from paper_2310_01655_amd import inputs
from test_gpu_f32_states import reference

pytestmark = pytest.mark.gpu

# rows that share a tile with the odd token take their sums in another order: fp32 sums differ by
# about 1e-6, their roundings to bf16 by at most 2^-8
SAME = {"f32": 1e-5, "bf16": 4e-3}
SHAPES = [(2, 1300, 325), (12, 600, 150), (40, 1000, 200)]      # 42, 120 and 640 workgroups of 64 rows


def same(x, y, dtype):
    x, y = x.double(), y.double()
    return bool(x.isfinite().all()) and float((x - y).norm()) <= SAME[dtype] * float(y.norm())


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("heads,n,b", SHAPES)
def test_an_infinite_value_stays_in_its_place(heads, n, b, dtype):
    at = n // 2 + 7
    q, k, v = (x.cuda() for x in inputs.make_qkv(1, heads, n, 64, seed=5, dtype=dtype))
    G = inputs.make_sketch_matrices(heads, 64, 32, 4, per_head=True, seed=3, dtype=dtype).cuda()
    dO = inputs.make_dout(1, heads, n, 64, seed=5, dtype=dtype).cuda()
    desc = psf.make_desc(1, heads, n, 64, 4, 32, b, dtype, per_head=True)
    assert psf.kernel_path(desc) == 0
    want = psf.psf_causal_attn_fwd(desc, q, k, v, G)
    grads = psf.psf_causal_attn_bwd(desc, q, k, v, G, dO)
    v2 = v.clone()
    v2[:, :, at, 5], v2[:, :, at, 6] = float("inf"), float("nan")
    got = psf.psf_causal_attn_fwd(desc, q, k, v2, G)
    assert same(got[:, :, :at], want[:, :, :at], dtype)
    own = got[:, :, at:at // b * b + b]                     # the rest of the block: weights are positive
    assert (own[..., 5] == float("inf")).all() and own[..., 6].isnan().all()
    assert not got[:, :, at:, 5:7].isfinite().any()
    others = [c for c in range(64) if c not in (5, 6)]
    assert got[..., others].isfinite().all()
    # the odd gradient of one row reaches the keys up to it and no later one
    dO2 = dO.clone()
    dO2[:, :, at, 3] = float("inf")
    dq, dk, dv = psf.psf_causal_attn_bwd(desc, q, k, v, G, dO2)
    for x, y in ((dk, grads[1]), (dv, grads[2])):
        assert same(x[:, :, at + 1:], y[:, :, at + 1:], dtype)
    rows = [i for i in range(n) if i != at]
    assert same(dq[:, :, rows], grads[0][:, :, rows], dtype) and not dv[:, :, at, 3].isfinite().any()


def cut(x):
    """x without its third part: 16 to 17 of its 24 bits."""
    h = (x.view(torch.int32) & -65536).view(torch.float32)
    return h + (x - h).bfloat16().float()


@pytest.mark.parametrize("heads,n,r,b", [(3, 330, 16, 110), (2, 3024, 16, 48), (5, 3131, 32, 101), (2, 4650, 64, 150)])
def test_every_part_counts(heads, n, r, b):
    """Rows of V, and columns of Q and K, over many binades.  Bound: fp32 sums err by 3e-7 to 6e-7 here; without its
    third part an operand is off by 2^-18.5 = 2.7e-6 in the mean, which the float64 evaluation of cut operands
    shows to be visible in some result of this case for each of Q, K, V, G and dO."""
    q, k, v = (x.cuda() for x in inputs.make_qkv(1, heads, n, 64, seed=9, dtype="f32"))
    g = torch.Generator(device="cuda")
    g.manual_seed(4)
    binades = lambda *shape: torch.randint(-6, 7, shape, generator=g, device="cuda").float().exp2()
    v = v * binades(1, heads, n, 1)
    q, k = ((x * c) / (x * c).norm(dim=-1, keepdim=True) for x, c in ((q, binades(64)), (k, binades(64))))
    G = inputs.make_sketch_matrices(heads, 64, r, 4, per_head=True, seed=3, dtype="f32").cuda()
    dO = inputs.make_dout(1, heads, n, 64, seed=9, dtype="f32").cuda()
    desc = psf.make_desc(1, heads, n, 64, 4, r, b, "f32", per_head=True)
    assert psf.kernel_path(desc) == 0
    got = [psf.psf_causal_attn_fwd(desc, q, k, v, G), psf.psf_noncausal_attn_fwd(desc, q, k, v, G),
           *psf.psf_causal_attn_bwd(desc, q, k, v, G, dO)]
    u = heads - 1
    operands = [q[0, u], k[0, u], v[0, u], G[u], dO[0, u]]
    want = reference(*operands, 4, r, b)

    def far(results):
        return [float((x.double() - w).norm() / w.norm()) for x, w in zip(results, want)]

    bound = 1e-6
    assert max(far([x[0, u] for x in got])) <= bound, far([x[0, u] for x in got])
    for i in range(5):
        changed = [cut(x) if i == j else x for j, x in enumerate(operands)]
        assert max(far(reference(*changed, 4, r, b))) > 1.5 * bound, i


@pytest.mark.parametrize("scale", [2.0 ** -40, 2.0 ** 30])
def test_small_and_large_values_scale(scale):
    # V enters linearly: scaled by a power of two, every output is scaled by it, to the bit, and no part
    # leaves bf16's range
    heads, n = 3, 330
    q, k, v = (x.cuda() for x in inputs.make_qkv(1, heads, n, 64, seed=9, dtype="f32"))
    G = inputs.make_sketch_matrices(heads, 64, 16, 4, per_head=True, seed=3, dtype="f32").cuda()
    desc = psf.make_desc(1, heads, n, 64, 4, 16, 110, "f32", per_head=True)
    O = psf.psf_causal_attn_fwd(desc, q, k, v, G)
    assert torch.equal(psf.psf_causal_attn_fwd(desc, q, k, v * scale, G), O * scale)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("heads,n,d,r,b", [
    (2, 3024, 64, 16, 48), (8, 3150, 64, 32, 150), (40, 1350, 64, 16, 150), (9, 4545, 64, 64, 101), (4, 5959, 128, 32, 59),
    (1, 14529, 128, 128, 29),
])
def test_an_infinite_value_keeps_its_sign_through_a_state(heads, n, d, r, b, dtype):
    """Sketches and rows of one sign: every weight is positive, so an infinity of V arrives as itself in
    its column of all later rows, and one of dO in dV of all earlier tokens, spans between them or not."""
    at = 7
    q, k, v = (x.cuda() for x in inputs.make_qkv(1, heads, n, d, seed=5, dtype=dtype))
    q, k = q.abs(), k.abs()
    G = inputs.make_sketch_matrices(heads, d, r, 4, per_head=True, seed=3, dtype=dtype).cuda().abs()
    dO = inputs.make_dout(1, heads, n, d, seed=5, dtype=dtype).cuda()
    desc = psf.make_desc(1, heads, n, d, 4, r, b, dtype, per_head=True)
    assert psf.kernel_path(desc) == 0 and psf.general_spans(desc, 0) > 1 and psf.general_spans(desc, 2) > 1
    v[:, :, at, 5], v[:, :, at, 6], v[:, :, at, 7] = float("inf"), float("-inf"), float("nan")
    calls = [psf.psf_causal_attn_fwd(desc, q, k, v, G)[:, :, at:], psf.psf_noncausal_attn_fwd(desc, q, k, v, G)]
    others = [c for c in range(d) if c not in (5, 6, 7)]
    for got in calls:
        assert (got[..., 5] == float("inf")).all() and (got[..., 6] == float("-inf")).all() and got[..., 7].isnan().all()
        assert got[..., others].isfinite().all()
    v = inputs.make_qkv(1, heads, n, d, seed=5, dtype=dtype)[2].cuda()
    dO[:, :, n - at, 3], dO[:, :, n - at, 4] = float("inf"), float("-inf")
    dV = psf.psf_causal_attn_bwd(desc, q, k, v, G, dO)[2][:, :, :n - at]
    assert (dV[..., 3] == float("inf")).all() and (dV[..., 4] == float("-inf")).all()
    assert dV[..., [c for c in range(d) if c not in (3, 4)]].isfinite().all()
