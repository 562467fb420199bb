"""The forms of the MFMA backward kernels that go by shape and number of units."""
import pytest
import torch

import oracle
from paper_2310_01655_amd import binding as psf
from paper_2310_01655_amd import inputs
from parity import as_f64, assert_close_scaled
from test_gpu_learned_backward import run_case as learned_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("r,filled,empty", [
    (32, ("query_side", "key_side"), ("in_block_and_dv", "cross_block_and_sketch_gradient")),
    (64, ("in_block_and_dv", "cross_block_and_sketch_gradient"), ()),
])
def test_stages_are_named_by_what_ran(r, filled, empty):
    desc = psf.make_desc(4, 12, 2048, 64, 4, r, 256, "bf16", per_head=False)
    q, k, v = (x.cuda() for x in inputs.make_qkv(4, 12, 2048, 64, seed=1, dtype="bf16"))
    dO = inputs.make_dout(4, 12, 2048, 64, seed=1, dtype="bf16").cuda()
    G = inputs.make_sketch_matrices(12, 64, r, 4, per_head=False, seed=0, dtype="bf16").cuda()
    psf.psf_causal_attn_bwd(desc, q, k, v, G, dO)                     # kernels load on first use
    _, ms = psf.psf_causal_attn_bwd_timed(desc, q, k, v, G, dO)
    assert list(ms) == ["forward_again", "g_c_and_layouts", "mirror_states", "in_block_and_dv",
                        "cross_block_and_sketch_gradient"] + [nm for nm in filled if nm.endswith("_side")]
    # (every filled stage is a kernel of 50 us and more, an empty one two events in a row)
    for nm in empty:
        assert all(ms[nm] < ms[other] for other in filled), ms


# The mirror states' deals (their blocks in reverse): one tile a wave, two and four, by the number of units, every width;
# dV's cross-block part inside the in-block kernel (d = 128, and r = 32) and as a kernel of its own (d = r = 64).
# Three and more blocks; first, middle and last unit against the float64 oracle.
@pytest.mark.parametrize("units,n,d,p,r,b", [
    (1, 768, 64, 4, 32, 256), (42, 768, 64, 4, 32, 256), (43, 768, 64, 4, 32, 256), (86, 768, 64, 4, 32, 256),
    (129, 768, 64, 4, 32, 256), (171, 768, 64, 4, 32, 256),
    (12, 768, 64, 4, 64, 256), (13, 768, 64, 4, 64, 256), (26, 768, 64, 8, 64, 256), (81, 768, 64, 4, 64, 256),
    (1, 1024, 128, 4, 32, 256), (42, 768, 128, 4, 32, 256), (43, 768, 128, 4, 32, 256), (3, 1536, 128, 4, 32, 512),
    (12, 768, 128, 4, 64, 256), (13, 768, 128, 8, 64, 256), (43, 768, 64, 8, 32, 256),
])
def test_gradients_by_units(units, n, d, p, r, b):
    q, k, v = inputs.make_qkv(1, units, n, d, seed=units + d, dtype="bf16")
    dO = inputs.make_dout(1, units, n, d, seed=units + d, dtype="bf16")
    G = inputs.make_sketch_matrices(units, d, r, p, per_head=False, seed=0, dtype="bf16")
    desc = psf.make_desc(1, units, n, d, p, r, b, "bf16", per_head=False)
    assert psf.bwd_kernel_path(desc) == 3
    got = psf.psf_causal_attn_bwd(desc, *(x.cuda() for x in (q, k, v, G, dO)))
    torch.cuda.synchronize()
    for h in sorted({0, units // 2, units - 1}):
        want = oracle.attn_bwd(*(as_f64(x[0, h]) for x in (q, k, v)), as_f64(G[0]), as_f64(dO[0, h]), p, r, b)
        for name, x, w in zip(("dQ", "dK", "dV"), got, want):
            assert_close_scaled(x[0, h].float().cpu().numpy(), w, "bf16", "%s, unit %d" % (name, h))


# One shared set: slices of three tiles of 256 rows where a unit has five, so that slices cross units; units of one
# tile each, their number without a divisor.
@pytest.mark.parametrize("heads,n,r", [(3, 1280, 32), (3, 1280, 64), (7, 256, 32), (13, 256, 64)])
def test_parameter_sums_by_slices(heads, n, r):
    learned_case(1, heads, n, 64, 64, 4, r, 256, "bf16", per_head=False, path=3)
