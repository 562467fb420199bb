"""The forms of the MFMA backward kernels that go by shape and number of units."""
import pytest
import torch

from paper_2310_01655_amd import binding as psf
from paper_2310_01655_amd import inputs

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
