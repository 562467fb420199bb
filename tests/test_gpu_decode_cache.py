"""The decode step's walk over the cached rows of the current block: 128 rows a trip at d = 64, 64 at d = 128, the last one
masked.  Slots on either side of one and of two trips, one workgroup a unit (many units) and several, with and
without a state before the block; rows against the float64 oracle (tolerance of bf16 storage)."""
import pytest
import torch

import oracle
from paper_2310_01655_amd import binding as psf
from paper_2310_01655_amd import inputs
from parity import as_f64, assert_close

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,heads,d,r,b,slots", [
    (64, 12, 64, 32, 300, (127, 255)), (64, 12, 64, 64, 300, (127, 255)), (64, 12, 128, 64, 200, (63, 127)),
    (64, 12, 128, 32, 200, (63, 127)),
    (1, 2, 64, 32, 520, (256, 512)),      # two workgroups a unit: their shares of the cache pass a trip, and two
    (1, 1, 64, 64, 1200, (1026,)),        # eight
    (1, 2, 128, 32, 300, (128, 256)),
])
def test_slots_past_a_trip(batch, heads, d, r, b, slots):
    steps, n = 4, 2 * b
    q, k, v = inputs.make_qkv(batch, heads, n, d, seed=b + r, dtype="bf16")
    G = inputs.make_sketch_matrices(heads, d, r, 4, per_head=False, seed=0, dtype="bf16")
    desc = psf.make_desc(batch, heads, n, d, 4, r, b, "bf16", per_head=False)
    qd, kd, vd, Gd = (x.cuda() for x in (q, k, v, G))
    state = psf.decode_new_state(desc, torch.device("cuda:0"))
    units = sorted({(0, 0), (batch // 2, heads - 1), (batch - 1, heads - 1)})
    for first in [s - 1 for s in slots] + [b + s - 1 for s in slots]:
        psf.psf_decode_prefill(desc, kd[:, :, :first].contiguous(), vd[:, :, :first].contiguous(), Gd, state)
        out = [psf.psf_decode_step(desc, *(x[:, :, pos:pos + 1].contiguous() for x in (qd, kd, vd)), Gd, pos, state)
               for pos in range(first, first + steps)]
        got = torch.cat(out, 2).float().cpu().numpy()
        for bi, h in units:
            want = oracle.attn_def(as_f64(q[bi, h]), as_f64(k[bi, h]), as_f64(v[bi, h]), as_f64(G[0]), 4, r, b,
                                   rows=list(range(first, first + steps)))
            assert_close(got[bi, h], want, "bf16", "unit %d %d, positions from %d" % (bi, h, first))
