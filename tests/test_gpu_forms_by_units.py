"""Kernels whose form goes by the number of units, at the numbers where it changes: the state kernel's deals (one or
two tiles a wave, two waves a SIMD, the full deal), the sketches as one launch or two, and the decode step for few and
many units.  First, middle and last unit against the float64 oracle."""
import pytest
import torch

import oracle
from paper_2310_01655_amd import binding as psf
from paper_2310_01655_amd import inputs
from parity import as_f64, assert_close, oracle_units_rows
from test_gpu_decode import prefill_then_decode

pytestmark = pytest.mark.gpu


# r = 32 deals 3 workgroups a unit, r = 64 10; d = 128 the same: at most 128 or 256 of them, twice as many, and past it;
# more than 384 parts (of 256 rows with b = 256) are two launches of the sketches
@pytest.mark.parametrize("units,n,d,r,b", [
    (1, 512, 64, 32, 256), (42, 512, 64, 32, 256), (43, 512, 64, 32, 256), (85, 512, 64, 32, 256), (86, 768, 64, 32, 256),
    (129, 512, 64, 32, 256), (171, 512, 64, 32, 256), (12, 768, 64, 64, 256), (13, 512, 64, 64, 256),
    (26, 512, 64, 64, 256), (81, 512, 64, 64, 256), (25, 512, 128, 64, 256), (43, 512, 128, 32, 256), (47, 1024, 64, 32, 1024),
    (192, 512, 64, 32, 256), (193, 512, 64, 32, 256), (192, 512, 64, 64, 256), (193, 512, 64, 64, 256),
    (16, 6144, 64, 64, 256), (17, 6144, 64, 64, 256),       # the same with the values' role: fp16 states beside the rows
])
def test_states_and_sketches_by_units(units, n, d, r, b):
    cfg = dict(batch=1, heads=units, n=n, d=d, p=4, r=r, b=b, dtype="bf16", per_head=False)
    q, k, v = inputs.make_qkv(1, units, n, d, seed=units + r, dtype="bf16")
    G = inputs.make_sketch_matrices(units, d, r, 4, per_head=False, seed=0, dtype="bf16")
    desc = psf.make_desc(1, units, n, d, 4, r, b, "bf16", per_head=False)
    assert psf.kernel_path(desc) == 1
    args = [x.cuda() for x in (q, k, v, G)]
    causal, plain = psf.psf_causal_attn_fwd(desc, *args), psf.psf_noncausal_attn_fwd(desc, *args)
    torch.cuda.synchronize()
    at = sorted({0, units // 2, units - 1})
    rows = [0, 31, 127, 128, b - 1, n - b, n - b + 1, n - 129, n - 1]
    want = oracle_units_rows(cfg, q, k, v, G, [(0, h) for h in at], rows)
    for h in at:
        assert_close(causal[0, h, rows].float().cpu().numpy(), want[(0, h)], "bf16", "causal, unit %d" % h)
        full = oracle.attn_noncausal(as_f64(q[0, h]), as_f64(k[0, h]), as_f64(v[0, h]), as_f64(G[0]), 4, r)
        assert_close(plain[0, h].float().cpu().numpy(), full, "bf16", "no mask, unit %d" % h)


# both widths of rows and of sketches, a cache of no, few and many rows, a state and none, alone and one workgroup a unit
# (where the cache goes through the kernel's loop more than once: test_gpu_decode_cache.py)
@pytest.mark.parametrize("batch,heads,n,n_prompt,d,r,b", [
    (1, 1, 192, 126, 128, 64, 64), (1, 2, 99, 65, 128, 32, 33), (1, 3, 140, 70, 64, 64, 70), (1, 2, 64, 31, 64, 32, 64),
    (16, 16, 36, 30, 128, 64, 12), (16, 17, 36, 33, 64, 64, 12),
])
def test_decode_step_widths_and_slots(batch, heads, n, n_prompt, d, r, b):
    prefill_then_decode(batch, heads, n, n_prompt, d, d, 4, r, b, "bf16", per_head=False)


def test_decode_step_of_rows_off_the_16_byte_grid():
    batch, heads, n, d, r, b = 1, 2, 48, 64, 64, 16
    q, k, v = inputs.make_qkv(batch, heads, n, d, seed=5, dtype="bf16")
    G = inputs.make_sketch_matrices(heads, d, r, 4, per_head=False, seed=0, dtype="bf16")
    desc = psf.make_desc(batch, heads, n, d, 4, r, b, "bf16", per_head=False)
    state, out = psf.decode_new_state(desc, torch.device("cuda:0")), []
    room = torch.empty(3, heads * d + 1, dtype=torch.bfloat16, device="cuda")
    for pos in range(n):
        room[:, 1:] = torch.stack([x[0, :, pos].reshape(-1) for x in (q, k, v)]).cuda()
        rows = [room[i, 1:].view(batch, heads, 1, d) for i in range(3)]
        assert rows[0].data_ptr() % 16 != 0
        out.append(psf.psf_decode_step(desc, *rows, G.cuda(), pos, state))
    torch.cuda.synchronize()
    want, _ = oracle.attn_def_batch(as_f64(q), as_f64(k), as_f64(v), as_f64(G), 4, r, b)
    assert_close(torch.cat(out, 2).float().cpu().numpy(), want, "bf16", "rows off the grid")
