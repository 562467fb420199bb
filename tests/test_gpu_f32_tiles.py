"""The fp32 matrix-core kernels of the general path at the edges of their tiles: sketch and head
widths around multiples of 16 and 64, blocks around 16 and 64 tokens, last tiles with one row,
spans with and without states.  Against the float64 oracle with the
bounds of parity.py (1e-4 for fp32 storage; sums of non-negative fp32 terms err by about 1e-6)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2310_01655_amd import binding as psf
from paper_2310_01655_amd import inputs
from parity import as_f64, assert_close, assert_close_scaled, gpu_attn, oracle_attn

pytestmark = pytest.mark.gpu

CASES = [
    # batch, heads, n, d, dv, p, r, b, dtype, local
    (1, 2, 2046, 64, 64, 4, 16, 66, "f32", psf.LOCAL_EXACT),       # many spans
    (2, 3, 1040, 64, 64, 4, 17, 65, "f32", psf.LOCAL_EXACT),       # a sketch tile with one column
    (1, 1, 2400, 60, 62, 4, 33, 48, "bf16", psf.LOCAL_EXACT),      # widths that four does not divide
    (1, 2, 2040, 65, 64, 4, 16, 120, "f32", psf.LOCAL_EXACT),      # wide tiles, one column over
    (1, 1, 1530, 128, 128, 8, 32, 255, "f32", psf.LOCAL_SKETCH),
    (1, 1, 2600, 100, 128, 2, 100, 100, "f32", psf.LOCAL_EXACT),     # m(x) = x, 100 columns
    (1, 1, 390, 128, 128, 16, 128, 130, "bf16", psf.LOCAL_EXACT),  # largest sizes, three levels
    (40, 14, 66, 16, 8, 4, 8, 33, "f32", psf.LOCAL_EXACT),         # many tiny sequences
    (16, 34, 65, 128, 16, 4, 16, 65, "bf16", psf.LOCAL_EXACT),
    (1, 1, 1, 64, 64, 4, 32, 1, "f32", psf.LOCAL_EXACT),
    (1, 2, 1300, 64, 64, 4, 32, 13, "f32", psf.LOCAL_SKETCH),
]


def case_inputs(batch, heads, n, d, dv, p, r, b, dtype):
    q, k, v = inputs.make_qkv(batch, heads, n, d, dv=dv, seed=7, dtype=dtype)
    G = inputs.make_sketch_matrices(heads, d, r, p, per_head=True, seed=3, dtype=dtype) if p > 2 else None
    return q, k, v, G


@pytest.mark.parametrize("batch,heads,n,d,dv,p,r,b,dtype,local", CASES)
def test_forward_and_backward_at_tile_edges(batch, heads, n, d, dv, p, r, b, dtype, local):
    q, k, v, G = case_inputs(batch, heads, n, d, dv, p, r, b, dtype)
    dO = inputs.make_dout(batch, heads, n, dv, seed=7, dtype=dtype)
    desc = psf.make_desc(batch, heads, n, d, p, r, b, dtype, dv=dv, local=local, per_head=True)
    assert psf.kernel_path(desc) == 0
    args = [x.cuda() if x is not None else None for x in (q, k, v, G)]
    O = psf.psf_causal_attn_fwd(desc, *args)
    N = psf.psf_noncausal_attn_fwd(desc, *args)
    grads = psf.psf_causal_attn_bwd(desc, *args, dO.cuda())
    ol = oracle.LOCAL_EXACT if local == psf.LOCAL_EXACT else oracle.LOCAL_SKETCH
    f = [as_f64(x) if x is not None else None for x in (q, k, v, G)]
    want, _ = oracle.attn_def_batch(*f, p, r, b, local=ol)
    assert_close(O.float().cpu().numpy(), want, dtype, "forward")
    last = heads - 1
    want = oracle.attn_noncausal(f[0][0, last], f[1][0, last], f[2][0, last],
                                 f[3][last] if G is not None else None, p, r)
    want = want[0] if isinstance(want, tuple) else want
    assert_close(N[0, last].float().cpu().numpy(), want, dtype, "noncausal")
    wants = oracle.attn_bwd_batch(*f, as_f64(dO), p, r, b, local=ol)
    for name, got, w in zip(("dQ", "dK", "dV"), grads, wants):
        assert_close_scaled(got.float().cpu().numpy(), w, dtype, name)


@pytest.mark.parametrize("n,at", [(96, 37), (1300, 901)])
def test_a_later_infinity_does_not_reach_earlier_rows(n, at):
    cfg = dict(batch=1, heads=2, n=n, d=64, p=4, r=32, b=n // 4, dtype="f32", per_head=True)
    q, k, v, G = case_inputs(1, 2, n, 64, 64, 4, 32, n // 4, "f32")
    want, _ = gpu_attn(cfg, q, k, v, G)
    v[:, :, at, 5] = float("inf")
    v[:, :, at, 6] = float("nan")
    got, _ = gpu_attn(cfg, q, k, v, G)
    assert torch.isfinite(got[:, :, :at]).all()
    torch.testing.assert_close(got[:, :, :at], want[:, :, :at], rtol=1e-5, atol=1e-6)   # fp32 sums in another order
    assert not torch.isfinite(got[:, :, at:, 5:7]).any()


@pytest.mark.parametrize("heads,n,d,dv,r,b,spans", [
    (2, 4096, 16, 16, 16, 4096, (0, 16, 0)),        # without a mask, one block: the records outgrow the states' room
    (1, 4096, 128, 16, 8, 512, (8, 16, 8)),         # causal and backward too; the upper half of a record is empty
    (1, 4096, 64, 1, 16, 1024, (4, 16, 4)),         # one value column
])
def test_records_that_need_more_room_than_the_vector_kernels_states(heads, n, d, dv, r, b, spans):
    q, k, v, G = case_inputs(1, heads, n, d, dv, 4, r, b, "f32")
    dO = inputs.make_dout(1, heads, n, dv, seed=7, dtype="f32")
    desc = psf.make_desc(1, heads, n, d, 4, r, b, "f32", dv=dv, per_head=True)
    assert tuple(psf.general_spans(desc, i) for i in range(3)) == spans
    args = [x.cuda() for x in (q, k, v, G)]
    O = psf.psf_causal_attn_fwd(desc, *args)
    N = psf.psf_noncausal_attn_fwd(desc, *args)
    grads = psf.psf_causal_attn_bwd(desc, *args, dO.cuda())
    f, rows = [as_f64(x) for x in (q, k, v, G)], [0, 1, b - 1, b % n, n // 2 + 1, n - 2, n - 1]
    want, _ = oracle.attn_def_batch(*f, 4, r, b, rows=rows)
    assert_close(O[:, :, rows].float().cpu().numpy(), want, "f32", "forward")
    last = heads - 1
    want = oracle.attn_noncausal(f[0][0, last, rows], *(x[0, last] for x in f[1:3]), f[3][last], 4, r)
    assert_close(N[0, last, rows].float().cpu().numpy(), want[0] if isinstance(want, tuple) else want, "f32", "noncausal")
    for name, got, w in zip(("dQ", "dK", "dV"), grads, oracle.attn_bwd_batch(*f, as_f64(dO), 4, r, b)):
        assert_close_scaled(got.float().cpu().numpy(), w, "f32", name)


def test_the_static_scratch_takes_a_call_whose_records_do_not_fit_it():
    desc = psf.make_desc(1, 40, 16384, 128, 4, 4, 16, "f32", dv=1)
    assert psf.general_spans(desc) == -1 and psf.workspace_bytes(desc) <= psf.STATIC_SCRATCH_BYTES
    q, k, v = inputs.make_qkv(1, 40, 16384, 128, dv=1, seed=7, dtype="f32")
    G = inputs.make_sketch_matrices(40, 128, 4, 4, per_head=False, seed=3, dtype="f32")
    args = [x.cuda() for x in (q, k, v, G)]
    O = psf.psf_causal_attn_fwd(desc, *args)
    again = torch.empty_like(O)
    psf.psf_causal_attn_fwd_static(desc, *args, again)
    assert torch.equal(O, again)
    rows = [0, 15, 16, 8000, 16383]
    want, _ = oracle.attn_def_batch(*(as_f64(x) for x in (q, k, v, G)), 4, 4, 16, rows=rows)
    assert_close(O[:, :, rows].float().cpu().numpy(), want, "f32", "forward")
