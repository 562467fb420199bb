"""Prompt hand-over and steps where their kernels change shape: rows that cannot be copied in
16-byte pieces, the largest number of state slices (added up by a second launch) and the smaller
ones (added up by the slice that arrives last, whose counter must be back at zero for the next
step), block ends inside the steps, prompts whose complete blocks are read in place.  Against the
float64 oracle with the bounds of parity.py."""
import numpy as np
import pytest
import torch

import oracle
from paper_2310_01655_amd import binding as psf
from paper_2310_01655_amd import inputs
from parity import as_f64, assert_close

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,heads,d,dv,p,r,b,prompt,dtype", [
    (1, 2, 33, 21, 4, 16, 40, 75, "bf16"),        # odd widths: element by element
    (1, 1, 100, 100, 2, 100, 24, 50, "f32"),      # 16 slices a unit: second launch
    (1, 3, 64, 64, 4, 64, 48, 130, "bf16"),       # 8 slices, last one finishes; fold inside the steps
    (2, 2, 64, 64, 4, 32, 256, 300, "bf16"),      # complete block read in place, tail of 44
    (1, 1, 128, 128, 8, 64, 64, 17, "bf16"),      # prompt inside the first block
    (3, 1, 64, 64, 4, 32, 100, 200, "f32"),       # no tail
    (1, 1, 136, 64, 4, 16, 30, 47, "f32"),        # above the matrix kernels' widths
])
def test_prompt_then_steps(batch, heads, d, dv, p, r, b, prompt, dtype):
    steps, n = 20, (prompt + 20 + b - 1) // b * b
    q, k, v = inputs.make_qkv(batch, heads, n, d, dv=dv, seed=5, dtype=dtype)
    G = inputs.make_sketch_matrices(heads, d, r, p, per_head=True, seed=2, dtype=dtype) if p > 2 else None
    desc = psf.make_desc(batch, heads, n, d, p, r, b, dtype, dv=dv, per_head=True)
    Gd = G.cuda() if G is not None else None
    state = psf.decode_new_state(desc)
    rows = list(range(prompt, prompt + steps))
    want, _ = oracle.attn_def_batch(as_f64(q), as_f64(k), as_f64(v), as_f64(G) if G is not None else None, p, r, b,
                                    rows=rows)
    for _ in range(2):                            # the second hand-over starts from a used state
        psf.psf_decode_prefill(desc, k[:, :, :prompt].contiguous().cuda(), v[:, :, :prompt].contiguous().cuda(), Gd,
                               state)
        got = [psf.psf_decode_step(desc, *(x[:, :, i].unsqueeze(2).contiguous().cuda() for x in (q, k, v)), Gd, i,
                                   state) for i in rows]
        got = torch.stack([g.reshape(batch, heads, dv) for g in got], 2).float().cpu().numpy()
        assert_close(got, want, dtype, "steps")
