"""psf_decode_prefill where the complete blocks are folded together (bf16 storage, blocks whose tokens
are no multiple of 256, or p = 2): decoded rows against the float64 oracle, and against the same
prompt folded block by block."""
import ctypes

import pytest
import torch

from paper_2310_01655_amd import binding as psf
from paper_2310_01655_amd import inputs
from test_gpu_decode import prefill_then_decode

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("heads,n,n_prompt,d,dv,p,r,b,per_head,learned", [
    (2, 1000, 950, 64, 64, 4, 64, 50, True, False),     # three slices, no tail
    (3, 462, 455, 64, 64, 4, 32, 77, False, False),     # one slice, odd chunk ends, a tail in the cache
    (1, 1536, 1500, 64, 64, 2, 64, 256, False, False),  # p = 2: the rows themselves are the sketches
    (2, 650, 640, 128, 128, 8, 64, 65, True, False),    # two-level sketch, the widest state
    (2, 390, 380, 40, 96, 4, 32, 39, True, False),      # d no multiple of 16, three value tiles
    (1, 192, 149, 64, 64, 4, 64, 48, True, True),       # learned sketches
    (1, 12, 10, 32, 32, 4, 32, 3, True, False),         # less than one chunk of tokens
])
def test_blocks_folded_together(heads, n, n_prompt, d, dv, p, r, b, per_head, learned):
    prefill_then_decode(1, heads, n, n_prompt, d, dv, p, r, b, "bf16", per_head=per_head, learned=learned)


@pytest.mark.parametrize("batch,heads,n_prompt,r,b", [
    (64, 12, 6000, 64, 1000),    # more sketches than the workspace holds at once: two chunks
    (1, 3, 3000, 32, 48),        # eleven slices
])
def test_together_as_block_by_block(batch, heads, n_prompt, r, b):
    """The state's bf16 copy rounds sums of another order: two roundings of 2^-9 apart at most."""
    n, d = n_prompt + b - n_prompt % b, 64
    desc = psf.make_desc(batch, heads, n, d, 4, r, b, "bf16")
    g = torch.Generator(device="cuda")
    g.manual_seed(5)

    def rows(t):
        x = torch.randn(batch, heads, t, d, generator=g, device="cuda")
        return (x / x.norm(dim=-1, keepdim=True)).bfloat16()

    K, V, step = rows(n_prompt), rows(n_prompt), [rows(1) for _ in range(3)]
    G = inputs.make_sketch_matrices(heads, d, r, 4, per_head=False, seed=0, dtype="bf16").cuda()
    assert psf.lib().psf_decode_prefill_workspace_bytes(ctypes.byref(desc), n_prompt) > 0
    out = []
    for together in (True, False):
        state = psf.decode_new_state(desc)
        if together:
            ws = psf.psf_decode_prefill(desc, K, V, G, state)
        else:                                            # no workspace: block by block
            st = psf.lib().psf_decode_prefill(
                ctypes.byref(desc), ctypes.c_void_p(K.data_ptr()), ctypes.c_void_p(V.data_ptr()),
                ctypes.c_void_p(G.data_ptr()), n_prompt, ctypes.c_void_p(state.data_ptr()),
                ctypes.c_size_t(state.numel()), None, ctypes.c_size_t(0),
                ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
            assert st == psf.PSF_OK
        out.append(psf.psf_decode_step(desc, step[0], step[1], step[2], G, n_prompt, state).float())
        torch.cuda.synchronize()
    del ws
    assert torch.isfinite(out[0]).all()
    assert (out[0] - out[1]).norm() <= 2 * 2.0 ** -9 * out[1].norm()
