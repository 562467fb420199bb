"""Distance of the fp32 matrix-core kernels from float64 (fp32 storage, relative 2-norm of the
difference, against the oracle).  The bounds are the errors of the vector kernels on the same inputs
(psf_general.hip, psf_backward.hip with one running sum per result), which the matrix-core kernels
must not exceed: where their sums were longer, gradients came out up to a quarter further off."""
import numpy as np
import pytest

import oracle
from paper_2310_01655_amd import binding as psf
from paper_2310_01655_amd import inputs
from parity import as_f64, errors

pytestmark = pytest.mark.gpu

CASES = [
    # heads, n, d, p, r, b; errors of O, dQ, dK, dV on the vector kernels
    (2, 2400, 128, 8, 32, 240, (9.78e-7, 8.03e-7, 6.75e-7, 6.00e-7)),       # long sums over 128 columns, 8th powers
    (12, 3000, 64, 4, 64, 200, (1.62e-6, 4.66e-7, 4.24e-7, 3.62e-7)),       # 15 blocks
    (30, 1200, 64, 2, 64, 48, (1.36e-6, 2.41e-7, 2.36e-7, 2.18e-7)),        # m(x) = x, pairs across 25 blocks
    (30, 1200, 64, 4, 32, 48, (8.54e-7, 3.96e-7, 3.39e-7, 3.18e-7)),
]


def relative_errors(heads, n, d, p, r, b):
    q, k, v = inputs.make_qkv(1, heads, n, d, seed=11, dtype="f32")
    G = inputs.make_sketch_matrices(heads, d, r, p, per_head=True, seed=3, dtype="f32") if p > 2 else None
    dO = inputs.make_dout(1, heads, n, d, seed=11, dtype="f32")
    desc = psf.make_desc(1, heads, n, d, p, r, b, "f32", per_head=True)
    assert psf.kernel_path(desc) == 0
    args = [x.cuda() if x is not None else None for x in (q, k, v, G)]
    got = [psf.psf_causal_attn_fwd(desc, *args), *psf.psf_causal_attn_bwd(desc, *args, dO.cuda())]
    f = [as_f64(x) if x is not None else None for x in (q, k, v, G)]
    rows = sorted(set(np.random.default_rng(1).integers(0, n, 300)))
    want = [oracle.attn_def_batch(*f, p, r, b, rows=rows)[0], *oracle.attn_bwd_batch(*f, as_f64(dO), p, r, b)[:3]]
    got[0] = got[0][:, :, rows]
    return [errors(x.cpu().numpy(), w)[1] for x, w in zip(got, want)]


@pytest.mark.parametrize("heads,n,d,p,r,b,bounds", CASES)
def test_no_further_from_float64_than_the_vector_kernels(heads, n, d, p, r, b, bounds):
    found = relative_errors(heads, n, d, p, r, b)
    for name, err, bound in zip(("O", "dQ", "dK", "dV"), found, bounds):
        assert err <= bound, "%s: %.3e > %.3e" % (name, err, bound)
