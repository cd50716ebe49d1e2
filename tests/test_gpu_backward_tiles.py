"""Backward tile pipeline: lengths around one, two, three and four 64-row
tiles (first, inner and last tile of either pass, full and ragged), at every
width, against the float64 closed forms.

Tolerance, per gradient: 2e-2 of its largest value (bf16 dS in the dQ / dK
products and the forward's bf16-rounded p, as in the other backward tests),
1e-3 for dV and dbeta, whose operands carry hi + lo parts (2^-16) and which
read the normalised posterior.
"""

import numpy as np
import pytest
import torch

import oracle
from paper_2602_07160_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [32, 64, 128])
@pytest.mark.parametrize("T", [63, 65, 127, 128, 129, 191, 193, 256])
def test_tile_edges(fem, T, d):
    print("[case]", T, d, flush=True)
    q, k, v, b = inputs.draw(7100 + T + d, 2, 2, T, d, beta_lo=0.1, beta_hi=8.0)
    g = torch.randn(q.shape, generator=torch.Generator().manual_seed(T))
    x = [t.cuda() for t in (q, k, v, b)]
    out, lse = fem.fem_softmax_fwd_train(*x)
    got = fem.fem_softmax_bwd(*x, out, lse, g.cuda())
    torch.cuda.synchronize()
    want = oracle.fem_softmax_grads(*(t.double().numpy() for t in (q, k, v, b, g)))
    for name, a, w in zip(("dq", "dk", "dv", "dbeta"), got, want):
        a = a.cpu().double().numpy()
        tol = (2e-2 if name in ("dq", "dk") else 1e-3) * np.abs(w).max()
        assert np.abs(a - w).max() <= tol, name
