"""The softmax read with two key groups per 32-row block (small launches)
against the oracle, and against the one-group kernel on the same rows.

Edges: a first tile whose second half is masked for every row of a block, a
tile with no key in the second half (T <= 32, encoder), ragged last tiles,
both sides of the dispatch rule.  Tolerance 2e-2 (the bf16 budget); between
the two kernels, 2^-7 (their P and E round at different shifts: 2^-9 of P and
at most 2^-8 / beta <= 2^-7 of E).
"""

import numpy as np
import pytest
import torch

import oracle
from paper_2602_07160_amd import inputs

pytestmark = pytest.mark.gpu

TOL = 2e-2


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("dk,dv", [(32, 32), (64, 64), (128, 128), (64, 32), (128, 64)])
@pytest.mark.parametrize("T", [1, 31, 33, 63, 97, 128, 129, 255, 300])
def test_small_launches(fem, T, dk, dv, causal):
    print("[case]", T, dk, dv, causal, flush=True)
    q, k, v, b = inputs.draw(8100 + T + dk + dv, 1, 2, T, dk, dv, beta_lo=0.1, beta_hi=8.0)
    out = fem.fem_softmax_fwd_ex(*(t.cuda() for t in (q, k, v, b)), causal=causal)
    torch.cuda.synchronize()
    ref = oracle.fem_softmax if causal else oracle.fem_softmax_encoder
    want = ref(*(t.double().numpy() for t in (q, k, v, b)))
    assert np.abs(out.cpu().double().numpy() - want).max() <= TOL


@pytest.mark.parametrize("d", [32, 64, 128])
def test_both_kernels_agree(fem, d):
    """The same heads alone (two key groups) and among many (one)."""
    q, k, v, b = (t.cuda() for t in inputs.draw(8300 + d, 20, 16, 300, d, beta_lo=0.5, beta_hi=8.0))
    many = fem.fem_softmax_fwd(q, k, v, b)
    few = fem.fem_softmax_fwd(*(t[:1].contiguous() for t in (q, k, v)), b)
    lam = torch.rand(q.shape, device="cuda")
    gmany = fem.fem_softmax_gated_fwd(q, k, v, b, lam)
    gfew = fem.fem_softmax_gated_fwd(*(t[:1].contiguous() for t in (q, k, v)), b,
                                     lam[:1].contiguous())
    torch.cuda.synchronize()
    assert (many[:1] - few).abs().max().item() <= 2.0 ** -7
    assert (gmany[:1] - gfew).abs().max().item() <= 2.0 ** -7


def test_repair_and_lse_with_two_groups(fem):
    """Rows that underflow against the shared column shift, and the
    log-normaliser merged from the two groups."""
    q, k, v, _ = inputs.draw(8400, 1, 2, 200, 64)
    v = (-5.0 + 0.1 * v.float()).to(torch.bfloat16)
    v[:, :, -1] = 5.0
    b = torch.full((2, 64), 16.0)
    out, lse = fem.fem_softmax_fwd_train(*(t.cuda() for t in (q, k, v, b)))
    torch.cuda.synchronize()
    want = oracle.fem_softmax(*(t.double().numpy() for t in (q, k, v, b)))
    assert np.abs(out.cpu().double().numpy() - want).max() <= TOL
    s = torch.matmul(q.double(), k.double().transpose(2, 3)) / 8.0
    s = s.masked_fill(torch.ones(200, 200, dtype=torch.bool).triu(1), -np.inf)
    assert (lse.cpu().double() - torch.logsumexp(s, -1)).abs().max().item() <= 1e-2


# Which kernel a launch takes, from the bits: the same heads in a launch of many
# (one key group) are equal where the smaller one takes one group too, and
# differ (P is rounded at other shifts) where it takes two.
@pytest.mark.parametrize("dk,dv,T,heads,two", [
    (64, 64, 256, 128, True), (64, 64, 256, 146, False), (128, 128, 200, 140, False),
    (64, 32, 256, 140, False), (32, 32, 256, 146, True), (128, 128, 500, 70, True),
    (128, 128, 400, 76, False), (64, 64, 512, 92, False), (32, 32, 500, 96, True),
    (32, 32, 500, 98, False), (128, 64, 768, 60, True), (64, 64, 768, 66, False),
    (128, 128, 1000, 52, True), (128, 128, 1000, 56, False), (128, 128, 2048, 32, True),
    (128, 128, 60, 128, True), (128, 128, 60, 300, False),
])
def test_rule(fem, dk, dv, T, heads, two):
    many = 2 * (max(300, heads) if T <= 256 else 160)
    q, k, v, b = (t.cuda() for t in inputs.draw(8500 + T + dk + dv, many // 2, 2, T, dk, dv,
                                                beta_lo=0.1, beta_hi=8.0))
    ref = fem.fem_softmax_fwd_ex(q, k, v, b)[: heads // 2]
    got = fem.fem_softmax_fwd_ex(*(t[: heads // 2].contiguous() for t in (q, k, v)), b)
    torch.cuda.synchronize()
    assert torch.equal(ref, got) != two
