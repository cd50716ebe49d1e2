"""The softmax reads with one key group a workgroup (launches that fill the
chip) against the oracle: encoder, half widths, bf16 output, the training pair,
the channel split of the lo products and the repair of underflow, at a ragged
length.  Heads of the first and the last batch are compared; that a launch took
one group shows in the bits, which differ from the same heads' alone (two
groups round P and E at other shifts).

Tolerance 2e-2 (the bf16 budget); gradients as in test_gpu_backward.
"""

import numpy as np
import pytest
import torch

import oracle
from paper_2602_07160_amd import inputs
from test_gpu_backward import check_grads, dbeta_floor, grad_scales, lse_ref
from test_gpu_softmax import SPLIT_PATTERNS, split_beta

pytestmark = pytest.mark.gpu

TOL = 2e-2
PAIRS = [(32, 32), (64, 64), (128, 128), (64, 32), (128, 64)]


def f64(*x):
    return [t.cpu().double().numpy() for t in x]


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("dk,dv", PAIRS)
def test_read(fem, dk, dv, causal):
    B, H, T = 20, len(SPLIT_PATTERNS), 300  # 280 workgroups of 256 rows
    print("[case]", B, H, T, dk, dv, causal, flush=True)
    q, k, v, _ = inputs.draw(8600 + dk + dv, B, H, T, dk, dv)
    b = split_beta(dv, 8610 + dk + dv)
    x = [t.cuda() for t in (q, k, v)]
    out = fem.fem_softmax_fwd_ex(*x, b.cuda(), causal=causal)
    half = fem.fem_softmax_fwd_ex(*x, b.cuda(), causal=causal, out_dtype=torch.bfloat16)
    alone = fem.fem_softmax_fwd_ex(*(t[:1].contiguous() for t in x), b.cuda(), causal=causal)
    torch.cuda.synchronize()
    assert not torch.equal(out[:1], alone)
    assert torch.equal(half, out.to(torch.bfloat16))
    ref = oracle.fem_softmax if causal else oracle.fem_softmax_encoder
    for s in (slice(0, 1), slice(B - 1, B)):
        want = ref(*f64(q[s], k[s], v[s], b))
        assert np.abs(f64(out[s])[0] - want).max() <= TOL


@pytest.mark.parametrize("d", [32, 64, 128])
def test_gated(fem, d):
    B, H, T = 20, len(SPLIT_PATTERNS), 300
    print("[case]", B, H, T, d, flush=True)
    q, k, v, _ = inputs.draw(8630 + d, B, H, T, d)
    b = split_beta(d, 8640 + d)
    lam, g = inputs.draw_gates(8650 + d, B, H, T, d)
    x = [t.cuda() for t in (q, k, v)]
    out = fem.fem_softmax_gated_fwd(*x, b.cuda(), lam.cuda(), g.cuda())
    alone = fem.fem_softmax_gated_fwd(*(t[:1].contiguous() for t in x), b.cuda(),
                                      lam[:1].cuda(), g[:1].cuda())
    torch.cuda.synchronize()
    assert not torch.equal(out[:1], alone)
    for s in (slice(0, 1), slice(B - 1, B)):
        n = f64(q[s], k[s], v[s], b, lam[s], g[s])
        err = np.abs(f64(out[s])[0] - oracle.fem_softmax_ltl(*n)) / np.maximum(1.0, n[-1])
        assert err.max() <= TOL


@pytest.mark.parametrize("d", [32, 64, 128])
def test_training_pair(fem, d):
    """Output gradients only in two batches, so that dbeta is theirs too."""
    B, H, T = 80, 2, 300  # 320 workgroups
    print("[case]", B, H, T, d, flush=True)
    q, k, v, b = inputs.draw(8660 + d, B, H, T, d, beta_lo=0.1, beta_hi=8.0)
    some = [0, B - 1]
    g = torch.zeros(B, H, T, d)
    g[some] = torch.randn(2, H, T, d, generator=torch.Generator().manual_seed(8670 + d))
    x = [t.cuda() for t in (q, k, v, b)]
    out, lse = fem.fem_softmax_fwd_train(*x)
    grads = fem.fem_softmax_bwd(*x, out, lse, g.cuda())
    alone, _ = fem.fem_softmax_fwd_train(*(t[:1].contiguous() for t in x[:3]), x[3])
    torch.cuda.synchronize()
    assert not torch.equal(out[:1], alone)
    qs, ks, vs, gs = q[some], k[some], v[some], g[some]
    assert np.abs(f64(out[some])[0] - oracle.fem_softmax(*f64(qs, ks, vs, b))).max() <= TOL
    assert np.abs(f64(lse[some])[0] - lse_ref(qs, ks)).max() <= 1e-2
    got = f64(*(t[some] for t in grads[:3]), grads[3])
    want = oracle.fem_softmax_grads(*f64(qs, ks, vs, b, gs))
    check_grads(got, want, f"one group d{d}", dbeta_floor(vs, b, gs), grad_scales(qs, ks, vs, b, gs))
    assert all((t[1:-1] == 0).all() for t in grads[:3])


@pytest.mark.parametrize("d", [32, 64, 128])
def test_repair(fem, d):
    """Rows that underflow against the shared column shift, in the last batch."""
    B, H, T = 150, 2, 200  # 300 workgroups
    print("[case]", B, H, T, d, flush=True)
    q, k, v, _ = inputs.draw(8680 + d, B, H, T, d)
    v[-1] = (-5.0 + 0.1 * v[-1].float()).to(torch.bfloat16)
    v[-1, :, -1] = 5.0
    b = torch.full((H, d), 16.0)
    x = [t.cuda() for t in (q, k, v)]
    out = fem.fem_softmax_fwd(*x, b.cuda())
    alone = fem.fem_softmax_fwd(*(t[:1].contiguous() for t in x), b.cuda())
    torch.cuda.synchronize()
    assert not torch.equal(out[:1], alone)
    for s in (slice(0, 1), slice(B - 1, B)):
        assert np.abs(f64(out[s])[0] - oracle.fem_softmax(*f64(q[s], k[s], v[s], b))).max() <= TOL


# the encoder's rule: two groups up to 128 workgroups of 256 rows
@pytest.mark.parametrize("dk,dv", PAIRS)
@pytest.mark.parametrize("heads,two", [(64, True), (66, False)])
def test_encoder_rule(fem, dk, dv, heads, two):
    q, k, v, b = (t.cuda() for t in inputs.draw(8690 + dk + dv, 80, 2, 300, dk, dv,
                                                beta_lo=0.1, beta_hi=8.0))
    many = fem.fem_softmax_fwd_ex(q, k, v, b, causal=False)[: heads // 2]
    got = fem.fem_softmax_fwd_ex(*(t[: heads // 2].contiguous() for t in (q, k, v)), b,
                                 causal=False)
    torch.cuda.synchronize()
    assert torch.equal(many, got) != two


def test_gated_and_plain_read_by_different_rules(fem):
    """lam = 1 and g = 1 give the plain read; here the plain read takes two key
    groups and the gated pass one, so they agree to the rounding of P and E at
    different shifts (2^-9 of P, at most 2^-8 / beta of E; beta >= 0.5)."""
    q, k, v, b = (t.cuda() for t in inputs.draw(8700, 2, 16, 2048, 128, beta_lo=0.5, beta_hi=8.0))
    one = torch.ones(q.shape, device="cuda")
    plain = fem.fem_softmax_fwd(q, k, v, b)
    gated = fem.fem_softmax_gated_fwd(q, k, v, b, one, one)
    torch.cuda.synchronize()
    assert (plain - gated).abs().max().item() <= 2.0 ** -7
