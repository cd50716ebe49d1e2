"""The fp32 read on the fp32 matrix instructions against the float64 oracle:
tile and width edges, the exact recomputation, and NaN confined to its rows.

Tolerance 1e-4 (max abs), the fp32 budget; the kernel's own rounding is about
2^-22 of an output at beta >= 0.25.
"""

import numpy as np
import pytest
import torch

import oracle
from paper_2602_07160_amd import inputs

pytestmark = pytest.mark.gpu

TOL = 1e-4


def read(fem, *x):
    print("[case]", [tuple(t.shape) for t in x], flush=True)
    out = fem.fem_softmax_fwd(*(t.cuda() for t in x))
    torch.cuda.synchronize()
    return out.cpu().double().numpy()


def ref(*x):
    return oracle.fem_softmax(*(t.double().numpy() for t in x))


# 32-row blocks and 32-key tiles over four waves: one wave only, a full and a
# ragged last tile, a second tile per wave; widths: each padded width, a
# multiple of four and a ragged one below it
@pytest.mark.parametrize("T", [1, 31, 32, 33, 127, 129, 161])
@pytest.mark.parametrize("d", [1, 7, 32, 36, 64, 100, 128, 130, 252, 256])
def test_edges(fem, T, d):
    x = inputs.draw(9000 + 300 * T + d, 1, 2, T, d, dtype="f32", beta_lo=0.25, beta_hi=4.0)
    assert np.abs(read(fem, *x) - ref(*x)).max() <= TOL


@pytest.mark.parametrize("T,d", [(70, 32), (300, 64), (200, 100), (130, 256)])
def test_late_maximum_is_recomputed(fem, T, d):
    """Values far below the last key's: every earlier row's weighted mean of E
    underflows against the shared column maximum."""
    q, k, v, _ = inputs.draw(9500 + d, 1, 2, T, d, dtype="f32")
    v = -5.0 + 0.1 * v
    v[:, :, -1] = 5.0
    b = torch.full((2, d), 16.0)
    assert np.abs(read(fem, q, k, v, b) - ref(q, k, v, b)).max() <= TOL


def test_nan_value_reaches_its_rows_only(fem):
    q, k, v, b = inputs.draw(9600, 1, 1, 100, 64, dtype="f32", beta_lo=0.25, beta_hi=4.0)
    want = ref(q, k, v, b)
    v[0, 0, 70, 5] = float("nan")
    got = read(fem, q, k, v, b)
    assert np.isnan(got[0, 0, 70:, 5]).all()
    got[0, 0, 70:, 5] = want[0, 0, 70:, 5]
    assert np.abs(got - want).max() <= TOL


# a second tile per wave at the widths whose loads take the narrow forms
@pytest.mark.parametrize("T", [160, 257])
@pytest.mark.parametrize("d", [33, 70, 101, 132, 200, 255])
def test_ragged_widths(fem, T, d):
    x = inputs.draw(9650 + 300 * T + d, 1, 2, T, d, dtype="f32", beta_lo=0.25, beta_hi=4.0)
    assert np.abs(read(fem, *x) - ref(*x)).max() <= TOL


# From |beta v| of about 2^30 on, the rounding of the shift beta max(v) alone
# passes the exponent's range.  Relative to the column's largest value: 2^-20
# (a few roundings of the exponents and of the result).
@pytest.mark.parametrize("size", [1e9, 1e10, 1e30])
@pytest.mark.parametrize("T,d", [(32, 32), (100, 64), (300, 20), (200, 128)])
def test_large_values(fem, T, d, size):
    q, k, v, b = inputs.draw(9700 + T, 1, 2, T, d, dtype="f32", beta_lo=0.25, beta_hi=4.0)
    v[:, :, :, : d // 2] *= size
    v[:, :, :, d // 2] = -size  # a column that holds a mask value
    got, want = read(fem, q, k, v, b), ref(q, k, v, b)
    scale = np.maximum(1.0, np.abs(v.double().numpy()).max(2, keepdims=True))
    assert (np.abs(got - want) / scale).max() <= 2.0 ** -20


@pytest.mark.parametrize("key", [0, 10, 70])
@pytest.mark.parametrize("where", ["k", "v"])
@pytest.mark.parametrize("d", [64, 20, 70])  # 20, 70: a key's row is read on into the next one's
def test_nan_reaches_every_row_that_sees_it(fem, d, where, key):
    q, k, v, b = inputs.draw(9750, 1, 1, 150, d, dtype="f32", beta_lo=0.25, beta_hi=4.0)
    want = ref(q, k, v, b)
    ch = slice(None) if where == "k" else slice(5, 6)
    (k if where == "k" else v)[0, 0, key, 5] = float("nan")
    got = read(fem, q, k, v, b)
    assert np.isnan(got[0, 0, key:, ch]).all()
    got[0, 0, key:, ch] = want[0, 0, key:, ch]
    assert np.abs(got - want).max() <= TOL


def test_infinite_and_lowest_values(fem):
    """+inf in V gives +inf to the rows that see it; the type's lowest value
    (a mask) has no weight, also where it fills a tile or a lane's first keys."""
    q, k, v, b = inputs.draw(9760, 1, 1, 150, 64, dtype="f32", beta_lo=1.0, beta_hi=4.0)
    low = torch.finfo(torch.float32).min
    v[0, 0, 20, 1] = float("inf")
    v[0, 0, 1:10, 2] = low
    v[0, 0, 32:96, 3] = low
    v[0, 0, 1:140, 4] = low
    got = read(fem, q, k, v, b)
    w = v.clone()
    w[0, 0, 20, 1] = 0.0
    want = ref(q, k, w, b)
    assert np.isposinf(got[0, 0, 20:, 1]).all()
    got[0, 0, 20:, 1] = want[0, 0, 20:, 1]
    assert np.abs(got - want).max() <= TOL


@pytest.mark.parametrize("d", [32, 40, 64, 128, 200, 256])
def test_some_outputs_recomputed(fem, d):
    """A few columns of a long context whose maximum comes late: single
    channels of single 32-row blocks, over several rounds of key tiles."""
    q, k, v, b = inputs.draw(9770 + d, 1, 1, 330, d, dtype="f32", beta_lo=1.0, beta_hi=4.0)
    v[0, 0, 31, 3] = v[0, 0, 150, 17] = v[0, 0, 329, d - 1] = 90.0
    b[0, [3, 17, d - 1]] = 4.0
    assert np.abs(read(fem, q, k, v, b) - ref(q, k, v, b)).max() <= TOL


# Launches of many rows, whose short contexts take the 32-row tiles too (the
# cases above are few rows: one workgroup each), at the same edges; first and
# last head.
@pytest.mark.parametrize("T", [1, 31, 32, 33, 127, 129, 161])
@pytest.mark.parametrize("d", [1, 7, 32, 36, 64, 100, 128, 130, 252, 256])
def test_edges_of_tiles(fem, T, d):
    H = 6200 // T + 1
    x = inputs.draw(9000 + 300 * T + d, 1, H, T, d, dtype="f32", beta_lo=0.25, beta_hi=4.0)
    got = read(fem, *x)
    for s in (slice(0, 1), slice(H - 1, H)):
        assert np.abs(got[:, s] - ref(*(t[:, s] for t in x[:3]), x[3][s])).max() <= TOL


@pytest.mark.parametrize("T,d", [(70, 32), (300, 64), (200, 100), (130, 256)])
def test_late_maximum_in_tiles(fem, T, d):
    H = 6200 // T + 1
    q, k, v, _ = inputs.draw(9500 + d, 1, H, T, d, dtype="f32")
    v = -5.0 + 0.1 * v
    v[:, :, -1] = 5.0
    b = torch.full((H, d), 16.0)
    got = read(fem, q, k, v, b)
    assert np.abs(got[:, :2] - ref(q[:, :2], k[:, :2], v[:, :2], b[:2])).max() <= TOL


@pytest.mark.parametrize("d", [64, 20, 70])
@pytest.mark.parametrize("where", ["k", "v", "inf", "lowest", "large"])
def test_special_values_in_tiles(fem, d, where):
    """NaN, +inf, the lowest and large values as above, among many heads."""
    H, T, key = 50, 150, 70
    q, k, v, b = inputs.draw(9780, 1, H, T, d, dtype="f32", beta_lo=1.0, beta_hi=4.0)
    if where == "large":
        v[:, :, :, : d // 2] *= 1e10
        v[:, :, :, d // 2] = -1e30
    if where == "lowest":
        v[0, 0, 1:140, 5] = torch.finfo(torch.float32).min
    want = ref(q[:, :1], k[:, :1], v[:, :1], b[:1])
    ch = slice(None) if where == "k" else slice(5, 6)
    if where in ("k", "v", "inf"):
        (k if where == "k" else v)[0, 0, key, 5] = float("inf" if where == "inf" else "nan")
    got = read(fem, q, k, v, b)[:, :1]
    if where in ("k", "v", "inf"):
        bad = got[0, 0, key:, ch]
        assert (np.isposinf(bad) if where == "inf" else np.isnan(bad)).all()
        got[0, 0, key:, ch] = want[0, 0, key:, ch]
    scale = 1.0
    if where == "large":
        scale = np.maximum(1.0, np.abs(v[:, :1].double().numpy()).max(2, keepdims=True))
    assert (np.abs(got - want) / scale).max() <= TOL


# One workgroup per row or tiles, from the bits: heads of a launch of many rows
# (tiles) are equal alone where that takes tiles too.  Limits of rows, work and T.
@pytest.mark.parametrize("T,d,heads,rows", [
    (32, 32, 32, True), (32, 32, 33, False), (33, 32, 1, False), (48, 20, 8, True),
    (49, 20, 1, False), (16, 20, 72, True), (16, 20, 73, False), (192, 64, 2, True), (193, 64, 1, False),
    (48, 64, 32, True), (48, 64, 33, False), (8, 64, 193, False), (64, 50, 32, True),
    (64, 50, 33, False), (256, 128, 1, True), (257, 128, 1, False), (96, 128, 9, False),
    (96, 96, 14, True), (96, 96, 15, False), (512, 130, 1, True), (513, 130, 1, False),
    (48, 200, 128, True), (48, 200, 129, False), (32, 256, 128, True), (32, 256, 129, False),
])
def test_rows_or_tiles(fem, T, d, heads, rows):
    H = heads + 300_000 // (T * T) + 6200 // T + 1
    x = inputs.draw(9800 + T + d, 1, H, T, d, dtype="f32", beta_lo=0.25, beta_hi=4.0)
    many, few = read(fem, *x)[:, :heads], read(fem, *(t[:, :heads].contiguous() for t in x[:3]),
                                               x[3][:heads])
    assert np.array_equal(many, few) != rows
    assert np.abs(few[:, -1:] - ref(*(t[:, heads - 1 : heads] for t in x[:3]),
                                    x[3][heads - 1 : heads])).max() <= TOL
