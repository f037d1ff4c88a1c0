"""GPU accuracy of the fp32 kernels whose operands are sums of 16-bit terms, where
one value of a row, a column or a tile is far larger than the others: every row,
feature and basis whose result does not hold the large value keeps the fp32
accuracy it has without it (compared part by part: a norm over the tensor would
hide it).  Against the float64 oracle at the fp32 tolerance 1e-5, relative to the
largest value of the part compared."""
import numpy as np
import pytest

import oracle
from gpu_common import F32_LAYER_TOL, normwise, say
from test_gpu_backward import _case
from test_gpu_backward import _run as _run_backward
from test_gpu_window import _inputs, _planned
from test_gpu_window import _run as _run_forward

pytestmark = pytest.mark.gpu

F32_MAX = float(np.finfo(np.float32).max)


def _rows_close(y, ref):
    """Every row against its own largest value."""
    scale = np.abs(ref).max(axis=1, keepdims=True)
    err = np.abs(y - ref) / np.where(scale > 0, scale, 1.0)
    assert err.max() <= F32_LAYER_TOL, (float(err.max()), int(err.max(axis=1).argmax()))


WINDOW = [(4096, 161, 64, 10, 3), (4096, 140, 140, 30, 3), (8192, 96, 100, 12, 1)]


@pytest.mark.parametrize("big", [1e4, 1e6, 1e10, F32_MAX])
@pytest.mark.parametrize("B,n_in,n_out,G,k", WINDOW)
def test_forward_one_large_coefficient(B, n_in, n_out, G, k, big):
    """One large coefficient in every output column: the rows whose input is outside
    its support.  (Those inside it are right to the large term's own rounding.)"""
    x, C, Wb = _inputs(B, n_in, n_out, G, k, "f32")
    C[np.arange(n_out), 3, 2] = np.float32(big)
    assert _planned(B, n_in, n_out, G, k, "f32")
    say(f"range forward coefficient {big:g} {n_in}->{n_out} G={G} k={k}")
    y = _run_forward(x, C, Wb, G, k, "f32")
    rows = np.r_[0:96, B - 32:B]
    ref = oracle.layer(x[rows], C, Wb, G, k=k)
    u = (x[rows, 3].astype(np.float64) + 1) * (G / 2) + k - 2
    out = (u <= -1e-3) | (u >= k + 1 + 1e-3)
    assert out.sum() > 20 and (~out).sum() > 5
    _rows_close(y[rows][out], ref[out])
    _rows_close(y[rows][~out], ref[~out])


@pytest.mark.parametrize("big", [1e6, 1e10, 1e30])
@pytest.mark.parametrize("B,n_in,n_out,G,k", WINDOW[:2])
def test_forward_one_large_silu_weight(B, n_in, n_out, G, k, big):
    """One large SiLU weight in every column, met by a SiLU value of 0 in half the rows."""
    x, C, Wb = _inputs(B, n_in, n_out, G, k, "f32")
    Wb[:, 5] = np.float32(big)
    x[::2, 5] = 0.0
    say(f"range forward silu weight {big:g} {n_in}->{n_out} G={G}")
    y = _run_forward(x, C, Wb, G, k, "f32")
    rows = np.r_[0:64]
    _rows_close(y[rows], oracle.layer(x[rows], C, Wb, G, k=k))


@pytest.mark.parametrize("small", [1e-3, 1e-6, 1e-9, 1e-20])
@pytest.mark.parametrize("B,n_in,n_out,G,k", WINDOW)
def test_forward_small_coefficients_beside_normal_ones(B, n_in, n_out, G, k, small):
    """All features but one with small weights, and rows that meet only those (the
    one feature off the grid, without a SiLU weight); then only some bases small."""
    x, C, Wb = _inputs(B, n_in, n_out, G, k, "f32")
    C[:, 1:] *= np.float32(small)
    Wb[:, 1:] *= np.float32(small)
    Wb[:, 0] = 0.0
    x[::2, 0] = 3.0
    say(f"range forward small {small:g} {n_in}->{n_out} G={G} k={k}")
    rows = np.r_[0:64]
    y = _run_forward(x, C, Wb, G, k, "f32")
    _rows_close(y[rows], oracle.layer(x[rows], C, Wb, G, k=k))
    x, C, Wb = _inputs(B, n_in, n_out, G, k, "f32")
    C[:, :, G // 2:] *= np.float32(small)
    Wb *= np.float32(small)
    x[::2] = np.float32(0.5) + np.abs(x[::2]) / 2  # past the large bases
    x[::2] = np.clip(x[::2], 0.5 + 2.0 * (k + 1) / G if G > 20 else 0.9, 1.0)
    y = _run_forward(x, C, Wb, G, k, "f32")
    _rows_close(y[rows], oracle.layer(x[rows], C, Wb, G, k=k))


@pytest.mark.parametrize("B,n_in,n_out,G,k", WINDOW)
@pytest.mark.parametrize("cs,ws,xs", [(0.0, 1.0, 1e30), (0.25, 1e-3, 1e36), (1.0, 1e-3, 1e38),
                                      (1e12, 1e-20, 1e3), (1e-20, 1.0, 1e20), (1e30, 1.0, 30.0)])
def test_forward_large_inputs(B, n_in, n_out, G, k, cs, ws, xs):
    """Inputs far past the grid, where only the SiLU term counts: finite while the
    layer's sum is, whatever the coefficients' scale."""
    x, C, Wb = _inputs(B, n_in, n_out, G, k, "f32")
    C = (C * cs / 0.1).astype(np.float32)
    Wb = (Wb * ws).astype(np.float32)
    x[::7] = np.where(np.arange(n_in) % 5 == 0, xs, np.where(np.arange(n_in) % 2, 0.0, -60.0))
    say(f"range forward inputs {xs:g} coefficients {cs:g} {ws:g} {n_in}->{n_out} G={G}")
    y = _run_forward(x, C, Wb, G, k, "f32")
    rows = np.r_[0:70]
    ref = oracle.layer(x[rows], C, Wb, G, k=k)
    assert np.abs(ref).max() < 1e38 and np.isfinite(y).all()
    _rows_close(y[rows], ref)


BACK = [(300, 9, 40, 10), (257, 6, 10, 10), (260, 5, 300, 10), (200, 5, 130, 30), (150, 3, 20, 60)]


@pytest.mark.parametrize("big", [1e6, 1e10, 1e30])
@pytest.mark.parametrize("B,n_in,n_out,G", BACK)
def test_dx_one_large_weight(B, n_in, n_out, G, big):
    """One large coefficient, or SiLU weight: dx of the other features, and of its own
    where its derivative is 0 there."""
    x, C, Wb, dy = _case(B, n_in, n_out, G, seed=11, dtype_name="f32")
    say(f"range dx weight {big:g} {n_in}->{n_out} G={G}")
    C1 = C.copy()
    C1[n_out // 2, 1, 2] = np.float32(big)
    got = _run_backward(x, C1, Wb, dy, G, "f32", need_dw=False)[0]
    ref = oracle.layer_backward(x, C1, Wb, dy, G)[0]
    u = (x[:, 1].astype(np.float64) + 1) * (G / 2) + 3 - 2
    out = (u <= -1e-3) | (u >= 4 + 1e-3)
    assert out.sum() > 20 and (~out).sum() > 3
    for f in range(n_in):
        if f != 1:
            assert normwise(got[:, f], ref[:, f]) <= F32_LAYER_TOL, f
    assert normwise(got[out, 1], ref[out, 1]) <= F32_LAYER_TOL
    assert normwise(got[~out, 1], ref[~out, 1]) <= F32_LAYER_TOL
    W1 = Wb.copy()
    W1[n_out // 3, 2] = np.float32(big)
    got = _run_backward(x, C, W1, dy, G, "f32", need_dw=False)[0]
    ref = oracle.layer_backward(x, C, W1, dy, G)[0]
    for f in range(n_in):
        assert normwise(got[:, f], ref[:, f]) <= F32_LAYER_TOL, f


@pytest.mark.parametrize("small", [1e-6, 1e-12])
@pytest.mark.parametrize("B,n_in,n_out,G", BACK)
def test_dx_pruned_and_small_edges(B, n_in, n_out, G, small):
    """One output's gradient far larger than the others', and features whose edges to
    that output are zero, or small: their dx is made of the small gradients.  Then
    one feature of small weights beside ones of normal weights."""
    x, C, Wb, dy = _case(B, n_in, n_out, G, seed=12, dtype_name="f32")
    o1 = n_out // 2
    dy[:, np.arange(n_out) != o1] *= np.float32(small)
    say(f"range dx edges {small:g} {n_in}->{n_out} G={G}")
    for edge in (0.0, small):
        C1, W1 = C.copy(), Wb.copy()
        C1[o1, ::2] *= np.float32(edge)
        W1[o1, ::2] *= np.float32(edge)
        got = _run_backward(x, C1, W1, dy, G, "f32", need_dw=False)[0]
        ref = oracle.layer_backward(x, C1, W1, dy, G)[0]
        for f in range(n_in):
            assert normwise(got[:, f], ref[:, f]) <= F32_LAYER_TOL, (edge, f)
    x, C, Wb, dy = _case(B, n_in, n_out, G, seed=13, dtype_name="f32")
    C[:, 2], Wb[:, 2] = C[:, 2] * np.float32(small), Wb[:, 2] * np.float32(small)
    C[:, 1, : G // 2] *= np.float32(small)
    Wb[:, 1] *= np.float32(small)
    got = _run_backward(x, C, Wb, dy, G, "f32", need_dw=False)[0]
    ref = oracle.layer_backward(x, C, Wb, dy, G)[0]
    for f in range(n_in):
        assert normwise(got[:, f], ref[:, f]) <= F32_LAYER_TOL, f
    low = (x[:, 1] > -1 + 1e-3) & (x[:, 1] < -1 + 2.0 / G * (G // 2 - 3) - 1e-3)
    if low.sum() > 3:
        assert normwise(got[low, 1], ref[low, 1]) <= F32_LAYER_TOL


DW = [(8192, 9, 40, 10), (8300, 5, 130, 30), (8200, 3, 20, 60), (20000, 33, 10, 12), (8257, 7, 300, 8)]


def _columns_close(x, C, Wb, dy, G):
    """Every column of the weight gradients (a feature's basis, or its SiLU weight)
    against its own largest value over the outputs, and every output of it where all
    of its own terms have one sign (else its sum may cancel)."""
    _, dC, dW = _run_backward(x, C, Wb, dy, G, "f32", need_dx=False)
    _, rC, rW = oracle.layer_backward(x, C, Wb, dy, G)
    got, ref = np.concatenate([dC, dW[:, :, None]], 2), np.concatenate([rC, rW[:, :, None]], 2)
    scale = np.abs(ref).max(axis=0, keepdims=True)
    if (dy >= 0).all():
        scale = np.repeat(scale, ref.shape[0], 0)
        scale[..., :-1] = np.abs(rC)
    err = np.abs(got - ref) / np.where(scale > 0, scale, 1.0)
    assert err.max() <= F32_LAYER_TOL, (float(err.max()), np.unravel_index(err.argmax(), err.shape))


# (the SiLU weight's gradient, up to 1.5 times the large one, stays finite in fp32)
@pytest.mark.parametrize("big", [1e4, 1e6, 1e10, 1e15, F32_MAX / 4])
@pytest.mark.parametrize("B,n_in,n_out,G", DW)
def test_dw_one_large_gradient(B, n_in, n_out, G, big):
    """One row of large gradients, for all outputs and for every third."""
    x, C, Wb, dy = _case(B, n_in, n_out, G, seed=21, dtype_name="f32")
    for step in (1, 3):
        d = dy.copy()
        d[B // 2 + 5, ::step] = np.float32(big)
        say(f"range dw gradient {big:g} step {step} B={B} {n_in}->{n_out} G={G}")
        _columns_close(x, C, Wb, d, G)


@pytest.mark.parametrize("small", [1e-3, 1e-6, 1e-9, 1e-12, 1e-20])
@pytest.mark.parametrize("B,n_in,n_out,G", DW)
def test_dw_columns_of_small_gradients(B, n_in, n_out, G, small):
    """Bases that only rows of small gradients meet: many rows, then three; with
    gradients of both signs and of one."""
    x, C, Wb, dy = _case(B, n_in, n_out, G, seed=22, dtype_name="f32", off=0.0)
    rng = np.random.default_rng(5)
    for rows in (np.arange(B) % 2 == 0, np.isin(np.arange(B), [7, B // 2, B - 2])):
        x1, d = x.copy(), dy.copy()
        d[rows] *= np.float32(small)
        # odd features: the rows of small gradients in the upper half, the others below
        x1[:, 1::2] = -np.abs(x1[:, 1::2])
        x1[np.ix_(rows, np.arange(n_in) % 2 == 1)] *= -1
        say(f"range dw small {small:g} rows {int(rows.sum())} B={B} {n_in}->{n_out} G={G}")
        _columns_close(x1, C, Wb, d, G)
        _columns_close(x1, C, Wb, np.abs(d), G)
    # gradients over a wide range in every row, as a softmax leaves them
    d = np.exp(-rng.uniform(0, -np.log(small), dy.shape)).astype(np.float32)
    _columns_close(x, C, Wb, d, G)


@pytest.mark.parametrize("xs", [1e4, 1e8, 1e12])
@pytest.mark.parametrize("B,n_in,n_out,G", DW[:3])
def test_dw_large_input_without_gradient(B, n_in, n_out, G, xs):
    """Inputs far past the grid in rows that some outputs have no gradient in, and a
    feature of tiny inputs beside them."""
    x, C, Wb, dy = _case(B, n_in, n_out, G, seed=23, dtype_name="f32")
    x[11, 1] = xs
    x[12:, 2] *= np.float32(1 / xs)
    x[13:, 0] = np.where(np.arange(B - 13) % 2, 0.0, -40.0)
    dy[11:13, ::2] = 0.0
    dy[:13, 1::4] = 0.0
    say(f"range dw input {xs:g} B={B} {n_in}->{n_out} G={G}")
    _, dC, dW = _run_backward(x, C, Wb, dy, G, "f32", need_dx=False)
    _, rC, rW = oracle.layer_backward(x, C, Wb, dy, G)
    for o in (slice(0, None, 2), slice(1, None, 4), slice(3, None, 4)):
        for f in range(n_in):
            assert normwise(dW[o, f], rW[o, f]) <= F32_LAYER_TOL, f
            assert normwise(dC[o, f], rC[o, f]) <= F32_LAYER_TOL, f


@pytest.mark.parametrize("edge", [0.0, 1e-9, 1e-30])
@pytest.mark.parametrize("B,n_in,n_out,G", BACK)
def test_dx_silu_weights_past_the_grid(B, n_in, n_out, G, edge):
    """Inputs past the grid, where only the SiLU weights count: those of the output with
    the large gradient are zero or small for some features, whose coefficients are not."""
    x, C, Wb, dy = _case(B, n_in, n_out, G, seed=14, dtype_name="f32")
    x[::2] = np.where(x[::2] > 0, 3.0, -2.5) + x[::2]
    o1 = n_out // 2
    dy[:, np.arange(n_out) != o1] *= np.float32(1e-12)
    Wb[o1, ::2] *= np.float32(edge)
    say(f"range dx silu edges {edge:g} {n_in}->{n_out} G={G}")
    got = _run_backward(x, C, Wb, dy, G, "f32", need_dw=False)[0]
    ref = oracle.layer_backward(x, C, Wb, dy, G)[0]
    for f in range(n_in):
        assert normwise(got[::2, f], ref[::2, f]) <= F32_LAYER_TOL, f
        assert normwise(got[1::2, f], ref[1::2, f]) <= F32_LAYER_TOL, f
