"""GPU parity of the backward's matrix-core kernels against the float64 oracle
where they can go wrong: the weight gradient on whole features per 256 K rows
(bf16; fp32 from 8192 rows on, as two fp16 terms per operand scaled per output
and per feature) and dx (fp32 likewise, scaled per row and per K tile; bf16 with
two row tiles per wave): features of 16, 32, 64, 128 and 256 K rows, and ones
that do not divide 256; column tiles and chunks of outputs, whole, ragged and
several; odd feature counts; ragged batches; dx alone and the weights alone;
scales far from 1; non-finite inputs, gradients and weights.  Tolerances as in
test_gpu_backward.py: 1e-5 in fp32, 2e-2 in bf16, normwise per gradient."""
import numpy as np
import pytest

import oracle
from gpu_common import device, normwise, say, torch
from paper_2609_01956_amd import binding as kb
from test_gpu_backward import _case, _check, _run

pytestmark = pytest.mark.gpu

F32 = [
    # (B, in, out, G)
    (8192, 9, 10, 12), (8193, 17, 33, 5), (8300, 33, 64, 10), (9000, 16, 100, 3),
    (8192, 12, 128, 10), (8200, 5, 129, 10), (8257, 7, 300, 8), (8192, 9, 40, 13),
    (8999, 3, 33, 50), (8192, 3, 70, 100), (8200, 2, 20, 200), (8192, 2, 17, 250),
    (40000, 3, 20, 10), (8192, 1, 1, 1),
]
BF16 = [(300, 9, 10, 12), (1000, 33, 130, 10), (8257, 7, 300, 8), (513, 40, 600, 5),
        (999, 3, 33, 50), (700, 3, 70, 100), (200, 2, 20, 200), (512, 2, 17, 250),
        (40000, 3, 20, 10), (2049, 18, 256, 10)]


@pytest.mark.parametrize("dtype_name,B,n_in,n_out,G",
                         [("f32", *c) for c in F32] + [("bf16", *c) for c in BF16])
def test_backward_matrix_kernels_match_oracle(dtype_name, B, n_in, n_out, G):
    x, C, Wb, dy = _case(B, n_in, n_out, G, seed=B + n_in + G, dtype_name=dtype_name)
    say(f"backward split {dtype_name} B={B} {n_in}->{n_out} G={G}")
    got = _run(x, C, Wb, dy, G, dtype_name)
    ref = oracle.layer_backward(x, C, Wb, dy, G)
    for g, r, what in zip(got, ref, ("dx", "dC", "dWb")):
        _check(g, r, dtype_name, what)
    only_dx = _run(x, C, Wb, dy, G, dtype_name, need_dw=False)
    only_dw = _run(x, C, Wb, dy, G, dtype_name, need_dx=False)
    assert np.array_equal(only_dx[0], got[0])
    assert np.array_equal(only_dw[1], got[1]) and np.array_equal(only_dw[2], got[2])


@pytest.mark.parametrize("ey,ex,ew", [(-100, 0, 0), (60, 0, -60), (0, 20, 0), (0, -30, 90), (-20, 3, -60)])  # (products stay normal fp32 values)
def test_backward_f32_scales(ey, ex, ew):
    """dy, x (past the grid: SiLU values up to 2^ex) and weights of other
    magnitudes, each mixed with far smaller ones in other rows and features."""
    B, n_in, n_out, G = 8192, 6, 40, 10
    x, C, Wb, dy = _case(B, n_in, n_out, G, seed=5, dtype_name="f32")
    dy = (dy * 2.0 ** ey).astype(np.float32)
    dy[::3] *= np.float32(2.0 ** -20)
    x[:, 1] *= np.float32(2.0 ** ex)
    C = (C * 2.0 ** ew).astype(np.float32)
    Wb = (Wb * 2.0 ** ew).astype(np.float32)
    C[:, 4], Wb[:, 4] = C[:, 4] * np.float32(2.0 ** -9), Wb[:, 4] * np.float32(2.0 ** -9)
    say(f"backward scales {ey} {ex} {ew}")
    got = _run(x, C, Wb, dy, G, "f32")
    ref = oracle.layer_backward(x, C, Wb, dy, G)
    for f in range(n_in):
        _check(got[0][:, f], ref[0][:, f], "f32", f"dx {f}")
        _check(got[1][:, f], ref[1][:, f], "f32", f"dC {f}")
        _check(got[2][:, f], ref[2][:, f], "f32", f"dWb {f}")
    _check(got[0][::3], ref[0][::3], "f32", "dx of the small rows")


@pytest.mark.parametrize("n_out,G", [(40, 10), (140, 30)])
def test_backward_f32_non_finite(n_out, G):
    """Non-finite dy, x and coefficients: the weight gradients have the NaN and
    infinities of the fp32 instruction's kernel (the same rows as a small batch,
    the others' dy being 0), dx is non-finite exactly in the rows (or windows) it
    reaches, and everything else is as without them."""
    B, n_in, S = 8200, 6, 500
    x, C, Wb, dy = _case(B, n_in, n_out, G, seed=6, dtype_name="f32")
    dy[S:] = 0.0
    clean = _run(x, C, Wb, dy, G, "f32")
    x2, dy2, C2 = x.copy(), dy.copy(), C.copy()
    dy2[3, 1], dy2[4, 2], dy2[5, 2], dy2[6, 3] = np.inf, np.inf, np.inf, np.nan
    x2[7, 0], x2[8, 1], x2[9, 2] = np.inf, np.nan, -np.inf
    C2[5, 3, 4] = np.inf
    say(f"backward non-finite out={n_out} G={G}")
    dx, dC, dW = _run(x2, C2, Wb, dy2, G, "f32")
    _, sC, sW = _run(x2[:S], C2, Wb, dy2[:S], G, "f32")
    for a, b in ((dC, sC), (dW, sW)):
        assert np.array_equal(np.isnan(a), np.isnan(b))
        inf = np.isinf(b)
        assert np.array_equal(inf, np.isinf(a)) and np.array_equal(a[inf], b[inf])
        ok = np.isfinite(b)
        assert normwise(a[ok], b[ok]) <= 2e-5
    assert not np.isfinite(dx[3:7]).any()
    assert np.isnan(dx[8, 1]) and np.isnan(dx[9, 2])
    bad = np.zeros_like(dx, dtype=bool)
    bad[3:7] = True
    bad[7, 0] = bad[8, 1] = bad[9, 2] = True
    # the infinite coefficient reaches the rows whose window holds its basis
    u = (x2[:, 3].astype(np.float64) + 1) * (G / 2) + 3 - 4
    bad[:, 3] |= (u > -1e-3) & (u < 4 + 1e-3)
    assert np.isfinite(dx[~bad]).all()
    assert normwise(dx[~bad], clean[0][~bad]) <= 1e-5
    inside = (u > 0.01) & (u < 1.9) & (np.arange(B) < S) & (dy2[:, 5] != 0)
    assert not np.isfinite(dx[inside, 3]).any()


def test_backward_f32_non_finite_late_row():
    """Infinite gradients in one late row of a batch split (3328 rows): infinities where the basis holds the row, NaN (0 times infinity)
    elsewhere, the outputs without one bitwise as before, and about the same time (the
    flagged outputs are summed again over the 64-row blocks that hold a non-finite
    value, not over every row)."""
    B, n_in, n_out, G, row = 16384, 784, 256, 10, 6600
    g = torch.Generator(device=device()).manual_seed(3)
    x = torch.rand(B, n_in, device=device(), generator=g) * 2 - 1
    C = torch.randn(n_out, n_in, G + 3, device=device(), generator=g) * 0.1
    Wb = torch.randn(n_out, n_in, device=device(), generator=g)
    dy = torch.randn(B, n_out, device=device(), generator=g)
    bad = dy.clone()
    bad[row, ::2] = float("inf")
    times = {}
    say("backward non-finite late row 16384 x 784 -> 256")
    for name, d in (("clean", dy), ("bad", bad), ("clean", dy), ("bad", bad)):
        start, end = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        start.record()
        out = kb.layer_backward(x, C, Wb, d, G, need_dx=False)
        end.record()
        torch.cuda.synchronize()
        times[name] = (start.elapsed_time(end), out)
    (t0, (_, cC, cW)), (t1, (_, dC, dW)) = times["clean"], times["bad"]
    assert torch.equal(dC[1::2], cC[1::2]) and torch.equal(dW[1::2], cW[1::2])
    assert torch.equal(torch.isposinf(dW[::2]), (x[row] > 0).expand(n_out // 2, -1))
    assert torch.equal(torch.isneginf(dW[::2]), (x[row] < 0).expand(n_out // 2, -1))
    u = (x[row].double()[:, None] + 1) * (G / 2) + 3 - torch.arange(G + 3, device=device())
    inside, edge = (u > 1e-3) & (u < 4 - 1e-3), (u.abs() <= 1e-3) | ((u - 4).abs() <= 1e-3)
    assert torch.isposinf(dC[::2])[:, inside].all()
    assert torch.isnan(dC[::2])[:, ~(inside | edge)].all()
    assert t1 < 4 * t0, (t0, t1)
