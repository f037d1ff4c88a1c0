"""GPU parity of the window kernel (the fused forward on the structured-sparse
matrix instruction for degrees 1 .. 3 and any grid: fp32 as two fp16 terms per
operand with the SiLU column in fp32, bf16 on grids outside 5 .. 12) against
the float64 oracle on sampled rows, at the layer tolerances 1e-5 (fp32) and
2e-2 (bf16, on the bf16-rounded tensors); its scaling over the range of fp32
weights; and its treatment of non-finite inputs and coefficients against the
kernels that read the packed weights (the same call without a workspace)."""
import numpy as np
import pytest

import oracle
from paper_2609_01956_amd import binding as kb
from paper_2609_01956_amd import workloads as wl
from gpu_common import (BF16_LAYER_TOL, F32_LAYER_TOL, device, normwise, say, to_dev, to_host64,
                        torch)

pytestmark = pytest.mark.gpu

TD = {"f32": torch.float32, "bf16": torch.bfloat16}


def _planned(B, n_in, n_out, G, k, dtype_name):
    """Whether the call runs the window kernel: its workspace is not a split's partials."""
    args = (kb.make_grid(G, spline_order=k), {"f32": kb.KAN_F32, "bf16": kb.KAN_BF16}[dtype_name],
            B, n_in, n_out)
    st, need = kb.kan_layer_forward_packed_full_workspace_bytes(*args)
    st2, least = kb.kan_layer_forward_packed_workspace_bytes(*args)
    assert st == st2 == kb.KAN_OK
    return need != least


def _inputs(B, n_in, n_out, G, k, dtype_name, seed=7):
    x, C, Wb = wl.make_layer(wl.LayerShape(B, n_in, n_out, G, off_grid_frac=0.1), seed, k=k)
    if dtype_name == "bf16":
        x, C, Wb = (wl.round_to_bf16_f32(a) for a in (x, C, Wb))
    return x, C, Wb


def _run(x, C, Wb, G, k, dtype_name, split=True):
    t = TD[dtype_name]
    p = kb.pack_layer(to_dev(C, t), to_dev(Wb, t), G, spline_order=k)
    y = kb.layer_forward_packed(to_dev(x, t), p, split=split)
    torch.cuda.synchronize()
    return to_host64(y)


CASES = [
    # (B, in, out, G, k): one, two and more 16-column blocks per feature (G + k + 1
    # = 16, 17, 32, 33); column tiles of 64, 128 and 256, whole, ragged and several;
    # an odd feature count; ragged row blocks; K splits and none
    ("f32", 4096, 256, 64, 12, 3), ("f32", 4099, 255, 33, 13, 3), ("f32", 1024, 131, 129, 28, 3),
    ("f32", 1500, 67, 300, 29, 3), ("f32", 90001, 7, 64, 10, 3), ("f32", 12000, 300, 17, 1, 3),
    ("f32", 2000, 101, 257, 14, 1), ("f32", 6003, 64, 100, 9, 2), ("f32", 16500, 40, 65, 5, 3),
    ("f32", 1024, 41, 200, 200, 3), ("f32", 1025, 41, 190, 200, 1),
    ("f32", 70000, 3, 256, 10, 3),
    ("bf16", 4099, 65, 75, 20, 2), ("bf16", 1111, 200, 64, 13, 1), ("bf16", 2050, 31, 260, 30, 2),
    ("bf16", 9001, 129, 129, 100, 3), ("bf16", 70001, 64, 256, 13, 3),
    ("bf16", 30001, 256, 64, 28, 3), ("bf16", 70000, 101, 255, 3, 3), ("bf16", 30001, 33, 40, 3, 1),
]


@pytest.mark.parametrize("dtype_name,B,n_in,n_out,G,k", CASES)
def test_window_kernel_matches_oracle(dtype_name, B, n_in, n_out, G, k):
    assert _planned(B, n_in, n_out, G, k, dtype_name)
    x, C, Wb = _inputs(B, n_in, n_out, G, k, dtype_name)
    say(f"window {dtype_name} B={B} {n_in}->{n_out} G={G} k={k}")
    y = _run(x, C, Wb, G, k, dtype_name)
    rows = np.unique(np.r_[0:8, B // 2:B // 2 + 8, 250:262, B - 40:B])
    ref = oracle.layer(x[rows], C, Wb, G, k=k)
    if dtype_name == "bf16":
        ref = oracle.round_bf16(ref)
    tol = F32_LAYER_TOL if dtype_name == "f32" else BF16_LAYER_TOL
    assert normwise(y[rows], ref) <= tol
    # every row against the packed-weight kernels (both within tol of the exact layer)
    assert normwise(y, _run(x, C, Wb, G, k, dtype_name, split=False)) <= 2 * tol


@pytest.mark.parametrize("ec,eb", [(-120, -120), (-149, 0), (0, -40), (40, 40), (-30, 10), (100, 90)])
def test_window_kernel_weight_scales(ec, eb):
    """Coefficients around 2^ec and SiLU weights around 2^eb: the two-term split
    follows each column's scale, so the tolerance is the layer's own."""
    B, n_in, n_out, G = 4096, 161, 64, 10
    x, C, Wb = _inputs(B, n_in, n_out, G, 3, "f32")
    C = (C * 2.0 ** ec).astype(np.float32)
    Wb = (Wb * 2.0 ** eb).astype(np.float32)
    C[:, :, 1] *= np.float32(2.0 ** -12)  # and some far below the column's largest
    assert _planned(B, n_in, n_out, G, 3, "f32")
    say(f"window scales {ec} {eb}")
    y = _run(x, C, Wb, G, 3, "f32")
    rows = np.r_[0:64]
    assert normwise(y[rows], oracle.layer(x[rows], C, Wb, G)) <= F32_LAYER_TOL


@pytest.mark.parametrize("dtype_name,n_out,G,k", [
    ("f32", 64, 10, 3), ("f32", 140, 30, 3), ("bf16", 140, 30, 3), ("bf16", 140, 14, 2),
    ("bf16", 60, 9, 1)])
def test_window_kernel_non_finite(dtype_name, n_out, G, k):
    """NaN and infinite inputs, and NaN and infinite weights: NaN where the
    dense kernel gives NaN, the same infinities, and unaffected rows and outputs
    as without them.  (An infinite coefficient times a basis value of exactly 0 is
    NaN in the dense contraction, and so here.)"""
    B, n_in = (65536, 64) if dtype_name == "bf16" else (4096, 140)
    x, C, Wb = _inputs(B, n_in, n_out, G, k, dtype_name)
    x[5, 3] = np.nan
    x[6, 2] = np.inf
    x[7, 2] = -np.inf
    x[B - 1, n_in - 1] = np.inf
    C2, Wb2 = C.copy(), Wb.copy()
    C2[3, 1, 4] = np.inf
    C2[4, 9, 0] = -np.inf
    C2[5, 20, G + k - 1] = np.nan
    Wb2[6, 2] = np.inf
    Wb2[7, 33] = np.nan
    cases = [(C, Wb), (C2, Wb2)]
    assert _planned(B, n_in, n_out, G, k, dtype_name)
    for c, w in cases:
        say(f"window non-finite {dtype_name} out={n_out} G={G} k={k}")
        y = _run(x, c, w, G, k, dtype_name)
        ref = _run(x, c, w, G, k, dtype_name, split=False)
        assert np.array_equal(np.isnan(y), np.isnan(ref))
        inf = np.isinf(ref)
        assert np.array_equal(y[inf], ref[inf]) and np.array_equal(inf, np.isinf(y))
        ok = np.isfinite(ref)
        assert normwise(y[ok], ref[ok]) <= 2 * (F32_LAYER_TOL if dtype_name == "f32" else
                                                BF16_LAYER_TOL)


def test_window_kernel_workspace_and_guard():
    """A dirty workspace, two runs bitwise equal, nothing written past y, and a
    workspace that is one byte short or misaligned runs the packed-weight kernel."""
    B, n_in, n_out, G = 4100, 200, 70, 10
    x, C, Wb = _inputs(B, n_in, n_out, G, 3, "f32")
    g = kb.make_grid(G)
    st, need = kb.kan_layer_forward_packed_full_workspace_bytes(g, kb.KAN_F32, B, n_in, n_out)
    assert st == kb.KAN_OK
    p = kb.pack_layer(to_dev(C, TD["f32"]), to_dev(Wb, TD["f32"]), G)
    xd = to_dev(x, TD["f32"])
    plain = kb.layer_forward_packed(xd, p, split=False)
    runs = []
    for fill, off, nbytes in ((0, 0, need), (255, 0, need), (0, 0, need - 1), (0, 4, need)):
        ws = torch.full((need + 64,), fill, dtype=torch.uint8, device=device())
        y = torch.full((B * n_out + 64,), 7.0, dtype=torch.float32, device=device())
        say(f"window workspace fill={fill} off={off} bytes={nbytes - need}")
        rc = kb.kan_layer_forward_packed(g, kb.KAN_F32, B, n_in, n_out, xd.data_ptr(),
                                         p.buf.data_ptr(), p.nbytes, y.data_ptr(),
                                         int(torch.cuda.current_stream().cuda_stream),
                                         workspace=ws.data_ptr() + off, workspace_bytes=nbytes)
        if off:  # (misaligned: as refused as for a split contraction's partial sums)
            st, plan = kb.kan_layer_plan(g, kb.KAN_F32, B, n_in, n_out)
            assert rc == (kb.KAN_ERR_INVALID_ARG if plan[5] > 1 else kb.KAN_OK)
            continue
        assert rc == kb.KAN_OK
        torch.cuda.synchronize()
        assert bool((y[B * n_out:] == 7.0).all()) and bool((ws[need:] == fill).all())
        runs.append(y[:B * n_out].reshape(B, n_out))
    assert torch.equal(runs[0], runs[1])
    assert normwise(to_host64(runs[2]), to_host64(plain)) <= F32_LAYER_TOL
    assert normwise(to_host64(runs[0]), to_host64(plain)) <= 2 * F32_LAYER_TOL
