"""Performance cases of the KAN layer: what a user's program calls, over the
sizes, grids, degrees and dtypes it calls it with.

    listed()            the fixed cases
    draw(rng)           one more case of the same ranges
    prepare(case, seed) inputs and weights on the GPU, from the seed alone
    run(state)          one pass through the public entry points
    work(case)          bytes and operations the pass cannot do without
    tolerance(case)     what another correct implementation would differ by
    exact(case, seed)   the same outputs from plain float64 torch

A case names its kind: "forward" (weights given as they are, packed by the
call), "packed" (weights packed once, the serving form), "span" (the
span-sparse forward), "basis" (the basis tensor alone), "backward" (gradients
of one layer), "train" (forward and backward of one layer) and "mlp_train"
(forward and backward of a stack).
"""
import math

import torch

from paper_2609_01956_amd import binding as kb

DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16}


def listed():
    return [
        # A tiny regression network's layer under training: a few launches, no work.
        layer("fit_2x5_g5_b1024_f32", "train", "f32", 1024, 2, 5, 5),
        # A served request batch on the first layer of the 784-256-256-10 network.
        layer("serve_784x256_g10_b64_bf16", "packed", "bf16", 64, 784, 256, 10),
        # The paper's timing layer: MNIST-sized rows at batch 256, weights not packed.
        layer("table1_784x64_g5_b256_f32", "forward", "f32", 256, 784, 64, 5),
        # A mid-sized layer's training step.
        layer("train_64x64_g5_b4096_bf16", "train", "bf16", 4096, 64, 64, 5),
        # A hidden layer whose inputs leave the grid now and then (offline inference).
        layer("offgrid_256x256_g10_b16384_bf16", "packed", "bf16", 16384, 256, 256, 10, off=0.1),
        # Grid refinement: the same layer on a large grid, by the dense entry point ...
        layer("grid_128x128_g100_b8192_f32", "forward", "f32", 8192, 128, 128, 100),
        # ... and by the span-sparse one.
        layer("span_128x128_g200_b8192_bf16", "span", "bf16", 8192, 128, 128, 200),
        # Another degree, with sizes that are multiples of nothing.
        layer("ragged_101x75_g20_k2_b30001_bf16", "forward", "bf16", 30001, 101, 75, 20, k=2),
        # The basis tensor alone, as the method is usually timed.
        dict(name="basis_784_g10_b65536_bf16", kind="basis", dtype="bf16", batch=65536, n_in=784,
             G=10, k=3, off=0.0),
        # The 784-256-256-10 network's training step in full precision.
        dict(name="mlp_train_784_256_256_10_g10_b16384_f32", kind="mlp_train", dtype="f32",
             batch=16384, sizes="784,256,256,10", G=10, k=3, off=0.0),
        # Its first layer at the largest batch: forward with packed weights, and gradients.
        layer("layer_784x256_g10_b65536_bf16", "packed", "bf16", 65536, 784, 256, 10),
        layer("backward_784x256_g10_b65536_bf16", "backward", "bf16", 65536, 784, 256, 10),
    ]


def layer(name, kind, dtype, batch, n_in, n_out, G, k=3, off=0.0):
    return dict(name=name, kind=kind, dtype=dtype, batch=batch, n_in=n_in, n_out=n_out, G=G, k=k,
                off=off)


def _log(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _cost(c):
    """Multiply-adds of the dense contraction, weighted by the dtype's matrix rate."""
    s = sizes(c)
    n = sum(a * b for a, b in zip(s, s[1:])) if c["kind"] != "basis" else s[0]
    per = {"forward": 1, "packed": 1, "span": 1, "basis": 8, "backward": 2, "train": 3,
           "mlp_train": 3}[c["kind"]]
    return c["batch"] * n * (c["G"] + c["k"] + 1) * per * (8 if c["dtype"] == "f32" else 1)


def draw(rng):
    """Batches 1 to 65536, widths 1 to 1024, grids 3 to 200 (the backward to 50), degrees 1 to 7
    (the backward: 3); at most the cost of the largest listed case."""
    most = _cost(listed()[-1])
    while True:
        kind = rng.choice(["forward", "packed", "packed", "span", "basis", "backward", "train",
                           "train", "mlp_train"])
        c = dict(kind=kind, dtype=rng.choice(["f32", "bf16"]), batch=_log(rng, 1, 65536),
                 k=3, off=rng.choice([0.0, 0.1]))
        back = kind in ("backward", "train", "mlp_train")
        # (most layers are on the small grids that networks are trained with)
        c["G"] = _log(rng, 3, 20) if rng.random() < 0.7 else _log(rng, 13, 50 if back else 200)
        if kind == "span":
            c["G"] = _log(rng, 20, 200)
        if not back and rng.random() < 0.25:
            c["k"] = rng.choice([1, 2, 4, 5, 6, 7])
        if kind == "mlp_train":
            c["sizes"] = ",".join(str(_log(rng, 2, 784)) for _ in range(rng.choice([3, 4])))
        else:
            c["n_in"] = _log(rng, 1, 1024)
            if kind != "basis":
                c["n_out"] = _log(rng, 1, 512)
        if _cost(c) <= most and c["batch"] * sum(sizes(c)) >= 64:
            return c


def sizes(c):
    if "sizes" in c:
        return [int(v) for v in c["sizes"].split(",")]
    return [c["n_in"], c.get("n_out", c["n_in"])]


def _inputs(case, seed):
    """x, the layers' (coef, base_w) and the upstream gradient, in the case's dtype: x uniform on
    the grid [-1, 1] with a share from U(-4, 4); coefficients N(0, 0.1) (over sqrt(G) on large
    grids, and in a stack scaled so that hidden values stay mostly on the grid); base weights
    N(0, 1 / in); the gradient N(0, 1)."""
    dev, dt = torch.device("cuda"), DTYPES[case["dtype"]]
    g = torch.Generator(device=dev)
    g.manual_seed(seed)
    B, G, k, s = case["batch"], case["G"], case["k"], sizes(case)
    x = torch.empty(B, s[0], device=dev).uniform_(-1, 1, generator=g)
    if case["off"] > 0:
        far = torch.rand(B, s[0], device=dev, generator=g) < case["off"]
        x = torch.where(far, torch.empty_like(x).uniform_(-4, 4, generator=g), x)
    layers = []
    if case["kind"] != "basis":
        for n_in, n_out in zip(s, s[1:]):
            std = 0.1 if G < 50 else 0.1 / math.sqrt(G)
            if case["kind"] == "mlp_train":
                std = 0.7 / math.sqrt(n_in)
            coef = torch.randn(n_out, n_in, G + k, device=dev, generator=g) * std
            base = torch.randn(n_out, n_in, device=dev, generator=g) / n_in
            layers.append((coef.to(dt), base.to(dt)))
    dy = torch.randn(B, s[-1], device=dev, generator=g)
    return x.to(dt), layers, dy.to(dt)


def prepare(case, seed):
    x, layers, dy = _inputs(case, seed)
    state = dict(case=case, x=x, layers=layers, dy=dy)
    if case["kind"] == "packed":
        coef, base = layers[0]
        state["packed"] = kb.pack_layer(coef, base, case["G"], spline_order=case["k"])
    return state


def run(state):
    case, x, layers, dy = state["case"], state["x"], state["layers"], state["dy"]
    kind, G, k = case["kind"], case["G"], case["k"]
    if kind == "basis":
        return kb.basis(x, G, spline_order=k)
    if kind == "packed":
        return kb.layer_forward_packed(x, state["packed"])
    if kind == "mlp_train":
        ys = kb.mlp_forward(x, layers, G, return_all=True)
        grads, d = [], dy
        for i in reversed(range(len(layers))):
            d, dc, dw = kb.layer_backward(x if i == 0 else ys[i - 1], *layers[i], d, G)
            grads += [dc, dw]
        return ys, d, grads
    coef, base = layers[0]
    if kind == "forward":
        return kb.layer_forward(x, coef, base, G, spline_order=k)
    if kind == "span":
        return kb.layer_forward_span(x, coef, base, G, spline_order=k)
    if kind == "backward":
        return kb.layer_backward(x, coef, base, dy, G)
    y = kb.layer_forward(x, coef, base, G)
    return y, kb.layer_backward(x, coef, base, dy, G)


def work(case):
    """Each tensor read or written once; per (row, input, output) the multiply-adds of the k + 1
    nonzero bases and the SiLU term, in each contraction of the pass; per basis value ten
    operations."""
    e = 4 if case["dtype"] == "f32" else 2
    B, s, nb = case["batch"], sizes(case), case["G"] + case["k"]
    if case["kind"] == "basis":
        return {"bytes": B * s[0] * (1 + nb) * e, "flops": B * s[0] * nb * 10}
    pairs = sum(a * b for a, b in zip(s, s[1:]))
    weights = pairs * (nb + 1)
    passes = {"backward": 2, "train": 3, "mlp_train": 3}.get(case["kind"], 1)
    rows = B * (s[0] + sum(s[1:]))
    if passes == 2:
        n = 2 * B * s[0] + B * s[-1] + 2 * weights
    elif passes == 3:
        n = rows + B * s[0] + B * s[-1] + 2 * weights
    else:
        n = rows + weights
    return {"bytes": n * e, "flops": 2 * B * pairs * (case["k"] + 2) * passes}


def tolerance(case):
    deep = case["kind"] == "mlp_train"  # (a rounding in one layer travels through all that follow)
    if case["dtype"] == "bf16":
        return {"rel": 3e-2 if deep else 1e-2}
    return {"rel": 5e-5 if deep else 1e-5}


# ---------------------------------------------------------------- float64

def _powers(x, G, k, p):
    """sum_m (-1)^m C(k + 1, m) (u_j - m)_+^p for every basis j, u_j clamped to [0, k + 1]."""
    j = torch.arange(G + k, device=x.device, dtype=torch.float64)
    u = ((x.unsqueeze(-1) + 1.0) * (G / 2.0) + k - j).clamp_(0, k + 1)
    # (the sum is symmetric up to the sign (-1)^(p - k) at k + 1 - u: the half with fewer terms)
    w = torch.minimum(u, k + 1 - u)
    n = torch.zeros_like(w)
    for m in range((k + 1) // 2 + 1):
        n.add_((w - m).clamp_(min=0).pow_(p), alpha=(-1) ** m * math.comb(k + 1, m))
    if (p - k) % 2:
        n.mul_(torch.where(u > (k + 1) / 2, -1.0, 1.0))
    return n


def _columns(x, G, k):
    """[silu(x), N_0(x), ...] per input."""
    n = _powers(x, G, k, k) / math.factorial(k)
    return torch.cat([(x * torch.sigmoid(x)).unsqueeze(-1), n], -1)


def _slopes(x, G, k):
    """d/dx of _columns."""
    s = torch.sigmoid(x)
    n = _powers(x, G, k, k - 1) * (G / 2.0 / math.factorial(k - 1))
    return torch.cat([(s * (1 + x * (1 - s))).unsqueeze(-1), n], -1)


def _exact_layer(x, coef, base, G, k, dy=None, forward=True):
    """y, and with dy also (dx, dcoef, dbase), a few rows at a time."""
    n_out, n_in = base.shape
    w = torch.cat([base.unsqueeze(-1), coef], -1).double().reshape(n_out, -1)
    step = max(1, (1 << 27) // w.shape[1])
    ys, dxs, dw = [], [], torch.zeros_like(w)
    for i in range(0, x.shape[0], step):
        xr = x[i:i + step].double()
        a = _columns(xr, G, k).reshape(xr.shape[0], -1)
        if forward:
            ys.append(a @ w.t())
        if dy is not None:
            d = dy[i:i + step].double()
            dw += d.t() @ a
            del a
            slopes = _slopes(xr, G, k)
            dxs.append((slopes * (d @ w).reshape(slopes.shape)).sum(-1))
    y = torch.cat(ys) if forward else None
    if dy is None:
        return y, None
    dw = dw.reshape(n_out, n_in, -1)
    return y, (torch.cat(dxs), dw[..., 1:].contiguous(), dw[..., 0].contiguous())


def exact(case, seed):
    x, layers, dy = _inputs(case, seed)
    kind, G, k = case["kind"], case["G"], case["k"]
    if kind == "basis":
        step = max(1, (1 << 26) // x.shape[1])
        return torch.cat([_powers(r.double(), G, k, k) / math.factorial(k) for r in x.split(step)])
    if kind == "mlp_train":
        hs = [x]
        for coef, base in layers:
            hs.append(_exact_layer(hs[-1], coef, base, G, k)[0])
        grads, d = [], dy
        for i in reversed(range(len(layers))):
            d, dc, dw = _exact_layer(hs[i], *layers[i], G, k, d, forward=False)[1]
            grads += [dc, dw]
        return hs[1:], d, grads
    y, grads = _exact_layer(x, *layers[0], G, k, dy if kind in ("backward", "train") else None,
                            forward=kind != "backward")
    return grads if kind == "backward" else (y, grads) if kind == "train" else y
