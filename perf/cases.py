"""The calls whose time matters to a user of the fused MLPs, as measurable cases.

A case names a net (width, depth, in_dim, out_dim, hidden and output
activation), a batch of `rows` rows and a mode:

  infer    one inference call, forward(packed, X)
  train    one training step, train_step(packed, X, T, ws)
  fit      one iteration of a training loop: train_step, then adam_step on the
           fp32 master weights, which also writes the bf16 weights and re-packs them
  seed     forward(packed, X, stash=ws), then backward from the caller's own dY
           (a loss that the library does not have)
  seed_dx  the same with the input gradient, backward_dx (nets that are chained,
           or that sit behind a trained encoding)
"""
import math

import torch

import paper_2403_17607_amd as ffmlp


def _case(name, mode, width, depth, in_dim, out_dim, rows, act="relu", out_act="linear"):
    return {"name": name, "mode": mode, "width": width, "depth": depth, "in_dim": in_dim,
            "out_dim": out_dim, "rows": rows, "act": act, "out_act": out_act}


def listed():
    return [
        # The smallest calls: a few thousand rows of the 64-wide default net,
        # once as a query and once as an iteration of a small training loop,
        # where launches and latency are most of the time.
        _case("infer_w64_4k", "infer", 64, 4, 64, 64, 4096),
        _case("fit_w64_4k", "fit", 64, 4, 64, 64, 4096),
        # Narrowest net of the width sweep over a large batch: streaming.
        _case("infer_w16_1m", "infer", 16, 4, 16, 16, 1 << 20),
        # An image held in a net, decoded: one row per pixel of a 1280 x 720
        # frame, sinusoidal features of the coordinates, three colours.
        _case("infer_image", "infer", 64, 2, 64, 3, 1280 * 720, out_act="sigmoid"),
        # The largest net of the width sweep: the headline inference.
        _case("infer_w128_1m", "infer", 128, 4, 128, 16, 1 << 20),
        # A wide, deeper net on positionally encoded 3-D points (3 + 6 * 10
        # features, not a multiple of eight), density and colour out, ragged batch.
        _case("infer_w128_points", "infer", 128, 6, 63, 4, 300001),
        # Training: a middle width of the sweep at a ragged middle batch, ...
        _case("train_w32_ragged", "train", 32, 4, 32, 16, 200003),
        # ... sine layers on 3-D points with one output (a solution field), ...
        _case("fit_sine_64k", "fit", 64, 4, 3, 1, 1 << 16, act="sine"),
        # ... the headline training step, ...
        _case("train_w128_1m", "train", 128, 4, 128, 16, 1 << 20),
        # ... and the deepest and widest net of the benchmark.
        _case("train_deep", "train", 128, 16, 128, 128, 1 << 19),
        # A colour net chained behind another net: forward, backward from the
        # renderer's gradient, gradient to the net before it.
        _case("chain_dx_w64", "seed_dx", 64, 2, 32, 3, 1 << 18, out_act="sigmoid"),
        # A caller's own loss on a deeper narrow sigmoid net with ragged sizes.
        _case("seed_w32_deep", "seed", 32, 8, 27, 3, 100003, act="sigmoid"),
    ]


def draw(rng):
    mode = rng.choice(["infer", "infer", "infer", "train", "train", "fit", "seed", "seed_dx"])
    width = rng.choice([16, 32, 64, 128])
    depth = rng.choice([1, 2, 3, 4, 4, 5, 6, 8, 16])
    # Half the nets have sizes that fit vector loads, half have any size.
    in_dim = rng.choice([width, 8 * rng.randint(1, width // 8)]) if rng.random() < 0.5 else rng.randint(1, width)
    out_dim = rng.choice([1, 3, 4, 16]) if rng.random() < 0.6 else rng.randint(1, width)
    act = rng.choice(["relu", "relu", "relu", "sine", "sigmoid"])
    out_act = rng.choice(["linear", "linear", "linear", "sigmoid", "relu"])
    # 2^12 .. 2^20 rows, 2^18 for the deepest wide nets (whose sine form does
    # about twice the work of the ReLU one), in any remainder.
    top = 18 if width * depth > 1024 else 20
    rows = int(2 ** rng.uniform(12, top))
    return {"mode": mode, "width": width, "depth": depth, "in_dim": in_dim, "out_dim": out_dim,
            "rows": rows, "act": act, "out_act": out_act}


def _shapes(case):
    w, n = case["width"], case["depth"] + 1
    return [(case["in_dim"] if l == 0 else w, case["out_dim"] if l == n - 1 else w) for l in range(n)]


def _data(case, seed):
    """Weights and inputs of a case: Xavier-uniform bf16 weights, features in
    [-1, 1], targets in the range of the output activation, and for the seeded
    modes the gradient of a mean over the batch."""
    g = torch.Generator(device="cuda").manual_seed(int(seed))

    def uniform(*shape):
        return torch.rand(*shape, generator=g, device="cuda") * 2 - 1

    rows, out = case["rows"], case["out_dim"]
    W = torch.cat([uniform(fi * fo) * math.sqrt(6.0 / (fi + fo)) for fi, fo in _shapes(case)]).to(torch.bfloat16)
    X = uniform(rows, case["in_dim"]).to(torch.bfloat16)
    T = uniform(rows, out)
    if case["out_act"] in ("sigmoid", "relu"):
        T = T * 0.5 + 0.5
    if case["mode"].startswith("seed"):
        T = T * (2.0 / (rows * out))
    return W, X, T.contiguous()


def prepare(case, seed):
    net = ffmlp.FusedMLP(case["width"], case["depth"], case["in_dim"], case["out_dim"], case["act"],
                         case["out_act"])
    W, X, T = _data(case, seed)
    s = {"mode": case["mode"], "net": net, "X": X, "packed": net.pack(W)}
    if case["mode"] != "infer":
        s["T"] = T
        s["ws"] = net.workspace(case["rows"], X.device)
    if case["mode"] == "fit":
        s["W"] = W
        s["master"] = W.float()
        s["m"] = torch.zeros_like(s["master"])
        s["v"] = torch.zeros_like(s["master"])
        s["t"] = 0
    return s


_LR = 1e-3


def run(s):
    net, mode = s["net"], s["mode"]
    if mode == "infer":
        return {"Y": net.forward(s["packed"], s["X"])}
    if mode == "train":
        G, loss = net.train_step(s["packed"], s["X"], s["T"], s["ws"])
        return {"G": G, "loss": loss}
    if mode == "fit":
        G, loss = net.train_step(s["packed"], s["X"], s["T"], s["ws"])
        s["t"] += 1
        net.adam_step(s["master"], s["m"], s["v"], G, s["W"], s["packed"], _LR, t=s["t"])
        return {"G": G, "loss": loss, "master": s["master"], "m": s["m"], "v": s["v"], "W": s["W"],
                "packed": s["packed"].view(torch.bfloat16)}
    Y = net.forward(s["packed"], s["X"], stash=s["ws"])
    if mode == "seed":
        return {"Y": Y, "G": net.backward(s["packed"], s["X"], s["T"], s["ws"])}
    G, dX = net.backward_dx(s["packed"], s["X"], s["T"], s["ws"])
    return {"Y": Y, "G": G, "dX": dX}


def work(case):
    rows, mode = case["rows"], case["mode"]
    p = sum(a * b for a, b in _shapes(case))
    p0 = case["in_dim"] * _shapes(case)[0][1]
    byts = rows * 2 * case["in_dim"] + 2 * p
    flops = 2 * p
    if mode == "infer" or mode.startswith("seed"):
        byts += rows * 2 * case["out_dim"]
    if mode != "infer":
        byts += rows * 4 * case["out_dim"] + 4 * p
        flops += 2 * (p - p0) + 2 * p
    if mode == "fit":
        byts += 24 * p + 2 * p + 4 * p  # master and moments in and out, W, both packed orientations
    if mode == "seed_dx":
        byts += rows * 4 * case["in_dim"]
        flops += 2 * p0
    return {"bytes": byts, "flops": flops * rows}


def tolerance(case):
    """Two correct paths with the same bf16 rounding points differ where their
    sums fall on different sides of a rounding boundary; each such flip travels
    through the layers after it.  Measured against float64 sums with the same
    rounding points, over these ranges: up to 4e-4 for nets of up to 7 matrices
    and 1.7e-3 at 17; single values up to 2.6e-2, and 6e-2 for dX, where one
    flip can switch a whole ReLU term of its row on or off."""
    s = max(1.0, (case["depth"] + 1) / 5)
    return {"rel": 1.5e-3 * s ** 1.25, "max": 0.9 if case["mode"] == "seed_dx" else min(0.9, 0.1 * s)}


def _act(a, c):
    return {"linear": lambda t: t, "relu": torch.relu, "sigmoid": torch.sigmoid, "sine": torch.sin}[a](c)


def _grad(a, c, y):
    if a == "relu":
        return (c > 0).to(c.dtype)
    return {"linear": lambda: torch.ones_like(c), "sigmoid": lambda: y * (1 - y), "sine": lambda: torch.cos(c)}[a]()


def exact(case, seed):
    """run()'s first answer in 64 bits throughout, from the same bf16 weights
    and inputs."""
    W, X, T = _data(case, seed)
    mode, rows, out = case["mode"], case["rows"], case["out_dim"]
    mats, o = [], 0
    for fi, fo in _shapes(case):
        mats.append(W[o:o + fi * fo].view(fi, fo).double())
        o += fi * fo
    n = len(mats)
    Y, dX, loss = [], [], 0.0
    G = [torch.zeros_like(w) for w in mats]
    for r in range(0, rows, 1 << 17):
        a, pre = [X[r:r + (1 << 17)].double()], []
        t = T[r:r + (1 << 17)].double()
        for l, w in enumerate(mats):
            pre.append(a[-1] @ w)
            a.append(_act(case["act"] if l < n - 1 else case["out_act"], pre[-1]))
        Y.append(a[-1])
        if mode == "infer":
            continue
        d = t
        if not mode.startswith("seed"):
            loss = loss + ((a[-1] - t) ** 2).sum() / (rows * out)
            d = 2 * (a[-1] - t) / (rows * out)
        d = d * _grad(case["out_act"], pre[-1], a[-1])
        for l in range(n - 1, -1, -1):
            G[l] += a[l].t() @ d
            if l > 0:
                d = (d @ mats[l].t()) * _grad(case["act"], pre[l - 1], a[l])
            elif mode == "seed_dx":
                dX.append(d @ mats[0].t())
    res = {}
    if mode == "infer" or mode.startswith("seed"):
        res["Y"] = torch.cat(Y)
    if mode != "infer":
        res["G"] = torch.cat([g.reshape(-1) for g in G])
    if mode in ("train", "fit"):
        res["loss"] = loss.reshape(1)
    if mode == "seed_dx":
        res["dX"] = torch.cat(dX)
    if mode == "fit":
        g = res["G"]
        res["m"] = 0.1 * g
        res["v"] = 0.001 * g * g
        w = W.double() - _LR * (res["m"] / 0.1) / ((res["v"] / 0.001).sqrt() + 1e-8)
        res["master"] = w
        res["W"] = w
        res["packed"] = None
    return res
