"""Timing cases of the framework: what its users run, through the public entry points.

Each case is one call (or the calls of one training iteration) on seeded inputs of the shapes that the
package's workloads, tests and the paper's experiments use: single PyraMiD-LSTM layers, forward and
forward + backward, volumes and images, fp32 and bf16 storage, 3x3 and larger filters, and whole stacked
networks.  `listed()` gives the fixed cases, `draw(rng)` further ones of the same ranges.
"""
import math

import torch

from paper_1506_07452_amd.network import (LayerW, layer2d_backward, layer2d_forward, layer_backward,
                                          layer_forward, network_forward, network_train_step,
                                          workspace_for_layers)

DT = {"f32": torch.float32, "bf16": torch.bfloat16}
GATES = 4

# kind: "fwd" (a layer's inference forward), "step" (a layer's training forward + backward, with dL/dx
# where `dx`), "step2d" (the same for an image layer), "net" (a stacked network's inference forward) and
# "train" (a stacked network's training iteration).  `values`: "mr" (a smoothed normal volume), "em"
# (uniform), "normal", "act" (tanh activations of the layer before).


def listed():
    return [
        # a smoke-size call: launch latency only
        {"name": "tiny-fwd", "kind": "fwd", "N": 1, "D": 8, "H": 8, "W": 8, "C": 1, "O": 4, "K": 3,
         "dtype": "f32", "values": "normal"},
        # the first training stage's sub-volumes (64 x 64 x 8), a small batch, first layer
        {"name": "cube-step", "kind": "step", "N": 2, "D": 8, "H": 64, "W": 64, "C": 1, "O": 16, "K": 3,
         "dtype": "f32", "values": "em", "dx": False},
        # inference of one layer over a whole MR volume
        {"name": "mr-fwd", "kind": "fwd", "N": 1, "D": 48, "H": 240, "W": 240, "C": 3, "O": 16, "K": 3,
         "dtype": "f32", "values": "mr"},
        # and over a whole EM stack
        {"name": "em-fwd", "kind": "fwd", "N": 1, "D": 30, "H": 512, "W": 512, "C": 1, "O": 16, "K": 3,
         "dtype": "f32", "values": "em"},
        # an inner 16-unit layer on odd extents (a cropped scan), with the gradient of its input
        {"name": "odd-step", "kind": "step", "N": 1, "D": 19, "H": 101, "W": 75, "C": 6, "O": 16, "K": 3,
         "dtype": "f32", "values": "act", "dx": True},
        # the second layer of the MR networks on the last training stage's sub-volume
        {"name": "hidden32-step", "kind": "step", "N": 1, "D": 25, "H": 240, "W": 240, "C": 32, "O": 32,
         "K": 3, "dtype": "f32", "values": "act", "dx": True},
        # the widest layer, on cubes
        {"name": "wide64-step", "kind": "step", "N": 1, "D": 20, "H": 64, "W": 64, "C": 64, "O": 64, "K": 3,
         "dtype": "f32", "values": "act", "dx": True},
        # a wide layer of a bf16 network on a cropped scan
        {"name": "odd-bf16-fwd", "kind": "fwd", "N": 2, "D": 21, "H": 75, "W": 90, "C": 32, "O": 32, "K": 3,
         "dtype": "bf16", "values": "act"},
        # a batch of slices through an image layer
        {"name": "images-step", "kind": "step2d", "N": 30, "H": 512, "W": 512, "C": 1, "O": 16, "K": 3,
         "dtype": "f32", "values": "em", "dx": True},
        # batched inference of the three-layer network with bf16 storage
        {"name": "stacked-bf16", "kind": "net", "N": 8, "D": 64, "H": 64, "W": 64, "C": 3,
         "hidden": "16,32,64", "fc": "32,64,128", "classes": 4, "K": 3, "dtype": "bf16", "values": "normal"},
        # a training iteration of the two-layer network on a whole MR volume
        {"name": "mr-train", "kind": "train", "N": 1, "D": 48, "H": 240, "W": 240, "C": 3,
         "hidden": "16,32", "fc": "32,64", "classes": 4, "K": 3, "dtype": "f32", "values": "mr",
         "loss": "ce"},
        # the second layer of the paper's 7x7 network on the second training stage's sub-volume
        {"name": "paper32-step", "kind": "step", "N": 1, "D": 15, "H": 128, "W": 128, "C": 25, "O": 32,
         "K": 7, "dtype": "f32", "values": "act", "dx": True},
    ]


def _span(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed ranges, at most as much work as the largest listed one."""
    top = max(_cost(c) for c in listed())
    while True:
        kind = rng.choice(["fwd", "fwd", "step", "step", "step", "step2d", "net", "train"])
        c = {"kind": kind, "N": rng.choice([1, 1, 1, 2, 3])}
        if kind == "step2d":
            c.update(N=_span(rng, 1, 30), H=_span(rng, 40, 512), W=_span(rng, 40, 512), C=_span(rng, 1, 4),
                     O=16, K=rng.choice([3, 3, 5]), dtype="f32", values=rng.choice(["em", "normal"]),
                     dx=rng.random() < 0.5)
        else:
            c.update(D=_span(rng, 8, 64), H=_span(rng, 24, 320), W=_span(rng, 24, 320))
        if kind in ("fwd", "step"):
            c["O"] = rng.choice([16, 16, 32, 64])
            inner = rng.random() < 0.6
            c["C"] = rng.choice([c["O"], c["O"] // 2, c["O"] // 2 + 9]) if inner else _span(rng, 1, 6)
            c["K"] = rng.choice([3, 3, 3, 5, 7])
            c["dtype"] = "bf16" if kind == "fwd" and rng.random() < 0.4 else "f32"
            c["values"] = "act" if inner else rng.choice(["mr", "em", "normal"])
            if kind == "step":
                c["dx"] = inner
        elif kind == "net":
            c.update(C=_span(rng, 1, 5), hidden=rng.choice(["16,32", "16,32,64"]), classes=rng.choice([2, 4, 5]),
                     K=3, dtype=rng.choice(["bf16", "f32"]), values=rng.choice(["mr", "em", "normal"]))
        elif kind == "train":
            c.update(C=_span(rng, 1, 5), classes=rng.choice([2, 4, 5]), K=3, dtype="f32",
                     values=rng.choice(["mr", "em"]), hidden="16,32", loss=rng.choice(["ce", "sq"]))
        if kind in ("net", "train") and "fc" not in c:
            c["fc"] = ",".join(str(2 * int(o)) for o in c["hidden"].split(","))
        if _cost(c) <= top:
            return c


def _ints(text):
    return [int(v) for v in text.split(",")]


def _voxels(case):
    return case["N"] * case.get("D", 1) * case["H"] * case["W"]


def _layers(case):
    """(input channels, hidden units) of each layer, and the hidden FC widths."""
    if "O" in case:
        return [(case["C"], case["O"])], []
    fc = _ints(case["fc"])
    c, out = case["C"], []
    for i, o in enumerate(_ints(case["hidden"])):
        out.append((c, o))
        c = fc[i] if i < len(fc) else o
    return out, fc


def work(case):
    """Dense contraction flops (input and recurrent convolutions, their transposes and the weight gradients,
    the FC layers), and each input, output and parameter once."""
    M = _voxels(case)
    nd, taps = (4, case["K"]) if case["kind"] == "step2d" else (6, case["K"] ** 2)
    train = case["kind"] in ("step", "step2d", "train")
    size = 2 if case["dtype"] == "bf16" else 4
    layers, fc = _layers(case)
    flops = params = 0
    for i, (C, O) in enumerate(layers):
        unit = nd * M * 2 * taps * GATES * O
        flops += unit * (C + O)
        params += nd * GATES * O * (taps * (C + O) + 1)
        if train:
            flops += unit * O + unit * (C + O)
            if i > 0 or case.get("dx"):
                flops += unit * C
    for i, f in enumerate(fc):
        flops += 2 * M * layers[i][1] * f * (3 if train else 1)
        params += (layers[i][1] + 1) * f
    last = layers[-1][1]
    nbytes = params * size * (2 if train else 1) + M * layers[0][0] * size
    if "classes" in case:
        feed = fc[-1] if len(fc) == len(layers) else last
        flops += 2 * M * feed * case["classes"] * (3 if train else 1)
        nbytes += M * case["classes"] * 4 + (M * 4 if train else 0)
    else:
        nbytes += M * last * size + (M * last * size if train else 0)
        if case.get("dx"):
            nbytes += M * case["C"] * size
    return {"bytes": float(nbytes), "flops": float(flops)}


def _cost(case):
    return work(case)["flops"] * (1.0 if case["dtype"] == "f32" else 0.2)


def tolerance(case):
    """About four times what the path differs from 64 bits by, the worst of some forty inputs: 2.1e-6 for a
    forward (sums of up to 4000 terms through a recurrence of up to 512 planes), 8e-6 for a layer's gradients
    (sums over all voxels), 2.7e-5 for those of a whole network;
    2.5e-3 with each direction's h and the output rounded to bf16."""
    if case["dtype"] == "bf16":
        return {"rel": 1e-2}
    return {"rel": {"fwd": 1e-5, "net": 1e-5, "step": 3e-5, "step2d": 1e-5, "train": 1e-4}[case["kind"]]}


# ------------------------------------------------------------------------------------------------ inputs
def _smooth(v):
    """Mean over the in-bounds voxels of a 5 x 5 x 5 box, per channel."""
    v = v.permute(0, 4, 1, 2, 3)
    v = torch.nn.functional.avg_pool3d(v, 5, 1, 2, count_include_pad=False)
    return v.permute(0, 2, 3, 4, 1)


def _volume(shape, values, gen):
    if values == "em":
        return torch.rand(shape, generator=gen, device="cuda")
    v = torch.randn(shape, generator=gen, device="cuda")
    if values == "mr":
        return _smooth(v)
    return torch.tanh(0.5 * v) if values == "act" else v


def _uniform(shape, gen, dtype, bound=0.1):
    return ((torch.rand(shape, generator=gen, device="cuda") * 2 - 1) * bound).to(dtype)


def _layer(nd, C, O, taps, gen, dtype):
    # U(-0.1, 0.1), the paper's initialisation; filters larger than 3 x 3 keep the reach of 3 x 3 ones, since
    # at 0.1 their recurrence is chaotic and no two orders of summation agree after a few dozen planes
    bound = 0.1 * min(1.0, 3.0 / taps[-1])
    b = torch.zeros(nd, GATES * O, device="cuda")
    b[:, O:2 * O] = 1.0
    return LayerW(_uniform((nd, GATES * O, C) + taps, gen, dtype, bound),
                  _uniform((nd, GATES * O, O) + taps, gen, dtype, bound), b.to(dtype))


def _labels(x, classes):
    """Class labels that follow the intensities, as those of a segmentation do (under random labels the
    voxels' gradients cancel and what is left of them is rounding)."""
    v = x.mean(-1).reshape(-1)
    z = (v - v.mean()) / v.std()
    return torch.clamp(torch.floor(z + classes / 2), 0, classes - 1).to(torch.int32)


def _fc(C, F, gen, dtype):
    return _uniform((F, C), gen, dtype), torch.zeros(F, device="cuda", dtype=dtype)


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1506 + 7919 * seed)
    dt, K, N = DT[case["dtype"]], case["K"], case["N"]
    two = case["kind"] == "step2d"
    dims = (N, case["H"], case["W"]) if two else (N, case["D"], case["H"], case["W"])
    layers, fc = _layers(case)
    s = {"case": case, "x": _volume(dims + (case["C"],), case["values"], gen).to(dt).contiguous()}
    s["layers"] = [_layer(4 if two else 6, C, O, (K,) if two else (K, K), gen, dt) for C, O in layers]
    if case["kind"] in ("step", "step2d"):
        s["dh"] = torch.randn(dims + (case["O"],), generator=gen, device="cuda")
    if "classes" in case:
        s["fcs"] = [_fc(layers[i][1], f, gen, dt) for i, f in enumerate(fc)]
        s["head"] = _fc(fc[-1] if len(fc) == len(layers) else layers[-1][1], case["classes"], gen, dt)
        train = case["kind"] == "train"
        if train:
            s["labels"] = _labels(s["x"], case["classes"])
        s["ws"] = workspace_for_layers(s["x"].shape, [(C, O, K) for C, O in layers], dt, train, "cuda")
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "net":
        return network_forward(s["x"], s["layers"], s["fcs"], s["head"], ws=s["ws"])["p"]
    if kind == "train":
        return network_train_step(s["x"], s["layers"], s["fcs"], s["head"], s["labels"], ws=s["ws"],
                                  loss=case["loss"])
    x, L = s["x"], s["layers"][0]
    if kind == "fwd":
        return layer_forward(x, L)[0]
    fwd, bwd = (layer2d_forward, layer2d_backward) if kind == "step2d" else (layer_forward, layer_backward)
    h, saved = fwd(x, L, training=True)
    dx, dwx, dwh, db = bwd(x, L, saved, s["dh"], want_dx=case["dx"])
    out = {"h": h, "dwx": dwx, "dwh": dwh, "db": db}
    if case["dx"]:
        out["dx"] = dx
    return out


# --------------------------------------------------------------------------------- the same in 64 bits
def _im2col(a):
    """[B][P][Q][C] zero-padded by its filter's radius -> function of the filter's extents."""
    def cols(KP, KQ, flip=False):
        p = torch.nn.functional.pad(a, (0, 0, KQ // 2, KQ // 2, KP // 2, KP // 2))
        u = p.unfold(1, KP, 1).unfold(2, KQ, 1)                      # [B][P][Q][C][KP][KQ]
        if flip:
            u = u.flip(4, 5)
        return u.reshape(u.shape[0] * u.shape[1] * u.shape[2], -1)
    return cols


def _sweep(x, wx, wh, b, keep):
    """One direction over planes x [T][N][P][Q][C]: h [T][N][P][Q][O], and (gates, c) where `keep`."""
    T, N, P, Q, C = x.shape
    O, KP, KQ = wh.shape[1], wh.shape[2], wh.shape[3]
    Wx, Wh = wx.reshape(GATES * O, -1).t().contiguous(), wh.reshape(GATES * O, -1).t().contiguous()
    h = x.new_empty(T, N, P, Q, O)
    gates = x.new_empty(T, N * P * Q, GATES * O) if keep else None
    cells = x.new_empty(T, N * P * Q, O) if keep else None
    hp, c = None, None
    for t in range(T):
        a = _im2col(x[t])(KP, KQ) @ Wx + b
        if hp is not None:
            a += _im2col(hp)(KP, KQ) @ Wh
        i, f, g, o = a.view(-1, GATES, O).unbind(1)
        i, f, g, o = torch.sigmoid(i), torch.sigmoid(f), torch.tanh(g), torch.sigmoid(o)
        c = g * i if c is None else g * i + c * f
        h[t] = (o * torch.tanh(c)).view(N, P, Q, O)
        hp = h[t]
        if keep:
            gates[t] = torch.cat([i, f, g, o], 1)
            cells[t] = c
    return h, gates, cells


def _sweep_back(x, wx, wh, b, dh, want_dx):
    """dL/dx (or None), dwx, dwh, db of one direction from dL/dh [T][N][P][Q][O]."""
    T, N, P, Q, C = x.shape
    O, KP, KQ = wh.shape[1], wh.shape[2], wh.shape[3]
    h, gates, cells = _sweep(x, wx, wh, b, True)
    # transposed convolution: columns of dA with flipped taps times [4O KP KQ][C or O]
    back = lambda w: w.permute(0, 2, 3, 1).reshape(GATES * O * KP * KQ, -1).contiguous()  # noqa: E731
    Bh, Bx = back(wh), back(wx)
    dwx, dwh, db = torch.zeros_like(wx), torch.zeros_like(wh), torch.zeros_like(b)
    dx = torch.empty_like(x) if want_dx else None
    nxt, carry = None, None                    # columns of dA_{t+1}; dL/dc_{t+1} f_{t+1}
    for t in range(T - 1, -1, -1):
        gh = dh[t].reshape(-1, O)
        if nxt is not None:
            gh = gh + nxt @ Bh
        i, f, g, o = gates[t].view(-1, GATES, O).unbind(1)
        tc = torch.tanh(cells[t])
        gc = gh * o * (1 - tc * tc)
        if carry is not None:
            gc = gc + carry
        cp = cells[t - 1] if t > 0 else torch.zeros_like(tc)
        dA = torch.cat([gc * g * i * (1 - i), gc * cp * f * (1 - f), gc * i * (1 - g * g), gh * tc * o * (1 - o)], 1)
        carry = gc * f
        nxt = _im2col(dA.view(N, P, Q, GATES * O))(KP, KQ, flip=True)
        dwx += (dA.t() @ _im2col(x[t])(KP, KQ)).view_as(dwx)
        if t > 0:
            dwh += (dA.t() @ _im2col(h[t - 1])(KP, KQ)).view_as(dwh)
        db += dA.sum(0)
        if want_dx:
            dx[t] = (nxt @ Bx).view(N, P, Q, C)
    return dx, dwx, dwh, db


def _directions(two):
    """(sweep axis, forward) of each direction over [N][D][H][W][C] (an image has D = 1)."""
    return [(ax, s) for ax in ((2, 3) if two else (1, 2, 3)) for s in (True, False)]


def _planes(v, axis, ahead):
    v = v.movedim(axis, 0)
    return v if ahead else v.flip(0)


def _unplanes(v, axis, ahead):
    return (v if ahead else v.flip(0)).movedim(0, axis)


def _double(L, two):
    wx, wh = L.wx.double(), L.wh.double()
    return (wx.unsqueeze(-2), wh.unsqueeze(-2), L.b.double()) if two else (wx, wh, L.b.double())


def _exact_forward(x, L, two):
    wx, wh, b = _double(L, two)
    h = None
    for d, (axis, ahead) in enumerate(_directions(two)):
        hd = _unplanes(_sweep(_planes(x, axis, ahead), wx[d], wh[d], b[d], False)[0], axis, ahead)
        h = hd if h is None else h + hd
    return h


def _exact_backward(x, L, dh, want_dx, two):
    wx, wh, b = _double(L, two)
    dwx, dwh, db = torch.empty_like(wx), torch.empty_like(wh), torch.empty_like(b)
    dx = None
    for d, (axis, ahead) in enumerate(_directions(two)):
        g, dwx[d], dwh[d], db[d] = _sweep_back(_planes(x, axis, ahead), wx[d], wh[d], b[d],
                                               _planes(dh, axis, ahead), want_dx)
        if want_dx:
            g = _unplanes(g, axis, ahead)
            dx = g if dx is None else dx + g
    return dx, dwx.view(L.wx.shape), dwh.view(L.wh.shape), db


def _exact_train(s, case):
    two = False
    a, ins, hs, ys = s["x"].double(), [], [], []
    for li, L in enumerate(s["layers"]):
        ins.append(a)
        a = _exact_forward(a, L, two)
        hs.append(a)
        if li < len(s["fcs"]):
            w, b = s["fcs"][li]
            a = torch.tanh(a @ w.double().t() + b.double())
            ys.append(a)
    hw, hb = s["head"][0].double(), s["head"][1].double()
    flat = a.reshape(-1, a.shape[-1])
    p = torch.softmax(flat @ hw.t() + hb, 1)
    if case["kind"] == "net":
        return p
    M = flat.shape[0]
    hot = torch.nn.functional.one_hot(s["labels"].long(), case["classes"]).double()
    if case["loss"] == "ce":
        loss = -torch.log((p * hot).sum(1)).mean()
        dl = (p - hot) / M
    else:
        loss = (hot - p).square().sum(1).mean()
        dp = 2 * (p - hot) / M
        dl = p * (dp - (p * dp).sum(1, keepdim=True))
    out = {"loss": loss.reshape(1), "p": p, "head": (dl.t() @ flat, dl.sum(0)), "fcs": [None] * len(s["fcs"]),
           "layers": [None] * len(s["layers"])}
    g = (dl @ hw).view(a.shape)
    for li in range(len(s["layers"]) - 1, -1, -1):
        if li < len(s["fcs"]):
            w = s["fcs"][li][0].double()
            dz = (g * (1 - ys[li].square())).reshape(-1, w.shape[0])
            out["fcs"][li] = (dz.t() @ hs[li].reshape(-1, w.shape[1]), dz.sum(0))
            g = (dz @ w).view(hs[li].shape)
        g, dwx, dwh, db = _exact_backward(ins[li], s["layers"][li], g, li > 0, two)
        out["layers"][li] = (dwx, dwh, db)
    return out


def exact(case, seed):
    s = prepare(case, seed)
    if case["kind"] in ("net", "train"):
        return _exact_train(s, case)
    two = case["kind"] == "step2d"
    x, L = s["x"].double(), s["layers"][0]
    if two:
        x = x.unsqueeze(1)
    h = _exact_forward(x, L, two)
    if case["kind"] == "fwd":
        return h
    dh = s["dh"].double().unsqueeze(1) if two else s["dh"].double()
    dx, dwx, dwh, db = _exact_backward(x, L, dh, case["dx"], two)
    out = {"h": h.squeeze(1) if two else h, "dwx": dwx, "dwh": dwh, "db": db}
    if case["dx"]:
        out["dx"] = dx.squeeze(1) if two else dx
    return out
