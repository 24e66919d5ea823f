"""The workloads whose speed this repository is judged by.

Each case is one pass through the library's public entry points as a program
that trains or serves quadratic layers calls them: the per-layer C ABI calls
(forward with saved maps, input gradient, weight gradient), the forward with
a fused epilogue, the autograd layers, and the CIFAR ResNet-20 training step.
Inputs are synthetic (normal activations and gradients, He-scaled weights).

``exact`` computes the same outputs in float64 with plain torch.
"""
from __future__ import annotations

import math

import torch

import paper_2204_01701_amd as ql
from paper_2204_01701_amd.autograd import quad_conv2d, quad_linear
from paper_2204_01701_amd.resnet import ResNet20Step, resnet20_geometry

DEV = "cuda:0"
NEURONS = {"quadra": ql.QL_NEURON_QUADRA, "t4": ql.QL_NEURON_T4, "t4_identity": ql.QL_NEURON_T4_IDENTITY,
           "t3": ql.QL_NEURON_T3, "t2": ql.QL_NEURON_T2, "t24": ql.QL_NEURON_T24}
TERMS = {"quadra": 3, "t4": 2, "t4_identity": 2, "t3": 1, "t2": 1, "t24": 3}
MAPS = {"quadra": 2, "t4": 2, "t4_identity": 2, "t3": 1, "t2": 0, "t24": 2}  # saved term maps


def _conv(name, n, c, hw, o, k=3, stride=1, dtype="bf16", neuron="quadra", kind="conv", **more):
    """A convolution case; the padding is that of a "same" convolution."""
    d = dict(kind=kind, n=n, c=c, hw=hw, o=o, k=k, stride=stride, pad=k // 2, dtype=dtype, neuron=neuron, **more)
    return dict(d, name=name) if name else d


def _dense(name, b, i, o, dtype="bf16", neuron="quadra", kind="dense", **more):
    d = dict(kind=kind, b=b, i=i, o=o, dtype=dtype, neuron=neuron, **more)
    return dict(d, name=name) if name else d


def listed():
    return [
        # The smallest layer of the configurations, forward and backward: launches and host time.
        _conv("small_fp32", 2, 16, 8, 16, dtype="fp32"),
        # The RGB stem of a CIFAR VGG-16 at its training batch.
        _conv("vgg_stem", 128, 3, 32, 64),
        # Training passes of one VGG-16 layer per kind of map: large and few channels ...
        _conv("vgg_64ch_32x32", 128, 64, 32, 64),
        # ... the middle of the network ...
        _conv("vgg_256ch_8x8", 128, 256, 8, 256),
        # ... and small maps with large weights.
        _conv("vgg_512ch_4x4", 128, 512, 4, 512),
        # A layer at ImageNet-style resolution: the largest convolution.
        _conv("large_conv", 64, 256, 56, 256),
        # The large fully-connected layer.
        _dense("dense_4096", 8192, 4096, 4096),
        # The classifier of a CIFAR network, trained through autograd.
        _dense("head_autograd", 128, 512, 10, kind="auto_dense", relu=False, recompute=False),
        # A depthwise layer at the same resolution as the large convolution.
        _conv("depthwise_56x56", 64, 256, 56, 256, kind="dw"),
        # Inference with a folded batch normalization and ReLU: odd maps, an odd batch, and
        # channel counts of a slimmed network, off the 16-byte vector.
        _conv("infer_ragged", 50, 60, 27, 100, kind="infer"),
        # A layer of a ReLU network trained through autograd with hybrid back-propagation.
        _conv("autograd_relu_recompute", 256, 64, 16, 128, kind="auto_conv", relu=True, recompute=True),
        # The whole CIFAR ResNet-20 training step, replayed as a HIP graph.
        dict(name="resnet20_step_fp32", kind="resnet", n=256, dtype="fp32", graph=True),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _channels(rng, lo, hi):
    """Channel counts: mostly multiples of 16, some of 8, some of any kind."""
    c, p = _log(rng, lo, hi), rng.random()
    q = 16 if p < 0.6 else 8 if p < 0.75 else 1
    return max(lo, c // q * q) if c >= q else c


def draw(rng):
    kind = rng.choices(["conv", "dense", "dw", "infer", "auto_conv", "auto_dense", "resnet"], [9, 3, 3, 3, 3, 2, 1])[0]
    if kind == "resnet":
        return dict(kind=kind, n=_log(rng, 8, 256), dtype="fp32", graph=rng.random() < 0.7)
    dtype = "bf16" if rng.random() < 0.7 or kind.startswith("auto") else "fp32"
    neuron = "quadra" if rng.random() < 0.75 else rng.choice(["t4", "t4_identity", "t3", "t2", "t24"])
    flops = 2.0e12 if dtype == "bf16" else 5.0e10
    if kind in ("dense", "auto_dense"):
        b, i = _log(rng, 1, 8192), _channels(rng, 16, 4096)
        o = rng.choice([10, 100, 200]) if kind == "auto_dense" else _channels(rng, 16, 4096)
        if neuron == "t4_identity":
            neuron = "t4"
        more = dict(relu=rng.random() < 0.5, recompute=rng.random() < 0.5) if kind == "auto_dense" else {}
        case = _dense(None, b, i, o, dtype, neuron, kind, **more)
        while work(case)["flops"] > flops and case["b"] > 1:
            case["b"] //= 2
        return case
    n, hw = _log(rng, 1, 256), _log(rng, 2, 56)
    k = rng.choices([1, 3, 5], [2, 9, 1])[0]
    stride = 1 if rng.random() < 0.75 else 2
    if kind == "dw":
        c = o = 16 * _log(rng, 1, 32) if rng.random() < 0.8 else _log(rng, 8, 300)
        k = 3 if k == 1 else k
        neuron = "t4" if neuron == "t24" else neuron
    else:
        c = 3 if rng.random() < 0.12 else _channels(rng, 8, 512)
        o = _channels(rng, 16, 512)
    if neuron == "t4_identity":
        o, stride = c, 1
    if c % 8 or o % 8:
        flops /= 20
    more = dict(relu=rng.random() < 0.5, recompute=rng.random() < 0.5) if kind == "auto_conv" else {}
    case = _conv(None, n, c, hw, o, k, stride, dtype, neuron, kind, **more)
    while case["n"] > 1 and (work(case)["flops"] > flops or work(case)["bytes"] > 7e8):
        case["n"] //= 2
    return case


# --- inputs ----------------------------------------------------------------------

def _dtype(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def _code(case):
    return ql.QL_BF16 if case["dtype"] == "bf16" else ql.QL_F32


def _randn(seed, i, shape, std, dtype):
    g = torch.Generator(device=DEV).manual_seed(seed * 1009 + i)
    return (torch.randn(shape, generator=g, device=DEV) * std).to(dtype)


def _out_hw(case):
    return (case["hw"] + 2 * case["pad"] - case["k"]) // case["stride"] + 1


def _dims(case):
    """Shapes of X, each weight, Y and the reduction length of one term."""
    if "b" in case:
        return (case["b"], case["i"]), (case["o"], case["i"]), (case["b"], case["o"]), case["i"]
    n, c, hw, o, k, ho = case["n"], case["c"], case["hw"], case["o"], case["k"], _out_hw(case)
    cw = 1 if case["kind"] == "dw" else c
    return (n, hw, hw, c), (o, k, k, cw), (n, ho, ho, o), k * k * cw


def _inputs(case, seed):
    """X, weights, biases (float32), dl/dY and the epilogue's scale and shift, channels last."""
    xs, ws, ys, red = _dims(case)
    dt, nt = _dtype(case), TERMS[case["neuron"]]
    std = math.sqrt((1.0 if "b" in case else 2.0) / red)
    return dict(x=_randn(seed, 0, xs, 1.0, dt),
                w=[_randn(seed, 1 + t, ws, std, dt) for t in range(nt)],
                b=[_randn(seed, 4 + t, (ws[0],), 0.1, torch.float32) for t in range(nt)],
                g=_randn(seed, 7, ys, 1.0, dt),
                scale=1.0 + _randn(seed, 8, (ws[0],), 0.1, torch.float32),
                shift=_randn(seed, 9, (ws[0],), 0.1, torch.float32))


def _resnet_inputs(case, seed):
    geo = resnet20_geometry(case["n"])
    dt, params = _dtype(case), {}

    def layer(i, shape, std):
        p = {k: _randn(seed, 16 * i + t, shape, std, dt).float() for t, k in enumerate(("wa", "wb", "wc"))}
        p.update({k: _randn(seed, 16 * i + 3 + t, (shape[0],), 0.1, torch.float32) for t, k in enumerate(("ba", "bb", "bc"))})
        return p

    for i, (c, _, _, o, _) in enumerate(geo):
        params[i] = layer(i, (o, c, 3, 3), math.sqrt(2.0 / (9 * c)))
    params["head"] = layer(len(geo), (10, geo[-1][3]), math.sqrt(1.0 / geo[-1][3]))
    x = _randn(seed, 900, (case["n"], 3, 32, 32), 1.0, dt)
    g = _randn(seed, 901, (case["n"], 10), 1.0, dt)
    return geo, params, x, g


def _pad3(v):
    return list(v) + [None] * (3 - len(v))


def prepare(case, seed):
    kind = case["kind"]
    if kind == "resnet":
        geo, params, x, g = _resnet_inputs(case, seed)
        net = ResNet20Step(params, x, g, dtype=_dtype(case), device=DEV)
        # the three terms' gradients of a layer side by side, as an optimizer or an all-reduce takes them
        grads = []
        for L, (c, _, _, o, _) in zip(net.layers, geo):
            dw = torch.empty((3, o, 3, 3, c), device=DEV)
            db = torch.empty((3, o), device=DEV)
            L["dw"], L["db"] = list(dw.unbind(0)), list(db.unbind(0))
            grads += [dw, db]
        dw, db = torch.empty((3, 10, geo[-1][3]), device=DEV), torch.empty((3, 12), device=DEV)
        net.hdw, net.hdb = list(dw.unbind(0)), [v[:10] for v in db.unbind(0)]
        grads += [dw, db[:, :10]]
        if case["graph"]:
            net.capture()
        return dict(case=case, net=net, out=[net.logits] + grads)
    s = _inputs(case, seed)
    xs, ws, ys, _ = _dims(case)
    nt, neuron, dt = TERMS[case["neuron"]], NEURONS[case["neuron"]], _dtype(case)
    st = dict(case=case, neuron=neuron)
    if kind in ("auto_conv", "auto_dense"):
        view = (lambda t: t.permute(0, 3, 1, 2)) if kind == "auto_conv" else (lambda t: t)
        st.update(x=view(s["x"]).requires_grad_(), w=_pad3([view(w).requires_grad_() for w in s["w"]]),
                  b=_pad3([b.requires_grad_() for b in s["b"]]), g=view(s["g"]))
        return st

    def new(shape, dtype=dt):
        return torch.empty(shape, device=DEV, dtype=dtype)

    st.update(x=s["x"], w=_pad3(s["w"]), b=_pad3(s["b"]), g=s["g"], y=new(ys))
    if "b" in case:
        st["desc"] = d = ql.linear_desc(case["b"], case["i"], case["o"], _code(case), neuron)
        sizes = [ql.qlayer_linear_fwd_workspace_size(d), ql.qlayer_linear_bwd_workspace_size(d)]
    else:
        st["desc"] = d = ql.conv_desc(case["n"], case["c"], case["hw"], case["hw"], case["o"], case["k"], case["k"],
                                      case["stride"], case["pad"], _code(case), neuron,
                                      groups=case["c"] if kind == "dw" else 1)
        if kind == "infer":
            st["keep"] = s["scale"], s["shift"]
            st["epi"] = ql.epilogue(s["scale"], s["shift"], relu=True)
            sizes = [ql.qlayer_conv2d_fwd_ex_workspace_size(d, st["epi"])]
        else:
            sizes = [ql.qlayer_conv2d_fwd_workspace_size(d), ql.qlayer_conv2d_bwd_data_workspace_size(d),
                     ql.qlayer_conv2d_bwd_weight_workspace_size(d)]
    st["ws"] = torch.empty(max(256, *sizes), device=DEV, dtype=torch.uint8)
    if kind != "infer":
        maps = [new(ys) for _ in range(MAPS[case["neuron"]])]
        st["maps"] = (maps + [None, None])[:2]
        st["dx"] = new(xs)
        st["dw"] = _pad3([new(ws, torch.float32) for _ in range(nt)])
        st["db"] = _pad3([new((ws[0],), torch.float32) for _ in range(nt)])
    return st


# --- one pass ----------------------------------------------------------------------

def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "resnet":
        if case["graph"]:
            st["net"].replay()
        else:
            st["net"].step(torch.cuda.current_stream())
        return st["out"]
    if kind in ("auto_conv", "auto_dense"):
        if kind == "auto_conv":
            y = quad_conv2d(st["x"], *st["w"], *st["b"], stride=case["stride"], pad=case["pad"],
                            recompute=case["recompute"], neuron=st["neuron"], relu=case["relu"])
        else:
            y = quad_linear(st["x"], *st["w"], *st["b"], recompute=case["recompute"], neuron=st["neuron"],
                            relu=case["relu"])
        leaves = [st["x"]] + [t for t in st["w"] + st["b"] if t is not None]
        return [y.detach(), *torch.autograd.grad(y, leaves, st["g"])]
    d, x, w, b, ws = st["desc"], st["x"], st["w"], st["b"], st["ws"]
    if kind == "infer":
        ql.qlayer_conv2d_fwd_ex(d, x, *w, *b, st["y"], epi=st["epi"], workspace=ws)
        return [st["y"]]
    (ta, tb), g = st["maps"], st["g"]
    if kind == "dense":
        ql.qlayer_linear_fwd(d, x, *w, *b, st["y"], ta, tb, workspace=ws)
        ql.qlayer_linear_bwd(d, x, g, ta, tb, *w, st["dx"], *st["dw"], *st["db"], workspace=ws)
    else:
        ql.qlayer_conv2d_fwd(d, x, *w, *b, st["y"], ta, tb, workspace=ws)
        if case["neuron"] == "t24":
            ql.qlayer_conv2d_bwd_data_ex(d, g, ta, tb, x, *w, st["dx"], workspace=ws)
        else:
            ql.qlayer_conv2d_bwd_data(d, g, x if case["neuron"] == "t2" else ta, tb, *w, st["dx"], workspace=ws)
        ql.qlayer_conv2d_bwd_weight(d, x, g, ta, tb, *st["dw"], *st["db"], workspace=ws)
    return [t for t in (st["y"], ta, tb, st["dx"], *st["dw"], *st["db"]) if t is not None]


# --- what a pass cannot do without ---------------------------------------------------

def _count(shape):
    return math.prod(shape)


def work(case):
    if case["kind"] == "resnet":
        # every layer's operands and results once per pass (they are kept for the backward), the glue's maps once
        eb, flops, nbytes = 2 if case["dtype"] == "bf16" else 4, 0, 0
        for i, (c, h, _, o, s) in enumerate(resnet20_geometry(case["n"])):
            m, x, wt = case["n"] * (h // s) ** 2 * o, case["n"] * h * h * c, 9 * c * o
            flops += 3 * 2 * m * 9 * c * (3 if i else 2)
            nbytes += eb * (x + 3 * wt + 3 * m) + eb * (x + 3 * m) + 12 * wt  # forward, weight gradient
            nbytes += eb * (3 * m + 3 * wt + x) if i else 0                   # input gradient
            nbytes += eb * (2 * m) + eb * (4 * m)                             # normalization, forward and backward
        return dict(bytes=nbytes, flops=flops)
    xs, ws, ys, red = _dims(case)
    x, wt, y = _count(xs), _count(ws), _count(ys)
    nt, nm, eb = TERMS[case["neuron"]], MAPS[case["neuron"]], 2 if case["dtype"] == "bf16" else 4
    unit = 2 * y * red  # one term of one pass
    if case["kind"] == "infer":
        return dict(bytes=eb * (x + nt * wt + y) + 4 * (nt + 2) * ws[0], flops=nt * unit)
    passes = 3 * nt
    if case.get("recompute"):
        passes += min(nm, nt)
    gbytes = eb if case["kind"].startswith("auto") else 4  # weight gradients
    nbytes = eb * (x + nt * wt + (1 + nm) * y)             # forward
    nbytes += eb * ((1 + nm) * y + nt * wt + x)            # input gradient
    nbytes += eb * (x + (1 + nm) * y) + gbytes * nt * wt + 4 * nt * ws[0]
    if case.get("relu"):
        nbytes += eb * y
    return dict(bytes=nbytes, flops=passes * unit)


def tolerance(case):
    if case["kind"] == "resnet":
        return {"rel": 1e-3}
    if case["dtype"] == "fp32":
        return {"rel": 1e-5}
    return {"rel": 1e-2}


# --- float64 -------------------------------------------------------------------------

def _patch(xp, r, q, s, ho):
    return xp[:, r:r + s * (ho - 1) + 1:s, q:q + s * (ho - 1) + 1:s, :]


def _corr(xp, w, s, ho, dw):
    """Correlation of the padded channels-last map with w (O, K, K, C)."""
    out = 0
    for r in range(w.shape[1]):
        for q in range(w.shape[2]):
            p = _patch(xp, r, q, s, ho)
            out = out + (p * w[:, r, q, 0] if dw else (p.reshape(-1, p.shape[-1]) @ w[:, r, q].T).reshape(*p.shape[:3], -1))
    return out


def _corr_dw(xp, g, k, s, dw):
    """Gradient of that correlation in w."""
    ho, o = g.shape[1], g.shape[3]
    out = torch.empty((o, k, k, 1 if dw else xp.shape[3]), device=g.device, dtype=g.dtype)
    for r in range(k):
        for q in range(k):
            p = _patch(xp, r, q, s, ho)
            out[:, r, q] = ((p * g).sum((0, 1, 2)).unsqueeze(1) if dw
                            else g.reshape(-1, o).T.contiguous() @ p.reshape(-1, p.shape[-1]))
    return out


def _corr_dx(g, w, xp_shape, s, dw):
    """Gradient of that correlation in the padded map."""
    out = torch.zeros(xp_shape, device=g.device, dtype=g.dtype)
    ho = g.shape[1]
    for r in range(w.shape[1]):
        for q in range(w.shape[2]):
            _patch(out, r, q, s, ho).add_(
                g * w[:, r, q, 0] if dw else (g.reshape(-1, g.shape[3]) @ w[:, r, q].contiguous()).reshape(*g.shape[:3], -1))
    return out


def _exact_resnet(case, seed):
    geo, params, x, g = _resnet_inputs(case, seed)

    def leaf(t):
        return t.double().requires_grad_()

    def quad(cols, p, b):
        ta, tb, tc = (cols @ p[t].reshape(p[t].shape[0], -1).T + b[t] for t in range(3))
        return ta * tb + tc

    ws = [[leaf(params[i][k].permute(0, 2, 3, 1).contiguous()) for k in ("wa", "wb", "wc")] for i in range(len(geo))]
    bs = [[leaf(params[i][k]) for k in ("ba", "bb", "bc")] for i in range(len(geo))]
    hw = [leaf(params["head"][k]) for k in ("wa", "wb", "wc")]
    hb = [leaf(params["head"][k]) for k in ("ba", "bb", "bc")]
    a, block = x.double().permute(0, 2, 3, 1).contiguous(), None
    for i, (c, h, _, o, s) in enumerate(geo):
        xin, ho = a, h // s
        xp = torch.nn.functional.pad(a, (0, 0, 1, 1, 1, 1))
        cols = torch.cat([_patch(xp, r, q, s, ho).reshape(-1, c) for r in range(3) for q in range(3)], 1)
        y = quad(cols, ws[i], bs[i]).reshape(case["n"], ho, ho, o)
        z = (y - y.mean((0, 1, 2))) / torch.sqrt(y.var((0, 1, 2), unbiased=False) + 1e-5)
        if i % 2 == 1:
            block = xin
        elif i > 0:
            if block.shape != z.shape:
                cb = block.shape[3]
                block = torch.nn.functional.pad(block[:, ::2, ::2], ((o - cb) // 2, (o - cb) // 2))
            z = z + block
        a = torch.relu(z)
    logits = quad(a.mean((1, 2)), hw, hb)
    flat = [t for p, b in zip(ws + [hw], bs + [hb]) for t in p + b]
    grads = torch.autograd.grad(logits, flat, g.double())
    out = [logits.detach()]
    for i in range(0, len(grads), 6):
        out += [torch.stack(grads[i:i + 3]), torch.stack(grads[i + 3:i + 6])]
    return out


def exact(case, seed):
    kind, neuron = case["kind"], case["neuron"] if "neuron" in case else None
    if kind == "resnet":
        return _exact_resnet(case, seed)
    s = _inputs(case, seed)
    x, g = s["x"].double(), s["g"].double()
    w, b = [t.double() for t in s["w"]], [t.double() for t in s["b"]]
    dense, dw, nt = "b" in case, kind == "dw", len(s["w"])
    if dense:
        x, g, w = x[:, None, None], g[:, None, None], [t[:, None, None] for t in w]
        k, st, pad = 1, 1, 0
    else:
        k, st, pad = case["k"], case["stride"], case["pad"]
    ho = g.shape[1]
    xp = torch.nn.functional.pad(x, (0, 0, pad, pad, pad, pad)) if pad else x
    on_square = neuron == "t2"
    tm = [_corr(xp * xp if on_square or (neuron == "t24" and t == 2) else xp, w[t], st, ho, dw) + b[t] for t in range(nt)]
    if neuron in ("quadra", "t24"):
        y = tm[0] * tm[1] + tm[2]
    elif neuron in ("t4", "t4_identity"):
        y = tm[0] * tm[1] + (x if neuron == "t4_identity" else 0)
    else:
        y = tm[0] * tm[0] if neuron == "t3" else tm[0]
    if kind == "infer":
        return [torch.relu(y * s["scale"].double() + s["shift"].double())]
    relu = bool(case.get("relu"))
    if relu:
        y = torch.relu(y)
        g = g * (y > 0)
    if neuron in ("quadra", "t24"):
        gt = [g * tm[1], g * tm[0], g]
    elif neuron in ("t4", "t4_identity"):
        gt = [g * tm[1], g * tm[0]]
    else:
        gt = [2 * g * tm[0]] if neuron == "t3" else [g]
    dxp, dws = 0, []
    for t in range(nt):
        square = on_square or (neuron == "t24" and t == 2)
        part = _corr_dx(gt[t], w[t], xp.shape, st, dw)
        dxp = dxp + (2 * xp * part if square else part)
        dws.append(_corr_dw(xp * xp if square else xp, gt[t], k, st, dw))
    dx = dxp[:, pad:pad + x.shape[1], pad:pad + x.shape[2]] if pad else dxp
    if neuron == "t4_identity":
        dx = dx + g
    dbs = [v.sum((0, 1, 2)) for v in gt]
    if dense:
        y, dx, dws, tm = y[:, 0, 0], dx[:, 0, 0], [v[:, 0, 0] for v in dws], [v[:, 0, 0] for v in tm]
    if kind.startswith("auto"):
        if not dense:
            y, dx, dws = y.permute(0, 3, 1, 2), dx.permute(0, 3, 1, 2), [v.permute(0, 3, 1, 2) for v in dws]
        return [y, dx, *dws, *dbs]
    return [y, *tm[:MAPS[neuron]], dx, *dws, *dbs]
