"""Cases by which the framework's speed and accuracy are measured.

Each case is one pass through the public entry points, on the sizes, types and
options that a training program uses:

  net    one SGD step of a layer chain (``Net.step``): the fp32 MLP, the
         LeNet-style bf16 network, the wide fp16 MLP with dynamic loss scaling,
         and networks of sizes between and around them;
  fc     one fully connected layer of a program that drives its own loop:
         forward with bias + ReLU, backward data with the ReLU mask, weight and
         bias gradients;
  conv   one convolution layer, the same passes (backward data left out for a
         network's first layer, which has no use for it);
  head   softmax cross-entropy over many classes, loss and gradient;
  split3 an fp32 product on the fp16 matrix cores (three products of the
         two-term splits).

``listed`` covers the smallest calls (the fp32 MLP step), ordinary and the
largest ones, with sizes that are multiples of the tiles and sizes that are
not; ``draw`` takes sizes from the same ranges.
"""
import math

import torch

import paper_2011_11188_amd as mdnn
import workloads as W

DEV = "cuda"
CODE = {"f32": mdnn.F32, "f16": mdnn.F16, "bf16": mdnn.BF16}
TORCH = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
BYTES = {"f32": 4, "f16": 2, "bf16": 2}


# --------------------------------------------------------------------------
# the cases
# --------------------------------------------------------------------------

def _net(name, chain, batch, dtype, **kw):
    c = {"name": name, "kind": "net", "chain": chain, "batch": batch, "dtype": dtype, "graph": False}
    c.update(kw)
    return c


def _fc(name, dtype, batch, n_in, n_out):
    return {"name": name, "kind": "fc", "dtype": dtype, "batch": batch, "n_in": n_in, "n_out": n_out}


def _conv(name, dtype, n, h, w, c_in, c_out, r, pad, first=False):
    return {"name": name, "kind": "conv", "dtype": dtype, "n": n, "h": h, "w": w, "c_in": c_in, "c_out": c_out,
            "r": r, "pad": pad, "first": first}


def listed():
    return [
        # the smallest step: an MNIST-sized MLP in fp32, batch 64 (launches and latency)
        _net("mlp_fp32_step_b64", "mlp", 64, "f32", n_in=784, hidden=128, depth=1, classes=10),
        # the LeNet-style network: convolutions, pooling, a wide and a narrow FC layer, two dozen launches
        _net("lenet_bf16_step_b256", "lenet", 256, "bf16", side=28, c1=32, c2=64, fc=1024, classes=10),
        # the largest single-GPU training step: regression MLP, loss scaling, momentum, update in the products
        _net("wide_mlp_fp16_step_b4096", "wide", 4096, "f16", n_in=1024, width=4096, depth=4),
        # one hidden layer of a wide network, driven by the program itself
        _fc("fc_f16_b4096_4096x4096", "f16", 4096, 4096, 4096),
        # feature counts and a batch that divide by nothing (vocabulary or table sizes, last batch of an epoch)
        _fc("fc_bf16_b1000_1531x777", "bf16", 1000, 1531, 777),
        # full-precision layer
        _fc("fc_f32_b1024_2048x2048", "f32", 1024, 2048, 2048),
        # residual-network 3x3 layer, 64 channels at 32x32
        _conv("conv_f16_b128_32x32_64x64_3x3", "f16", 128, 32, 32, 64, 64, 3, 1),
        # odd image, 5x5 filter, pixel count that is no multiple of a K step
        _conv("conv_bf16_b50_27x27_96x160_5x5", "bf16", 50, 27, 27, 96, 160, 5, 2),
        # a network's first layer on colour images, 7x7 filter
        _conv("conv_f16_b64_64x64_3x64_7x7_first", "f16", 64, 64, 64, 3, 64, 7, 3, True),
        # full-precision convolution layer
        _conv("conv_f32_b64_16x16_64x128_3x3", "f32", 64, 16, 16, 64, 128, 3, 1),
        # classifier over a thousand classes
        {"name": "head_b4096_c1000", "kind": "head", "batch": 4096, "classes": 1000, "dtype": "f16"},
        # fp32 product through the fp16 matrix cores
        {"name": "split3_nn_2048", "kind": "split3", "layout": "NN", "m": 2048, "n": 2048, "k": 2048,
         "auto_scale": False},
    ]


def _log(rng, lo, hi):
    """An integer whose logarithm is spread evenly; half of them multiples of a power of two (as sizes mostly are)."""
    v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    if rng.random() < 0.5:
        q = 8 if v < 128 else 64
        v = max(q, v // q * q) if v >= q else v
    return min(max(v, lo), hi)


def draw(rng):
    kind = rng.choice(["net", "fc", "fc", "conv", "conv", "conv", "head", "split3"])
    if kind == "net":
        chain = rng.choice(["mlp", "lenet", "wide"])
        if chain == "mlp":
            c = _net("", "mlp", _log(rng, 16, 512), rng.choice(["f32", "f16", "bf16"]), n_in=_log(rng, 64, 2048),
                     hidden=_log(rng, 32, 1024), depth=rng.randint(1, 3), classes=rng.randint(2, 100))
        elif chain == "lenet":
            c = _net("", "lenet", _log(rng, 32, 512), rng.choice(["f32", "f16", "bf16"]), side=rng.choice([16, 20, 28, 32]),
                     c1=rng.choice([16, 20, 32]), c2=rng.choice([32, 50, 64]), fc=_log(rng, 84, 1024),
                     classes=rng.randint(2, 100))
            if c["dtype"] == "f32":
                c["batch"] = min(c["batch"], 256)
        else:
            c = _net("", "wide", _log(rng, 256, 4096), rng.choice(["f16", "bf16"]), n_in=_log(rng, 256, 1024),
                     width=_log(rng, 256, 4096), depth=rng.randint(1, 4))
        c["graph"] = rng.random() < 0.25
    elif kind == "fc":
        dtype = rng.choice(["f16", "f16", "bf16", "bf16", "f32"])
        while True:
            c = _fc("", dtype, _log(rng, 16, 8192), _log(rng, 32, 8192), _log(rng, 32, 8192))
            if c["batch"] * c["n_in"] * c["n_out"] <= (1 << 36 if dtype != "f32" else 1 << 33):
                break
    elif kind == "conv":
        dtype = rng.choice(["f16", "f16", "bf16", "bf16", "f32"])
        while True:
            first = rng.random() < 0.2
            r = rng.choice([1, 3, 3, 3, 5, 7])
            h = _log(rng, 7, 64)
            w = h if rng.random() < 0.7 else _log(rng, 7, 64)
            c = _conv("", dtype, _log(rng, 8, 256), h, w, rng.choice([1, 3, 3, 4]) if first else _log(rng, 16, 512),
                      _log(rng, 16, 512), r, r // 2 if rng.random() < 0.8 else 0, first)
            macs = c["n"] * h * w * c["c_in"] * c["c_out"] * r * r
            if macs <= (1 << 34 if dtype != "f32" else 1 << 31) and c["n"] * h * w * max(c["c_in"], c["c_out"]) <= 1 << 25:
                break
    elif kind == "head":
        c = {"kind": "head", "batch": _log(rng, 32, 16384), "classes": _log(rng, 10, 1024),
             "dtype": rng.choice(["f32", "f16", "bf16"])}
    else:
        c = {"kind": "split3", "layout": rng.choice(["NN", "NT", "TN"]), "m": _log(rng, 256, 4096),
             "n": _log(rng, 256, 4096), "k": _log(rng, 256, 4096), "auto_scale": rng.random() < 0.5}
    c.pop("name", None)
    return c


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------

class _Rng:
    """Draws on the GPU, from the seed alone."""

    def __init__(self, seed):
        self.g = torch.Generator(device=DEV)
        self.g.manual_seed(int(seed))

    def normal(self, *shape, scale=1.0, dtype="f32"):
        return (torch.randn(shape, generator=self.g, device=DEV) * scale).to(TORCH[dtype])

    def relu(self, *shape, dtype="f32"):
        """A stored post-ReLU activation."""
        return torch.randn(shape, generator=self.g, device=DEV).clamp_(min=0).to(TORCH[dtype])

    def uniform(self, *shape):
        return torch.rand(shape, generator=self.g, device=DEV)

    def labels(self, n, classes):
        return torch.randint(0, classes, (n,), generator=self.g, device=DEV, dtype=torch.int32)


def _layers(case):
    """The layer chain of a net case, its loss and its hyperparameters."""
    if case["chain"] == "lenet":
        s, c1, c2 = case["side"], case["c1"], case["c2"]
        q = s // 4
        return (W.Layer(W.CONV, 1, s, s, c1, 5, 5, 2, W.ACT_RELU), W.Layer(W.MAXPOOL2, c1, s, s, c1),
                W.Layer(W.CONV, c1, s // 2, s // 2, c2, 5, 5, 2, W.ACT_RELU),
                W.Layer(W.MAXPOOL2, c2, s // 2, s // 2, c2),
                W.Layer(W.FC, q * q * c2, c_out=case["fc"], act=W.ACT_RELU),
                W.Layer(W.FC, case["fc"], c_out=case["classes"]))
    if case["chain"] == "mlp":
        widths = [case["n_in"]] + [case["hidden"]] * case["depth"] + [case["classes"]]
    else:
        widths = [case["n_in"]] + [case["width"]] * case["depth"] + [1]
    n = len(widths) - 1
    return tuple(W.Layer(W.FC, a, c_out=b, act=W.ACT_RELU if i < n - 1 else W.ACT_NONE)
                 for i, (a, b) in enumerate(zip(widths, widths[1:])))


def _hyper(case):
    if case["chain"] == "wide":
        return {"lr": 1e-4, "momentum": 0.9, "scaled": case["dtype"] == "f16", "fused": True}
    if case["chain"] == "lenet":
        return {"lr": 0.01, "momentum": 0.0, "scaled": case["dtype"] == "f16", "fused": False}
    return {"lr": 0.05, "momentum": 0.0, "scaled": case["dtype"] == "f16", "fused": False}


def _net_inputs(case, seed):
    """fp32 master parameters (He-normal weights, zero biases), the batch and its targets."""
    layers, g = _layers(case), _Rng(seed)
    parts = []
    for l in layers:
        if l.n_weight:
            parts += [g.normal(l.n_weight, scale=math.sqrt(2.0 / l.fan_in)),
                      torch.zeros(l.n_bias, dtype=torch.float32, device=DEV)]
    b, n_in = case["batch"], layers[0].c_in * layers[0].h * layers[0].w
    if case["chain"] == "wide":
        return layers, torch.cat(parts), g.normal(b, n_in), g.normal(b, 1)
    return layers, torch.cat(parts), g.uniform(b, n_in), g.labels(b, case["classes"])


def _fc_inputs(case, seed):
    g, dt = _Rng(seed), case["dtype"]
    b, i, o = case["batch"], case["n_in"], case["n_out"]
    x = g.relu(b, i, dtype=dt)
    w = g.normal(i, o, scale=math.sqrt(2.0 / i), dtype=dt)
    bias = g.normal(o, scale=0.1)
    dz = g.normal(b, o, scale=1.0 / math.sqrt(o), dtype=dt)
    return x, w, bias, dz


def _conv_inputs(case, seed):
    g, dt, r = _Rng(seed), case["dtype"], case["r"]
    ho, wo = case["h"] + 2 * case["pad"] - r + 1, case["w"] + 2 * case["pad"] - r + 1
    shape = (case["n"], case["h"], case["w"], case["c_in"])
    x = g.normal(*shape, dtype=dt) if case["first"] else g.relu(*shape, dtype=dt)
    k = r * r * case["c_in"]
    w = g.normal(case["c_out"], r, r, case["c_in"], scale=math.sqrt(2.0 / k), dtype=dt)
    bias = g.normal(case["c_out"], scale=0.1)
    dz = g.normal(case["n"], ho, wo, case["c_out"], scale=1.0 / math.sqrt(case["c_out"]), dtype=dt)
    return x, w, bias, dz


def _head_inputs(case, seed):
    g = _Rng(seed)
    return g.normal(case["batch"], case["classes"], scale=2.0), g.labels(case["batch"], case["classes"])


def _split3_inputs(case, seed):
    g = _Rng(seed)
    m, n, k, lay = case["m"], case["n"], case["k"], case["layout"]
    # an automatic scale is for data whose magnitude the program does not know
    sa, sb = (300.0, 0.01) if case["auto_scale"] else (1.0, 1.0 / math.sqrt(k))
    a = g.normal(*((k, m) if lay == "TN" else (m, k)), scale=sa)
    b = g.normal(*((n, k) if lay == "NT" else (k, n)), scale=sb)
    return a, b


def prepare(case, seed):
    kind, dt = case["kind"], case.get("dtype", "f32")
    s = {"case": case}
    if kind == "net":
        layers, params, x, t = _net_inputs(case, seed)
        h = _hyper(case)
        net = mdnn.Net(layers, case["batch"], CODE[dt], mdnn.LOSS_MSE if case["chain"] == "wide" else mdnn.LOSS_XENT,
                       h["lr"], h["momentum"], h["scaled"], 2.0 ** 16 if case["chain"] == "wide" else 2.0 ** 10,
                       n_classes=case.get("classes", 10), device=DEV, fuse_update=h["fused"])
        net.set_params(params)
        # the logits (fp32, the last layer's stored output) inside the net's workspace
        out = layers[-1].c_out
        at = net.activation_ptr(len(layers)) - net.ws.data_ptr()
        logits = net.ws[at:at + case["batch"] * out * 4].view(torch.float32).view(case["batch"], out)
        s.update(net=net, x=x, t=t, logits=logits)
        if case["graph"]:
            s["graph"] = net.record_step(x, t)
        outs = {"loss": net.loss, "logits": logits, "weights": net.master}
        if net.mom is not None:
            outs["momentum"] = net.mom
        else:
            outs["grads"] = net.grads
        s["outs"] = outs
    elif kind == "fc":
        x, w, bias, dz = _fc_inputs(case, seed)
        b, i, o = case["batch"], case["n_in"], case["n_out"]
        code = CODE[dt]
        nb = max(mdnn.mdnn_gemm_workspace(code, b, o, i), mdnn.mdnn_gemm_workspace(code, b, i, o),
                 mdnn.mdnn_gemm_workspace(code, i, o, b), mdnn.mdnn_bias_act_bwd_workspace(b, o), 256)
        s.update(x=x, w=w, bias=bias, dz=dz, ws=torch.empty(nb, dtype=torch.uint8, device=DEV),
                 y=torch.empty(b, o, dtype=TORCH[dt], device=DEV), dx=torch.empty(b, i, dtype=TORCH[dt], device=DEV),
                 dw=torch.empty(i, o, device=DEV), db=torch.empty(o, device=DEV))
    elif kind == "conv":
        x, w, bias, dz = _conv_inputs(case, seed)
        sh = mdnn.conv_shape(tuple(x.shape), case["c_out"], case["r"], case["r"], case["pad"])
        nb = max(mdnn.mdnn_conv2d_bwd_filter_workspace(sh, CODE[dt]), 256)
        s.update(x=x, w=w, bias=bias, dz=dz, sh=sh, ws=torch.empty(nb, dtype=torch.uint8, device=DEV),
                 y=torch.empty_like(dz), dx=torch.empty_like(x), dw=torch.empty(tuple(w.shape), device=DEV),
                 db=torch.empty(case["c_out"], device=DEV))
    elif kind == "head":
        logits, labels = _head_inputs(case, seed)
        s.update(logits=logits, labels=labels, scale=torch.full((1,), 1024.0, device=DEV),
                 loss=torch.empty(1, device=DEV), dz=torch.empty(tuple(logits.shape), dtype=TORCH[dt], device=DEV))
    else:
        a, b = _split3_inputs(case, seed)
        s.update(a=a, b=b, out=torch.empty(case["m"], case["n"], device=DEV))
    return s


# --------------------------------------------------------------------------
# one pass
# --------------------------------------------------------------------------

def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "net":
        if case["graph"]:
            s["graph"].launch()
        else:
            s["net"].step(s["x"], s["t"])
        return s["outs"]
    if kind == "fc":
        code, ws = CODE[case["dtype"]], s["ws"]
        mdnn.gemm(mdnn.NN, s["x"], s["w"], bias=s["bias"], act=mdnn.ACT_RELU, out=s["y"], workspace=ws)
        mdnn.mdnn_bias_act_bwd(case["batch"], case["n_out"], s["dz"], None, mdnn.ACT_NONE, None, s["db"], code, ws,
                               ws.numel())
        mdnn.gemm(mdnn.TN, s["x"], s["dz"], out=s["dw"], workspace=ws)
        mdnn.gemm(mdnn.NT, s["dz"], s["w"], mask=s["x"], out=s["dx"], workspace=ws)
        return {"y": s["y"], "db": s["db"], "dw": s["dw"], "dx": s["dx"]}
    if kind == "conv":
        sh, code, ws = s["sh"], CODE[case["dtype"]], s["ws"]
        mdnn.mdnn_conv2d_fwd(sh, s["x"], s["w"], code, s["bias"], mdnn.ACT_RELU, s["y"], code)
        mdnn.mdnn_conv2d_bwd_filter(sh, s["x"], s["dz"], code, s["dw"], s["db"], ws, ws.numel())
        out = {"y": s["y"], "db": s["db"], "dw": s["dw"]}
        if not case["first"]:
            mdnn.mdnn_conv2d_bwd_data(sh, s["dz"], s["w"], code, s["x"], s["dx"], code)
            out["dx"] = s["dx"]
        return out
    if kind == "head":
        b, c = case["batch"], case["classes"]
        mdnn.mdnn_softmax_xent(b, c, s["logits"], c, s["labels"], s["scale"], s["loss"], s["dz"], c,
                               CODE[case["dtype"]])
        return {"loss": s["loss"], "dz": s["dz"]}
    scale = 0.0 if case["auto_scale"] else 1.0
    return mdnn.gemm_split3(getattr(mdnn, case["layout"]), s["a"], s["b"], a_scale=scale, b_scale=scale, out=s["out"])


# --------------------------------------------------------------------------
# what a pass cannot do without, and how far two correct ones may differ
# --------------------------------------------------------------------------

def work(case):
    kind, es = case["kind"], BYTES[case.get("dtype", "f32")]
    if kind == "net":
        layers, b = _layers(case), case["batch"]
        h = _hyper(case)
        flops = W.TrainConfig("", 0, layers, b, 0, case["dtype"], 0, 0.0).flops_per_step()
        n = sum(l.n_weight + l.n_bias for l in layers)
        # input, weights read and written (momentum too), the 16-bit copy read and written, the output
        per = 8 + (8 if h["momentum"] else 0) + (4 if es == 2 else 0)
        return {"bytes": b * layers[0].c_in * layers[0].h * layers[0].w * 4 + n * per + b * layers[-1].c_out * 4,
                "flops": flops}
    if kind == "fc":
        b, i, o = case["batch"], case["n_in"], case["n_out"]
        return {"bytes": es * (2 * b * i + i * o + 2 * b * o) + 4 * (i * o + 2 * o), "flops": 6 * b * i * o}
    if kind == "conv":
        r, p = case["r"], case["pad"]
        px_in = case["n"] * case["h"] * case["w"]
        px_out = case["n"] * (case["h"] + 2 * p - r + 1) * (case["w"] + 2 * p - r + 1)
        ci, co, k = case["c_in"], case["c_out"], r * r * case["c_in"]
        ops = 2 if case["first"] else 3
        return {"bytes": es * ((ops - 1) * px_in * ci + co * k + 2 * px_out * co) + 4 * (co * k + 2 * co),
                "flops": ops * 2 * px_out * co * k}
    if kind == "head":
        n = case["batch"] * case["classes"]
        return {"bytes": n * (4 + es) + case["batch"] * 4, "flops": 6 * n}
    m, n, k = case["m"], case["n"], case["k"]
    return {"bytes": 4 * (m * k + k * n + m * n), "flops": 6 * m * n * k}


def tolerance(case):
    """About four times the distance between this path and 64-bit results."""
    kind, dt = case["kind"], case.get("dtype", "f32")
    if kind == "net":
        return {"rel": {"f32": 1e-5, "f16": 1e-2, "bf16": 5e-2}[dt]}
    if kind in ("fc", "conv"):
        return {"rel": {"f32": 5e-6, "f16": 1e-3, "bf16": 8e-3}[dt]}
    if kind == "head":
        return {"rel": {"f32": 5e-6, "f16": 5e-4, "bf16": 4e-3}[dt]}
    return {"rel": 5e-6}


# --------------------------------------------------------------------------
# the same results in 64 bits
# --------------------------------------------------------------------------

def _windows(h, w, r, pad):
    """(tap, rows and columns of the output, rows and columns of the input) of a stride-1 convolution."""
    ho, wo = h + 2 * pad - r + 1, w + 2 * pad - r + 1
    for a in range(r):
        for b in range(r):
            i0, i1 = max(0, pad - a), min(ho, h + pad - a)
            j0, j1 = max(0, pad - b), min(wo, w + pad - b)
            if i0 < i1 and j0 < j1:
                yield (a, b, slice(i0, i1), slice(j0, j1), slice(i0 + a - pad, i1 + a - pad),
                       slice(j0 + b - pad, j1 + b - pad))


def _conv64(x, w, pad):
    n, h, wd, c = x.shape
    k, r = w.shape[0], w.shape[1]
    y = torch.zeros(n, h + 2 * pad - r + 1, wd + 2 * pad - r + 1, k, dtype=torch.float64, device=x.device)
    for a, b, oi, oj, ii, ij in _windows(h, wd, r, pad):
        v = x[:, ii, ij, :]
        y[:, oi, oj, :] += (v.reshape(-1, c) @ w[:, a, b, :].t().contiguous()).view(*v.shape[:3], k)
    return y


def _conv64_back(x, w, dz, pad, data=True):
    n, h, wd, c = x.shape
    k, r = w.shape[0], w.shape[1]
    dx, dw = torch.zeros_like(x), torch.zeros_like(w)
    for a, b, oi, oj, ii, ij in _windows(h, wd, r, pad):
        v, d = x[:, ii, ij, :].reshape(-1, c), dz[:, oi, oj, :]
        dw[:, a, b, :] = d.reshape(-1, k).t().contiguous() @ v
        if data:
            dx[:, ii, ij, :] += (d.reshape(-1, k) @ w[:, a, b, :].contiguous()).view(*d.shape[:3], c)
    return dx, dw, dz.sum(dim=(0, 1, 2))


def _xent64(z, labels):
    b = z.shape[0]
    lp = torch.log_softmax(z, dim=1)
    rows = torch.arange(b, device=z.device)
    loss = -lp[rows, labels.long()].mean()
    g = lp.exp()
    g[rows, labels.long()] -= 1.0
    return loss, g / b


def _net64(case, seed):
    layers, params, x, t = _net_inputs(case, seed)
    h = _hyper(case)
    p, b, a = params.double(), case["batch"], x.double()
    offs, off = [], 0
    for l in layers:
        offs.append(off)
        off += l.n_weight + l.n_bias
    acts, picks = [a], {}
    for i, l in enumerate(layers):
        w, bias = p[offs[i]:offs[i] + l.n_weight], p[offs[i] + l.n_weight:offs[i] + l.n_weight + l.n_bias]
        if l.kind == W.FC:
            a = a.reshape(b, l.c_in) @ w.view(l.c_in, l.c_out) + bias
        elif l.kind == W.CONV:
            a = _conv64(a.reshape(b, l.h, l.w, l.c_in), w.view(l.c_out, l.r, l.s, l.c_in), l.pad) + bias
        else:
            v = a.reshape(b, l.h // 2, 2, l.w // 2, 2, l.c_in).permute(0, 1, 3, 5, 2, 4).reshape(
                b, l.h // 2, l.w // 2, l.c_in, 4)
            a, picks[i] = v.max(dim=-1)
        if l.kind != W.MAXPOOL2 and l.act == W.ACT_RELU:
            a = a.clamp(min=0)
        acts.append(a)
    logits = a
    if case["chain"] == "wide":
        loss, dz = ((a - t.double()) ** 2).sum() / b, 2 * (a - t.double()) / b
    else:
        loss, dz = _xent64(a, t)
    grads = torch.zeros_like(p)
    for i in range(len(layers) - 1, -1, -1):
        l, a_in = layers[i], acts[i]
        w = p[offs[i]:offs[i] + l.n_weight]
        gw, gb = grads[offs[i]:offs[i] + l.n_weight], grads[offs[i] + l.n_weight:offs[i] + l.n_weight + l.n_bias]
        if l.kind == W.FC:
            a_in = a_in.reshape(b, l.c_in)
            dz = dz.reshape(b, l.c_out)
            gw.copy_((a_in.t().contiguous() @ dz).reshape(-1))
            gb.copy_(dz.sum(dim=0))
            dx = dz @ w.view(l.c_in, l.c_out).t().contiguous() if i else None
        elif l.kind == W.CONV:
            a_in = a_in.reshape(b, l.h, l.w, l.c_in)
            dx, dw, db = _conv64_back(a_in, w.view(l.c_out, l.r, l.s, l.c_in), dz.reshape(b, l.h, l.w, l.c_out), l.pad,
                                      i > 0)
            gw.copy_(dw.reshape(-1))
            gb.copy_(db)
        else:
            d = torch.zeros(b, l.h // 2, l.w // 2, l.c_in, 4, dtype=torch.float64, device=dz.device)
            d.scatter_(-1, picks[i].unsqueeze(-1), dz.reshape(b, l.h // 2, l.w // 2, l.c_in, 1))
            dx = d.view(b, l.h // 2, l.w // 2, l.c_in, 2, 2).permute(0, 1, 4, 2, 5, 3).reshape(b, l.h, l.w, l.c_in)
        if i:
            prev = layers[i - 1]
            relu = prev.act == W.ACT_RELU if prev.kind != W.MAXPOOL2 else True
            dz = dx.reshape(acts[i].shape)
            if relu and l.kind != W.MAXPOOL2:
                dz = dz * (acts[i] > 0)
    out = {"loss": loss.reshape(1), "logits": logits, "weights": p - h["lr"] * grads}
    if h["momentum"]:
        out["momentum"] = grads
    else:
        # what the step stores is scaled by the loss scale
        out["grads"] = grads * (2.0 ** 10 if h["scaled"] else 1.0)
    return out


def exact(case, seed):
    kind = case["kind"]
    if kind == "net":
        return _net64(case, seed)
    if kind == "fc":
        x, w, bias, dz = (v.double() for v in _fc_inputs(case, seed))
        return {"y": (x @ w + bias).clamp(min=0), "db": dz.sum(dim=0), "dw": x.t().contiguous() @ dz,
                "dx": (dz @ w.t().contiguous()) * (x > 0)}
    if kind == "conv":
        x, w, bias, dz = (v.double() for v in _conv_inputs(case, seed))
        dx, dw, db = _conv64_back(x, w, dz, case["pad"], not case["first"])
        out = {"y": (_conv64(x, w, case["pad"]) + bias).clamp(min=0), "db": db, "dw": dw}
        if not case["first"]:
            out["dx"] = dx * (x > 0)
        return out
    if kind == "head":
        logits, labels = _head_inputs(case, seed)
        loss, dz = _xent64(logits.double(), labels)
        return {"loss": loss.reshape(1), "dz": dz * 1024.0}
    a, b = (v.double() for v in _split3_inputs(case, seed))
    lay = case["layout"]
    return (a.t().contiguous() if lay == "TN" else a) @ (b.t().contiguous() if lay == "NT" else b)
