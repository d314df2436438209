"""Performance cases: the work that programs built on this library have it do, through the public
entry points of paper_2002_09481_amd.

Every case is a dict of plain values; its "kind" says which part of the library it exercises:

  conv      one layer on 8-bit codes, one call that prepares its constants itself (ax_conv2d,
            ax_conv2d_ex with signed codes or dilation) or a prepared layer handle
  dense     one dense layer on 8-bit codes, one call or a handle
  network   inference with prepared handles, one after another on one stream: the 54 layers of the
            ResNet-50-shaped workload or the seven of the CIFAR-shaped stack
  float     the CIFAR-shaped stack chained from float32: ranges, quantization and ReLU on the device
  depthwise one depthwise layer on 8-bit codes
  sweep     two layers ranked over many multiplier tables that arrive from host memory
  backward  gradients of the three convolutions of a bottleneck block

Operands have the distributions of the repository's synthetic workloads: uniform codes for images,
per-tensor quantized ReLU of normal values for hidden activations, quantized normal filters.  Tables
are the truncated array multiplier, the exact one and exact-plus-random-error ones.
"""

import math

import numpy as np
import torch

from paper_2002_09481_amd import binding as ax
from paper_2002_09481_amd import inputs as I
from paper_2002_09481_amd.sweep import TableSweep

DEV = "cuda"


def listed():
    return [
        # the smallest call: latency of one layer of the size unit tests and toy networks use
        {"name": "tiny_conv", "kind": "conv", "call": "once", "table": "truncated4", "N": 1, "H": 16, "W": 16, "Cin": 8,
         "k": 3, "Cout": 8, "stride": 1, "pad": 1, "dilation": 1, "signed": False},
        # sizes that fit no tile: odd image, channels that are no multiple of 16 on either side
        {"name": "ragged_conv", "kind": "conv", "call": "once", "table": "random", "N": 5, "H": 45, "W": 37, "Cin": 50,
         "k": 3, "Cout": 70, "stride": 2, "pad": 1, "dilation": 1, "signed": False},
        # operator variants: signed multiplier, dilated filter (segmentation networks)
        {"name": "signed_dilated_conv", "kind": "conv", "call": "once", "table": "random", "N": 32, "H": 56, "W": 56,
         "Cin": 64, "k": 3, "Cout": 64, "stride": 1, "pad": 2, "dilation": 2, "signed": True},
        # the classifier of a network at serving batch size: few rows, one handle kept by the server
        {"name": "classifier", "kind": "dense", "call": "handle", "table": "truncated6", "M": 32, "K": 2048, "N": 1000},
        # a large square matrix product, constants prepared in the call
        {"name": "dense_square", "kind": "dense", "call": "once", "table": "exact", "M": 256, "K": 4096, "N": 4096},
        # small-image network, evaluation batch
        {"name": "cifar_stack", "kind": "network", "net": "cifar", "batch": 128, "table": "truncated6"},
        # one image through the large network: serving latency
        {"name": "resnet50_one_image", "kind": "network", "net": "resnet50", "batch": 1, "table": "truncated6"},
        # the headline workload
        {"name": "resnet50", "kind": "network", "net": "resnet50", "batch": 32, "table": "truncated6"},
        # ranking of candidate multipliers: tables from host memory, layers prepared again per table
        {"name": "table_sweep", "kind": "sweep", "batch": 32, "hw": 28, "wide": 512, "mid": 128, "tables": 16, "chunk": 1},
        # float network as the paper's operator runs it, its batch of 1000 images
        {"name": "float_stack", "kind": "float", "batch": 1000, "table": "truncated6"},
        # first depthwise layer of a mobile-style network
        {"name": "depthwise", "kind": "depthwise", "table": "truncated6", "N": 32, "H": 112, "W": 112, "C": 32, "mult": 1,
         "k": 3, "stride": 1, "signed": False},
        # training: both gradients of the convolutions of one bottleneck block
        {"name": "block_backward", "kind": "backward", "batch": 32, "hw": 14, "cin": 1024, "mid": 256, "stride": 1},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _tab(rng):
    return rng.choice(["truncated4", "truncated6", "random", "exact"])


def draw(rng):
    kind = rng.choice(["conv", "conv", "dense", "network", "network", "float", "depthwise", "sweep", "backward"])
    if kind == "conv":
        while True:
            k = rng.choice([1, 3, 3, 5, 7])
            d = rng.choice([1, 1, 1, 2]) if k > 1 else 1
            c = {"kind": kind, "call": rng.choice(["once", "handle"]), "table": _tab(rng), "N": _log(rng, 1, 64),
                 "H": _log(rng, 7, 112), "W": _log(rng, 7, 112), "Cin": _log(rng, 3, 512), "k": k,
                 "Cout": _log(rng, 8, 512), "stride": rng.choice([1, 1, 2]), "pad": d * (k // 2), "dilation": d,
                 "signed": rng.random() < 0.25}
            if 1e5 <= _conv_layer(c).macs <= 3e10 and c["N"] * c["H"] * c["W"] * c["Cin"] < 1e8:
                return c
    if kind == "dense":
        while True:
            c = {"kind": kind, "call": rng.choice(["once", "handle"]), "table": _tab(rng), "M": _log(rng, 1, 4096),
                 "K": _log(rng, 64, 8192), "N": _log(rng, 10, 8192)}
            if 1e5 <= c["M"] * c["K"] * c["N"] <= 3e10:
                return c
    if kind == "network":
        net = rng.choice(["cifar", "resnet50"])
        return {"kind": kind, "net": net, "batch": _log(rng, 1, 1000) if net == "cifar" else _log(rng, 1, 30), "table": _tab(rng)}
    if kind == "float":
        return {"kind": kind, "batch": _log(rng, 1, 2000), "table": _tab(rng)}
    if kind == "depthwise":
        while True:
            c = {"kind": kind, "table": _tab(rng), "N": _log(rng, 1, 64), "H": _log(rng, 7, 150), "W": _log(rng, 7, 150),
                 "C": rng.choice([_log(rng, 8, 1024), 8 * _log(rng, 1, 128), 32, 128, 512]), "mult": rng.choice([1, 1, 1, 2]),
                 "k": rng.choice([3, 3, 5]), "stride": rng.choice([1, 2]), "signed": rng.random() < 0.25}
            if c["N"] * c["H"] * c["W"] * c["C"] * c["mult"] <= 1e8:
                return c
    if kind == "sweep":
        return {"kind": kind, "batch": _log(rng, 1, 32), "hw": rng.choice([7, 14, 21, 28]), "wide": _log(rng, 64, 512),
                "mid": _log(rng, 32, 128), "tables": rng.randint(3, 16), "chunk": rng.choice([1, 1, 4, 8])}
    while True:
        c = {"kind": "backward", "batch": _log(rng, 1, 32), "hw": rng.choice([7, 14, 20, 28, 56]), "cin": _log(rng, 32, 1024),
             "mid": _log(rng, 16, 512), "stride": rng.choice([1, 1, 2])}
        if sum(l.macs for l in _block_layers(c)) <= 3e10:
            return c


# ---- layers of a case ------------------------------------------------------------------------


def _conv_layer(c):
    span = (c["k"] - 1) * c["dilation"] + 1  # extent of the dilated filter: gives OH and OW of the plain formula

    class Conv(I.Layer):
        @property
        def OH(self):
            return (self.H + 2 * self.pad - span) // self.stride + 1

        @property
        def OW(self):
            return (self.W + 2 * self.pad - span) // self.stride + 1

    return Conv("conv", c["N"], c["H"], c["W"], c["Cin"], c["k"], c["k"], c["Cout"], c["stride"], c["pad"],
                x_dist="relu" if c["Cin"] > 4 else "uniform", w_dist="normal")


def _dense_layer(c):
    return I.Layer("dense", c["M"], 1, 1, c["K"], 1, 1, c["N"], dense=True, x_dist="relu", w_dist="normal")


def _net_layers(c):
    return I.config_resnet50(c["batch"]) if c.get("net") == "resnet50" else I.config_resnet8_cifar(c["batch"])


def _sweep_layers(c):
    b, hw, wide, mid = c["batch"], c["hw"], c["wide"], c["mid"]
    return [I.Layer("a", b, hw, hw, wide, 1, 1, mid), I.Layer("b", b, hw, hw, mid, 3, 3, mid, 1, 1)]


def _block_layers(c):
    b, hw, cin, mid, s = c["batch"], c["hw"], c["cin"], c["mid"], c["stride"]
    return [I.Layer("a", b, hw, hw, cin, 1, 1, mid, x_dist="relu", w_dist="normal"),
            I.Layer("b", b, hw, hw, mid, 3, 3, mid, s, 1, x_dist="relu", w_dist="normal"),
            I.Layer("c", b, (hw - 1) // s + 1, (hw - 1) // s + 1, mid, 1, 1, cin, x_dist="relu", w_dist="normal")]


def _dw_layer(c):
    return I.Layer("dw", c["N"], c["H"], c["W"], c["C"], c["k"], c["k"], c["mult"], c["stride"], c["k"] // 2,
                   x_dist="relu6", w_dist="normal")


def _layers(c):
    return {"conv": lambda: [_conv_layer(c)], "dense": lambda: [_dense_layer(c)], "network": lambda: _net_layers(c),
            "float": lambda: _net_layers(c), "depthwise": lambda: [_dw_layer(c)], "sweep": lambda: _sweep_layers(c),
            "backward": lambda: _block_layers(c)}[c["kind"]]()


# ---- inputs, made on the GPU from the seed ----------------------------------------------------


def _gen(seed, i=0):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed * 1009 + i)
    return g


def _table(name, seed, signed=False):
    if name == "random":
        t = I.lut_signed_random_error(seed) if signed else I.lut_random_error(seed)
    elif signed:
        t = I.lut_signed_exact().astype(np.int64)
        if name != "exact":  # low bits of the magnitude dropped
            t = np.sign(t) * (np.abs(t) >> int(name[-1]) << int(name[-1]))
        t = t.astype(np.int16)
    else:
        t = I.lut_exact() if name == "exact" else I.lut_truncated(int(name[-1]))
    return ax.lut_to_device(t)


def _quantized(r):
    lo, hi = min(float(r.min()), 0.0), max(float(r.max()), 0.0)
    scale = (hi - lo) / 255.0 or 1.0
    zp = int(min(255, max(0, round(-lo / scale))))
    return (torch.round(r / scale) + zp).clamp_(0, 255).to(torch.uint8), scale, zp


def _codes(dist, shape, g):
    if dist == "uniform":
        return torch.randint(0, 256, shape, generator=g, device=DEV, dtype=torch.uint8), 1.0 / 64.0, 128
    r = torch.randn(shape, generator=g, device=DEV)
    if dist == "relu":
        r.clamp_(min=0.0)
    elif dist == "relu6":
        r.clamp_(0.0, 6.0)
    return _quantized(r)


def _operands(l, g, signed=False):
    x, xs, xz = _codes(l.x_dist, (l.N, l.H, l.W, l.Cin), g)
    w, ws, wz = _codes("uniform" if l.w_dist == "uniform" else "normal", (l.KH, l.KW, l.Cin, l.Cout), g)
    q = I.Quant(xs, xz, ws, wz, None)
    if signed:  # the same real values on codes lowered by 128
        x, w = ((t.to(torch.int16) - 128).to(torch.int8) for t in (x, w))
        q.x_zp, q.w_zp = q.x_zp - 128, q.w_zp - 128
    return x, w, q


def _outs(shape):
    return torch.empty(shape, dtype=torch.int32, device=DEV), torch.empty(shape, dtype=torch.float32, device=DEV)


def _scratch(n):
    return torch.empty(max(256, int(n)), dtype=torch.uint8, device=DEV)


def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case}
    g = _gen(seed)
    if kind in ("conv", "dense", "depthwise"):
        l = _layers(case)[0]
        signed = bool(case.get("signed"))
        x, w, q = _operands(l, g, signed)
        lut = _table(case["table"], seed, signed)
        cout = l.Cin * l.Cout if kind == "depthwise" else l.Cout
        if kind == "dense":
            x, w = x.view(l.N, l.K), w.view(l.K, l.Cout)
            desc = ax._dense_desc(l.N, l.K, l.Cout)
        else:
            desc = ax._conv_desc(x.shape, w.shape, l.stride, l.pad, case.get("dilation", 1), kind == "depthwise", signed)
        acc, y = _outs((l.N, cout) if kind == "dense" else (l.N, l.OH, l.OW, cout))
        s.update(l=l, x=x, w=w, q=q, lut=lut, acc=acc, y=y)
        if case.get("call", "handle") == "handle":
            h = s["h"] = ax.AxLayer(desc, q)
            h.prepare(w, lut)
            s["ws"] = _scratch(h.workspace_bytes)
        elif kind == "dense":
            s["ws"] = _scratch(ax.ax_dense_workspace_bytes(l.N, l.K, l.Cout))
        else:
            s["ws"] = _scratch(ax.lib().ax_conv2d_ex_workspace_bytes(desc, None))
    elif kind == "network":
        lut = _table(case["table"], seed)
        s["layers"], most = [], 256
        for i, l in enumerate(_layers(case)):
            x, w, q = _operands(l, _gen(seed, i))
            if l.dense:
                x, w, desc = x.view(l.N, l.K), w.view(l.K, l.Cout), ax._dense_desc(l.N, l.K, l.Cout)
            else:
                desc = ax._conv_desc(x.shape, w.shape, l.stride, l.pad)
            h = ax.AxLayer(desc, q)
            h.prepare(w, lut)
            most = max(most, h.workspace_bytes)
            s["layers"].append((h, x, torch.empty(h.out_shape(), dtype=torch.float32, device=DEV)))
        s["ws"] = _scratch(most)  # one stream: the layers take turns
    elif kind == "float":
        s["lut"], s["layers"], most = _table(case["table"], seed), [], 256
        for i, l in enumerate(_layers(case)):
            w = torch.randn((l.KH, l.KW, l.Cin, l.Cout), generator=_gen(seed, 1 + i), device=DEV) * 0.1
            s["layers"].append((l, w) + _outs((l.N, l.OH, l.OW, l.Cout)))
            most = max(most, ax.ax_conv2d_f32_workspace_bytes((l.N, l.H, l.W, l.Cin), w.shape, l.stride, l.pad))
        l = s["layers"][0][0]
        s["x"] = torch.randn((l.N, l.H, l.W, l.Cin), generator=g, device=DEV)
        s["ws"] = _scratch(most)
    elif kind == "sweep":
        layers = []
        for i, l in enumerate(_layers(case)):
            x, w, q = _operands(l, _gen(seed, i))
            layers.append((ax._conv_desc(x.shape, w.shape, l.stride, l.pad), q, x, w))
        s["sweep"] = TableSweep(layers, chunk=case["chunk"])
        tables = np.stack([I.lut_random_error(seed * 64 + t) for t in range(case["tables"])]).view(np.int16)
        s["tables"] = torch.empty(tables.shape, dtype=torch.int16, pin_memory=True)
        s["tables"].copy_(torch.from_numpy(tables))
        outs = [_outs(s["sweep"].out_shape(i, case["tables"])) for i in range(len(layers))]
        s["acc"], s["y"] = [o[0] for o in outs], [o[1] for o in outs]
    else:
        s["layers"], most = [], 256
        for i, l in enumerate(_layers(case)):
            x, w, q = _operands(l, _gen(seed, i))
            gy = torch.randn((l.N, l.OH, l.OW, l.Cout), generator=_gen(seed, 100 + i), device=DEV)
            gx, gw = (torch.empty(t.shape, dtype=torch.float32, device=DEV) for t in (x, w))
            most = max(most, int(ax.lib().ax_conv2d_backward_workspace_bytes(ax._conv_desc(x.shape, w.shape, l.stride, l.pad))))
            s["layers"].append((l, x, w, q, gy, gx, gw))
        s["ws"] = _scratch(most)
    return s


def run(s):
    c = s["case"]
    kind = c["kind"]
    if "h" in s:
        return s["h"].run(s["x"], s["acc"], s["y"], s["ws"])
    if kind == "dense":
        return ax.ax_dense(s["x"], s["w"], s["lut"], s["q"], s["acc"], s["y"], s["ws"])
    if kind == "conv":
        l = s["l"]
        if c["signed"] or c["dilation"] > 1:
            return ax.ax_conv2d_ex(s["x"], s["w"], s["lut"], l.stride, l.pad, s["q"], c["dilation"], False, s["acc"], s["y"], s["ws"])
        return ax.ax_conv2d(s["x"], s["w"], s["lut"], l.stride, l.pad, s["q"], s["acc"], s["y"], s["ws"])
    if kind == "network":
        return [h.run(x, False, y, s["ws"])[1] for h, x, y in s["layers"]]
    if kind == "float":
        x, outs = s["x"], []
        for i, (l, w, acc, y) in enumerate(s["layers"]):
            ax.ax_conv2d_f32(x, w, s["lut"], l.stride, l.pad, relu=i > 0, acc_out=acc, y_out=y, workspace=s["ws"])
            x = y
            outs.append((acc, y))
        return outs
    if kind == "sweep":
        return s["sweep"].run(s["tables"], s["acc"], s["y"])
    return [ax.ax_conv2d_backward(x, w, gy, l.stride, l.pad, q, gx_out=gx, gw_out=gw, workspace=s["ws"])
            for l, x, w, q, gy, gx, gw in s["layers"]]


def work(case):
    """Operands read once, outputs written once; two operations (a table lookup or a product, and an
    addition) per term of every sum."""
    kind = case["kind"]
    nbytes = flops = 0.0
    for l in _layers(case):
        nx, nw = l.N * l.H * l.W * l.Cin, l.KH * l.KW * l.Cin * l.Cout
        ny = l.M * l.Cout
        if kind == "depthwise":
            nw, ny = l.KH * l.KW * l.Cin * l.Cout, l.M * l.Cin * l.Cout
            nbytes += nx + nw + 131072 + 8 * ny
            flops += 2.0 * ny * l.KH * l.KW
        elif kind == "backward":
            nbytes += nx + nw + 4.0 * (ny + nx + nw)
            flops += 4.0 * l.macs
        elif kind == "sweep":
            nbytes += nx + nw + case["tables"] * (131072 + 8.0 * ny)
            flops += 2.0 * case["tables"] * l.macs
        elif kind == "float":
            nbytes += 4.0 * (nx + nw) + 131072 + 8.0 * ny
            flops += 2.0 * l.macs
        else:  # a network's layers return the float tensor only
            nbytes += nx + nw + (0 if kind == "network" else 131072) + (4.0 if kind == "network" else 8.0) * ny
            flops += 2.0 * l.macs
    return {"bytes": nbytes + (131072 if kind == "network" else 0), "flops": flops}


def tolerance(case):
    """Integer sums are exact.  The float output is the rounded integer times a rounded product of
    the scales: at most three roundings of 2^-24 each.  Gradients are sums of exact products in 32-bit
    floating point: against the same convolutions in 64 bits they measure up to rel 1.9e-7, max 1.2e-6."""
    if case["kind"] == "backward":
        return {"rel": 8e-7, "max": 6e-6}
    return {"rel": 3e-7, "max": 6e-7}
