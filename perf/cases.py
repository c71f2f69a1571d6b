"""The work this framework is measured on: what users of the convolution library call, through its
public entry points, over the range of sizes it is used at.

A case is a dict of plain values; `kind` says which entry points it goes through:

* "graph": one forward + backward pass of a workload bi-graph on the executor (`build_workload`, `run`);
* "conv":  the three passes of one convolution layer (fused operators; grouped where groups > 1), or
  only its forward pass where `train` is false;
* "fc":    the three passes of one fully-connected layer;
* "pool":  max pooling of a ReLU output, forward and backward.

Inputs follow what training meets: images and activations behind a ReLU (non-negative, half of the
values zero), He-scaled filters, output gradients of about 1e-3.
"""
import math
import zlib

import torch
import torch.nn.functional as F

import paper_1412_6249_amd as pa
from paper_1412_6249_amd.layers import build_workload
from synth.configs import CONV_LAYERS

DEV = "cuda:0"
MAX_FLOPS = 3.0e11          # a drawn case stays below the largest listed one
MAX_BYTES = 2.0e9


def _conv(name, dtype, N, C, H, W, K, R, stride, pad, groups=1, train=True):
    return {"name": name, "kind": "conv", "dtype": dtype, "N": N, "C": C, "H": H, "W": W, "K": K, "R": R,
            "stride": stride, "pad": pad, "groups": groups, "train": train}


def listed():
    return [
        # one small layer stepped through the executor: the latency of a pass (launches, event waits,
        # the host's part) and nothing else
        {"name": "graph_single_conv_f32", "kind": "graph", "cfg": 1, "batch": 2, "sgd": False},
        # the inception module as a training step runs it: five streams, merged 1x1 operator,
        # concatenation by address, 3x3 / 5x5 / pooling branches
        {"name": "graph_inception_f32", "kind": "graph", "cfg": 3, "batch": 128, "sgd": False},
        # one GPU's share of an AlexNet training iteration: five conv layers, pooling, SGD updates
        {"name": "graph_alexnet_f32", "kind": "graph", "cfg": 4, "batch": 128, "sgd": True},
        # GoogLeNet's stem layers in bf16 at the largest batch
        {"name": "graph_stem_bf16", "kind": "graph", "cfg": 5, "batch": 256, "sgd": False},
        # inference at a batch of two on a deep layer: long reduction, few output tiles
        _conv("conv_infer_f32", "f32", 2, 384, 13, 13, 384, 3, 1, 1, train=False),
        # no extent is a multiple of anything: ragged tiles in every direction, partial batch share
        _conv("conv_odd_f32", "f32", 29, 75, 29, 31, 150, 5, 1, 2),
        # NIN's cccp layer: 1x1, close to the memory roof
        _conv("conv_1x1_f32", "f32", 64, 96, 54, 54, 96, 1, 1, 0),
        # AlexNet's two-group conv2
        _conv("conv_grouped_f32", "f32", 128, 96, 27, 27, 256, 5, 1, 2, groups=2),
        # the inception module's 3x3 in bf16: rows of 28 elements, not whole 16-byte packets
        _conv("conv_28_bf16", "bf16", 128, 96, 28, 28, 128, 3, 1, 1),
        # AlexNet's fc6 in both types: bound by the weight matrix
        {"name": "fc_f32", "kind": "fc", "dtype": "f32", "N": 128, "C": 9216, "K": 4096},
        {"name": "fc_bf16", "kind": "fc", "dtype": "bf16", "N": 128, "C": 9216, "K": 4096},
        # AlexNet's first pooling layer, 3x3 / stride 2 on odd planes
        {"name": "pool_f32", "kind": "pool", "dtype": "f32", "N": 128, "C": 96, "H": 55, "W": 55, "window": 3,
         "stride": 2, "pad": 0},
    ]


# ------------------------------------------------------------------------------------------ drawn
def _spread(rng, lo, hi):
    """An integer of [lo, hi], spread over its logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _draw_conv(rng):
    dtype = rng.choice(["f32", "f32", "bf16"])
    R = rng.choice([1, 3, 3, 3, 5, 7, 11])
    stride = rng.choice([1, 1, 1, 2]) if R < 7 else rng.choice([2, 4])
    pad = rng.choice([0, R // 2, R // 2])
    groups = rng.choice([1, 1, 1, 2]) if R in (3, 5) else 1
    if R >= 7:
        C, HW = 3, _spread(rng, 64, 232)
    else:
        C, HW = _spread(rng, 16, 512), _spread(rng, 7, 64)
    K = _spread(rng, 16, 512)
    H = HW
    W = max(R, HW + rng.choice([0, 0, 0, 1, 2]))
    if groups == 2:                    # slices keep whole 16-byte packets
        C, K = max(16, C // 16 * 16), max(16, K // 16 * 16)
    c = _conv("", dtype, _spread(rng, 1, 256), C, H, W, K, R, stride, pad, groups, rng.random() < 0.8)
    del c["name"]
    return c


def draw(rng):
    while True:
        kind = rng.choice(["conv"] * 7 + ["fc"] * 2 + ["pool"] * 2 + ["graph"])
        if kind == "conv":
            c = _draw_conv(rng)
        elif kind == "fc":
            c = {"kind": "fc", "dtype": rng.choice(["f32", "bf16"]), "N": _spread(rng, 1, 256),
                 "C": _spread(rng, 64, 9216), "K": _spread(rng, 10, 4096)}
        elif kind == "pool":
            w, s, p = rng.choice([(3, 2, 0), (3, 2, 1), (3, 1, 1), (2, 2, 0)])
            c = {"kind": "pool", "dtype": rng.choice(["f32", "bf16"]), "N": _spread(rng, 1, 256), "C": _spread(rng, 16, 512),
                 "H": _spread(rng, 7, 112), "W": _spread(rng, 7, 112), "window": w, "stride": s, "pad": p}
        else:
            cfg = rng.choice([1, 2, 3, 4])
            c = {"kind": "graph", "cfg": cfg, "batch": _spread(rng, 1, 64), "sgd": rng.random() < 0.5}
        w = work(c)
        if w["flops"] <= MAX_FLOPS and w["bytes"] <= MAX_BYTES:
            return c


# ----------------------------------------------------------------------------------------- inputs
def _gen(seed, name):
    g = torch.Generator(device=DEV)
    g.manual_seed((int(seed) * 1000003 + zlib.crc32(name.encode())) % (1 << 62))
    return g


def _td(dtype):
    return torch.bfloat16 if dtype == "bf16" else torch.float32


def _code(dtype):
    return pa.PURINE_BF16 if dtype == "bf16" else pa.PURINE_F32


def _make(seed, name, shape, dtype, kind, fan_in=1):
    """kind: "image" in [0, 1), "act" (a ReLU output), "w" (He scale), "b", "dy"."""
    g, shape = _gen(seed, name), tuple(int(v) for v in shape)
    if kind == "image":
        t = torch.rand(shape, generator=g, device=DEV)
    else:
        t = torch.randn(shape, generator=g, device=DEV)
        if kind == "act":
            t = t.clamp_(min=0)
        elif kind == "w":
            t = t * math.sqrt(2.0 / fan_in)
        elif kind == "b":
            t = t * 0.1
        else:
            t = t * 1e-3
    return t.to(_td(dtype)).contiguous()


def _graph_init(seed):
    def init(name, shape, dtype, kind):
        fan_in = shape[1] * shape[2] * shape[3] if kind == "w" else 1
        return _make(seed, name, shape, dtype, {"x": "image", "w": "w", "b": "b", "dy": "dy"}[kind], fan_in)
    return init


def _scratch(nbytes):
    return torch.empty(max(256, int(nbytes)), dtype=torch.uint8, device=DEV)


class _Graph:
    """A workload graph that is given back when the program drops it."""

    def __init__(self, case, seed):
        # the way bench.py builds them: fused vertices, several streams, config 3 with the merged 1x1;
        # a training iteration does not need the gradient of the images
        self.cfg, self.sgd = case["cfg"], case["sgd"]
        self.gb = build_workload(case["cfg"], batch=case["batch"], init=_graph_init(seed), fuse=True,
                                 merge_1x1=case["cfg"] == 3, fan_in_add=case["cfg"] == 3,
                                 first_layer_dx=not (case["sgd"] and case["cfg"] in (2, 4)),
                                 sgd_lr=0.01 if case["sgd"] else None)

    def run(self):
        gb, out = self.gb, {}
        gb.run()
        if self.cfg == 3:
            out["y"], out["dx"] = gb.t["cat"], gb.t["dx"]
        for i, rec in enumerate(gb.conv_records):
            p = rec["prefix"]
            if self.cfg in (1, 5) or (self.cfg == 2 and i == len(gb.conv_records) - 1):
                out[p + ".y"] = gb.t[rec["out"]]
            if self.cfg in (1, 2, 5) and rec["dx"] is not None and (self.cfg != 2 or i == 0):
                out[p + ".dx"] = gb.t[rec["dx"]]
            out[p + ".dw"], out[p + ".db"] = gb.t[rec["dw"]], gb.t[rec["db"]]
            if self.sgd:
                out[p + ".w.new"], out[p + ".b.new"] = gb.t[p + ".w.new"], gb.t[p + ".b.new"]
        if self.cfg == 4:
            out["y"] = gb.t["conv5.pool.y"]
        return out

    def __del__(self):
        gb = getattr(self, "gb", None)
        if gb is not None:
            gb.close()


def _out_hw(c):
    return ((c["H"] + 2 * c["pad"] - c["R"]) // c["stride"] + 1, (c["W"] + 2 * c["pad"] - c["R"]) // c["stride"] + 1)


def _conv_inputs(c, seed):
    P, Q = _out_hw(c)
    cg = c["C"] // c["groups"]
    kind = "image" if c["C"] == 3 else "act"
    return {"x": _make(seed, "x", (c["N"], c["C"], c["H"], c["W"]), c["dtype"], kind),
            "w": _make(seed, "w", (c["K"], cg, c["R"], c["R"]), c["dtype"], "w", cg * c["R"] * c["R"]),
            "b": _make(seed, "b", (c["K"],), c["dtype"], "b"),
            "dy": _make(seed, "dy", (c["N"], c["K"], P, Q), c["dtype"], "dy")}


def _fc_inputs(c, seed):
    return {"x": _make(seed, "x", (c["N"], c["C"]), c["dtype"], "act"),
            "w": _make(seed, "w", (c["K"], c["C"]), c["dtype"], "w", c["C"]),
            "b": _make(seed, "b", (c["K"],), c["dtype"], "b"),
            "dy": _make(seed, "dy", (c["N"], c["K"]), c["dtype"], "dy")}


def _pool_hw(c):
    return ((c["H"] + 2 * c["pad"] - c["window"]) // c["stride"] + 1,
            (c["W"] + 2 * c["pad"] - c["window"]) // c["stride"] + 1)


def _pool_inputs(c, seed):
    P, Q = _pool_hw(c)
    return {"x": _make(seed, "x", (c["N"], c["C"], c["H"], c["W"]), c["dtype"], "act"),
            "dy": _make(seed, "dy", (c["N"], c["C"], P, Q), c["dtype"], "dy")}


def prepare(case, seed):
    kind = case["kind"]
    if kind == "graph":
        return {"case": case, "graph": _Graph(case, seed)}
    c, td, code = case, _td(case["dtype"]), _code(case["dtype"])
    if kind == "pool":
        s = _pool_inputs(c, seed)
        s.update(case=c, desc=pa.pool_desc(c["window"], c["stride"], c["pad"]), y=torch.empty_like(s["dy"]),
                 arg=torch.empty(s["dy"].shape, dtype=torch.int32, device=DEV), dx=torch.empty_like(s["x"]))
        return s
    s = _conv_inputs(c, seed) if kind == "conv" else _fc_inputs(c, seed)
    s.update(case=c, y=torch.empty(s["dy"].shape, dtype=td, device=DEV), dx=torch.empty_like(s["x"]),
             dw=torch.empty(s["w"].shape, device=DEV), db=torch.empty(s["b"].shape, device=DEV))
    if kind == "fc":
        q = lambda which: _scratch(pa.purine_fc_workspace_bytes(which, c["N"], c["C"], c["K"], code))
        s["ws"] = [q(p) for p in (pa.PURINE_CONV_FWD, pa.PURINE_CONV_BWD_DATA, pa.PURINE_CONV_BWD_WEIGHT)]
        return s
    s["desc"] = pa.conv_desc(c["stride"], c["pad"])
    passes = (pa.PURINE_CONV_FWD, pa.PURINE_CONV_BWD_DATA, pa.PURINE_CONV_BWD_WEIGHT_BIAS)
    if c["groups"] > 1:
        s["ws"] = [_scratch(pa.purine_grouped_conv_workspace_bytes(p, s["desc"], c["groups"], s["x"].shape, s["w"].shape, code))
                   for p in passes]
    else:
        s["ws"] = [_scratch(pa.purine_conv_workspace_bytes(p, s["desc"], s["x"].shape, s["w"].shape, code)) for p in passes]
    return s


# ------------------------------------------------------------------------------------------- run
def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind == "graph":
        return s["graph"].run()
    if kind == "pool":
        pa.purine_maxpool_fwd(s["desc"], s["x"], s["y"], s["arg"])
        pa.purine_maxpool_bwd_relu(s["desc"], s["dy"], s["arg"], s["y"], s["dx"])
        return {"y": s["y"], "arg": s["arg"], "dx": s["dx"]}
    x, w, b, dy, y, dx, dw, db, ws = (s[k] for k in ("x", "w", "b", "dy", "y", "dx", "dw", "db", "ws"))
    if kind == "fc":
        pa.purine_fc_fwd(x, w, b, y, ws=ws[0])
        pa.purine_fc_bwd_data(dy, w, dx, ws=ws[1])
        pa.purine_fc_bwd_weight(x, dy, dw, db, ws=ws[2])
        return {"y": y, "dx": dx, "dw": dw, "db": db}
    desc, groups = s["desc"], c["groups"]
    if groups > 1:
        pa.purine_grouped_conv_fwd(desc, groups, x, w, b, y, relu=True, ws=ws[0])
    else:
        pa.purine_conv_fwd_bias_relu(desc, x, w, b, y, relu=True, ws=ws[0])
    if not c["train"]:
        return {"y": y}
    if groups > 1:
        pa.purine_grouped_conv_bwd_data(desc, groups, dy, w, dx, ws=ws[1])
        pa.purine_grouped_conv_bwd_weight(desc, groups, x, dy, dw, db, ws=ws[2])
    else:
        pa.purine_conv_bwd_data_relu(desc, dy, w, x, dx, ws=ws[1])
        pa.purine_conv_bwd_weight_bias(desc, x, dy, dw, db, ws=ws[2])
    return {"y": y, "dx": dx, "dw": dw, "db": db}


# ------------------------------------------------------------------------------------------ work
def work(case):
    kind = case["kind"]
    es = 2 if case.get("dtype") == "bf16" else 4
    if kind == "graph":
        flops = nbytes = 0
        for i, L in enumerate(CONV_LAYERS[case["cfg"]]):
            L = L.with_batch(case["batch"])
            e = 2 if L.dtype == "bf16" else 4
            n = lambda s: math.prod(s)
            no_dx = i == 0 and case["sgd"] and case["cfg"] in (2, 4)
            flops += L.flop_per_pass * (2 if no_dx else 3)
            nbytes += e * (n(L.x_shape) * (1 if no_dx else 2) + 2 * n(L.y_shape) + n(L.w_shape)) + 4 * n(L.w_shape)
            nbytes += 4 * n(L.w_shape) if case["sgd"] else 0
        return {"bytes": nbytes, "flops": flops}
    if kind == "pool":
        P, Q = _pool_hw(case)
        planes = case["N"] * case["C"]
        return {"bytes": planes * (2 * es * case["H"] * case["W"] + (2 * es + 4) * P * Q),
                "flops": planes * P * Q * case["window"] ** 2}
    if kind == "fc":
        N, C, K = case["N"], case["C"], case["K"]
        return {"bytes": es * (2 * N * C + 2 * N * K + K * C) + 4 * K * C, "flops": 6 * N * C * K}
    P, Q = _out_hw(case)
    x, y = case["N"] * case["C"] * case["H"] * case["W"], case["N"] * case["K"] * P * Q
    w = case["K"] * (case["C"] // case["groups"]) * case["R"] ** 2
    flops = 2 * w * case["N"] * P * Q
    if not case["train"]:
        return {"bytes": es * (x + y + w), "flops": flops}
    return {"bytes": es * (2 * x + 2 * y + w) + 4 * w, "flops": 3 * flops}


def tolerance(case):
    if case["kind"] == "pool":
        return "exact"              # the winner and the order of the sums are part of the operator
    if case["kind"] == "graph" and case["cfg"] != 5:
        # fp32 through several layers: a last-bit difference moves a ReLU's zero or a pooling winner
        # here and there, which moves single gradient entries whole
        return {"rel": 1e-5, "max": 0.1} if case["cfg"] == 1 else {"rel": 2e-3, "max": 0.9}
    if case["kind"] == "graph" or case["dtype"] == "bf16":
        return {"rel": 8e-3, "max": 0.1}   # bf16 results are rounded once: 1.7e-3 from the exact value
    return {"rel": 1e-5}


# ----------------------------------------------------------------------------------------- exact
def _conv64(x, w, b, stride, pad):
    K, R, S = w.shape[0], w.shape[2], w.shape[3]
    P, Q = (x.shape[2] + 2 * pad - R) // stride + 1, (x.shape[3] + 2 * pad - S) // stride + 1
    y = torch.matmul(w.reshape(K, -1), F.unfold(x, (R, S), padding=pad, stride=stride)).reshape(-1, K, P, Q)
    return y + b.reshape(1, -1, 1, 1)


def _exact_graph(case, seed):
    cfg, layers = case["cfg"], [L.with_batch(case["batch"]) for L in CONV_LAYERS[case["cfg"]]]
    init = _graph_init(seed)
    par = {}
    for L in layers:
        par[L.name] = [init(L.name + s, sh, L.dtype, k).double().requires_grad_() for s, sh, k in
                       ((".w", L.w_shape, "w"), (".b", (L.K,), "b"))]
    conv = lambda L, t: _conv64(t, par[L.name][0], par[L.name][1], L.stride, L.pad)
    out, want = {}, {}
    if cfg in (1, 5):
        for L in layers:
            x = init(L.name + ".x", L.x_shape, L.dtype, "x").double().requires_grad_()
            y = conv(L, x)
            dy = init(L.name + ".dout", L.y_shape, L.dtype, "dy").double()
            gx, gw, gb = torch.autograd.grad(y, [x] + par[L.name], dy)
            out.update({L.name + ".y": y.detach(), L.name + ".dx": gx, L.name + ".dw": gw, L.name + ".db": gb})
            del y
    else:
        x = init("x", layers[0].x_shape, "f32", "x").double().requires_grad_()
        if cfg == 2:
            y = conv(layers[2], F.relu(conv(layers[1], F.relu(conv(layers[0], x)))))
            dy = init("dout", layers[2].y_shape, "f32", "dy").double()
            want = {"x": None if case["sgd"] else layers[0].name + ".dx"}
            out[layers[2].name + ".y"] = y.detach()
        elif cfg == 3:
            b1, b2r, b2, b3r, b3, b4 = layers
            o1 = F.relu(conv(b1, x))
            o2 = F.relu(conv(b2, F.relu(conv(b2r, x))))
            o3 = F.relu(conv(b3, F.relu(conv(b3r, x))))
            o4 = F.relu(conv(b4, F.max_pool2d(x, 3, 1, 1)))
            y = torch.cat([o1, o2, o3, o4], 1)
            dy = init("dout", y.shape, "f32", "dy").double()
            want = {"x": "dx"}
            out["y"] = y.detach()
        else:
            t = x
            for L, pool in zip(layers, (True, True, False, False, True)):
                t = F.relu(conv(L, t))
                t = F.max_pool2d(t, 3, 2) if pool else t
            y = t
            dy = init("dout", y.shape, "f32", "dy").double()
            out["y"] = y.detach()
        flat = [v for L in layers for v in par[L.name]]
        grads = torch.autograd.grad(y, [x] + flat, dy)
        if want.get("x"):
            out[want["x"]] = grads[0]
        for i, L in enumerate(layers):
            out[L.name + ".dw"], out[L.name + ".db"] = grads[1 + 2 * i], grads[2 + 2 * i]
    if cfg == 3:                       # the three 1x1 layers on the module input are one operator there
        order = [layers[i].name for i in (1, 3, 0)]
        for s, i in ((".dw", 0), (".db", 1)):
            out["merged_1x1" + s] = torch.cat([out.pop(n + s) for n in order], 0)
            par.setdefault("merged_1x1", [None, None])[i] = torch.cat([par[n][i].detach() for n in order], 0)
    if case["sgd"]:
        for k in [k for k in out if k.endswith(".dw")]:
            p = k[:-3]
            out[p + ".w.new"] = par[p][0].detach() - 0.01 * out[p + ".dw"]
            out[p + ".b.new"] = par[p][1].detach() - 0.01 * out[p + ".db"]
    return out


def exact(case, seed):
    kind = case["kind"]
    if kind == "graph":
        return _exact_graph(case, seed)
    if kind == "pool":
        t = _pool_inputs(case, seed)
        x = t["x"].double().requires_grad_()
        y, arg = F.max_pool2d(x, case["window"], case["stride"], case["pad"], return_indices=True)
        dx, = torch.autograd.grad(y, [x], t["dy"].double() * (y.detach() > 0))
        return {"y": y.detach(), "arg": None, "dx": dx}
    if kind == "fc":
        t = {k: v.double() for k, v in _fc_inputs(case, seed).items()}
        return {"y": t["x"] @ t["w"].t() + t["b"], "dx": t["dy"] @ t["w"], "dw": t["dy"].t() @ t["x"], "db": t["dy"].sum(0)}
    t = {k: v.double().requires_grad_(k != "dy") for k, v in _conv_inputs(case, seed).items()}
    G = case["groups"]
    y = torch.cat([_conv64(xg, wg, bg, case["stride"], case["pad"]) for xg, wg, bg in
                   zip(t["x"].chunk(G, 1), t["w"].chunk(G, 0), t["b"].chunk(G, 0))], 1)
    if not case["train"]:
        return {"y": F.relu(y).detach()}
    dx, dw, db = torch.autograd.grad(y, [t["x"], t["w"], t["b"]], t["dy"])
    if G == 1:                         # the plain layer's backward-data carries the ReLU mask of its input
        dx = dx * (t["x"].detach() > 0)
    return {"y": F.relu(y).detach(), "dx": dx, "dw": dw, "db": db}
