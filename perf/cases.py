"""The calls whose speed is measured: single layers through the operation entry
points and networks through the plan, over the sizes this library is used at.

A case is a dict of plain values.  ``kind`` names the entry point:

``conv``     ``neo.conv2d_blocked`` (``neo.conv2d_nchwxc`` for inputs of at most
             four channels, which it reads as plain NCHW)
``wino``     ``neo.conv2d_winograd``
``int8``     ``neo.conv2d_int8_q``, the integer layer inside an integer network
``dense``    ``neo.dense``
``bottle``   a plan of two ResNet bottlenecks (projection, then identity)
``mixed``    a plan of one 17x17-style Inception block (1x7 / 7x1 branches)
``net``      a plan of the whole ResNet-50, float32 or int8

Inputs follow the networks' statistics: activations U[-1, 1] (post-ReLU maps
inside the integer layers), Kaiming-normal weights, N(0, 0.1) biases.  Plans
are built with the local search of launch configurations, the launch fusions
and Winograd offered to the search, and replayed as a graph: the way the
library's own benchmark runs a network.
"""
import math

import numpy as np
import torch

from paper_1809_02697_amd import neo
from paper_1809_02697_amd import workloads as wl

DEV = "cuda:0"
FUSED = (neo.PLAN_TUNE | neo.PLAN_HIPGRAPH | neo.PLAN_GROUP | neo.PLAN_FUSE_GAP |
         neo.PLAN_FUSE_PAIRS | neo.PLAN_FUSE_CHAINS | neo.PLAN_FUSE_POOL | neo.PLAN_WINOGRAD)
INT8 = neo.PLAN_INT8 | neo.PLAN_TUNE | neo.PLAN_HIPGRAPH | neo.PLAN_GROUP


def _conv(N, C, H, W, K, R, S, stride=1, ph=0, pw=0, relu=True, res=False, **kw):
    return dict(kw, N=N, C=C, H=H, W=W, K=K, R=R, S=S, stride=stride, ph=ph, pw=pw, relu=relu, res=res)


def listed():
    return [
        # one image through one 3x3 layer, the single-convolution workload of
        # the method's paper: launch latency against a small layer
        _conv(1, 64, 56, 56, 64, 3, 3, 1, 1, 1, kind="conv", name="conv3x3_b1"),
        # serving at batch 32: a 3x3 layer of ResNet-50's second stage
        _conv(32, 128, 28, 28, 128, 3, 3, 1, 1, 1, kind="conv", name="conv3x3_b32"),
        # ... and the third stage's pointwise expansion with its residual
        _conv(32, 256, 14, 14, 1024, 1, 1, 1, 0, 0, res=True, kind="conv", name="conv1x1_res_b32"),
        # ragged channels, an odd map and an asymmetric window, batch 3
        _conv(3, 100, 35, 33, 150, 1, 7, 1, 0, 3, relu=False, kind="conv", name="conv1x7_ragged"),
        # a network stem on camera frames as they arrive (NCHW), batch 8
        _conv(8, 3, 224, 224, 64, 7, 7, 2, 3, 3, kind="conv", name="stem7x7_b8"),
        # VGG-16's third stage with the fast algorithm, batch 8
        _conv(8, 256, 56, 56, 256, 3, 3, 1, 1, 1, kind="wino", name="winograd_b8"),
        # an integer layer at batch 32, its output requantized for the next
        _conv(32, 256, 14, 14, 256, 3, 3, 1, 1, 1, kind="int8", name="int8_3x3_b32"),
        # VGG-16's first fully connected layer at a serving batch
        dict(kind="dense", name="dense_fc6_b16", N=16, IN=25088, OUT=4096),
        # two bottlenecks of ResNet-50's second stage as a plan, batch 8
        dict(kind="bottle", name="bottleneck_b8", N=8, C=256, width=128, H=56, stride=2),
        # one Inception-v3 block (Mixed_6c) as a plan, batch 2
        dict(kind="mixed", name="inception_block_b2", N=2, C=768, c7=160, H=17),
        # whole networks: single-image latency, and batched throughput
        dict(kind="net", name="resnet50_b1", N=1, int8=False),
        dict(kind="net", name="resnet50_b32", N=32, int8=False),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _channels(rng, lo, hi):
    c = _log(rng, lo, hi)
    return max(16, c // 16 * 16) if rng.random() < 0.6 else c


def draw(rng):
    kind = rng.choices(["conv", "wino", "int8", "dense", "bottle", "mixed", "net"],
                       [46, 10, 12, 14, 8, 6, 4])[0]
    if kind == "dense":
        return dict(kind=kind, N=_log(rng, 1, 64), IN=_log(rng, 256, 25088), OUT=_log(rng, 10, 4096))
    if kind == "bottle":
        return dict(kind=kind, N=_log(rng, 1, 16), C=_channels(rng, 64, 512), width=16 * rng.randint(2, 12),
                    H=_log(rng, 7, 56), stride=rng.choice([1, 2]))
    if kind == "mixed":
        return dict(kind=kind, N=_log(rng, 1, 8), C=16 * rng.randint(8, 48), c7=16 * rng.randint(4, 12),
                    H=_log(rng, 8, 35))
    if kind == "net":
        return dict(kind=kind, N=_log(rng, 1, 16), int8=rng.random() < 0.5)
    stem = kind == "conv" and rng.random() < 0.1
    while True:
        H = _log(rng, 7, 112) if not stem else _log(rng, 64, 256)
        W = H if rng.random() < 0.6 else max(7, H + rng.randint(-5, 5))
        N = _log(rng, 1, 32)
        C = rng.choice([1, 3, 4]) if stem else _channels(rng, 16, 1024)
        K = _channels(rng, 16, 1024)
        R, S = (3, 3) if kind == "wino" else rng.choice(
            [(3, 3), (5, 5), (7, 7)] if stem else
            [(1, 1), (1, 1), (1, 1), (3, 3), (3, 3), (3, 3), (1, 7), (7, 1), (5, 5), (1, 3)])
        stride = 2 if kind != "wino" and rng.random() < (0.7 if stem else 0.2) else 1
        c = _conv(N, C, H, W, K, R, S, stride, R // 2, S // 2, relu=rng.random() < 0.7,
                  res=kind != "int8" and not stem and rng.random() < 0.25, kind=kind)
        w = work(c)
        if w["flops"] < 6e10 and w["bytes"] < 4e8:
            return c


# ---- what a user's program holds before the call ----------------------------------------
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _uniform(g, shape, lo=-1.0, hi=1.0):
    return torch.empty(shape, device=DEV).uniform_(lo, hi, generator=g)


def _normal(g, shape, std):
    return torch.empty(shape, device=DEV).normal_(0.0, std, generator=g)


def _out_hw(c):
    return ((c["H"] + 2 * c["ph"] - c["R"]) // c["stride"] + 1, (c["W"] + 2 * c["pw"] - c["S"]) // c["stride"] + 1)


def _conv_inputs(c, seed):
    """x, w, bias, residual of a convolution case in NCHW / KCRS."""
    g = _gen(seed)
    x = _uniform(g, (c["N"], c["C"], c["H"], c["W"]), 0.0 if c["kind"] == "int8" else -1.0)
    w = _normal(g, (c["K"], c["C"], c["R"], c["S"]), math.sqrt(2.0 / (c["C"] * c["R"] * c["S"])))
    b = _normal(g, (c["K"],), 0.1)
    r = _uniform(g, (c["N"], c["K"]) + _out_hw(c)) if c["res"] else None
    return x, w, b, r


def _dense_inputs(c, seed):
    g = _gen(seed)
    return (_uniform(g, (c["N"], c["IN"])), _normal(g, (c["OUT"], c["IN"]), math.sqrt(2.0 / c["IN"])),
            _normal(g, (c["OUT"],), 0.1))


def _pad16(b):
    p = torch.zeros(-(-b.numel() // 16) * 16, device=DEV)
    p[:b.numel()] = b
    return p


class _Net:
    """Builds a network description with parameters drawn on one generator."""

    def __init__(self, shape, seed):
        self.g = np.random.default_rng(seed)
        self.nodes = [wl.Node(op="input")]
        self.ch = [shape[1]]
        self.shape = shape

    def add(self, op, inputs, ch, **kw):
        self.nodes.append(wl.Node(op=op, inputs=inputs, **kw))
        self.ch.append(ch)
        return len(self.nodes) - 1

    def conv(self, x, K, R=1, S=None, stride=1, act="relu", residual=-1):
        S = R if S is None else S
        C = self.ch[x]
        w = self.g.standard_normal((K, C, R, S), dtype=np.float32) * np.float32(math.sqrt(2.0 / (C * R * S)))
        u = lambda lo, hi: self.g.uniform(lo, hi, K).astype(np.float32)  # noqa: E731
        n = lambda: (0.1 * self.g.standard_normal(K)).astype(np.float32)  # noqa: E731
        bn = dict(gamma=u(0.5, 1.5), beta=n(), mean=n(), var=u(0.5, 1.5), eps=1e-5)
        return self.add("conv", (x,), K, K=K, R=R, S=S, stride=(stride, stride), pad=(R // 2, S // 2), act=act,
                        residual=residual, w=w, bn=bn)

    def graph(self, name, out):
        self.add("output", (out,), self.ch[out])
        return wl.Graph(name=name, nodes=self.nodes, input_shape=self.shape)


def _graph(c, seed):
    N = c["N"]
    if c["kind"] == "net":
        return wl.resnet50(N=N, seed=seed)
    b = _Net((N, c["C"], c["H"], c["H"]), seed)
    if c["kind"] == "bottle":
        w = c["width"]
        sc = b.conv(0, 4 * w, stride=c["stride"], act="none")
        y = b.conv(b.conv(0, w), w, 3, stride=c["stride"])
        x = b.conv(y, 4 * w, residual=sc)
        y = b.conv(b.conv(x, w), w, 3)
        return b.graph("bottle", b.conv(y, 4 * w, residual=x))
    k = c["c7"]
    b1 = b.conv(0, 192)
    b7 = b.conv(b.conv(b.conv(0, k), k, 1, 7), 192, 7, 1)
    bd = b.conv(b.conv(b.conv(b.conv(b.conv(0, k), k, 7, 1), k, 1, 7), k, 7, 1), 192, 1, 7)
    bp = b.conv(b.add("avgpool", (0,), c["C"], R=3, S=3, stride=(1, 1), pad=(1, 1)), 192)
    return b.graph("mixed", b.add("concat", (b1, b7, bd, bp), 768))


def _net_input(c, g, seed):
    gen = _gen(seed)
    return _normal(gen, g.input_shape, 1.0) if c["kind"] == "net" else _uniform(gen, g.input_shape)


def prepare(case, seed):
    c = case
    if c["kind"] == "dense":
        x, w, b = _dense_inputs(c, seed)
        return dict(c, x=x, w=w, b=b, out=torch.empty((c["N"], c["OUT"]), device=DEV))
    if c["kind"] in ("bottle", "mixed", "net"):
        g = _graph(c, seed)
        int8 = c.get("int8", False)
        p = neo.Plan(g, flags=INT8 if int8 else FUSED)
        x = _net_input(c, g, seed)
        N, C, H, W = p.output_shape
        out = torch.empty((N, C) if (H, W) == (1, 1) else (N, C, H, W), device=DEV)
        if int8:
            p.calibrate_int8(x, out)
        return dict(c, plan=p, x=x, out=out)
    x, w, b, r = _conv_inputs(c, seed)
    OH, OW = _out_hw(c)
    KB = -(-c["K"] // 16)
    st = dict(c, bias=_pad16(b), act="relu" if c["relu"] else "none", pad=(c["ph"], c["pw"]))
    st["residual"] = None if r is None else neo.to_blocked(r)
    if c["kind"] == "int8":
        xb = neo.to_blocked(x)
        st["x_scale"] = 1.0 / 127
        st["xq"] = neo.quantize_int8(xb, c["C"], st["x_scale"], pad=st["pad"])
        st["wq"], st["ws"] = neo.pack_filter_int8(w)
        st["y_scale"] = 6.0 / 127
        st["out"] = torch.zeros((c["N"], KB, OH + 2 * c["ph"], OW + 2 * c["pw"], 16), device=DEV, dtype=torch.int8)
        return st
    st["out"] = torch.empty((c["N"], KB, OH, OW, 16), device=DEV)
    if c["kind"] == "wino":
        st["u"] = neo.winograd_filter(w)
    else:
        st["w"] = neo.pack_filter(w)
    # an input of at most four channels is read as it arrives: NCHW1c is NCHW
    st["x"] = x.unsqueeze(-1) if c["C"] <= 4 else neo.to_blocked(x)
    return st


def run(state):
    s = state
    kind = s["kind"]
    if kind in ("bottle", "mixed", "net"):
        return s["plan"].run(s["x"], s["out"])
    if kind == "dense":
        return neo.dense(s["x"], s["w"], s["b"], "relu", out=s["out"])
    if kind == "int8":
        return neo.conv2d_int8_q(s["xq"], s["C"], s["wq"], s["ws"], s["K"], s["R"], s["S"], s["x_scale"],
                                 s["y_scale"], s["bias"], s["stride"], s["pad"], s["act"], out_pad=s["pad"],
                                 out=s["out"])
    if kind == "wino":
        return neo.conv2d_winograd(s["x"], s["C"], s["u"], s["K"], s["bias"], s["pad"], s["act"], s["residual"],
                                   out=s["out"])
    f = neo.conv2d_nchwxc if s["C"] <= 4 else neo.conv2d_blocked
    return f(s["x"], s["C"], s["w"], s["K"], s["R"], s["S"], s["bias"], s["stride"], s["pad"], s["act"],
             s["residual"], out=s["out"])


# ---- what a pass cannot do without -------------------------------------------------------
def _conv_work(N, C, H, W, K, R, S, sh, OH, OW, res, in_b=4, out_b=4):
    touched = C * OH * OW if R == S == 1 else C * H * W  # a strided 1x1 reads the sampled pixels only
    return (N * touched * in_b + K * C * R * S * in_b + N * K * OH * OW * (out_b + 4 * bool(res)) + 4 * K,
            2.0 * N * K * C * R * S * OH * OW)


_SHAPES = {}  # descriptions without parameters, for work() of the plan cases


def _net_shapes(c):
    """(node, input shape, output shape) triples of a plan case's network."""
    key = tuple(sorted((k, v) for k, v in c.items() if k not in ("name", "int8")))
    if key not in _SHAPES:
        g = _graph(c, 0)
        shp, rows = [], []
        for n in g.nodes:
            if n.op == "input":
                shp.append(tuple(g.input_shape))
                continue
            N, C, H, W = shp[n.inputs[0]]
            i = (N, C, H, W)
            if n.op in ("conv", "maxpool", "avgpool"):
                o = (N, n.K if n.op == "conv" else C, (H + 2 * n.pad[0] - n.R) // n.stride[0] + 1,
                     (W + 2 * n.pad[1] - n.S) // n.stride[1] + 1)
            elif n.op == "concat":
                o = (N, sum(shp[j][1] for j in n.inputs), H, W)
            elif n.op == "gap":
                o = (N, C, 1, 1)
            elif n.op == "dense":
                o = (N, n.K, 1, 1)
            else:
                o = (N, C * H * W, 1, 1) if n.op == "flatten" else i
            shp.append(o)
            rows.append((n.op, n.K, n.R, n.S, i, o))
        _SHAPES[key] = rows
    return _SHAPES[key]


def work(case):
    c = case
    if c["kind"] == "dense":
        return {"bytes": 4.0 * (c["N"] * c["IN"] + c["OUT"] * c["IN"] + c["OUT"] + c["N"] * c["OUT"]),
                "flops": 2.0 * c["N"] * c["IN"] * c["OUT"]}
    if c["kind"] in ("bottle", "mixed", "net"):
        # the network's input, parameters and output; what lies between may stay on the chip
        rows = _net_shapes(c)
        wb = 1 if c.get("int8") else 4
        par = fl = 0.0
        for op, K, R, S, i, o in rows:
            if op in ("conv", "dense"):
                par += K * i[1] * R * S * wb + 4 * K
                fl += 2.0 * o[0] * K * i[1] * R * S * o[2] * o[3]
        first, last = rows[0][4], rows[-1][5]
        return {"bytes": par + 4.0 * (math.prod(first) + math.prod(last)), "flops": fl}
    OH, OW = _out_hw(c)
    q = 1 if c["kind"] == "int8" else 4
    b, f = _conv_work(c["N"], c["C"], c["H"], c["W"], c["K"], c["R"], c["S"], c["stride"], OH, OW, c["res"], q, q)
    return {"bytes": float(b), "flops": f}


def tolerance(case):
    if case["kind"] == "int8" or case.get("int8"):
        return "exact"  # integer sums and a float32 epilogue whose every rounding the interface fixes
    # float32 sums in another order: against 64 bits the relative error measured
    # 1.1e-7 to 9.5e-7 for the convolutions and networks, 1.4e-6 for the 25,088
    # products of the dense layer; about four times that between two orders
    return {"rel": 6e-6 if case["kind"] == "dense" else 4e-6, "max": 6e-5}


# ---- the same in 64 bits ------------------------------------------------------------------
def _conv64(x, w, b, r, sh, sw, ph, pw, relu):
    """NCHW convolution in float64 as unfolded windows times a matrix product, an image at a time."""
    N, C, H, W = x.shape
    K, _, R, S = w.shape
    OH, OW = (H + 2 * ph - R) // sh + 1, (W + 2 * pw - S) // sw + 1
    wm = w.reshape(K, -1).double()
    y = torch.empty((N, K, OH, OW), device=x.device, dtype=torch.float64)
    for n in range(N):
        xn = x[n:n + 1].double()
        cols = (xn[:, :, ::sh, ::sw].reshape(C, -1) if R == S == 1 and ph == pw == 0 else
                torch.nn.functional.unfold(xn, (R, S), padding=(ph, pw), stride=(sh, sw))[0])
        y[n] = (wm @ cols.contiguous()).reshape(K, OH, OW)
    if b is not None:
        y += b.double().reshape(1, -1, 1, 1)
    if r is not None:
        y += r.double()
    return y.relu_() if relu else y


def _blocked(y):
    N, K, H, W = y.shape
    KB = -(-K // 16)
    p = torch.zeros((N, KB * 16, H, W), device=y.device, dtype=y.dtype)
    p[:, :K] = y
    return p.reshape(N, KB, 16, H, W).permute(0, 1, 3, 4, 2).contiguous()


def _net64(g, x):
    F = torch.nn.functional
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV).double()  # noqa: E731
    vals, left = [], [0] * len(g.nodes)
    for n in g.nodes:
        for j in n.inputs + ((n.residual,) if n.residual >= 0 else ()):
            left[j] += 1
    for n in g.nodes:
        i = vals[n.inputs[0]] if n.inputs else None
        if n.op == "input":
            v = x.double()
        elif n.op == "conv":
            w, b = dev(n.w), None if n.bias is None else dev(n.bias)
            v = _conv64(i, w, b, None, *n.stride, *n.pad, False)
            if n.bn is not None:
                q = {k: (dev(a).reshape(1, -1, 1, 1) if k != "eps" else a) for k, a in n.bn.items()}
                v = (v - q["mean"]) / torch.sqrt(q["var"] + q["eps"]) * q["gamma"] + q["beta"]
            if n.residual >= 0:
                v = v + vals[n.residual]
        elif n.op == "maxpool":
            v = F.max_pool2d(i, (n.R, n.S), n.stride, n.pad)
        elif n.op == "avgpool":
            v = F.avg_pool2d(i, (n.R, n.S), n.stride, n.pad, count_include_pad=False)
        elif n.op == "gap":
            v = i.mean((2, 3), keepdim=True)
        elif n.op == "concat":
            v = torch.cat([vals[j] for j in n.inputs], 1)
        elif n.op == "flatten":
            v = i.reshape(i.shape[0], -1)
        elif n.op == "dense":
            v = i @ dev(n.w).t() + dev(n.bias)
        else:
            v = i
        vals.append(v.relu() if n.act == "relu" else v)
        for j in n.inputs + ((n.residual,) if n.residual >= 0 else ()):
            left[j] -= 1
            if not left[j]:
                vals[j] = None
    return vals[-1]


def exact(case, seed):
    c = case
    if c["kind"] == "int8" or c.get("int8"):
        return None  # whole numbers, and logits computed from them: compared bit for bit
    if c["kind"] == "dense":
        x, w, b = _dense_inputs(c, seed)
        return (x.double() @ w.double().t() + b.double()).relu_()
    if c["kind"] in ("bottle", "mixed", "net"):
        g = _graph(c, seed)
        return _net64(g, _net_input(c, g, seed))
    x, w, b, r = _conv_inputs(c, seed)
    return _blocked(_conv64(x, w, b, r, c["stride"], c["stride"], c["ph"], c["pw"], c["relu"]))
