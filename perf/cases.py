"""Timed cases of the framework: one training path per case, through the public entry points.

Each case is one layer (or one whole step) as a training program calls it: the `_lib` binding of the
C ABI with device pointers and a stream, or `Trainer.step`.  Sizes are those of `workloads/configs.py`
and of the sweeps in `bench.py`, and ragged ones beside them.  What a program keeps between calls
(parameters with their history, descriptors, workspaces of the queried size) is made in `prepare`.

Distributions: activations N(0, 1) (the positive half after a ReLU), weights Kaiming-uniform,
incoming gradients N(0, 1) scaled by 1 / rows (a mean loss), optimizer history at the scale of the
gradients it has averaged (a run some steps old).
"""
import math

import numpy as np
import torch

from paper_2104_00237_amd import _lib as L

DEV = "cuda:0"
LN_EPS = 1e-5
STEP0 = 20          # updates the history has seen before the first pass

OPTS = {
    "sgd": dict(kind="sgd", lr=1e-3, momentum=0.9, weight_decay=5e-4),
    "adam": dict(kind="adam", lr=1e-4, beta1=0.9, beta2=0.999, eps=1e-8, weight_decay=0.0),
    "adamw": dict(kind="adamw", lr=1e-4, beta1=0.9, beta2=0.999, eps=1e-8, weight_decay=0.01),
    "adagrad": dict(kind="adagrad", lr=1e-4, eps=1e-10, weight_decay=1e-4),
    "rmsprop": dict(kind="rmsprop", lr=1e-4, alpha=0.99, eps=1e-8, momentum=0.0, weight_decay=1e-4),
    "adadelta": dict(kind="adadelta", lr=1e-1, rho=0.9, eps=1e-6, weight_decay=1e-4),
}


# ---------------------------------------------------------------- the cases
def listed():
    return [
        # The smallest call: a whole step of the 3-layer MLP every ordering is checked on.
        dict(name="mlp3_step", path="mlp_step", dims="64-128-128-10", batch=32, ordering="bf"),
        # An ordinary fully connected layer, a batch that fills no whole tile.
        dict(name="linear_fwd_1000", path="linear_fwd", M=1000, N=1024, K=1024, act="relu", bias=True),
        # Backward and update of a wide layer at a larger batch.
        dict(name="linear_bwd_1024x2048", path="linear_bwd", M=1024, N=2048, K=2048, act="relu",
             bias=True, opt="adam"),
        # The parameter-bound stack: 8192 x 8192 layers at 64 rows, forward ...
        dict(name="wide_fwd_64x8192", path="linear_fwd", M=64, N=8192, K=8192, act="none", bias=False),
        # ... and the data gradient merged with the update.
        dict(name="wide_merged_64x8192", path="linear_merged", M=64, N=8192, K=8192, act="none",
             bias=False, opt="adam"),
        # The Transformer block's FC1 forward: bf16 operands kept as bf16, GELU, Z kept for backward.
        dict(name="bf16_fc1_fwd", path="bf16_fwd", M=4096, N=4096, K=1024, act="gelu", bias=True,
             x_bf16=True, y_bf16=True),
        # Its FC2 backward and update: the data gradient takes GELU's derivative.
        dict(name="bf16_fc2_bwd", path="bf16_bwd", M=4096, N=1024, K=4096, act="gelu", bias=True,
             opt="adamw", overlap=False),
        # A VGG-11 convolution at batch 128, forward, data gradient and fused update.
        dict(name="conv_128x8x8x256", path="conv", N=128, H=8, W=8, C=256, Cout=256, opt="sgd"),
        # MobileNetV2 at batch 32: a depthwise layer ...
        dict(name="depthwise_32x56x56x144", path="depthwise", N=32, H=56, W=56, C=144, stride=1,
             opt="adam"),
        # ... and a 1x1 expansion over its pixel rows, both directions.
        dict(name="pointwise_100352x24x144", path="pointwise", M=100352, N=144, K=24, act="relu",
             opt="adam"),
        # LayerNorm of the Transformer block: forward, backward, update of gamma and beta.
        dict(name="layernorm_4096x1024", path="layernorm", M=4096, D=1024, y_bf16=True, opt="adamw"),
        # The unfused optimizer stage with global-norm clipping, over one Transformer block's tensors.
        dict(name="optimizer_block", path="optimizer", width=1024, ffn=4096, layers=1, clip=True,
             opt="adamw"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _feat(rng, lo, hi):
    """A feature count: mostly a multiple of 8 as in real layers, sometimes odd."""
    n = _log(rng, lo, hi)
    return n if rng.random() < 0.3 else max(8, n // 8 * 8)


def draw(rng):
    path = rng.choice(["mlp_step", "linear_fwd", "linear_fwd", "linear_bwd", "linear_bwd", "linear_merged",
                       "bf16_fwd", "bf16_fwd", "bf16_bwd", "bf16_bwd", "conv", "conv", "depthwise",
                       "pointwise", "layernorm", "optimizer"])
    opt = rng.choice(["sgd", "adam", "adam", "adamw", "adamw", "adagrad", "rmsprop", "adadelta"])
    if path == "mlp_step":
        dims = [_feat(rng, 16, 512) for _ in range(rng.randint(2, 5))] + [rng.randint(4, 100)]
        return dict(path=path, dims="-".join(map(str, dims)), batch=_log(rng, 8, 256),
                    ordering=rng.choice(["eager", "ff", "bf"]))
    if path in ("linear_fwd", "linear_bwd"):
        while True:
            M, N, K = _log(rng, 1, 4096), _feat(rng, 10, 8192), _feat(rng, 10, 8192)
            if 2 * M * N * K <= 9.5e9 and N * K <= 2 ** 25:
                break
        c = dict(path=path, M=M, N=N, K=K, act=rng.choice(["none", "relu", "gelu"]),
                 bias=rng.random() < 0.7)
        return c if path == "linear_fwd" else dict(c, opt=opt)
    if path == "linear_merged":
        while True:
            N, K = _feat(rng, 64, 8192), _feat(rng, 64, 8192)
            if N * K <= 2 ** 25:
                break
        return dict(path=path, M=rng.randint(1, 64), N=N, K=K, act=rng.choice(["none", "relu", "gelu"]),
                    bias=rng.random() < 0.5, opt=opt)
    if path in ("bf16_fwd", "bf16_bwd"):
        while True:
            M, N, K = _log(rng, 64, 8192), _feat(rng, 96, 4096), _feat(rng, 96, 4096)
            if 2 * M * N * K <= 3.4e10:
                break
        c = dict(path=path, M=M, N=N, K=K, act=rng.choice(["none", "relu", "gelu"]),
                 bias=rng.random() < 0.8)
        if path == "bf16_fwd":
            return dict(c, x_bf16=rng.random() < 0.7, y_bf16=rng.random() < 0.6)
        return dict(c, opt=opt, overlap=rng.random() < 0.3)
    if path == "conv":
        while True:
            N, s = _log(rng, 3, 128), rng.choice([2, 4, 7, 8, 14, 15, 16, 28, 32])
            C, Co = rng.choice([3, 3, _feat(rng, 8, 512), _feat(rng, 8, 512)]), _feat(rng, 16, 512)
            if 18 * N * s * s * C * Co <= 9.6e9:
                break
        return dict(path=path, N=N, H=s, W=s if rng.random() < 0.7 else s + 1, C=C, Cout=Co,
                    opt=rng.choice(["sgd", "sgd", opt]))
    if path == "depthwise":
        while True:
            N, s, C = _log(rng, 2, 32), rng.choice([7, 14, 15, 28, 56, 57, 112]), _feat(rng, 16, 960)
            if N * s * s * C <= 1.45e7:
                break
        return dict(path=path, N=N, H=s, W=s, C=C, stride=rng.choice([1, 1, 2]), opt=opt)
    if path == "pointwise":
        while True:
            M, N, K = _log(rng, 1568, 401408), _feat(rng, 16, 960), _feat(rng, 16, 960)
            if M * (N + K) <= 1.68e7 and 2 * M * N * K <= 2e9:
                break
        return dict(path=path, M=M, N=N, K=K, act=rng.choice(["none", "relu"]), opt=opt)
    if path == "layernorm":
        while True:
            M, D = _log(rng, 16, 16384), _feat(rng, 64, 4096)
            if M * D <= 2 ** 22:
                break
        return dict(path=path, M=M, D=D, y_bf16=rng.random() < 0.5, opt=opt)
    w = _feat(rng, 64, 1024)
    return dict(path="optimizer", width=w, ffn=4 * w if rng.random() < 0.7 else _feat(rng, 64, 4096),
                layers=rng.randint(1, max(1, min(6, 2 ** 20 // (w * w)))), clip=rng.random() < 0.5, opt=opt)


# ------------------------------------------------------------------- inputs
class _Rng:
    def __init__(self, seed):
        self.g = torch.Generator(device=DEV).manual_seed(int(seed) * 7919 + 17)

    def normal(self, *shape, scale=1.0):
        return torch.randn(*shape, generator=self.g, device=DEV) * scale

    def uniform(self, *shape, lo=0.0, hi=1.0):
        return torch.rand(*shape, generator=self.g, device=DEV) * (hi - lo) + lo

    def weight(self, *shape, fan_in):
        b = math.sqrt(6.0 / fan_in)
        return self.uniform(*shape, lo=-b, hi=b)

    def history(self, shape, gscale, kind):
        """(m, v) of an optimizer some steps old whose gradients have the scale gscale."""
        m = self.normal(*shape, scale=0.3 * gscale)
        v = self.uniform(*shape, lo=0.5, hi=1.5) * gscale * gscale
        if kind == "adagrad":
            v = v * STEP0
        if kind == "adadelta":
            m = self.uniform(*shape, lo=0.5, hi=1.5) * 1e-6
        return m, v


def _activation(r, act, *shape):
    x = r.normal(*shape)
    return x.clamp_min(0) if act == "relu" else x


def _theta(r, name, shape, fan_in, gscale, kind):
    w = r.weight(*shape, fan_in=fan_in) if len(shape) > 1 else r.normal(*shape, scale=0.02)
    m, v = r.history(shape, gscale, kind)
    return {name: w, name + "_m": m, name + "_v": v}


def _inputs(c, seed):
    """The tensors a pass starts from, by name (fp32 unless said)."""
    r, p, d = _Rng(seed), c["path"], {}
    if p in ("linear_fwd", "bf16_fwd"):
        d["x"] = _activation(r, "none", c["M"], c["K"])
        d["W"] = r.weight(c["N"], c["K"], fan_in=c["K"])
        d["b"] = r.normal(c["N"], scale=0.02)
    elif p in ("linear_bwd", "linear_merged", "bf16_bwd", "pointwise"):
        M, N, K = c["M"], c["N"], c["K"]
        g = 1.0 / math.sqrt(M)
        d["prev"] = _activation(r, "relu" if p == "pointwise" else c["act"], M, K)
        d["x"] = d["prev"] if c["act"] != "gelu" else torch.nn.functional.gelu(d["prev"])
        d["dz"] = r.normal(M, N, scale=1.0 / M)
        d.update(_theta(r, "W", (N, K), K, g, c["opt"]))
        d.update(_theta(r, "b", (N,), K, g, c["opt"]))
    elif p in ("conv", "depthwise"):
        N, H, W, C, Co = c["N"], c["H"], c["W"], c["C"], c.get("Cout", c["C"])
        s = c.get("stride", 1)
        Ho, Wo = (H - 1) // s + 1, (W - 1) // s + 1
        rows = N * Ho * Wo
        g = 1.0 / math.sqrt(rows)
        d["x"] = _activation(r, "relu", N, H, W, C)
        d["dy"] = r.normal(N, Ho, Wo, Co, scale=1.0 / rows)
        shape = (Co, 3, 3, C) if p == "conv" else (3, 3, C)
        d.update(_theta(r, "W", shape, 9 * C if p == "conv" else 9, g, c["opt"]))
        d.update(_theta(r, "b", (Co,), 9, g, c["opt"]))
    elif p == "layernorm":
        M, D = c["M"], c["D"]
        g = 1.0 / math.sqrt(M)
        d["x"] = r.normal(M, D) + 0.3 * r.normal(1, D)
        d["dy"], d["dres"] = r.normal(M, D, scale=1.0 / M), r.normal(M, D, scale=1.0 / M)
        d.update(_theta(r, "gamma", (D,), D, g, c["opt"]))
        d["gamma"] += 1.0
        d.update(_theta(r, "beta", (D,), D, g, c["opt"]))
    elif p == "optimizer":
        for name, shape in _block_shapes(c):
            d.update(_theta(r, name, shape, shape[-1], 0.01, c["opt"]))
            d[name + "_g"] = r.normal(*shape, scale=0.01)
    elif p == "mlp_step":
        dims = _dims(c)
        for i in range(len(dims) - 1):
            d[f"fc{i + 1}.weight"] = r.weight(dims[i + 1], dims[i], fan_in=dims[i])
            d[f"fc{i + 1}.bias"] = r.normal(dims[i + 1], scale=0.02)
        d["x"] = r.normal(c["batch"], dims[0])
        d["labels"] = torch.randint(0, dims[-1], (c["batch"],), generator=r.g, device=DEV)
    else:
        raise ValueError(p)
    return d


def _dims(c):
    return [int(v) for v in c["dims"].split("-")]


def _block_shapes(c):
    w, f = c["width"], c["ffn"]
    out = []
    for i in range(c["layers"]):
        out += [(f"t{i}.{n}", s) for n, s in (("ln", (w,)), ("qkv", (3 * w, w)), ("qkv_b", (3 * w,)),
                                              ("proj", (w, w)), ("proj_b", (w,)), ("fc1", (f, w)),
                                              ("fc1_b", (f,)), ("fc2", (w, f)), ("fc2_b", (w,)))]
    return out


# ------------------------------------------------------- what a program keeps
class _State:
    """One prepared case: tensors by name, descriptors, workspaces and the update counter."""

    def __init__(self, c, seed):
        self.c, self.t = c, _inputs(c, seed)
        self.stream = torch.cuda.current_stream().cuda_stream
        self.step = STEP0
        self.hyper = OPTS.get(c.get("opt"))

    def buf(self, name, *shape, dtype=torch.float32):
        self.t[name] = torch.zeros(*shape, dtype=dtype, device=DEV)
        return self.t[name]

    def p(self, name):
        return self.t[name].data_ptr()

    def param(self, name, shadow=False):
        wb = None
        if shadow:
            wb = self.t[name + "_bf16"] = self.t[name].to(torch.bfloat16)
        q = L.param_of(self.t[name], self.t[name + "_m"], self.t[name + "_v"], wb)
        if self.hyper["kind"] in ("adagrad", "rmsprop"):
            q.m = None      # these keep no m
        return q

    def weight_only(self, name, shadow=False):
        q = L.OfParam(self.p(name), None, None, None, self.t[name].numel())
        if shadow:
            self.t[name + "_bf16"] = self.t[name].to(torch.bfloat16)
            q.w_bf16 = self.p(name + "_bf16")
        return q

    def ws(self, name, size):
        b = self.buf(name, (max(size, 16) + 15) // 16 * 4)
        return b.data_ptr(), b.numel() * 4

    def opt(self):
        """The optimizer argument of the next update."""
        self.step += 1
        return L.make_opt(self.hyper, self.step, None, self.t["scale"].data_ptr()
                          if "scale" in self.t else None)

    def updated(self, *names):
        out = {}
        for n in names:
            out[n] = self.t[n]
            if self.hyper["kind"] not in ("adagrad", "rmsprop"):
                out[n + "_m"] = self.t[n + "_m"]
            if self.hyper["kind"] != "sgd":
                out[n + "_v"] = self.t[n + "_v"]
            if n + "_bf16" in self.t:
                out[n + "_bf16"] = self.t[n + "_bf16"]
        return out


def prepare(case, seed):
    c, s, p = case, _State(case, seed), case["path"]
    if p in ("linear_fwd", "bf16_fwd"):
        M, N, K = c["M"], c["N"], c["K"]
        bf = p == "bf16_fwd"
        io = (L.OF_IO_X_BF16 if c.get("x_bf16") else 0) | (L.OF_IO_Y_BF16 if c.get("y_bf16") else 0)
        s.desc = L.OfLinearDesc(M, N, K, 0, 0, L.OF_BF16 if bf else L.OF_F32, L.ACTS[c["act"]],
                                int(c["bias"]), io)
        if c.get("x_bf16"):
            s.t["x"] = s.t["x"].to(torch.bfloat16)
        s.W = s.weight_only("W", shadow=bf)
        s.buf("y", M, N, dtype=torch.bfloat16 if c.get("y_bf16") else torch.float32)
        s.z = s.buf("z", M, N).data_ptr() if c["act"] == "gelu" else None
        s.wsm = s.ws("ws", L.of_linear_workspace_size(s.desc, L.OF_LINEAR_FWD))
    elif p in ("linear_bwd", "linear_merged", "bf16_bwd", "pointwise"):
        M, N, K = c["M"], c["N"], c["K"]
        bf = p == "bf16_bwd"
        s.desc = L.OfLinearDesc(M, N, K, 0, 0, L.OF_BF16 if bf else L.OF_F32,
                                L.ACTS[c["act"]] if p == "pointwise" else L.OF_ACT_NONE,
                                int(c.get("bias", True)), L.OF_IO_X_BF16 if bf else 0)
        if bf:
            s.t["x"] = s.t["x"].to(torch.bfloat16)
        s.W = s.param("W", shadow=bf)
        s.b = s.param("b") if c.get("bias", True) else None
        s.act_prev = L.OF_ACT_RELU if p == "pointwise" else L.ACTS[c["act"]]
        s.prev = s.p("prev") if s.act_prev != L.OF_ACT_NONE else None
        s.buf("dx", M, K)
        if p == "linear_merged":
            s.wsm = s.ws("ws", L.of_linear_workspace_size(s.desc, L.OF_LINEAR_BWD_MERGED))
        else:
            ops = (L.OF_LINEAR_FWD, L.OF_LINEAR_BWD_DATA)
            s.wsm = s.ws("ws", max(L.of_linear_workspace_size(s.desc, o) for o in ops))
            s.wsu = s.ws("ws_update", L.of_linear_workspace_size(s.desc, L.OF_LINEAR_BWD_WEIGHT))
        if p == "pointwise":
            s.buf("y", M, N)
        s.side = torch.cuda.Stream() if c.get("overlap") else None
        s.main = torch.cuda.current_stream()
    elif p == "conv":
        N, H, W, C, Co = c["N"], c["H"], c["W"], c["C"], c["Cout"]
        s.desc = L.OfConvDesc(N, H, W, C, Co, L.OF_ACT_RELU, 1, 1)
        s.W, s.b = s.param("W"), s.param("b")
        s.buf("y", N, H, W, Co)
        s.buf("dx", N, H, W, C)
        s.wsm = s.ws("ws", max(L.of_conv_workspace_size(s.desc, o) for o in (0, 1, 2)))
    elif p == "depthwise":
        N, H, W, C = c["N"], c["H"], c["W"], c["C"]
        s.desc = L.OfConvDesc(N, H, W, C, C, L.OF_ACT_RELU, 1, c["stride"])
        s.W, s.b = s.param("W"), s.param("b")
        s.buf("y", *s.t["dy"].shape)
        s.buf("dx", N, H, W, C)
        s.wsm = s.ws("ws", L.of_dwconv_workspace_size(s.desc))
    elif p == "layernorm":
        M, D = c["M"], c["D"]
        s.gamma, s.beta = s.param("gamma"), s.param("beta")
        s.buf("y", M, D, dtype=torch.bfloat16 if c["y_bf16"] else torch.float32)
        s.buf("dx", M, D)
        s.buf("mean", M), s.buf("rstd", M)
        s.G = L.of_layernorm_partial_rows(M)
        s.buf("dgamma", s.G, D), s.buf("dbeta", s.G, D)
    elif p == "optimizer":
        names = [n for n, _ in _block_shapes(c)]
        s.n = len(names)
        s.params = (L.OfParam * s.n)(*[s.param(n) for n in names])
        s.grads = (L.c_void_p * s.n)(*[s.p(n + "_g") for n in names])
        if c["clip"]:
            s.t["scale"], s.t["norm"] = torch.ones(1, device=DEV), torch.zeros(1, device=DEV)
            s.refs = L.grad_refs([(s.p(n + "_g"), s.t[n].numel(), 1, 0) for n in names])
            s.wsm = s.ws("ws", L.OF_CLIP_WS_BYTES)
    elif p == "mlp_step":
        from paper_2104_00237_amd.trainer import Trainer
        dims = _dims(c)
        cfg = dict(kind="mlp", dims=dims, act="relu", bias=True, batch=c["batch"], loss="xent",
                   classes=dims[-1], dtype="f32", steps=5, name="mlp",
                   opt=dict(kind="sgd", lr=0.01, momentum=0.9, weight_decay=1e-4))
        s.trainer = Trainer(cfg, {k: v.cpu().numpy() for k, v in s.t.items() if k.startswith("fc")}, DEV)
    return s


def run(s):
    c, p = s.c, s.c["path"]
    if p in ("linear_fwd", "bf16_fwd"):
        L.of_linear_fwd(s.desc, s.p("x"), s.W, s.p("b") if c["bias"] else None, s.z, s.p("y"),
                        *s.wsm, s.stream)
        return {"y": s.t["y"], "z": s.t["z"]} if s.z else {"y": s.t["y"]}
    if p == "linear_merged":
        L.of_linear_bwd_merged(s.desc, s.p("dz"), s.p("x"), s.W, s.b, None, None, s.opt(), s.prev,
                               s.act_prev, s.p("dx"), *s.wsm, s.stream)
        return {"dx": s.t["dx"], **s.updated("W", *(["b"] if s.b else []))}
    if p in ("linear_bwd", "bf16_bwd", "pointwise"):
        out = {}
        if p == "pointwise":
            L.of_linear_fwd(s.desc, s.p("x"), s.W, s.p("b"), None, s.p("y"), *s.wsm, s.stream)
            out["y"] = s.t["y"]
        L.of_linear_bwd_fused(s.desc, s.p("dz"), s.p("x"), s.W, s.b, None, None, s.opt(), s.prev,
                              s.act_prev, s.p("dx"), *s.wsm, *s.wsu, s.stream,
                              s.side.cuda_stream if s.side else None)
        if s.side:
            s.main.wait_stream(s.side)
        return {**out, "dx": s.t["dx"], **s.updated("W", *(["b"] if s.b else []))}
    if p == "conv":
        L.of_conv_fwd(s.desc, s.p("x"), s.W, s.p("b"), s.p("y"), *s.wsm, s.stream)
        L.of_conv_bwd_data(s.desc, s.p("dy"), s.W, s.p("x"), L.OF_ACT_RELU, s.p("dx"), *s.wsm, s.stream)
        L.of_conv_wgrad_fused(s.desc, s.p("dy"), s.p("x"), s.W, s.b, None, None, s.opt(), *s.wsm,
                              s.stream)
        return {"y": s.t["y"], "dx": s.t["dx"], **s.updated("W", "b")}
    if p == "depthwise":
        L.of_dwconv_fwd(s.desc, s.p("x"), s.p("W"), s.p("b"), s.p("y"), s.stream)
        L.of_dwconv_bwd_data(s.desc, s.p("dy"), s.p("W"), s.p("x"), L.OF_ACT_RELU, s.p("dx"), s.stream)
        L.of_dwconv_wgrad_fused(s.desc, s.p("dy"), s.p("x"), s.W, s.b, None, None, s.opt(), *s.wsm,
                                s.stream)
        return {"y": s.t["y"], "dx": s.t["dx"], **s.updated("W", "b")}
    if p == "layernorm":
        M, D = c["M"], c["D"]
        fwd = L.of_layernorm_fwd_bf16 if c["y_bf16"] else L.of_layernorm_fwd
        fwd(s.p("x"), M, D, s.p("gamma"), s.p("beta"), LN_EPS, s.p("y"), s.p("mean"), s.p("rstd"),
            s.stream)
        L.of_layernorm_bwd(s.p("dy"), s.p("x"), s.p("mean"), s.p("rstd"), s.p("gamma"), s.p("dres"),
                           M, D, s.p("dx"), s.p("dgamma"), s.p("dbeta"), s.stream)
        opt = s.opt()
        L.of_elementwise_fused_update(s.gamma, s.p("dgamma"), s.G, 0, opt, s.stream)
        L.of_elementwise_fused_update(s.beta, s.p("dbeta"), s.G, 0, opt, s.stream)
        return {"y": s.t["y"], "mean": s.t["mean"], "rstd": s.t["rstd"], "dx": s.t["dx"],
                **s.updated("gamma", "beta")}
    if p == "optimizer":
        if c["clip"]:
            L.of_grad_clip_scale(s.n, s.refs, 1.0, s.p("scale"), s.p("norm"), *s.wsm, s.stream)
        L.of_optimizer_step(s.n, s.params, s.grads, s.opt(), s.stream)
        out = s.updated(*[n for n, _ in _block_shapes(c)][:9])
        return {**out, "norm": s.t["norm"]} if c["clip"] else out
    tr = s.trainer
    tr.step(s.t["x"], s.t["labels"], c["ordering"])
    out = {"logits": tr.net.out}
    for k, q in tr.params.items():
        out[k] = q.w
        if c["ordering"] != "bf":
            out[k + ".grad"] = q.g
    return out


# --------------------------------------------------------------- what it costs
def _state_bytes(n, kind):
    """Bytes of one fused update of n elements: w and the history, read and written."""
    return 8 * n * (3 if kind in ("adam", "adamw", "adadelta") else 2)


def work(c):
    p = c["path"]
    if p in ("linear_fwd", "bf16_fwd"):
        M, N, K = c["M"], c["N"], c["K"]
        xb, yb = (2 if c.get("x_bf16") else 4), (2 if c.get("y_bf16") else 4)
        wb = 2 if p == "bf16_fwd" else 4
        return {"bytes": M * K * xb + N * K * wb + M * N * (yb + (4 if c["act"] == "gelu" else 0)) + 4 * N,
                "flops": 2 * M * N * K}
    if p in ("linear_bwd", "linear_merged", "bf16_bwd", "pointwise"):
        M, N, K = c["M"], c["N"], c["K"]
        bf = p == "bf16_bwd"
        act = "relu" if p == "pointwise" else c["act"]
        # ReLU's saved output is X itself; GELU's pre-activation is another tensor
        saved = 4 if act == "gelu" or (bf and act != "none") else 0
        b = 4 * M * N + M * K * ((2 if bf else 4) + 4 + saved) + _state_bytes(N * K + N, c["opt"])
        if bf:
            b += 4 * N * K      # the shadow read by the data gradient and rewritten
        if p == "pointwise":
            return {"bytes": b + 4 * M * N, "flops": 6 * M * N * K}
        return {"bytes": b, "flops": 4 * M * N * K}
    if p in ("conv", "depthwise"):
        s = c.get("stride", 1)
        Co = c.get("Cout", c["C"])
        nx = c["N"] * c["H"] * c["W"] * c["C"]
        rows = c["N"] * ((c["H"] - 1) // s + 1) * ((c["W"] - 1) // s + 1)
        nw = 9 * (c["C"] * Co if p == "conv" else Co)
        return {"bytes": 4 * (2 * nx + 2 * rows * Co) + _state_bytes(nw + Co, c["opt"]),
                "flops": 6 * rows * nw}
    if p == "layernorm":
        n = c["M"] * c["D"]
        return {"bytes": n * (4 * 4 + (2 if c["y_bf16"] else 4)) + _state_bytes(2 * c["D"], c["opt"]),
                "flops": 20 * n}
    if p == "optimizer":
        n = sum(int(np.prod(s)) for _, s in _block_shapes(c))
        return {"bytes": _state_bytes(n, c["opt"]) + 4 * n, "flops": 15 * n}
    d = _dims(c)
    n = sum(a * b + b for a, b in zip(d, d[1:]))
    return {"bytes": 4 * c["batch"] * (d[0] + d[-1]) + _state_bytes(n, "sgd"),
            "flops": 6 * c["batch"] * n}


def tolerance(c):
    """About four times the distance from `exact` of the paths as first measured: fp32 sums 0.6 to 0.8e-6
    at reductions of 1024 to 8192, outputs rounded to bf16 1.7e-3."""
    if c["path"] == "bf16_bwd" or c.get("y_bf16"):
        return {"rel": 7e-3}        # the shadow of the updated weight, or Y, is rounded to bf16
    if c["path"] == "mlp_step":
        return {"rel": 4e-6, "max": 1e-3}   # a pre-activation near 0 may take the other side
    return {"rel": 4e-6}


# ------------------------------------------------------------ in 64 bits
def _update64(hyper, w, g, m, v, t):
    k, lr, wd = hyper["kind"], hyper["lr"], hyper.get("weight_decay", 0.0)
    f = lambda x: float(np.float32(x))  # noqa: E731  (hyperparameters travel as fp32)
    lr, wd = f(lr), f(wd)
    if k == "sgd":
        m = f(hyper["momentum"]) * m + g + wd * w
        return w - lr * m, m, v
    eps = f(hyper["eps"])
    if k in ("adam", "adamw"):
        b1, b2 = f(hyper["beta1"]), f(hyper["beta2"])
        if k == "adamw":
            w = w * (1 - lr * wd)
        else:
            g = g + wd * w
        m, v = b1 * m + (1 - b1) * g, b2 * v + (1 - b2) * g * g
        return w - lr / (1 - b1 ** t) * m / (v.sqrt() / math.sqrt(1 - b2 ** t) + eps), m, v
    g = g + wd * w
    if k == "adagrad":
        v = v + g * g
        return w - lr * g / (v.sqrt() + eps), m, v
    if k == "rmsprop":
        a = f(hyper["alpha"])
        v = a * v + (1 - a) * g * g
        return w - lr * g / (v.sqrt() + eps), m, v
    a = f(hyper["rho"])
    v = a * v + (1 - a) * g * g
    d = ((m + eps) / (v + eps)).sqrt() * g
    return w - lr * d, a * m + (1 - a) * d * d, v


def _act64(act, z):
    if act == "relu":
        return z.clamp_min(0)
    return 0.5 * z * (1 + torch.erf(z / math.sqrt(2))) if act == "gelu" else z


def _dact64(act, prev):
    if act == "relu":
        return (prev > 0).double()
    if act == "gelu":
        return (0.5 * (1 + torch.erf(prev / math.sqrt(2)))
                + prev * torch.exp(-0.5 * prev * prev) / math.sqrt(2 * math.pi))
    return 1.0


def _bf16(x):
    return x.to(torch.bfloat16).double()


def _updated64(c, d, grads):
    out, h = {}, OPTS[c["opt"]]
    for n, g in grads.items():
        w, m, v = _update64(h, d[n].double(), g, d[n + "_m"].double(), d[n + "_v"].double(), STEP0 + 1)
        out[n] = w
        if h["kind"] not in ("adagrad", "rmsprop"):
            out[n + "_m"] = m
        if h["kind"] != "sgd":
            out[n + "_v"] = v
    return out


def _shift(x, dy, dx):
    """x[n, h + dy, w + dx, c], zero outside the image."""
    N, H, W, C = x.shape
    xp = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1))
    return xp[:, 1 + dy:1 + dy + H, 1 + dx:1 + dx + W, :]


def exact(case, seed):
    c, p, d = case, case["path"], _inputs(case, seed)
    if p in ("linear_fwd", "bf16_fwd"):
        r = _bf16 if p == "bf16_fwd" else torch.Tensor.double
        z = r(d["x"]) @ r(d["W"]).t()
        if c["bias"]:
            z = z + d["b"].double()
        y = _act64(c["act"], z)
        return {"y": y, "z": z} if c["act"] == "gelu" else {"y": y}
    if p in ("linear_bwd", "linear_merged", "bf16_bwd", "pointwise"):
        r = _bf16 if p == "bf16_bwd" else torch.Tensor.double
        act = "relu" if p == "pointwise" else c["act"]
        dz, x, W = r(d["dz"]), r(d["x"]), r(d["W"])
        out = {}
        if p == "pointwise":
            out["y"] = _act64(c["act"], x @ W.t() + d["b"].double())
        out["dx"] = (dz @ W) * _dact64(act, d["prev"].double())
        grads = {"W": dz.t() @ x}
        if c.get("bias", True):
            grads["b"] = d["dz"].double().sum(0)
        out.update(_updated64(c, d, grads))
        if p == "bf16_bwd":
            out["W_bf16"] = out["W"]
        return out
    if p == "conv":
        N, H, W, C, Co = c["N"], c["H"], c["W"], c["C"], c["Cout"]
        x, dy, w = d["x"].double(), d["dy"].double(), d["W"].double()
        y = torch.zeros(N * H * W, Co, dtype=torch.float64, device=DEV)
        dx, dw = torch.zeros_like(x), torch.zeros_like(w)
        dyf = dy.reshape(-1, Co)
        for i in range(3):
            for j in range(3):
                xs = _shift(x, i - 1, j - 1).reshape(-1, C)
                y += xs @ w[:, i, j, :].t()
                dw[:, i, j, :] = dyf.t() @ xs
                dx += (_shift(dy, 1 - i, 1 - j).reshape(-1, Co) @ w[:, i, j, :]).reshape(N, H, W, C)
        return {"y": _act64("relu", y + d["b"].double()).reshape(N, H, W, Co), "dx": dx * (x > 0),
                **_updated64(c, d, {"W": dw, "b": dyf.sum(0)})}
    if p == "depthwise":
        s, x, dy, w = c["stride"], d["x"].double(), d["dy"].double(), d["W"].double()
        full = torch.zeros_like(x)          # dy at the input pixels its output rows come from
        full[:, ::s, ::s, :] = dy
        y, dx, dw = torch.zeros_like(x), torch.zeros_like(x), torch.zeros_like(w)
        for i in range(3):
            for j in range(3):
                xs = _shift(x, i - 1, j - 1)
                y += xs * w[i, j]
                dw[i, j] = (full * xs).sum((0, 1, 2))
                dx += _shift(full, 1 - i, 1 - j) * w[i, j]
        y = _act64("relu", y[:, ::s, ::s, :] + d["b"].double())
        return {"y": y, "dx": dx * (x > 0), **_updated64(c, d, {"W": dw, "b": dy.sum((0, 1, 2))})}
    if p == "layernorm":
        x, dy = d["x"].double(), d["dy"].double()
        mean = x.mean(1)
        rstd = 1 / (x.var(1, unbiased=False) + float(np.float32(LN_EPS))).sqrt()
        xh = (x - mean[:, None]) * rstd[:, None]
        g = dy * d["gamma"].double()
        dx = d["dres"].double() + rstd[:, None] * (g - g.mean(1, True) - xh * (g * xh).mean(1, True))
        return {"y": xh * d["gamma"].double() + d["beta"].double(), "mean": mean, "rstd": rstd, "dx": dx,
                **_updated64(c, d, {"gamma": (dy * xh).sum(0), "beta": dy.sum(0)})}
    if p == "optimizer":
        names = [n for n, _ in _block_shapes(c)]
        grads = {n: d[n + "_g"].double() for n in names}
        norm = torch.stack([g.square().sum() for g in grads.values()]).sum().sqrt()
        scale = min(1.0, 1.0 / (float(norm) + 1e-6)) if c["clip"] else 1.0
        out = _updated64(c, d, {n: grads[n] * scale for n in names[:9]})
        return {**out, "norm": norm.reshape(1)} if c["clip"] else out
    dims, a, hs = _dims(c), d["x"].double(), []
    for i in range(1, len(dims)):
        hs.append(a)
        z = a @ d[f"fc{i}.weight"].double().t() + d[f"fc{i}.bias"].double()
        a = z if i == len(dims) - 1 else z.clamp_min(0)
    out = {"logits": a}
    g = torch.softmax(a, 1)
    g[torch.arange(c["batch"], device=DEV), d["labels"]] -= 1
    g = g / c["batch"]
    lr, wd = float(np.float32(0.01)), float(np.float32(1e-4))
    for i in range(len(dims) - 1, 0, -1):
        for n, gw in ((f"fc{i}.weight", g.t() @ hs[i - 1]), (f"fc{i}.bias", g.sum(0))):
            w = d[n].double()
            # the first update of a run (momentum starts at 0); forward-fusion leaves it pending
            out[n] = w if c["ordering"] == "ff" else w - lr * (gw + wd * w)
            if c["ordering"] != "bf":
                out[n + ".grad"] = gw
        g = (g @ d[f"fc{i}.weight"].double()) * (hs[i - 1] > 0)
    return out
