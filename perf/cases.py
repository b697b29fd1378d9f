"""The calls whose speed matters to a user of this framework, over the sizes they are used at.

Most of them are whole training steps (`s4tf_train_step`: forward, pullbacks, optimizer), which is what the framework
is for: the five networks of workloads/nets.py at their own sizes, and at other batch and image sizes.  The rest are the
per-op entry points that op-by-op programs and inference call: a convolution layer with its pullback, a BatchNorm
with its pullback, a residual block in inference mode with folded BatchNorms, indexing with its pullback.

A case is a dict with a `kind` and that kind's sizes; `draw` gives other cases of the same ranges."""
import math

import numpy as np
import torch

from paper_2102_13243_amd import binding as B
from workloads import nets

DEV = "cuda:0"


# ---- the cases -------------------------------------------------------------------------------------------------
def _step(net, batch, hw):
    return {"kind": "step", "net": net, "batch": batch, "hw": hw}


def listed():
    return [
        # The configurations that the benchmark runs: the smallest is launch latency alone, LeNet-5 little more ...
        dict(_step("tiny", 8, 16), name="step_tiny_b8"),
        dict(_step("lenet5", 128, 28), name="step_lenet5_b128"),
        # ... the CIFAR network is many small layers, the two ImageNet networks move gigabytes a step (fp32 and bf16)
        dict(_step("resnet56", 128, 32), name="step_resnet56_b128"),
        dict(_step("mobilenetv2", 32, 224), name="step_mobilenetv2_b32"),
        dict(_step("resnet50", 64, 224), name="step_resnet50_b64"),
        # Sizes off the beaten path: a data set of other images (40x40, so 20x20 and 10x10 maps) with the uneven last
        # minibatch of an epoch, and two steps of training at a reduced resolution (maps of 11x11, 6x6 and 5x5)
        dict(_step("resnet56", 50, 40), name="step_resnet56_b50_hw40"),
        dict(_step("mobilenetv2", 5, 160), name="step_mobilenetv2_b5_hw160"),
        dict(_step("resnet50", 13, 176), name="step_resnet50_b13_hw176"),
        # Op by op: one 3x3 layer in the middle of a bf16 network, forward and both pullbacks
        {"kind": "conv", "n": 32, "h": 28, "w": 28, "c": 128, "k": 128, "r": 3, "stride": 1, "dtype": "bf16",
         "name": "conv_bf16_28x28_128"},
        # ... the largest BatchNorm + residual + ReLU of that network, forward and pullback: memory bound
        {"kind": "bn", "n": 64, "h": 56, "w": 56, "c": 256, "residual": True, "act": "relu", "dtype": "bf16",
         "name": "bn_bf16_56x56_256"},
        # Inference of a bottleneck block at a serving batch, BatchNorms folded into its convolutions
        {"kind": "infer", "n": 8, "h": 14, "w": 14, "width": 256, "dtype": "bf16", "name": "infer_bf16_14x14_256"},
        # x[i] and its in-place pullback: an embedding table and the tokens of a minibatch
        {"kind": "gather", "rows": 50000, "cols": 128, "count": 8192, "dtype": "f32", "name": "gather_f32_8192x128"},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# batch and image sizes each network is used at; the last number bounds batch * hw^2 by the listed configuration's
_STEP_RANGE = {"tiny": ((1, 64), (8, 32), 64 * 256), "lenet5": ((16, 512), (28, 28), 512 * 784),
               "resnet56": ((16, 128), (24, 64), 128 * 1024), "mobilenetv2": ((1, 32), (96, 224), 32 * 224 * 224),
               "resnet50": ((12, 64), (128, 224), 64 * 224 * 224)}


def draw(rng):
    kind = rng.choice(["step"] * 6 + ["conv", "bn", "infer", "gather"])
    if kind == "step":
        net = rng.choice(sorted(_STEP_RANGE))
        (blo, bhi), (hlo, hhi), most = _STEP_RANGE[net]
        hw = rng.randint(hlo // 2, hhi // 2) * 2
        if net in ("mobilenetv2", "resnet50"):
            hw = hw // 16 * 16
        return _step(net, max(1, min(_log(rng, blo, bhi), most // (hw * hw))), hw)
    dtype = rng.choice(["f32", "bf16"])
    if kind == "conv":
        while True:
            c, k = 8 * _log(rng, 2, 64), 8 * _log(rng, 2, 64)
            case = {"kind": "conv", "n": _log(rng, 1, 64), "h": rng.randint(7, 56), "w": rng.randint(7, 56), "c": c, "k": k,
                    "r": rng.choice([1, 3]), "stride": rng.choice([1, 1, 2]), "dtype": dtype}
            if work(case)["flops"] <= (3e11 if dtype == "bf16" else 3e10):
                return case
    if kind == "bn":
        while True:
            case = {"kind": "bn", "n": _log(rng, 1, 64), "h": rng.randint(7, 112), "w": rng.randint(7, 112),
                    "c": 8 * _log(rng, 2, 256), "residual": rng.random() < 0.5, "act": rng.choice(["none", "relu", "relu6"]),
                    "dtype": dtype}
            if case["n"] * case["h"] * case["w"] * case["c"] <= 64 * 56 * 56 * 256:
                return case
    if kind == "infer":
        width = 64 * rng.choice([1, 2, 4, 8])
        return {"kind": "infer", "n": _log(rng, 1, 32), "h": rng.randint(7, 56), "w": rng.randint(7, 28), "width": width, "dtype": dtype}
    return {"kind": "gather", "rows": _log(rng, 1000, 100000), "cols": _log(rng, 16, 512), "count": _log(rng, 128, 16384),
            "dtype": dtype}


# ---- inputs ----------------------------------------------------------------------------------------------------
def _net(case):
    make = nets.CONFIGS[case["net"]]
    if case["net"] in ("resnet56", "mobilenetv2", "resnet50"):
        return make(batch=case["batch"], hw=case["hw"])
    net = make(batch=case["batch"])
    n, _, _, c = net["input"]
    net["input"] = (n, case["hw"], case["hw"], c)
    return net


def _code(case):
    return B.S4TF_BF16 if case["dtype"] == "bf16" else B.S4TF_F32


class _Draw:
    """Seeded tensors on the GPU in the case's storage type."""

    def __init__(self, case, seed):
        self.g = torch.Generator(device=DEV)
        self.g.manual_seed(seed)
        self.dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32

    def normal(self, shape, scale=1.0, dt=None):
        return (torch.randn(shape, generator=self.g, device=DEV) * scale).to(dt or self.dt)

    def f32(self, n, mean=0.0, scale=0.3):
        return torch.randn(n, generator=self.g, device=DEV) * scale + mean

    def empty(self, shape, dt=None):
        return torch.empty(shape, dtype=dt or self.dt, device=DEV)


def _ws(nbytes):
    return torch.empty(max(16, nbytes), dtype=torch.uint8, device=DEV)


def _clear_of_kinks(net, params, seed):
    """BatchNorm shifts that put every pre-activation on one side of its ReLU kink, some four of the channel's standard
    deviations from zero: half of the channels on, half off; all on where a residual or a depthwise layer would make
    something else of an off channel.  With pre-activations centred on the kink two correct implementations decide a
    few of a deep network's millions of activations differently, and their gradients then agree to 1e-2 in fp32 and
    not at all in bf16: nothing to compare results by."""
    rng = np.random.default_rng(seed)
    depthwise = {op["in"] for op in net["ops"] if op["kind"] == "conv" and op["groups"] > 1}
    for i, (op, p) in enumerate(zip(net["ops"], params)):
        if op["kind"] == "bn" and op["act"] != "none":
            on = rng.random(p[1].shape) < (0.5 if op["res"] < 0 and i + 1 not in depthwise else 1.0)
            p[0] *= np.float32(0.25)
            p[1] = np.where(on, 1.0, -1.0).astype(np.float32) + np.float32(0.25) * p[1]


def _prepare_step(case, seed):
    net = _net(case)
    net["seed"] = seed
    wl = nets.make_workload(net, perturb=True)
    _clear_of_kinks(net, wl["params"], seed)
    st = B.TrainState(net, wl["params"], DEV)
    x, labels = st.upload_batch(wl["x"], wl["labels"])
    # a step of an early warm-up in fp32, of training in full swing in bf16
    return {"kind": "step", "st": st, "x": x, "labels": labels, "lr": net["lr"] * (0.1 if st.lowp is None else 1.0)}


def _prepare_conv(case, seed):
    r = _Draw(case, seed)
    n, h, w, c, k, f = (case[v] for v in ("n", "h", "w", "c", "k", "r"))
    d = B.ConvDesc(n, h, w, c, k, f, f, case["stride"], f // 2, 1, _code(case), B.ACT["none"], 0)
    p, q = (h + 2 * (f // 2) - f) // case["stride"] + 1, (w + 2 * (f // 2) - f) // case["stride"] + 1
    return {"kind": "conv", "d": d, "x": r.normal((n, h, w, c)), "w": r.normal((f, f, c, k), (2.0 / (f * f * c)) ** 0.5),
            "dy": r.normal((n, p, q, k)), "y": r.empty((n, p, q, k)), "dx": r.empty((n, h, w, c)),
            "dw": r.empty((f, f, c, k), torch.float32),
            "ws": _ws(max(B.s4tf_conv2d_fwd_workspace_bytes(d), B.s4tf_conv2d_vjp_workspace_bytes(d)))}


def _prepare_bn(case, seed):
    r = _Draw(case, seed)
    shape, c = tuple(case[v] for v in ("n", "h", "w", "c")), case["c"]
    d = B.BnDesc(*shape, 1e-5, B.ACT[case["act"]], _code(case), 0)
    # convolution outputs: channel means of a fraction of the channel's spread
    x = (torch.randn(shape, generator=r.g, device=DEV) * (1.0 + r.f32(c, 0.0, 0.2).abs()) + r.f32(c)).to(r.dt)
    res = r.normal(shape) if case["residual"] else None
    gamma, beta = r.f32(c, 1.0), r.f32(c, 0.0, 0.2)
    # what the pullback captures is given: the statistics and the output of an earlier forward pass over the same input
    x32 = x.float()
    mean, var = x32.mean((0, 1, 2)), x32.var((0, 1, 2), unbiased=False)
    invstd = (var + 1e-5).rsqrt()
    z = (x32 - mean) * (gamma * invstd) + beta
    if res is not None:
        z += res.float()
    z = {"none": z, "relu": z.clamp(min=0.0), "relu6": z.clamp(0.0, 6.0)}[case["act"]]
    s = {"kind": "bn", "d": d, "x": x, "res": res, "gamma": gamma, "beta": beta, "y0": z.to(r.dt), "mean0": mean.contiguous(),
         "invstd0": invstd.contiguous(), "dy": r.normal(shape), "y": r.empty(shape), "dx": r.empty(shape),
         "dres": r.empty(shape) if case["residual"] else None, "ws": _ws(B.s4tf_bn_relu_workspace_bytes(d))}
    for v in ("mean", "invstd", "dgamma", "dbeta"):
        s[v] = r.empty((c,), torch.float32)
    return s


def _prepare_infer(case, seed):
    r = _Draw(case, seed)
    n, h, w, m = (case[v] for v in ("n", "h", "w", "width"))
    code, relu = _code(case), B.ACT["relu"]
    s = {"kind": "infer", "x": r.normal((n, h, w, 4 * m)).clamp_(min=0), "layers": []}
    for c, k, f, act in ((4 * m, m, 1, relu), (m, m, 3, relu), (m, 4 * m, 1, B.ACT["none"])):
        d = B.ConvDesc(n, h, w, c, k, f, f, 1, f // 2, 1, code, act, 0)
        wt = r.normal((f, f, c, k), (2.0 / (f * f * c)) ** 0.5)
        bn = (r.f32(k, 1.0), r.f32(k, 0.0, 0.2), r.f32(k), 0.5 + r.f32(k).abs())  # gamma, beta, running mean and variance
        y, bias = r.empty((n, h, w, k)), None
        if act == relu:  # the weights as an inference program keeps them: the BatchNorm inside them
            wf, bias = torch.empty_like(wt), r.empty((k,), torch.float32)
            B.s4tf_bn_fold_into_conv(d, wt, None, *bn, 1e-5, wf, bias)
            wt = wf
        s["layers"].append((d, wt, bias, y, _ws(B.s4tf_conv2d_fwd_workspace_bytes(d))))
    s["bnd"] = B.BnDesc(n, h, w, 4 * m, 1e-5, relu, code, 0)  # the last BatchNorm adds the residual
    s["bn"], s["out"] = bn, r.empty((n, h, w, 4 * m))
    return s


def _prepare_gather(case, seed):
    r = _Draw(case, seed)
    rows, cols, count = case["rows"], case["cols"], case["count"]
    return {"kind": "gather", "d": B.GatherDesc(rows, cols, count, _code(case)), "x": r.normal((rows, cols)),
            "index": torch.randint(0, rows, (count,), generator=r.g, device=DEV, dtype=torch.int32),
            "dy": r.normal((count, cols)), "y": r.empty((count, cols)), "dx": r.normal((rows, cols))}


_PREPARE = {"step": _prepare_step, "conv": _prepare_conv, "bn": _prepare_bn, "infer": _prepare_infer, "gather": _prepare_gather}


def prepare(case, seed):
    return _PREPARE[case["kind"]](case, int(seed))


# ---- one pass --------------------------------------------------------------------------------------------------
def _run_step(s):
    st = s["st"]
    st.step(s["x"], s["labels"], s["lr"])
    if st.lowp is None:
        return {"loss": st.loss, "grad": st.grad, "param": st.master, "velocity": st.velocity}
    # bf16: rounding leaves 1e-1 of uncertainty in a filter's gradient fifty layers down, so what is compared is the loss, the
    # updated model and its bf16 working copy, at a learning rate that moves the parameters by several times the tolerance
    return {"loss": st.loss, "param": st.master, "lowp": st.lowp}


def _run_conv(s):
    B.s4tf_conv2d_fwd(s["d"], s["x"], s["w"], None, s["y"], s["ws"])
    B.s4tf_conv2d_vjp(s["d"], s["x"], s["w"], None, s["dy"], s["dx"], s["dw"], None, s["ws"])
    return s["y"], s["dx"], s["dw"]


def _run_bn(s):
    B.s4tf_bn_relu_fwd(s["d"], s["x"], s["res"], s["gamma"], s["beta"], s["y"], s["mean"], s["invstd"], s["ws"])
    beta = s["beta"] if s["res"] is None else None  # without a residual the pullback need not read y
    B.s4tf_bn_relu_vjp(s["d"], s["x"], s["y0"], s["gamma"], beta, s["mean0"], s["invstd0"], s["dy"], s["dx"], s["dres"],
                       s["dgamma"], s["dbeta"], s["ws"])
    return {v: s[v] for v in ("y", "mean", "invstd", "dx", "dres", "dgamma", "dbeta")}


def _run_infer(s):
    t, outs = s["x"], []
    for d, w, bias, y, ws in s["layers"]:
        B.s4tf_conv2d_fwd(d, t, w, bias, y, ws)
        t = y
        outs.append(y)
    B.s4tf_bn_inference_fwd(s["bnd"], t, s["x"], *s["bn"], s["out"])
    return outs + [s["out"]]


def _run_gather(s):
    B.s4tf_gather_rows_fwd(s["d"], s["x"], s["index"], s["y"])
    B.s4tf_gather_rows_vjp(s["d"], s["dy"], s["index"], s["dx"])
    return s["y"], s["dx"]


_RUN = {"step": _run_step, "conv": _run_conv, "bn": _run_bn, "infer": _run_infer, "gather": _run_gather}


def run(state):
    return _RUN[state["kind"]](state)


# ---- what a pass cannot do without --------------------------------------------------------------------------------
def work(case):
    kind = case["kind"]
    if kind == "step":
        # The convolutions (each pass its multiplications; the first layer has no input pullback) and the dense head.
        # Activations do not fit on the chip, so each convolution reads its input and writes its output in the forward pass,
        # reads its input and its output's cotangent and writes its input's cotangent in the backward pass; everything
        # between two convolutions could ride along.  Parameters: value, velocity and gradient, 20 bytes each.
        net = _net(case)
        es = 2 if net["dtype"] == "bf16" else 4
        shapes = nets.tensor_shapes(net)
        flops = bytes_ = params = 0
        for i, op in enumerate(net["ops"]):
            a, b = shapes[op["in"]], shapes[i + 1]
            if op["kind"] == "conv":
                f = 2 * math.prod(b) * op["r"] * op["s"] * a[3] // op["groups"]
                first = op["in"] == 0
                flops += f * (2 if first else 3)
                bytes_ += es * (math.prod(a) * (2 if first else 3) + 2 * math.prod(b))
                params += op["r"] * op["s"] * a[3] // op["groups"] * op["k"]
            elif op["kind"] == "bn":
                params += 2 * a[3]
            elif op["kind"] == "head":
                params += (a[3] + 1) * op["classes"]
                flops += 6 * a[0] * a[3] * op["classes"]
                bytes_ += es * 2 * math.prod(a)
        return {"bytes": bytes_ + params * (20 + (2 if es == 2 else 0)), "flops": flops}
    es = 2 if case["dtype"] == "bf16" else 4
    if kind == "gather":
        e = case["count"] * case["cols"]
        return {"bytes": es * 5 * e + 8 * case["count"], "flops": e}
    if kind == "bn":
        e = case["n"] * case["h"] * case["w"] * case["c"]
        res = 2 if case["residual"] else 0  # residual in, its cotangent out
        y = 1 if case["residual"] and case["act"] != "none" else 0
        return {"bytes": es * e * (5 + res + y), "flops": 14 * e}
    n, h, w = case["n"], case["h"], case["w"]
    if kind == "infer":
        m, px = case["width"], n * h * w
        return {"bytes": es * (px * 18 * m + 17 * m * m), "flops": 2 * px * 17 * m * m + 8 * px * m}
    f, st, c, k = case["r"], case["stride"], case["c"], case["k"]
    px, po = n * h * w, n * ((h + 2 * (f // 2) - f) // st + 1) * ((w + 2 * (f // 2) - f) // st + 1)
    return {"bytes": es * (2 * px * c + 2 * po * k + f * f * c * k) + 4 * f * f * c * k, "flops": 6 * po * k * f * f * c}


def tolerance(case):
    if case["kind"] == "gather":
        return "exact"  # one addition per element, repeated rows in a stated order
    if case["kind"] == "step":
        # bf16: between two roundings of the same step the loss differs by up to 2e-3 and the updated model by 5e-4, of the
        # 2e-2 to 5e-2 that it moves; fp32: up to 3e-6 in a deep network's gradients, on single elements 1e-3 of their rms
        return {"rel": 1e-2} if case["net"] == "resnet50" else {"rel": 1e-4}
    # one op on given inputs: sums in fp32, outputs rounded to the storage type
    return {"rel": 1e-2} if case["dtype"] == "bf16" else {"rel": 2e-5}
