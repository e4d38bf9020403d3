"""The work a training loop has the optimizer-step library do, as cases that can be timed and compared.

A case is one call of ``triaccel_step`` (a training step's optimizer part) or ``triaccel_power_iter`` /
``triaccel_power_iter_static`` (one power iteration on every layer) on tensors of the caller's own.
The caller keeps its parameters, curvature, momentum and masks in flat arenas, as data-parallel
training loops do, and one prepared tensor table per set of input buffers; passes cycle through the
input sets, so that a probed step sees a new probe sample and its threshold moves as it does in a run.

``grad`` / ``store``: precision of the gradients / of the stored parameters.  The thresholds of the
precision rule are set so that every tensor keeps that precision ("mixed": per tensor, by the variance
band its gradients are drawn from; "switch": the gradients of the two input sets lie on either side of
the threshold, so every tensor is rewritten at another size on every step).
``warm``: steps the run has behind it when the case begins.  A run's first steps look for the curvature
threshold without a forecast; on the large sets, where few passes are made, the case is a run under way.
"""
from __future__ import annotations

import ctypes
import math
import random

import numpy as np
import torch

import paper_2508_16905_amd as ta
from workloads import shapes as _shapes

_CODE = {"fp16": ta.FP16, "bf16": ta.BF16, "fp32": ta.FP32}
_TORCH = {"fp16": torch.float16, "bf16": torch.bfloat16, "fp32": torch.float32}
_BYTES = {"fp16": 2, "bf16": 2, "fp32": 4}
_PAD = 128       # elements a tensor's place in an arena is rounded up to (a mask of whole 16-byte units)
_HUGE = 1e30
_LR, _MU, _WD, _ALPHA = 0.1, 0.9, 5e-4, 0.1


def _step(name, set_, **kw):
    c = dict(name=name, kind="step", set=set_, tensors=0, total=0, shape_seed=0, grad="fp32", store="fp32", probe=False,
             source="hutchinson", elementwise=False, topk=0, loss_scale=1.0, read_result=False, input_sets=2, warm=0)
    c.update(kw)
    return c


def listed():
    return [
        # the ordinary step of a small model, between two curvature refreshes: launches and host time only
        _step("mlp_step", "tiny_mlp"),
        # the same model while it refreshes its curvature every step and reads the loss scale after each
        _step("mlp_probe_scaled", "tiny_mlp", probe=True, grad="fp16", loss_scale=1024.0, read_result=True),
        # the two networks the paper trains: the ordinary step, and the step that refreshes the curvature
        _step("resnet18_step", "resnet18"),
        _step("resnet18_probe", "resnet18", probe=True, store="bf16", input_sets=3),
        _step("effnet_b0_step_bf16", "efficientnet_b0", grad="bf16", store="bf16"),
        _step("effnet_b0_probe", "efficientnet_b0", probe=True, loss_scale=65536.0, input_sets=3),
        # odd sizes from a few elements to some millions; Fisher curvature, the paper's fixed k = 5 entries
        _step("ragged_fisher_top5", "mix", tensors=41, total=9_700_003, shape_seed=7, grad="bf16", store="bf16", probe=True,
              source="fisher", topk=5, input_sets=3),
        # step sizes per entry of the masked curvature, odd sizes
        _step("ragged_elementwise", "mix", tensors=29, total=37_000_019, shape_seed=11, probe=True, elementwise=True),
        # every layer changes its storage size on every step (a run whose gradient scale moves)
        _step("switch_50m", "wide", tensors=12, total=12 * 1024 * 4096, store="switch"),
        # 352 M parameters in three storage formats with scaled fp16 gradients
        _step("mixed_state_probe", "mixed_state", grad="fp16", store="mixed", probe=True, loss_scale=32768.0,
              warm=64),
        # 64 matrices of 4096 x 4096, the largest set: parameters half BF16, half FP32, a probe every step
        _step("large_probe", "square", tensors=64, total=64 * 4096 * 4096, store="mixed", probe=True, warm=64),
        # top-5 eigenvalues of every layer of the ResNet-18 set (k = 5 as in the paper)
        dict(name="power_resnet18_k5", kind="power", set="resnet18", tensors=0, total=0, shape_seed=0, k=5, entry="handle"),
    ]


def draw(rng):
    if rng.random() < 0.2:
        k = rng.randint(1, 8)
        total = int(math.exp(rng.uniform(math.log(300), math.log(2.4e8 / k))))
        tensors = rng.randint(1, min(120, max(1, total // 50)))
        return dict(kind="power", set="mix", tensors=tensors, total=total, shape_seed=rng.randrange(1 << 20), k=k,
                    entry=rng.choice(("handle", "static")))
    total = int(math.exp(rng.uniform(math.log(300), math.log(4e8))))
    tensors = rng.randint(1, min(220, max(1, total // 50)))
    grad = rng.choice(("fp32", "fp32", "bf16", "fp16"))
    probe = rng.random() < 0.6
    c = _step("", "mix", tensors=tensors, total=total, shape_seed=rng.randrange(1 << 20), grad=grad,
              store=rng.choice(("fp32", "bf16", "fp16")), probe=probe,
              source="fisher" if probe and rng.random() < 0.25 else "hutchinson",
              elementwise=probe and rng.random() < 0.2, topk=5 if probe and rng.random() < 0.2 else 0,
              loss_scale=1024.0 if grad == "fp16" else 1.0, read_result=grad == "fp16" and rng.random() < 0.5,
              warm=64 if probe and total > 50_000_000 else 0)
    del c["name"]
    return c


# ---- shapes ------------------------------------------------------------------------------------

def _numels(case):
    kind = case["set"]
    if kind == "mix":
        # sizes spread over several decades, as biases and weights are, none of them round
        r = random.Random(case["shape_seed"])
        w = [r.lognormvariate(0.0, 2.0) for _ in range(case["tensors"])]
        least = 16 if case["kind"] == "power" else 1  # fewer elements than vectors have no k directions
        return [max(least, int(case["total"] * x / sum(w))) for x in w]
    if kind in ("square", "wide"):
        return [case["total"] // case["tensors"]] * case["tensors"]
    make = {"tiny_mlp": _shapes.tiny_mlp_shapes, "resnet18": _shapes.resnet18_cifar_shapes,
            "efficientnet_b0": _shapes.efficientnet_b0_shapes, "mixed_state": _shapes.mixed_state_shapes}[kind]
    return [_shapes.numel(s) for _, s in make()]


def _stores(case, n):
    """Storage precision of every tensor at the first step's end."""
    if case["store"] == "mixed":
        if case["set"] == "mixed_state":
            return [("fp32", "bf16", "fp32", "bf16", "fp16")[i % 5] for i in range(n)]
        return [("bf16", "fp32")[i % 2] for i in range(n)]
    if case["store"] == "switch":
        return ["bf16"] * n
    return [case["store"]] * n


def _sigma(case, store, which):
    if case["store"] == "mixed":  # inside the variance bands below 1e-6, up to 1e-4, above
        return {"fp16": 3e-4, "bf16": 3e-3, "fp32": 3e-2}[store]
    if case["store"] == "switch":
        return (1e-3, 1e-1)[which % 2]
    return 1e-2


def _taus(case):
    if case["store"] == "mixed":
        return 1e-6, 1e-4
    return {"fp32": (0.0, 0.0), "bf16": (0.0, _HUGE), "fp16": (_HUGE, _HUGE), "switch": (0.0, 1e-4)}[case["store"]]


def _offsets(numels):
    offs, o = [], 0
    for n in numels:
        offs.append(o)
        o += -(-n // _PAD) * _PAD
    return offs, o


# ---- inputs ------------------------------------------------------------------------------------

def _generator(seed, *more):
    g = torch.Generator(device="cuda")
    x = seed & 0x7FFFFFFF
    for m in more:
        x = (x * 1_000_003 + m + 1) & 0x7FFFFFFFFFFF
    g.manual_seed(x)
    return g


def _step_inputs(case, seed):
    numels = _numels(case)
    stores = _stores(case, len(numels))
    offs, size = _offsets(numels)
    level = random.Random(seed * 31 + 5)
    d = [10.0 ** level.uniform(-5.0, 0.0) for _ in numels]  # curvature level of each layer
    s = dict(numels=numels, stores=stores, offs=offs, size=size, dev=torch.device("cuda"))
    g = _generator(seed, 1)
    first = "fp32" if case["store"] == "switch" else None
    s["init"] = [first or st for st in stores]
    # one parameter arena per storage precision; a tensor owns 4 bytes per element of it
    s["where"], fill = [], {}
    for st, n in zip(s["init"], numels):
        s["where"].append((st, fill.get(st, 0)))
        fill[st] = fill.get(st, 0) + -(-n // _PAD) * _PAD
    s["params"] = {st: torch.zeros(4 * n, dtype=torch.uint8, device="cuda") for st, n in fill.items()}
    for (st, o), n in zip(s["where"], numels):
        view = s["params"][st][4 * o:4 * (o + n)].view(_TORCH[st])[:n]
        view.normal_(0.0, 0.1, generator=g)
    s["mom"] = torch.zeros(size, device="cuda")
    for o, n in zip(offs, numels):
        s["mom"][o:o + n].normal_(0.0, 0.01, generator=g)
    s["curv"] = torch.zeros(size, device="cuda")
    s["mask"] = torch.zeros(size // 32, dtype=torch.int32, device="cuda")
    pairs = case["probe"] and case["source"] == "hutchinson"
    s["sets"] = []
    for which in range(case["input_sets"]):
        g = _generator(seed, 2, which)
        grad = torch.zeros(size, dtype=_TORCH[case["grad"]], device="cuda")
        for st, o, n in zip(stores, offs, numels):
            grad[o:o + n].normal_(0.0, _sigma(case, st, which) * case["loss_scale"], generator=g)
        z = hz = None
        if pairs:
            z = torch.empty(size, device="cuda").random_(0, 2, generator=g).mul_(2.0).sub_(1.0)
            hz = torch.zeros(size, device="cuda")
            for dl, o, n in zip(d, offs, numels):
                hz[o:o + n].normal_(0.0, math.sqrt(0.1 * dl), generator=g).add_(z[o:o + n], alpha=dl)
            hz.mul_(case["loss_scale"])
        s["sets"].append((grad, z, hz))
    return s


def _power_inputs(case, seed):
    numels = _numels(case)
    k, g = case["k"], _generator(seed, 3)
    us, hus = [], []
    for n in numels:
        stride = -(-n // 4) * 4
        u = torch.zeros(k, stride, device="cuda")
        u[:, :n].normal_(generator=g)
        # a product with a symmetric matrix: a positive diagonal plus a few directions that stand out
        a = torch.rand(n, generator=g, device="cuda") * 0.5
        v = torch.randn(min(6, n), n, generator=g, device="cuda") / math.sqrt(n)
        spikes = torch.tensor([8.0, 5.0, 3.0, 2.0, 1.25, 0.75], device="cuda")[:v.shape[0]]
        hu = torch.zeros_like(u)
        hu[:, :n] = u[:, :n] * a + ((u[:, :n] @ v.T) * spikes) @ v
        us.append(u)
        hus.append(hu)
    return numels, us, hus


class _Handle:
    """A library handle that is released with the state that owns it."""

    def __init__(self, raw):
        self.raw = raw

    def __del__(self):
        ta.triaccel_destroy(self.raw)


def _hyper(case, **more):
    lo, hi = _taus(case) if case["kind"] == "step" else (0.0, 0.0)
    return dict(beta_var=0.0 if case.get("store") == "switch" else 0.9, beta_curv=0.9, tau_low=lo, tau_high=hi, tau_curv=_HUGE,
                alpha=_ALPHA, sparsity_ppm=950000, momentum=_MU, weight_decay=_WD, ctrl_interval=1, scale_backoff=0.5,
                scale_growth=2.0, growth_interval=1 << 30, rho_low=0.7, rho_high=0.9, delta_up=16, delta_down=16, b_min=16,
                b_max=4096, **more)


def prepare(case, seed):
    if case["kind"] == "power":
        return _prepare_power(case, seed)
    s = _step_inputs(case, seed)
    s["tables"] = []
    for grad, z, hz in s["sets"]:
        arr = (ta.Tensor * len(s["numels"]))()
        for i, (n, o, (st, po)) in enumerate(zip(s["numels"], s["offs"], s["where"])):
            t = arr[i]
            t.param = s["params"][st].data_ptr() + 4 * po
            t.grad = grad.data_ptr() + grad.element_size() * o
            t.z = z.data_ptr() + 4 * o if z is not None else None
            t.hz = hz.data_ptr() + 4 * o if hz is not None else None
            t.curv = s["curv"].data_ptr() + 4 * o
            t.mom = s["mom"].data_ptr() + 4 * o
            t.mask = s["mask"].data_ptr() + o // 8
            t.numel, t.grad_dtype, t.param_dtype = n, _CODE[case["grad"]], _CODE[st]
        s["tables"].append(arr)
    cfg = ta.Config.from_hyper(_hyper(case, curvature_source=int(case["source"] == "fisher"),
                                      elementwise_scale=int(case["elementwise"]), topk_abs=case["topk"]))
    s["handle"] = _Handle(ta.triaccel_init(cfg, s["tables"][0], torch.cuda.current_stream().cuda_stream))
    s["case"], s["pass"] = case, 0
    if case["warm"]:
        # the parameters and momenta of the case itself are the drawn ones
        kept = {st: raw.clone() for st, raw in s["params"].items()}, s["mom"].clone()
        for _ in range(case["warm"]):
            run(s)
        for st, raw in kept[0].items():
            s["params"][st].copy_(raw)
        s["mom"].copy_(kept[1])
    return s


def _prepare_power(case, seed):
    numels, us, hus = _power_inputs(case, seed)
    n = len(numels)
    s = dict(case=case, numels=numels, us=us, hus=hus)
    s["vectors"] = (ta.PowerTensor * n)()
    for i in range(n):
        s["vectors"][i].u, s["vectors"][i].hu = us[i].data_ptr(), hus[i].data_ptr()
        s["vectors"][i].stride = us[i].shape[1]
    if case["entry"] == "static":
        s["info"] = torch.zeros(n, ctypes.sizeof(ta.PowerInfo) // 4, device="cuda")
        return s
    # the handle of the training loop whose layers these are; the iteration reads no tensor of its table
    arr = (ta.Tensor * n)()
    s["own"] = [torch.zeros(3, -(-m // _PAD) * _PAD, device="cuda") for m in numels]
    for t, own, m in zip(arr, s["own"], numels):
        t.param = t.grad = own[0].data_ptr()
        t.curv, t.mom, t.mask = own[1].data_ptr(), own[2].data_ptr(), own[1].data_ptr()
        t.numel, t.grad_dtype, t.param_dtype = m, ta.FP32, ta.FP32
    cfg = ta.Config.from_hyper(_hyper(case, power_k=case["k"]))
    s["handle"] = _Handle(ta.triaccel_init(cfg, arr, torch.cuda.current_stream().cuda_stream))
    return s


def run(state):
    case = state["case"]
    if case["kind"] == "power":
        if case["entry"] == "static":
            ta.triaccel_power_iter_static(state["vectors"], state["numels"], case["k"], state["info"].data_ptr(),
                                          torch.cuda.current_stream().cuda_stream)
            return {"u": _merged(state["us"]), "info": state["info"]}
        ta.triaccel_power_iter(state["handle"].raw, state["vectors"], case["k"], False)
        return {"u": _merged(state["us"])}
    which = state["pass"] % case["input_sets"]
    state["pass"] += 1
    ta.triaccel_step(state["handle"].raw, state["tables"][which], _LR, case["loss_scale"], 96, 800, 1000, case["probe"])
    out = {"mom": state["mom"]}
    if case["probe"]:
        out["curv"], out["mask"] = state["curv"], state["mask"]
    if case["store"] == "switch":
        kind = _TORCH[("bf16", "fp32")[which]]
        out["params"] = [state["params"][st][4 * o:4 * (o + n)].view(kind)[:n] for (st, o), n in zip(state["where"], state["numels"])]
    else:
        out["params"] = {st: raw.view(_TORCH[st]) for st, raw in state["params"].items()}
    if case["read_result"]:
        res = ta.triaccel_result(state["handle"].raw)
        out["skipped"], out["next_scale"], out["next_batch"] = res.skipped, res.next_loss_scale, res.next_batch_size
    return out


def _merged(us):
    """At most 64 outputs: all vectors of the largest layers, the first of them up to 60."""
    order = sorted(range(len(us)), key=lambda i: -us[i].numel())[:60]
    return [us[i] for i in sorted(order)]


# ---- what the path cannot do without ------------------------------------------------------------

def work(case):
    numels = _numels(case)
    if case["kind"] == "power":
        k, n = case["k"], sum(numels)
        return {"bytes": 12.0 * k * n, "flops": 2.0 * n * (k * (k + 1) + 2 * k)}
    total = 0.0
    for n, st in zip(numels, _stores(case, len(numels))):
        store = 6 if case["store"] == "switch" else 2 * _BYTES[st]
        b = _BYTES[case["grad"]] + store + 8
        if case["probe"]:
            b += 8 + 0.125 + (8 if case["source"] == "hutchinson" else 0)
        total += float(b) * n
    per = 8 + (6 if case["probe"] else 0) + (4 if case["elementwise"] else 0)
    return {"bytes": total, "flops": float(per) * sum(numels)}


def tolerance(case):
    if case["kind"] == "power":
        # fp64 sums rounded once to fp32; a vector's direction error grows with the square of its
        # conditioning, the residual is formed from sums that cancel
        return {"rel": 1e-6, "max": 1e-5}
    if case["store"] == "fp32":
        # fp32 element-wise operations in another order: 4.3e-8 (largest: 2.4e-7) off 64 bits after one
        # step, and a little more in a curvature average of many steps
        return {"rel": 3e-7, "max": 2e-6, "differ": 1e-5}
    # a stored 16-bit value next to a rounding boundary may fall the other way: one unit (2^-7 of it at
    # most) in few elements, 2.4e-6 over all of them against the rounded 64-bit values
    return {"rel": 1e-5, "max": 1e-2, "differ": 1e-5}


# ---- the first pass on new inputs, in 64 bits -----------------------------------------------------

def exact(case, seed):
    if case["kind"] == "power":
        return _exact_power(case, seed)
    s = _step_inputs(case, seed)
    inv = 1.0 / case["loss_scale"]
    weight = [0.0] * case["input_sets"]  # of each input set in the curvature average after the case's pass
    for t in range(case["warm"] + 1):
        weight = [w * 0.9 if t else 0.0 for w in weight]
        weight[t % case["input_sets"]] += 0.1 if t else 1.0
    grad = s["sets"][case["warm"] % case["input_sets"]][0]
    mom = torch.zeros(s["size"], dtype=torch.float64, device="cuda")
    curv = torch.zeros_like(mom) if case["probe"] else None
    switch = case["store"] == "switch"
    out = {} if not switch else []
    if not switch:
        for st, raw in s["params"].items():
            out[st] = torch.zeros(raw.numel() // _BYTES[st], dtype=torch.float64, device="cuda")
    hyper = _hyper(case)
    for n, o, (st, po) in zip(s["numels"], s["offs"], s["where"]):
        x = grad[o:o + n].double() * inv
        theta = s["params"][st][4 * po:4 * (po + n)].view(_TORCH[st])[:n].double()
        lam, eta = 0.0, _LR
        if case["probe"]:
            h = curv[o:o + n]
            for w, (gs, zs, hzs) in zip(weight, s["sets"]):
                if w:
                    u = (gs[o:o + n].double() * inv).square() if case["source"] == "fisher" else zs[o:o + n].double() * hzs[o:o + n] * inv
                    h += w * u
            mag = h.abs()
            lam = float(mag.max())
            if case["elementwise"]:
                k = case["topk"] or n - n * hyper["sparsity_ppm"] // 1_000_000
                k = min(max(k, 1), n)
                kth = torch.topk(mag, k).values[-1]
                eta = _LR / (1.0 + _ALPHA * torch.where((mag >= kth) & (mag > 0), mag, torch.zeros_like(mag)))
            else:
                eta = _LR / (1.0 + _ALPHA * lam)
        m = _MU * s["mom"][o:o + n].double() + (_WD * theta + x)
        mom[o:o + n] = m
        theta = theta - eta * m
        if switch:
            out.append(theta)
        else:
            at = po * 4 // _BYTES[st]
            out[st][at:at + n] = theta
    got = {"mom": mom, "params": out}
    if case["probe"]:
        got["curv"], got["mask"] = curv, None
    if case["read_result"]:
        got["skipped"] = got["next_scale"] = got["next_batch"] = None
    return got


def _exact_power(case, seed):
    numels, us, hus = _power_inputs(case, seed)
    k, new, info = case["k"], [], torch.zeros(len(numels), 27, dtype=torch.float64, device="cuda")
    for i, (n, u, hu) in enumerate(zip(numels, us, hus)):
        w, uu = hu[:, :n].double(), u[:, :n].double()
        q = torch.zeros(k, u.shape[1], dtype=torch.float64, device="cuda")
        kept = []
        for j in range(k):  # ordered Gram-Schmidt, twice over
            v = w[j].clone()
            for _ in range(2):
                for p in kept:
                    v -= (p @ v) * p
            norm = float(v.norm())
            if norm <= 1e-6 * float(w[j].norm()):
                continue
            q[j, :n] = v / norm
            kept.append(q[j, :n])
        new.append(q)
        c, d = (uu * w).sum(1), (uu * uu).sum(1)
        ray = c / d
        info[i, 0:k] = ray
        info[i, 8:8 + k] = (w - ray[:, None] * uu).norm(dim=1) / d.sqrt()
        info[i, 16:16 + k] = w.norm(dim=1)
        info[i, 25] = ray.abs().max()
    got = {"u": _merged(new)}
    if case["entry"] == "static":
        got["info"] = info
    return got
