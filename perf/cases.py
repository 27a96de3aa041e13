"""The optimizer calls that a training program makes, as timed cases.

A case names one call of ``MtdaoOptimizer`` over K worker replicas of P
parameters:

    call   "step"       local step, nothing averaged (most steps of a run)
           "step_sync"  local step and averaging of ``mask`` in one call
           "sync"       averaging alone
           "stats"      averaging with its diagnostics (waits for them)
           "window"     one replay of a captured HIP graph of 16 steps whose
                        update number lives on the device
    form   "adam" / "adopt" / "sgdm"; n first moments; x, g storage types
    clip   global-norm clipping (rho = 1); prob: momenta averaged inside the
           step (Algorithm 4); outer: Nesterov OuterOpt on x
    mask   states averaged: "none", "x", "all"

All states are those of a run resumed in its middle: parameters that differ
a little between the workers, moments of the size that gradients of one
standard deviation leave, and update numbers above 1000.
"""

import math

import numpy as np
import torch

from paper_2510_05361_amd import mtdao as abi
from paper_2510_05361_amd.optimizer import MtdaoOptimizer

_DTYPE = {"f32": torch.float32, "bf16": torch.bfloat16}
_BYTES = {"f32": 4, "bf16": 2}
_BETA1 = (0.9, 0.99, 0.999)
_OMEGA = {1: (0.9,), 2: (0.3, 0.6), 3: (0.3, 0.3, 0.3)}
_BETA2, _EPS, _LR, _RHO = 0.999, 1e-8, 1e-3, 1.0
_OUTER_LR, _OUTER_MU = 0.7, 0.9
_G_STD = 1e-3
_START = 1008           # updates already applied; a multiple of the window
_WINDOW = 16            # steps of a captured window
_PERIODS = (4, 8, 16)   # of x, of the first moments, of v
_TABLE = 4096           # entries of the learning-rate table

_DEFAULTS = {"call": "step", "form": "adam", "n": 3, "k": 4, "x": "f32", "g": "f32", "clip": False,
             "prob": False, "outer": False, "mask": "none"}


def _case(**kw):
    return {**_DEFAULTS, **kw}


def listed():
    return [
        # a small model's step: launch latency and the host path
        _case(name="adam_k2_58k_step", n=2, k=2, p=58_296),
        # the 1M workload as a captured window of 16 steps with their averaging
        _case(name="adam_k2_1m_window", call="window", n=2, k=2, p=1_048_576),
        # 16.8M transformer, four workers: the plain step
        _case(name="adam_k4_16m_step", p=16_785_920),
        # the same with a ragged tail tensor, x due
        _case(name="adam_k4_16m_ragged_x", call="step_sync", p=16_785_957, mask="x"),
        # averaging with its diagnostics, every state due
        _case(name="adam_k4_16m_stats", call="stats", p=16_785_920, mask="all"),
        # sixteen workers with averaged momenta inside the step (Algorithm 4)
        _case(name="sgdm_k16_16m_prob", call="step_sync", form="sgdm", n=2, k=16, p=16_785_920, prob=True, mask="all"),
        # bf16 parameters and gradients, eight workers, ragged length: the plain step
        _case(name="adopt_k8_16m_bf16_ragged", form="adopt", n=2, k=8, p=16_785_957, x="bf16", g="bf16"),
        # 124M GPT, bf16: the plain step, and the averaging of every state alone
        _case(name="adopt_k8_124m_bf16_step", form="adopt", n=2, k=8, p=123_605_760, x="bf16", g="bf16"),
        _case(name="adopt_k8_124m_bf16_sync", call="sync", form="adopt", n=2, k=8, p=123_605_760, x="bf16", g="bf16",
              mask="all"),
        # 124M GPT under the Nesterov OuterOpt: the step at which x restarts
        _case(name="adam_k4_124m_outer_x", call="step_sync", p=123_605_760, outer=True, mask="x"),
        # sixteen workers with global-norm clipping, every state due
        _case(name="sgdm_k16_124m_clip_all", call="step_sync", form="sgdm", n=2, k=16, p=123_605_760, clip=True,
              mask="all"),
        # 354M GPT, four workers: the step at which every state is due
        _case(name="adam_k4_354m_all", call="step_sync", p=353_600_512, mask="all"),
    ]


def _step_bytes(c):
    """Bytes of one update of one element of one replica."""
    return 2 * _BYTES[c["x"]] + _BYTES[c["g"]] + 8 * c["n"] + (8 if c["form"] != "sgdm" else 0)


def work(case):
    c = case
    kp = c["k"] * c["p"]
    outer = 16 * c["p"] if c["outer"] and c["mask"] != "none" else 0
    if c["call"] in ("sync", "stats"):
        words = 4 * (c["n"] + (1 if c["form"] != "sgdm" else 0)) if c["mask"] == "all" else 0
        return {"bytes": 2 * kp * (_BYTES[c["x"]] + words) + outer, "flops": kp * 4}
    steps = _WINDOW if c["call"] == "window" else 1
    return {"bytes": steps * (kp * _step_bytes(c) + outer), "flops": steps * kp * (8 + 4 * c["n"])}


def draw(rng):
    big = work(listed()[-1])["bytes"]
    c = dict(_DEFAULTS)
    c["call"] = rng.choice(("step", "step", "step", "step_sync", "step_sync", "step_sync", "sync", "stats", "window"))
    c["form"] = rng.choice(("adam", "adam", "adopt", "sgdm"))
    c["n"] = rng.choice((1, 2, 2, 3, 3))
    c["k"] = rng.choice((1, 2, 3, 4, 4, 5, 6, 8, 8, 12, 16, 16, 24, 32))
    c["x"], c["g"] = rng.choice((("f32", "f32"), ("f32", "f32"), ("bf16", "bf16"), ("f32", "bf16")))
    c["clip"] = c["form"] != "adopt" and rng.random() < 0.5
    if c["call"] == "step_sync":
        c["mask"] = rng.choice(("x", "all"))
        if c["form"] == "sgdm" and rng.random() < 0.4:
            c["prob"], c["mask"] = True, "all"
        elif rng.random() < 0.3:
            c["outer"] = True
    elif c["call"] in ("sync", "stats"):
        c["mask"] = rng.choice(("x", "all"))
        c["k"] = rng.choice((2, 3, 4, 6, 8, 12, 16)) if c["call"] == "stats" else max(2, c["k"])
    most = 350_000_000
    while True:
        p = int(math.exp(rng.uniform(math.log(50_000), math.log(most))))
        # half the lengths are those of whole tensors of some width, half are ragged
        c["p"] = p if rng.random() < 0.5 else max(512, p // 512 * 512)
        if work(c)["bytes"] <= big and c["k"] * c["p"] <= 1_400_000_000:
            return c
        most = max(60_000, most // 2)


def _masks(c):
    bits = 1 + c["n"] + (1 if c["form"] != "sgdm" else 0)
    return {"none": 0, "x": 1, "all": (1 << bits) - 1}[c["mask"]]


def _fill(c, seed, x, g, u, v, outer):
    """The inputs of ``seed`` into the given [K][P] (outer: [P]) tensors."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    base = torch.empty(c["p"], dtype=torch.float32, device="cuda").normal_(0.0, 0.02, generator=gen)
    row = torch.empty_like(base)
    for m in range(c["k"]):
        x[m].copy_(row.normal_(0.0, 1e-3, generator=gen).add_(base))
    g.normal_(0.0, _G_STD, generator=gen)
    for b, a in zip(_BETA1, u):
        a.normal_(0.0, _G_STD * math.sqrt((1 - b) / (1 + b)), generator=gen)
    if v is not None:
        v.uniform_(0.5 * _G_STD ** 2, 1.5 * _G_STD ** 2, generator=gen)
    if outer is not None:
        outer[0].copy_(base)
        outer[1].normal_(0.0, 1e-3, generator=gen)


def _lr_table():
    return _LR * (0.5 + 0.5 * torch.cos(torch.arange(_TABLE, dtype=torch.float64) * (math.pi / _TABLE)))


def _adopt_clip(c):
    return float(np.float32(_START ** 0.25)) if c["form"] == "adopt" else 0.0


def prepare(case, seed):
    c = case
    px, pu, pv = _PERIODS
    cfg = abi.make_config(c["form"], c["k"], _BETA1[:c["n"]], _OMEGA[c["n"]], c["p"], beta2=_BETA2, eps=_EPS,
                          clip_rho=_RHO if c["clip"] else 0.0, param_dtype=c["x"], grad_dtype=c["g"],
                          period_x=px, period_u=(pu,) * c["n"], period_v=pv, start_step=_START,
                          sync_order=abi.MTDAO_SYNC_MOMENTA_IN_STEP if c["prob"] else abi.MTDAO_SYNC_AFTER_STEP,
                          outer_opt=abi.MTDAO_OUTER_NESTEROV if c["outer"] else abi.MTDAO_OUTER_AVERAGE,
                          outer_lr=_OUTER_LR, outer_momentum=_OUTER_MU)
    opt = MtdaoOptimizer(cfg, torch.device("cuda"), grad_buffer=True)
    _fill(c, seed, opt.x, opt.grad, opt.u, opt.v, (opt.x_outer, opt.x_outer_mom) if c["outer"] else None)
    state = {"call": c["call"], "opt": opt, "mask": _masks(c), "clip": _adopt_clip(c)}
    if c["call"] == "window":
        lr = _lr_table().float().cuda()
        ct = torch.full((_TABLE,), state["clip"], dtype=torch.float32, device="cuda") if c["form"] == "adopt" else None
        opt.device_step(lr, ct)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            for _ in range(_WINDOW):
                opt.step_sync_device(opt.grad)
            opt.device_step_advance()
        state["graph"] = graph
    return state


def run(state):
    opt, call = state["opt"], state["call"]
    out = {}
    if call == "step":
        opt.step(opt.grad, _LR, state["clip"])
    elif call == "step_sync":
        opt.step_sync(opt.grad, _LR, state["clip"], state["mask"])
    elif call == "sync":
        opt.sync(state["mask"])
    elif call == "stats":
        out["stats"] = list(opt.sync_stats(state["mask"])[1])
    else:
        state["graph"].replay()
    out["x"], out["u"] = opt.x, list(opt.u)
    if opt.v is not None:
        out["v"] = opt.v
    if opt.x_outer is not None:
        out["x_outer"], out["x_outer_mom"] = opt.x_outer, opt.x_outer_mom
    return out


def tolerance(case):
    # About four times the largest distance to 64 bits seen: 1e-7 for fp32
    # states (5.7e-7 for the outer momentum, a difference of parameters),
    # 1.7e-3 for bf16 parameters, which may round to their other neighbour.
    if case["x"] == "bf16":
        return {"rel": 7e-3, "max": 2e-2}
    return {"rel": 2.5e-6 if case["outer"] else 4e-7, "max": 1e-5}


# ------------------------------------------------------------- in 64 bits


def _mean(rows):
    return rows.mean(0, keepdim=True).expand_as(rows).clone()


def _update(c, s, lr, scale, x, g, u, v, outer, mask):
    """One update of [K][columns] fp64 values in place."""
    f32 = lambda a: float(np.float32(a))  # noqa: E731  hyper-parameters are fp32 values
    beta = [f32(b) for b in _BETA1[:c["n"]]]
    omega = [f32(w) for w in _OMEGA[c["n"]]]
    b2, eps = f32(_BETA2), f32(_EPS)
    due = lambda j: (mask >> j) & 1  # noqa: E731
    gh = g * scale[:, None] if scale is not None else g
    if c["form"] == "adopt":
        gh = g / (v.sqrt() + eps)
        v.mul_(b2).add_(g * g, alpha=1 - b2)
        gh = gh.clamp(-_adopt_clip(c), _adopt_clip(c))
    num = gh * (1 - sum(omega))
    for j in range(c["n"]):
        u[j].mul_(beta[j]).add_(gh, alpha=1 - beta[j])
        if c["prob"] and due(j + 1):
            u[j].copy_(_mean(u[j]))
        num += u[j] * (omega[j] / (1 - beta[j] ** s) if c["form"] == "adam" else omega[j])
    if c["form"] == "adam":
        v.mul_(b2).add_(gh * gh, alpha=1 - b2)
        num = num / ((v / (1 - b2 ** s)).sqrt() + eps)
    x.sub_(num, alpha=f32(lr))
    _average(c, x, u, v, outer, mask & 1 if c["prob"] else mask)


def _average(c, x, u, v, outer, mask):
    if mask & 1:
        if outer is not None:
            lr, mu = float(np.float32(_OUTER_LR)), float(np.float32(_OUTER_MU))
            xo, mom = outer
            d = xo - x.mean(0)
            mom.mul_(mu).add_(d)
            xo.sub_(lr * (d + mu * mom))
            x.copy_(xo[None].expand_as(x))
        else:
            x.copy_(_mean(x))
    for j in range(c["n"]):
        if (mask >> (j + 1)) & 1:
            u[j].copy_(_mean(u[j]))
    if v is not None and (mask >> (c["n"] + 1)) & 1:
        v.copy_(_mean(v))


def _stats_into(total, row, a):
    """Diagnostics sums of the [K][columns] values a, added to total[row]."""
    K = a.shape[0]
    mean = a.mean(0)
    total[row, abi.MTDAO_STAT_MEAN_SQ] += float((mean * mean).sum())
    total[row, abi.MTDAO_STAT_VARIANCE] += float(((a - mean) ** 2).sum()) / K
    for m in range(K):
        total[row, abi.MTDAO_STAT_WORKER_SQ + m] += float((a[m] * a[m]).sum())
        total[row, abi.MTDAO_STAT_WORKER_DOT + m] += float((a[m] * mean).sum())


def exact(case, seed):
    c = case
    K, P = c["k"], c["p"]
    has_v = c["form"] != "sgdm"
    x = torch.empty((K, P), dtype=_DTYPE[c["x"]], device="cuda")
    g = torch.empty((K, P), dtype=_DTYPE[c["g"]], device="cuda")
    u = [torch.empty((K, P), device="cuda") for _ in range(c["n"])]
    v = torch.empty((K, P), device="cuda") if has_v else None
    outer = [torch.empty(P, device="cuda") for _ in range(2)] if c["outer"] else None
    _fill(c, seed, x, g, u, v, outer)
    mask = _masks(c)
    scale = None
    if c["clip"] and c["call"] in ("step", "step_sync", "window"):
        norm = torch.zeros(K, dtype=torch.float64, device="cuda")
        for m in range(K):
            for part in g[m].split(1 << 24):
                norm[m] += part.double().square().sum()
        scale = (_RHO / norm.sqrt()).clamp(max=1.0)
    stats = np.full((abi.MTDAO_MAX_N + 2, abi.MTDAO_STATS_STRIDE), np.nan)
    ids = [k for k in range(2 + c["n"]) if (mask >> k) & 1]
    stats[ids] = 0.0
    lrs = _lr_table().float().tolist()
    made = [torch.empty((K, P), dtype=torch.float64, device="cuda") for _ in range(1 + c["n"] + has_v)]
    made_outer = [torch.empty(P, dtype=torch.float64, device="cuda") for _ in range(2)] if outer else None
    cols = max(1, (1 << 26) // K)
    for at in range(0, P, cols):
        cut = slice(at, min(P, at + cols))
        xs, gs = x[:, cut].double(), g[:, cut].double()
        us = [a[:, cut].double() for a in u]
        vs = v[:, cut].double() if has_v else None
        os = [a[cut].double() for a in outer] if outer else None
        if c["call"] in ("sync", "stats"):
            if c["call"] == "stats":
                for k, a in zip(range(2 + c["n"]), [xs] + us + ([vs] if has_v else [])):
                    if (mask >> k) & 1:
                        _stats_into(stats, k, a)
            _average(c, xs, us, vs, os, mask)
        elif c["call"] == "window":
            periods = (_PERIODS[0],) + (_PERIODS[1],) * c["n"] + ((_PERIODS[2],) if has_v else ())
            for s in range(_START + 1, _START + _WINDOW + 1):
                due = sum(1 << k for k, h in enumerate(periods) if s % h == 0)
                _update(c, s, lrs[s - 1], scale, xs, gs, us, vs, os, due)
                if c["x"] == "bf16":  # the parameters stored between the steps
                    xs = xs.bfloat16().double()
        else:
            _update(c, _START + 1, _LR, scale, xs, gs, us, vs, os, mask if c["call"] == "step_sync" else 0)
        for to, a in zip(made, [xs] + us + ([vs] if has_v else [])):
            to[:, cut] = a
        for to, a in zip(made_outer or [], os or []):
            to[cut] = a
    out = {"x": made[0], "u": made[1:1 + c["n"]]}
    if has_v:
        out["v"] = made[-1]
    if outer:
        out["x_outer"], out["x_outer_mom"] = made_outer
    if c["call"] == "stats":
        out["stats"] = list(stats)
    return out
