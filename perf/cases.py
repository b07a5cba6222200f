"""What a user of the framework has it do, as cases whose time is measured.

A case names a training graph (the ``model`` of ``workloads``, with its
workers or devices), a scenario count and a call; ``prepare`` makes the graph
and the inputs a program holds before the call, ``run`` makes the call,
``exact`` replays it in plain torch with 64-bit integers.  Results are whole
numbers with one right value, so every tolerance is "exact".
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

import paper_2002_06790_amd as mlsim
from paper_2002_06790_amd import workloads

#: relative spread of an op's duration around its profile (the workloads' 1 %)
SIGMA = 0.01


def listed():
    return [
        # the smallest call: one small model, a few profiled variations of it
        {"name": "mlp run 100", "model": "mlp", "workers": 2, "call": "run", "scen": 100, "finish": True},
        # an ordinary question about one ring all-reduce configuration (odd count)
        {"name": "inception run 4099", "model": "inception", "workers": 4, "call": "run", "scen": 4099, "finish": True},
        # the full sweeps of the benchmark's graphs, every op's finish time wanted
        {"name": "inception run 65536", "model": "inception", "workers": 4, "call": "run", "scen": 65536, "finish": True},
        {"name": "resnet run 65536", "model": "resnet", "workers": 8, "call": "run", "scen": 65536, "finish": True},
        {"name": "bert run 262144", "model": "bert", "workers": 16, "call": "run", "scen": 262144, "finish": True},
        # placements searched at random: every scenario puts every op elsewhere
        {"name": "random place 16384", "model": "random", "workers": 64, "call": "run", "scen": 16384, "finish": True},
        # what launch gaps and copies cost, iteration time only
        {"name": "bert device 20000", "model": "bert", "workers": 16, "call": "device", "scen": 20000, "finish": False},
        # strategy grid: durations drawn in the kernel, iteration time only
        {"name": "bert generated 262144", "model": "bert", "workers": 16, "call": "generated", "scen": 262144, "finish": False},
        # the bound with unlimited devices
        {"name": "bert critical 262144", "model": "bert", "workers": 16, "call": "critical", "scen": 262144, "finish": False},
        # a fixed launch order per device
        {"name": "resnet static 65536", "model": "resnet", "workers": 8, "call": "static", "scen": 65536, "finish": True},
        # transfers dividing their link's bandwidth
        {"name": "bert share 32768", "model": "bert", "workers": 16, "call": "share", "scen": 32768, "finish": False},
        # where the time goes: busy time and binding chain of every device
        {"name": "resnet attribute 16384", "model": "resnet", "workers": 8, "call": "attribute", "scen": 16384, "finish": True},
    ]


# per model: worker (or device, or resource) counts, and the scenario counts of
# its calls; a share call takes the same range divided by four
_RANGE = {"mlp": ((2, 2), (1, 100000)), "inception": ((2, 8), (64, 65536)), "resnet": ((2, 12), (64, 65536)),
          "bert": ((2, 16), (64, 262144)), "random": ((8, 96), (64, 8192))}


def draw(rng):
    model = rng.choice(["mlp", "inception", "resnet", "resnet", "bert", "bert", "random"])
    calls = ["run", "run", "run", "device", "generated", "critical", "static", "attribute"]
    if model in ("mlp", "bert"):
        calls.append("share")  # at most 64 transfers of one link are in flight there
    call = rng.choice(calls)
    (w0, w1), (s0, s1) = _RANGE[model]
    if call == "share":
        s1 //= 4
    if call == "attribute":
        s1 //= 2
    scen = int(round(math.exp(rng.uniform(math.log(s0), math.log(s1)))))
    case = {"model": model, "workers": rng.randint(w0, w1), "call": call, "scen": max(1, min(s1, scen + rng.randint(-3, 3))),
            "finish": call == "attribute" or (call in ("run", "static", "device", "generated") and rng.random() < 0.6)}
    if call in ("run", "device") and rng.random() < 0.25:
        case["prio"] = True  # the caller orders simultaneous arrivals itself
    return case


@functools.lru_cache(maxsize=64)
def _workload(model, workers):
    if model == "mlp":
        return workloads.tiny_dp_mlp()
    if model == "resnet":
        return workloads.resnet50_ps(workers=workers)
    if model == "inception":
        return workloads.inception_v3_ring(devices=workers)
    if model == "bert":
        return workloads.bert_large_ps(workers=workers)
    return workloads.random_layered(n_res=workers)


def _prio(case, w):
    """Later ops first among simultaneous arrivals, or None."""
    return -np.arange(w.n_ops, dtype=np.int32) if case.get("prio") else None


def _device_model(w):
    """Idle ns after each op (5 us on the first quarter of the resources, 2 us
    on the others), and 10 us until a transfer's outputs arrive."""
    gap = np.full(w.n_res, 2_000, np.int32)
    gap[: max(1, w.n_res // 4)] = 5_000
    delay = np.zeros(w.n_res, np.int32)
    delay[workloads.link_resources(w)] = 10_000
    return gap, delay


def _base(w):
    return torch.from_numpy(w.gen_base()).cuda()


def _durations(w, scen, seed):
    """int32 [n_ops, scen]: each op's profile (of the scenario's strategy) times
    lognormal noise; for the random graph log-uniform in [1 us, 10 ms]."""
    gen = torch.Generator(device="cuda").manual_seed(1 + seed)
    dur = torch.empty((w.n_ops, scen), dtype=torch.int32, device="cuda")
    base = _base(w).float()
    knob = (torch.arange(scen, device="cuda") // w.knob_block) % base.shape[0]
    step = max(1, (1 << 28) // max(scen, 1))  # rows at a time: a gigabyte of noise
    for v in range(0, w.n_ops, step):
        shape = (min(step, w.n_ops - v), scen)
        if w.name.startswith("random"):
            x = torch.rand(shape, generator=gen, device="cuda").mul_(math.log(1e4)).exp_().mul_(1e3)
        else:
            x = torch.randn(shape, generator=gen, device="cuda").mul_(SIGMA).exp_()
            rows = base[:, v:v + shape[0]]
            x.mul_(rows[0][:, None] if len(base) == 1 else rows.t()[:, knob])
        dur[v:v + shape[0]] = x.round_().clamp_(min=1.0).to(torch.int32)
    return dur


def _placement(w, scen, seed):
    gen = torch.Generator(device="cuda").manual_seed(2 + seed)
    return torch.randint(0, w.n_res, (w.n_ops, scen), generator=gen, device="cuda", dtype=torch.int32).to(torch.uint16)


def _placed(case):
    return case["model"] == "random" and case["call"] in ("run", "device", "attribute")


def prepare(case, seed):
    w, scen, call = _workload(case["model"], case["workers"]), case["scen"], case["call"]
    s = {"case": case, "graph": mlsim.Graph(w.succ_ptr, w.succ_idx, w.op_res, w.n_res, prio=_prio(case, w)),
         "makespan": torch.empty(scen, dtype=torch.int32, device="cuda"),
         "status": torch.empty(scen, dtype=torch.int32, device="cuda"), "finish": None}
    if case["finish"] and call != "attribute":
        s["finish"] = torch.empty((w.n_ops, scen), dtype=torch.int32, device="cuda")
    if call == "generated":
        s["gen"] = mlsim.Gen(_base(w), knob_block=w.knob_block, noise=mlsim.noise_for_sigma(SIGMA), seed=1 + seed)
    else:
        s["dur"] = _durations(w, scen, seed)
    s["place"] = _placement(w, scen, seed) if _placed(case) else None
    if call == "device":
        s["gap"], s["delay"] = _device_model(w)
    if call == "share":
        s["share"] = np.zeros(w.n_res, np.uint8)
        s["share"][workloads.link_resources(w)] = 1
    if call == "static":
        s["replay"] = s["graph"].static_order(np.arange(w.n_ops, dtype=np.int32))
    return s


def run(s):
    case, g = s["case"], s["graph"]
    call, out = case["call"], {"makespan": s["makespan"], "status": s["status"], "finish": s["finish"]}
    if call == "run":
        r = g.run(s["dur"], place=s["place"], **out)
    elif call == "device":
        r = g.run(s["dur"], place=s["place"], gap=s["gap"], delay=s["delay"], **out)
    elif call == "generated":
        r = g.run_generated(s["gen"], case["scen"], **out)
    elif call == "share":
        r = g.run_share(s["dur"], s["share"], **out)
    elif call == "static":
        r = s["replay"].run(s["dur"], **out)
    elif call == "critical":
        return {"critical": g.critical_path(s["dur"], cp_len=s["makespan"])[0]}
    else:
        r = g.attribute(s["dur"], place=s["place"])
        return {k: r[k] for k in ("makespan", "status", "finish", "prev", "busy", "chain", "chain_ops")}
    return {k: v for k, v in zip(("makespan", "finish", "status"), r) if v is not None}


def work(case):
    """Each duration (and placement) read once, each result written once."""
    w, S, call = _workload(case["model"], case["workers"]), case["scen"], case["call"]
    events = w.n_ops * S
    b = 0 if call == "generated" else 4 * events
    b += 2 * events if _placed(case) else 0
    b += 4 * S if call == "critical" else 8 * S
    if call == "attribute":
        b += 8 * events + 8 * w.n_res * S + 4 * S
    elif case["finish"]:
        b += 4 * events
    # integer operations: one max and one add per event, and the generator's
    # ten rounds (two products and four exclusive ors each) and its sum
    return {"bytes": b, "flops": events * (2 + (80 if call == "generated" else 0))}


def tolerance(case):
    return "exact"  # integer nanoseconds with one right value


# -- the same results in plain torch -----------------------------------------

def _philox_durations(w, scen, seed):
    """The generator's documented integers, for every op and scenario."""
    m = 0xFFFFFFFF
    s = torch.arange(scen, device="cuda")
    v = torch.arange(w.n_ops, device="cuda")
    zero = torch.zeros((w.n_ops, scen), dtype=torch.int64, device="cuda")
    x = [s[None, :] + zero, zero, v[:, None] + zero, zero]
    k0, k1 = (1 + seed) & m, (1 + seed) >> 32

    def product(a, b):  # the 32-bit halves of a 32 x 32-bit product
        lo, hi = a * (b & 0xFFFF), a * (b >> 16)
        mid = (lo >> 16) + hi
        return (mid >> 16) & m, ((mid << 16) | (lo & 0xFFFF)) & m

    for _ in range(10):
        h0, l0 = product(x[0], 0xD2511F53)
        h1, l1 = product(x[2], 0xCD9E8D57)
        x = [h1 ^ x[1] ^ k0, l1, h0 ^ x[3] ^ k1, l0]
        k0, k1 = (k0 + 0x9E3779B9) & m, (k1 + 0xBB67AE85) & m
    t = 2 * sum((y & 0xFFFF) + (y >> 16) for y in x) - 524280
    base = _base(w).long()
    b = base[(s // w.knob_block) % base.shape[0]].t()
    return b + ((b * t * mlsim.noise_for_sigma(SIGMA) + (1 << 39)) >> 40)


def _predecessors(w):
    pred = [[] for _ in range(w.n_ops)]
    for u in range(w.n_ops):
        for v in w.succ_idx[w.succ_ptr[u]:w.succ_ptr[u + 1]]:
            pred[int(v)].append(u)
    return pred


def _sweep(w, dur, pred):
    """Finish times (ids are a topological order) when an op starts at its
    latest predecessor's finish."""
    fin = dur.long()
    for v in range(w.n_ops):
        if pred[v]:
            fin[v] += fin[pred[v]].max(dim=0).values
    return fin


def _replay(w, dur, place, gap, delay, prio):
    """First in first out by (ready, priority, id): each step pops every
    scenario's smallest waiting key and releases the popped op's successors."""
    n, S = dur.shape
    dev = dur.device
    rank = torch.arange(n, device=dev)  # of (priority, id)
    if prio is not None:
        rank[torch.from_numpy(np.argsort(prio, kind="stable")).to(dev)] = torch.arange(n, device=dev)
    deg = np.bincount(w.succ_idx, minlength=n)
    fan = max(1, int(np.diff(w.succ_ptr).max()))
    table = np.full((n + 1, fan), n, np.int64)  # n: no successor
    for u in range(n):
        e = w.succ_idx[w.succ_ptr[u]:w.succ_ptr[u + 1]]
        table[u, :len(e)] = e
    table = torch.from_numpy(table).to(dev)
    left = torch.from_numpy(np.append(deg, 1 << 30)).to(dev)[:, None].repeat(1, S)
    ready = torch.zeros((n + 1, S), dtype=torch.int64, device=dev)
    never = 1 << 62
    key = torch.where((left[:n] == 0), rank[:, None], never)
    free = torch.zeros((w.n_res, S), dtype=torch.int64, device=dev)
    fin = torch.zeros((n, S), dtype=torch.int64, device=dev)
    res = torch.from_numpy(w.op_res.astype(np.int64)).to(dev)
    gap = torch.from_numpy(gap.astype(np.int64)).to(dev) if gap is not None else None
    delay = torch.from_numpy(delay.astype(np.int64)).to(dev) if delay is not None else None
    rank = torch.cat([rank, rank.new_zeros(1)])
    for _ in range(n):
        k, v = key.min(dim=0, keepdim=True)
        key.scatter_(0, v, never)
        r = place.gather(0, v).long() if place is not None else res[v]
        f = torch.maximum(k >> 24, free.gather(0, r)) + dur.gather(0, v)
        fin.scatter_(0, v, f)
        free.scatter_(0, r, f if gap is None else f + gap[r])
        out = f if delay is None else f + delay[r]
        for j in range(fan):
            x = table[:, j][v]
            left.scatter_add_(0, x, torch.full_like(x, -1))
            t = torch.maximum(ready.gather(0, x), out)
            ready.scatter_(0, x, t)
            go = (left.gather(0, x) == 0)
            y = x.clamp(max=n - 1)
            key.scatter_(0, y, torch.where(go, (t << 24) | rank[x], key.gather(0, y)))
    return fin


def exact(case, seed):
    w, S, call = _workload(case["model"], case["workers"]), case["scen"], case["call"]
    fan = max(1, int(np.diff(w.succ_ptr).max()))
    swept = call in ("critical", "static")
    steps = w.n_ops * (w.n_ops * S * 8 / 3e12 + (10 + 8 * fan) * max(1e-5, S * 2e-10))
    if call == "share" or not (swept or steps < 12) or w.n_ops * S > 2e9 or (call == "generated" and w.n_ops * S > 2e8):
        return None
    dur = _philox_durations(w, S, seed) if call == "generated" else _durations(w, S, seed)
    if swept:
        pred = _predecessors(w)
        if call == "static":  # devices run their ops in id order
            last = {}
            for v in range(w.n_ops):
                r = int(w.op_res[v])
                if r in last:
                    pred[v].append(last[r])
                last[r] = v
        fin = _sweep(w, dur, pred)
    else:
        gap, delay = _device_model(w) if call == "device" else (None, None)
        place = _placement(w, S, seed).to(torch.int32) if _placed(case) else None
        fin = _replay(w, dur, place, gap, delay, _prio(case, w))
    span = fin.max(dim=0).values
    if call == "critical":
        return {"critical": span}
    out = {"makespan": span, "status": torch.zeros_like(span)}
    if call == "attribute":
        return {"makespan": span, "status": out["status"], "finish": fin, "prev": None, "busy": None, "chain": None,
                "chain_ops": None}
    return {k: v for k, v in (("makespan", span), ("finish", fin if case["finish"] else None),
                              ("status", out["status"])) if v is not None}
