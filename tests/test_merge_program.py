"""CPU checks of the merge program the library builds (host code only).

A graph whose ops mostly run in one order in every scenario is compiled into
a fixed instruction list.  These tests take it through
sim_testing_merge_program (no device is used), interpret it and compare
every finish time with the oracle's replay: a wrong chain order, a release
or a visit too early, or a value slot freed too soon changes them.
"""
import collections
import os

import numpy as np
import pytest

import oracle
from merge_interp import FORCE, LOAD, MAX, RELEASE, VISIT, interpret
from paper_2002_06790_amd import workloads as W

mlsim = pytest.importorskip("paper_2002_06790_amd")
pytestmark = pytest.mark.skipif(not os.path.exists(mlsim.LIB_PATH), reason="libmlsim.so is not built")


def check(ptr, idx, res, R, dur, prio=None, gap=None, delay=None):
    """The program's kinds of instruction (empty: the graph has none)."""
    p = mlsim.merge_program(ptr, idx, res, R, prio=prio, device_model=gap is not None or delay is not None)
    if p is None:
        return collections.Counter()
    _, fin, _ = oracle.run_batch(ptr, idx, res, R, dur, prio=prio, gap=gap, delay=delay)
    for s in range(dur.shape[1]):
        got, _ = interpret(p, R, dur[:, s], gap, delay)
        assert np.array_equal(got, fin[:, s]), f"scenario {s}"
    return collections.Counter(p[1][:, 0].tolist())


@pytest.mark.parametrize("make", [W.resnet50_ps, W.bert_large_ps])
@pytest.mark.parametrize("workers", [1, 2, 5])
def test_parameter_server_workloads(make, workers):
    w = make(n_scen=4096, workers=workers)
    dur = w.durations()[:, ::1365]
    rng = np.random.default_rng(workers)
    kinds = check(w.succ_ptr, w.succ_idx, w.op_res, w.n_res, dur)
    assert kinds[VISIT] > w.n_ops // 2, "most ops have one place in every scenario"
    assert kinds[RELEASE] > 0 and (kinds[MAX] > 0) == (workers > 4)
    wild = rng.integers(1, 1000, size=dur.shape).astype(np.int32)  # nothing like the profile
    check(w.succ_ptr, w.succ_idx, w.op_res, w.n_res, wild, prio=-np.arange(w.n_ops, dtype=np.int32),
          gap=rng.integers(0, 50, w.n_res).astype(np.int32), delay=rng.integers(0, 90, w.n_res).astype(np.int32))


def ps_graph(rng):
    """A few workers whose chains feed links, aggregates and updates, some of
    them sharing a resource, with shuffled ids."""
    workers, layers, links, per = (int(rng.integers(1, h)) for h in (4, 5, 4, 4))
    links -= 1
    R = workers * (1 + links) + 1
    ops, edges = [], []

    def op(r, *preds):
        ops.append(r)
        edges.extend((p, len(ops) - 1) for p in preds)
        return len(ops) - 1

    def link(w, k):
        return w if links == 0 else workers + w * links + min(k, links - 1)

    grad = {}
    for w in range(workers):
        last = ()
        for layer in range(layers):
            for _ in range(per):
                last = (op(w, *last),)
                if rng.random() < 0.2:
                    op(w, *last)
            grad[w, layer] = last[0]
    push = {k: op(link(k[0], 0), g) for k, g in grad.items()}
    server = rng.random() < 0.5
    agg = [op(R - 1, *(push[w, layer] for w in range(workers))) for layer in range(layers)] if server else None
    for w in range(workers):
        for layer in range(layers):
            pull = op(link(w, 1), *([agg[layer]] if server else [push[v, layer] for v in range(workers)]))
            if rng.random() < 0.8:
                u = op(w, pull)
                if rng.random() < 0.2:
                    op(w, u)
    n = len(ops)
    perm = rng.permutation(n) if rng.random() < 0.5 else np.arange(n)
    e = np.array(sorted((perm[a], perm[b]) for a, b in edges), np.int64).reshape(-1, 2)
    ptr = np.concatenate([[0], np.cumsum(np.bincount(e[:, 0], minlength=n))]).astype(np.int64)
    res = np.zeros(n, np.int32)
    res[perm] = ops
    return ptr, e[:, 1].astype(np.int32), res, R


@pytest.mark.parametrize("family", ["random", "workers"])
def test_random_graphs(family):
    rng = np.random.default_rng(5)
    seen = collections.Counter()
    for it in range(250):
        if family == "random":
            n, R = int(rng.integers(1, 24)), int(rng.integers(1, 5))
            ptr, idx, res, prio = W.random_dag(n, R, float(rng.choice([0.05, 0.1, 0.2, 0.4])), rng, with_prio=it % 2 == 0)
        else:
            ptr, idx, res, R = ps_graph(rng)
            prio = rng.integers(-3, 4, res.size).astype(np.int32) if it % 2 else None
        dur = W.random_durations(res.size, 3, 1, (3, 8, 1000)[it % 3], rng)  # short ones tie
        gap = rng.integers(0, 4, R).astype(np.int32) if it % 4 == 1 else None
        delay = rng.integers(0, 6, R).astype(np.int32) if it % 5 == 1 else None
        seen.update(set(check(ptr, idx, res, R, dur, prio=prio, gap=gap, delay=delay)))
    assert all(seen[k] for k in (VISIT, RELEASE, FORCE)), seen
    if family == "workers":
        assert seen[LOAD], seen
