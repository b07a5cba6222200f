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


def ps_graph(rng, hops=1, extra=False):
    """A few workers whose chains feed links, aggregates and updates, some of
    them sharing a resource, with shuffled ids.  Some pulls take up to ``hops``
    transfers in a row; ``extra`` adds and drops a few edges."""
    workers, layers, links, per = (int(rng.integers(1, h)) for h in (4, 5, 3 + hops, 4))
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
            for k in range(int(rng.integers(0, hops)) if hops > 1 else 0):
                pull = op(link(w, 2 + k), pull)
            if rng.random() < 0.8:
                u = op(w, pull)
                if rng.random() < 0.2:
                    op(w, u)
    n = len(ops)
    if extra:
        if rng.random() < 0.4:
            edges = [e for e in edges if rng.random() > 0.08]
        edges += [tuple(sorted(rng.choice(n, 2, replace=False))) for _ in range(int(rng.integers(0, 4))) if n > 1]
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


def csr(succ):
    return np.cumsum([0] + [len(x) for x in succ]).astype(np.int64), np.array([w for x in succ for w in x], np.int32)


#: an op released by an op that another deferred op's run releases: op 11
#: (9 -> 10 -> 11) is ready before op 7 on resource 0
TWO_HOPS = (*csr([[1, 2], [3], [4], [8], [5], [6], [7], [], [9], [10], [11], []]),
            np.array([0, 0, 1, 1, 2, 3, 4, 0, 1, 3, 4, 0], np.int32), 6)
TWO_HOPS_DUR = np.array([[380, 268, 210, 22, 240, 416, 240, 381, 137, 83, 447, 305]], np.int32).T
#: the same with edges between the hops
TWO_HOPS_JOINED = (*csr([[1, 4], [5], [3, 6], [], [8], [9], [8], [8, 9], [10, 11, 14], [12, 16], [11], [], [13], [],
                         [15, 16], [], []]),
                   np.array([0, 0, 1, 1, 2, 2, 4, 4, 6, 6, 3, 0, 3, 0, 5, 1, 5], np.int32), 7)

def graph(ptr, idx, res, R):
    return np.array(ptr, np.int64), np.array(idx, np.int32), np.array(res, np.int32), R


#: deferred chains of which only some ops release an op of another chain, or
#: only some are released by one
PART_OF_A_CHAIN = {
    "leaders": graph([0, 2, 2, 4, 6, 6, 7, 8, 10, 10, 11, 12, 13], [3, 6, 5, 8, 7, 11, 4, 2, 9, 11, 5, 1, 10],
                     [0, 0, 2, 0, 0, 2, 1, 0, 0, 1, 2, 1], 5),
    "followers": graph([0, 1, 4, 5, 5, 7, 10, 10, 10, 10, 10, 11, 11], [1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11],
                       [1, 0, 0, 1, 0, 1, 0, 1, 0, 1, 1, 0], 2),
    "order": graph([0, 5, 12, 15, 17, 23, 26, 30, 30, 33, 34, 36, 36, 37, 37, 37],
                   [1, 4, 5, 6, 9, 2, 6, 7, 8, 10, 12, 13, 3, 5, 10, 5, 12, 5, 6, 7, 8, 11, 12, 10, 13, 14, 7, 9, 10, 11,
                    9, 10, 11, 14, 11, 14, 13], [1, 1, 0, 1, 1, 0, 1, 0, 0, 0, 1, 0, 1, 1, 0], 2)}


def stream_graph(rng):
    """Mostly ops of one predecessor, a few places back, on random resources."""
    n, R = int(rng.integers(4, 40)), int(rng.integers(2, 7))
    e = set()
    for v in range(1, n):
        for _ in range(1 if rng.random() < 0.85 else int(rng.integers(0, 4))):
            e.add((max(0, v - 1 - int(rng.integers(0, rng.integers(1, 9)))), v))
    e = np.array(sorted(e), np.int64).reshape(-1, 2)
    return graph(np.concatenate([[0], np.cumsum(np.bincount(e[:, 0], minlength=n))]), e[:, 1], rng.integers(0, R, n), R)


def test_streams():
    rng = np.random.default_rng(0)
    seen = collections.Counter()
    for it in range(6000):
        g = stream_graph(rng)
        seen.update(set(check(*g, W.random_durations(g[2].size, 4, 1, (3, 8, 500)[it % 3], rng))))
    assert all(seen[k] for k in (VISIT, RELEASE, LOAD, FORCE)), seen


@pytest.mark.parametrize("which", PART_OF_A_CHAIN)
def test_partners_in_part_of_a_chain(which):
    g = PART_OF_A_CHAIN[which]
    rng = np.random.default_rng(0)
    for hi in (3, 8, 500):
        check(*g, W.random_durations(g[2].size, 100, 1, hi, rng))


def test_deferred_op_released_by_a_released_one():
    check(*TWO_HOPS, TWO_HOPS_DUR)
    rng = np.random.default_rng(0)
    for g in (TWO_HOPS, TWO_HOPS_JOINED):
        for hi in (3, 8, 500):
            check(*g, W.random_durations(g[2].size, 100, 1, hi, rng))


@pytest.mark.parametrize("hops,extra,seed", [(3, False, 0), (3, False, 1), (1, True, 2), (3, True, 3)])
def test_worker_graphs_with_hops(hops, extra, seed):
    rng = np.random.default_rng(seed)
    seen = collections.Counter()
    for it in range(4000):
        ptr, idx, res, R = ps_graph(rng, hops, extra)
        dur = W.random_durations(res.size, 4, 1, (3, 8, 500)[it % 3], rng)
        gap = rng.integers(0, 4, R).astype(np.int32) if it % 4 == 1 else None
        delay = rng.integers(0, 6, R).astype(np.int32) if it % 5 == 1 else None
        seen.update(set(check(ptr, idx, res, R, dur, gap=gap, delay=delay)))
    assert all(seen[k] for k in (VISIT, RELEASE, LOAD, FORCE)), seen


#: 7 of 17 ops deferred in one cluster of six chains
MANY_CHAINS = graph([0, 4, 6, 7, 7, 8, 8, 9, 10, 10, 10, 12, 13, 16, 19, 19, 19, 19],
                    [1, 2, 4, 6, 3, 9, 5, 10, 7, 8, 11, 15, 14, 13, 14, 15, 14, 15, 16],
                    [1, 3, 3, 3, 0, 2, 0, 2, 2, 4, 0, 2, 4, 0, 1, 0, 3], 5)


def test_program_is_taken_where_it_pays():
    """A deferred op of a cluster of c > 2 chains counts 8 + c against 4 per op."""
    assert not mlsim.merge_program(*MANY_CHAINS)[0][8]
    for w in (W.resnet50_ps(n_scen=64), W.bert_large_ps(n_scen=64)):
        assert mlsim.merge_program(w.succ_ptr, w.succ_idx, w.op_res, w.n_res)[0][8]
    rng = np.random.default_rng(3)
    seen = collections.Counter()
    for it in range(3000):
        g = stream_graph(rng) if it % 2 else ps_graph(rng, 3, True)
        p = mlsim.merge_program(*g)
        if p is None:
            continue
        size = {c: c1 - c0 for c0, c1 in p[1][:, 8:10] for c in range(c0, c1)}
        cost = sum(8 + size[c] for c in p[2][:, 2] if size[c] > 2)
        assert p[0][8] == (cost < 4 * g[2].size)
        seen[int(p[0][8]), cost > 0] += 1
    assert len(seen) == 3, seen
