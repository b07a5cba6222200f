"""The merge kernel against the oracle: frames of every length and type,
tiles with a remainder, deferred ops that queue up, and scenarios whose times
do not fit."""
import numpy as np
import pytest
import torch

import oracle
import paper_2002_06790_amd as mlsim
from paper_2002_06790_amd import workloads as W
from test_merge_program import (MANY_CHAINS, PART_OF_A_CHAIN, TWO_HOPS, TWO_HOPS_DUR, TWO_HOPS_JOINED,
                                ps_graph, stream_graph)

pytestmark = pytest.mark.gpu


def run_all(ptr, idx, res, R, dur, prio=None, rng=None):
    """Every call that may take the merge kernel, each equal to the oracle."""
    g = mlsim.Graph(ptr, idx, res, R, prio=prio)
    g.pin_variant("merge", 1)  # also where the event list is faster
    d = torch.from_numpy(dur).cuda()
    S = dur.shape[1]
    gap, delay = (rng.integers(0, 9, R).astype(np.int32) for _ in range(2))
    for kw in ({}, {"gap": gap}, {"delay": delay}, {"gap": gap, "delay": delay}):
        omk, ofin, ost = oracle.run_batch(ptr, idx, res, R, dur, prio=prio, **kw)
        for want in (True, False):
            mk, fin, st = g.run(d, want_finish=want, **kw)
            assert np.array_equal(mk.cpu().numpy(), omk) and np.array_equal(st.cpu().numpy(), ost), (kw, want)
            if want:
                ok = ost == 0
                assert np.array_equal(fin.cpu().numpy()[:, ok], ofin[:, ok]), kw
    a = g.attribute(d)
    for k, o in zip(("makespan", "status", "busy", "chain", "chain_ops"), oracle.attribute(ptr, idx, res, R, dur, prio=prio)):
        assert np.array_equal(a[k].cpu().numpy(), o), k
    base = rng.integers(1, 5000, (2, res.size)).astype(np.int32)
    noise = mlsim.noise_for_sigma(0.02)
    gdur = oracle.generate(base, S, 32, noise, 11)
    omk, ofin, _ = oracle.run_batch(ptr, idx, res, R, gdur, prio=prio)
    mk, fin, _ = g.run_generated(mlsim.Gen(torch.from_numpy(base).cuda(), 32, noise, 11), S, want_finish=True)
    assert np.array_equal(mk.cpu().numpy(), omk) and np.array_equal(fin.cpu().numpy(), ofin)
    g.close()


@pytest.mark.parametrize("scen", [1, 63, 64, 65, 200])
def test_worker_graphs(scen):
    rng = np.random.default_rng(scen)
    built = 0
    for it in range(6):
        ptr, idx, res, R = ps_graph(rng)
        while mlsim.merge_program(ptr, idx, res, R) is None:
            ptr, idx, res, R = ps_graph(rng)
        prio = rng.integers(-3, 4, res.size).astype(np.int32) if it % 3 == 2 else None
        built += mlsim.merge_program(ptr, idx, res, R, prio=prio) is not None
        run_all(ptr, idx, res, R, W.random_durations(res.size, scen, 1, (4, 50, 5000)[it % 3], rng), prio, rng)
    assert built >= 4


@pytest.mark.parametrize("make,workers", [(W.resnet50_ps, 3), (W.bert_large_ps, 2)])
def test_scenarios_unlike_each_other(make, workers):
    """Durations that share nothing between lanes: deferred ops run everywhere
    and wait in long queues."""
    w = make(n_scen=64, workers=workers)
    rng = np.random.default_rng(workers)
    dur = np.exp(rng.uniform(0, 12, (w.n_ops, 130))).astype(np.int32) + 1
    run_all(w.succ_ptr, w.succ_idx, w.op_res, w.n_res, dur, None, rng)


def test_flagged_scenarios():
    """Bad durations and times past INT32_MAX, also ones that wrap around 32
    bits, beside good scenarios of one tile."""
    w = W.resnet50_ps(n_scen=64, workers=2)
    rng = np.random.default_rng(3)
    dur = rng.integers(1, 1000, (w.n_ops, 100)).astype(np.int32)
    dur[rng.integers(0, w.n_ops, 8), np.arange(8)] = [0, -1, -2**31, 0, -5, 0, -7, -2**31]
    dur[:, 8:12] = 2**31 - 1
    dur[rng.integers(0, w.n_ops, 4), np.arange(12, 16)] = 2**31 - 1
    dur[:, 16] = 1 << 20
    ptr, idx, res, R = w.succ_ptr, w.succ_idx, w.op_res, w.n_res
    g = mlsim.Graph.from_workload(w)
    d = torch.from_numpy(dur).cuda()
    big = np.full(R, 2**31 - 1, np.int32)
    for kw in ({}, {"gap": big}, {"delay": big}):
        omk, ofin, ost = oracle.run_batch(ptr, idx, res, R, dur, **kw)
        mk, fin, st = g.run(d, want_finish=True, **kw)
        assert np.array_equal(mk.cpu().numpy(), omk) and np.array_equal(st.cpu().numpy(), ost), kw
        assert np.array_equal(fin.cpu().numpy()[:, ost == 0], ofin[:, ost == 0])
    # the scratch is as it was: the event list runs in the same set
    mk, _, _ = g.run(d)
    g2 = mlsim.Graph.from_workload(w)
    g2.run(d)
    place = torch.from_numpy(np.repeat(w.op_res[:, None], 100, 1).astype(np.uint16)).cuda()
    for _ in range(2):
        pmk, _, _ = g2.run(d, place=place)
        assert torch.equal(pmk, mk)
        assert torch.equal(g2.run(d)[0], mk)


def test_free_time_that_wraps_to_all_ones():
    """2^31 - 1 twice and 1: the free time of a resource without deferred ops
    is then the value that stands for no waiting op."""
    n = 12
    ptr = np.minimum(np.arange(n + 1), n - 1).astype(np.int64)
    idx, res = np.arange(1, n, dtype=np.int32), np.zeros(n, np.int32)
    p = mlsim.merge_program(ptr, idx, res, 1)
    assert p is not None and not len(p[3])
    rng = np.random.default_rng(0)
    dur = rng.integers(1, 1000, (n, 70)).astype(np.int32)
    for s in range(0, 60, 3):  # the sum is 2^32 - 1 after op ``at``, at every place of the frames
        at = 2 + s // 3 % (n - 2)
        dur[:at + 1, s] = [*[1] * (at - 2), 2**31 - 1, 2**31 - 1 - (at - 2), 1]
        assert dur[:at + 1, s].sum(dtype=np.int64) == 2**32 - 1
    g = mlsim.Graph(ptr, idx, res, 1)
    omk, ofin, ost = oracle.run_batch(ptr, idx, res, 1, dur)
    mk, fin, st = g.run(torch.from_numpy(dur).cuda(), want_finish=True)
    assert np.array_equal(mk.cpu().numpy(), omk) and np.array_equal(st.cpu().numpy(), ost)
    assert np.array_equal(fin.cpu().numpy()[:, ost == 0], ofin[:, ost == 0])


def test_deferred_op_released_by_a_released_one():
    g = mlsim.Graph(*TWO_HOPS)
    g.pin_variant("merge", 1)
    mk, fin, _ = g.run(torch.from_numpy(TWO_HOPS_DUR).cuda(), want_finish=True)
    assert mk.item() == 2023 and fin[11].item() == 1642 and fin[7].item() == 2023
    rng = np.random.default_rng(1)
    for g in (TWO_HOPS, TWO_HOPS_JOINED, *PART_OF_A_CHAIN.values()):
        run_all(*g, W.random_durations(g[2].size, 70, 1, 300, rng), None, rng)


@pytest.mark.parametrize("seed", [0, 1])
def test_irregular_graphs(seed):
    """Worker graphs with several pull hops and edges added or dropped, and streams."""
    rng = np.random.default_rng(seed)
    built = 0
    for it in range(150):
        ptr, idx, res, R = stream_graph(rng) if it % 3 == 2 else ps_graph(rng, 3, it % 3 == 1)
        p = mlsim.merge_program(ptr, idx, res, R)
        if p is None or not len(p[3]) or (p[3][:, 2] < 0).all() and it % 2:
            continue  # programs with deferred ops, every second of them with partners
        built += 1
        own = np.random.default_rng(it)
        run_all(ptr, idx, res, R, W.random_durations(res.size, 100, 1, (4, 50, 5000)[it % 3], own), None, own)
    assert built > 10


def test_program_taken_or_not():
    """The library's choice, the event list and the program on a graph whose
    program costs more than the event list, and on one where it pays."""
    rng = np.random.default_rng(0)
    for graph, pays in ((MANY_CHAINS, 0), (TWO_HOPS, None), (PART_OF_A_CHAIN["followers"], None)):
        ptr, idx, res, R = graph
        p = mlsim.merge_program(*graph)
        dur = W.random_durations(res.size, 200, 1, 60, rng)
        omk, ofin, _ = oracle.run_batch(ptr, idx, res, R, dur)
        assert pays is None or p[0][8] == pays
        g = mlsim.Graph(*graph)
        for merge in (-1, 0, 1, -1):
            g.pin_variant("merge", merge)
            mk, fin, _ = g.run(torch.from_numpy(dur).cuda(), want_finish=True)
            assert np.array_equal(mk.cpu().numpy(), omk) and np.array_equal(fin.cpu().numpy(), ofin), merge
