"""The merge kernel against the oracle: frames of every length and type,
tiles with a remainder, deferred ops that queue up, and scenarios whose times
do not fit."""
import numpy as np
import pytest
import torch

import oracle
import paper_2002_06790_amd as mlsim
from paper_2002_06790_amd import workloads as W
from test_merge_program import ps_graph

pytestmark = pytest.mark.gpu


def run_all(ptr, idx, res, R, dur, prio=None, rng=None):
    """Every call that may take the merge kernel, each equal to the oracle."""
    g = mlsim.Graph(ptr, idx, res, R, prio=prio)
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
