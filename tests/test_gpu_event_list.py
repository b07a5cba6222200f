"""The event list, by its default plan, on graphs whose replays take a merge
program otherwise: the parity cases of every call that chooses between the
two, once more with the program turned off."""
import numpy as np
import pytest

import test_gpu_attr
import test_gpu_delay
import test_gpu_gap
import test_gpu_gen
import test_gpu_parity
from paper_2002_06790_amd import workloads as W
from test_gpu_parity import mlsim  # noqa: F401 (the fixture)

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def event_list(pin_variants):
    pin_variants(merge=0)


def test_plain(mlsim):
    test_gpu_parity._variant_cases(mlsim)


@pytest.mark.parametrize("k", [2, 4])
def test_full_size(mlsim, k):
    """Enough tiles for the heap root's children in registers."""
    test_gpu_parity.test_full_size_population(mlsim, k)


@pytest.mark.parametrize("k,S", [(2, 200), (4, 200)])
def test_device_model(mlsim, k, S):
    test_gpu_gap.test_workload_parity(mlsim, k, S)
    test_gpu_delay.test_workload_parity(mlsim, k, S)


def test_device_model_status(mlsim):
    test_gpu_gap.test_overflow_and_bad_durations(mlsim)
    test_gpu_delay.test_overflow_and_bad_durations(mlsim)
    test_gpu_parity.test_status_bits(mlsim)


@pytest.mark.parametrize("case", test_gpu_gen.CASES)
def test_generated(mlsim, case):
    test_gpu_gen.test_run_generated_matches_oracle(mlsim, *case)


@pytest.mark.parametrize("k,S", [(2, 130), (4, 130)])
def test_attribution(mlsim, k, S):
    test_gpu_attr.test_attr_workloads(mlsim, k, S)
    w = W.make_config(k, n_scen=64)
    rng = np.random.default_rng(k)
    wild = rng.integers(1, 1000, size=(w.n_ops, 70)).astype(np.int32)
    test_gpu_attr.check_attr(mlsim, w.succ_ptr, w.succ_idx, w.op_res, w.n_res, wild)
