"""Atoms ordered by the leading bits of their keys (k_fix_runs): runs of equal leading bits of no, a few, some and very many
atoms, in order and not, with second keys and without, keys that are all alike, and so many alike that the digests are
given up from the start (the sample of k_atom_keys) or after a run that the sample did not show, against the oracle."""
import numpy as np
import pytest

from gen import make_workload
from test_gpu_parity import full_tick_check

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def engine():
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    import paper_2509_19086_amd as P
    return P.Engine(0)


@pytest.mark.parametrize("step", [1 << 14, 1 << 9, 1 << 6, 1, 0])
@pytest.mark.parametrize("policy", [0, 1, 2, 3])
def test_runs(engine, oracle, step, policy):
    # jobs of one cut, F = 1000 x (2^24 + a number below 8000 steps): the leading bits tell them apart, or leave runs
    # of two to three, of some ten to forty, or of thousands; under MIXED jobs of equal scores differ in F
    jobs, gaps = 8000, 300
    rng = np.random.default_rng(step + policy)
    wl = make_workload("medium", 1, n_gaps=gaps, n_jobs=jobs)
    wl.seg_off = np.arange(jobs + 1, dtype=np.int64)
    wl.dur = np.full(jobs, 1000, dtype=np.int32)
    wl.mem = (2**24 + step * rng.integers(0, 8000, size=jobs)).astype(np.int32)
    wl.safe = np.ones(jobs, dtype=np.uint8)
    wl.progress = np.zeros(jobs, dtype=np.int32)
    wl.wait = np.full(jobs, 60000, dtype=np.int32)
    half = jobs // 2
    wl.mem[:half:2] = 2 * (wl.mem[:half:2] // 2)
    wl.mem[1:half:2] = wl.mem[:half:2] // 2         # half the memory, twice the weight
    wl.wait[1:half:2] = 2 * (60000 + wl.wait_scale) - wl.wait_scale
    wl.sla_class = rng.integers(0, 3, size=jobs).astype(np.uint8)
    wl.W = rng.integers(500, 1500, size=gaps).astype(np.int32)
    wl.C = rng.choice([2**23 + 100 * step, 2**24 + 4000 * step, 2**30], size=gaps).astype(np.int32)
    full_tick_check(engine, oracle, wl, policies=[policy], resolve_modes=(0,))


@pytest.mark.parametrize("spread", [10, 1000])
@pytest.mark.parametrize("jobs", [600, 9000])
@pytest.mark.parametrize("policy", [1, 3])
def test_jobs_of_one_profile(engine, oracle, spread, jobs, policy):
    # waits a thousandth apart or less: hundreds of atoms of different keys behind each 24 bits, few behind 32
    wl = make_workload("small", 3, n_gaps=300, n_jobs=jobs)
    n = int(wl.seg_off[1])
    for name in ("dur", "mem", "safe"):
        setattr(wl, name, np.tile(getattr(wl, name)[:n], jobs))
    wl.progress[:] = 0
    wl.wait = np.random.default_rng(spread).integers(10**6, 10**6 + spread, size=jobs).astype(np.int32)
    wl.max_rounds = 40
    full_tick_check(engine, oracle, wl, policies=[policy], resolve_modes=(0,))


@pytest.mark.parametrize("policy", [0, 1, 2, 3])
@pytest.mark.parametrize("close", ["keys", "second"])
def test_a_long_run_among_keys_that_differ(engine, oracle, policy, close):
    # 200 of 9000 jobs behind the same 24 bits, out of order: too few for the sample.  second: under MIXED the same score from
    # half the memory and twice the weight
    jobs, gaps = 9000, 300
    rng = np.random.default_rng(policy)
    wl = make_workload("medium", 1, n_gaps=gaps, n_jobs=jobs)
    wl.seg_off = np.arange(jobs + 1, dtype=np.int64)
    wl.dur = np.full(jobs, 1000, dtype=np.int32)
    wl.mem = np.floor(1000 * 2.0 ** (14 * rng.random(jobs))).astype(np.int32)
    wl.safe, wl.progress = np.ones(jobs, dtype=np.uint8), np.zeros(jobs, dtype=np.int32)
    wl.wait = np.full(jobs, 60000, dtype=np.int32)
    wl.sla_class = np.ones(jobs, dtype=np.uint8)
    some = np.sort(rng.choice(jobs, size=200, replace=False))
    if close == "keys":
        wl.mem[some] = 2**25 + rng.permutation(200)
    else:
        wl.mem[some] = np.where(np.arange(200) % 2, 2**25, 2**24)
        wl.wait[some] = np.where(np.arange(200) % 2, 60000, 2 * (60000 + wl.wait_scale) - wl.wait_scale)
    wl.W = rng.integers(900, 1500, size=gaps).astype(np.int32)
    wl.C = rng.choice([2**23, 2**30], size=gaps).astype(np.int32)
    full_tick_check(engine, oracle, wl, policies=[policy], resolve_modes=(0,))


@pytest.mark.parametrize("name,gaps,jobs", [("stress", 600, 5000), ("medium", 300, 12000), ("large", 1100, 20000)])
def test_drawn(engine, oracle, name, gaps, jobs):
    full_tick_check(engine, oracle, make_workload(name, 2, n_gaps=gaps, n_jobs=jobs), policies=[1, 3], resolve_modes=(0,))
