"""Grant-list records: four bytes while job ids fit 19 bits, eight beyond.  Both forms, on both
sides of the line, with the job in the list key and looked up through the rank, against the oracle."""
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


def _short_jobs(n_jobs, n_gaps, seed):
    """Jobs of one to three segments, so that half a million of them are quick; the best jobs sit at
    both ends of the id range, where a truncated id would show."""
    wl = make_workload("small", seed, n_gaps=n_gaps, n_jobs=8)
    rng = np.random.default_rng(seed)
    lens = rng.integers(1, 4, size=n_jobs)
    wl.n_jobs = n_jobs
    wl.seg_off = np.zeros(n_jobs + 1, dtype=np.int64)
    np.cumsum(lens, out=wl.seg_off[1:])
    S = int(wl.seg_off[-1])
    wl.dur = rng.integers(1, 700, size=S).astype(np.int32)
    wl.mem = rng.integers(256, 41000, size=S).astype(np.int32)
    wl.safe = (rng.random(S) < 0.5).astype(np.uint8)
    wl.progress = (rng.random(n_jobs) * lens).astype(np.int32)
    wl.wait = rng.integers(0, 1000, size=n_jobs).astype(np.int32)
    wl.wait[:40] += 900000
    wl.wait[-40:] += 900000
    wl.sla_class = rng.integers(0, 3, size=n_jobs).astype(np.uint8)
    return wl


@pytest.mark.parametrize("n_jobs", [(1 << 19) - 1, 1 << 19, (1 << 19) + 65])
def test_both_record_sizes(engine, oracle, n_jobs):
    wl = _short_jobs(n_jobs, 90, n_jobs & 7)
    t = full_tick_check(engine, oracle, wl, policies=[1], resolve_modes=(0, 2))
    jobs = t.grant_job.cpu().numpy()
    assert (jobs > n_jobs - 50).any() and (jobs < 50).any()


@pytest.mark.parametrize("classes,all_safe", [(64, True), (40, True), (1, False)])
def test_entries_by_groups_of_classes(engine, oracle, classes, all_safe):
    # every boundary safe and many capacities: an atom's places in all classes do not fit the buffer at once
    wl = make_workload("stress", 21, n_gaps=700, n_jobs=30)
    rng = np.random.default_rng(classes)
    if all_safe:
        wl.safe[:] = 1
        wl.progress[:] = 0
    caps = np.sort(rng.choice(np.arange(2000, 150000), size=classes, replace=False)).astype(np.int32)
    wl.C = caps[rng.integers(0, classes, size=700)]
    full_tick_check(engine, oracle, wl, policies=[0, 3], resolve_modes=(0,))


@pytest.mark.parametrize("n_jobs", [1, 63, 64, 65])
def test_atoms_around_the_sort_of_one_block(engine, oracle, n_jobs):
    # every cut of every job can be reached: 64 atoms a job, and one thread block sorts up to 4096
    wl = make_workload("tiny", n_jobs, n_gaps=70, n_jobs=n_jobs)
    wl.safe[:] = 1
    wl.progress[:] = 0
    wl.C[:] = 40960
    wl.C[:3] = 20480
    full_tick_check(engine, oracle, wl, policies=[0, 1, 2, 3], resolve_modes=(0,))


@pytest.mark.parametrize("n_gaps", [1, 2, 1023, 1025, 4095, 4096, 4097])
def test_gap_order_at_the_edges_of_a_tile(engine, oracle, n_gaps):
    # few distinct pairs, so that most are equal and the index decides; the largest pair equals the padding
    wl = make_workload("tiny", n_gaps, n_gaps=n_gaps, n_jobs=5)
    rng = np.random.default_rng(n_gaps)
    wl.W = rng.choice(np.array([50, 51, 700, 2**31 - 1], dtype=np.int32), size=n_gaps)
    wl.C = rng.choice(np.array([5120, 40960, 2**31 - 1], dtype=np.int32), size=n_gaps)
    full_tick_check(engine, oracle, wl, policies=[0], resolve_modes=(0,))
