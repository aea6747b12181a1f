"""The passes that put atoms and list entries in order (k_sort.h): one tile, the edges of a tile and of a group of
tiles, more tiles than are summed up in the scatter, keys with and without a payload, against the scanning rounds; and
the interest rows of short windows (k_fit_bits_low) at the edges of their tiles, against the oracle."""
import numpy as np
import pytest

from gen import make_workload

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def engine():
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    import paper_2509_19086_amd as P
    return P.Engine(0)


def _staircase(jobs, each, gaps, seed=1):
    """jobs * each atoms: every boundary is a cut, memory grows along a job, all gaps take all of it."""
    rng = np.random.default_rng(seed)
    wl = make_workload("tiny", 0, n_gaps=8, n_jobs=8)
    wl.n_gaps, wl.n_jobs = gaps, jobs
    wl.W = rng.integers(1, 40 * each, size=gaps).astype(np.int32)
    wl.C = rng.choice(np.array([60000, 70000], np.int32), size=gaps)
    wl.seg_off = (each * np.arange(jobs + 1)).astype(np.int64)
    wl.dur = rng.integers(1, 30, size=jobs * each).astype(np.int32)
    wl.mem = (rng.integers(1000, 40000, size=(jobs, 1)) + 10 * np.arange(each)[None]).reshape(-1).astype(np.int32)
    wl.safe = np.ones(jobs * each, dtype=np.uint8)
    wl.progress = np.zeros(jobs, dtype=np.int32)
    wl.wait = rng.integers(0, 10**6, size=jobs).astype(np.int32)
    wl.sla_class = rng.integers(0, 3, size=jobs).astype(np.uint8)
    return wl


def _replies(engine, wl, policy, max_rounds):
    import paper_2509_19086_amd as P
    t = P.DeviceTick(engine, wl)
    t.prepare(); t.fit()
    par = P.Params.make(policy, max_rounds=max_rounds)
    got = []
    try:
        for mode in (1, 0):
            engine.sja_set_resolve_mode(mode)
            t.resolve(par)
            got.append([x.cpu().numpy().copy() for x in (t.grant_job, t.grant_cut, t.grant_score, t.job_gap, t.rounds)])
    finally:
        engine.sja_set_resolve_mode(0)
    return t, got


# atoms: one tile and one more; 15 to 17 tiles (a group is 16); 1023, 1024 and 1025 tiles (beyond 1024 the columns are scanned)
@pytest.mark.parametrize("jobs,each,gaps", [
    (4096, 1, 600), (4097, 1, 600), (3840, 16, 600), (4096, 16, 600), (4097, 16, 600), (4352, 16, 600), (6001, 11, 400),
    (8184, 512, 300), (8192, 512, 300), (8200, 512, 300)])
@pytest.mark.parametrize("policy", [0, 3])
def test_order_by_tiles(engine, jobs, each, gaps, policy):
    _, got = _replies(engine, _staircase(jobs, each, gaps), policy, 12)
    for a, b in zip(*got):
        np.testing.assert_array_equal(a, b)


# words of 32 jobs: a block takes 256 of them, and 8, 16 or 32 rows
@pytest.mark.parametrize("gaps,jobs", [(1025, 4097), (1033, 8192), (1100, 8193), (4096, 8161), (16400, 8225), (2100, 33000)])
def test_rows_of_short_windows(engine, oracle, gaps, jobs):
    wl = _staircase(jobs, 6, gaps, seed=2)
    wl.W[: gaps // 2] = np.random.default_rng(5).integers(1, 30, size=gaps // 2)         # below many a job's first cut
    import paper_2509_19086_amd as P
    t = P.DeviceTick(engine, wl)
    t.prepare(); t.fit()
    rows = np.unique(np.concatenate([np.arange(0, gaps, max(1, gaps // 200)), [gaps - 1]]))
    _, bits = oracle.fit(wl.seg_off, wl.dur, wl.mem, wl.safe, wl.progress, wl.W[rows], wl.C[rows])
    np.testing.assert_array_equal(t.bits.cpu().numpy().view(np.uint32)[rows], bits)
