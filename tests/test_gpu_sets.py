"""Calm conflict rounds, played in batches (k_sets.h): one and several list blocks and classes, up to one,
two and four sets per lane, one launch and launches in turn, caps in the middle of a batch, jobs or gaps that
run out, equal keys, cuts that only some windows get, against the oracle.  Most batches here are small enough to be
served pair by pair: full_tick_check fits those a second time, in the mode that leaves them to these kernels."""
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


def _calm(caps, groups, gaps_each, jobs, mixed=0.1, max_rounds=0, seed=1):
    """Every capacity has gaps of the same `groups` windows (ten times as long each, so each is a list block of its
    own), every job a cut for each of them, and the jobs' order is the same in all windows but for the share
    `mixed` of them: nearly all gaps want the same few jobs, round after round."""
    rng = np.random.default_rng(seed)
    wl = make_workload("tiny", 0, n_gaps=8, n_jobs=8)
    wl.n_gaps, wl.n_jobs = caps * groups * gaps_each, jobs
    window = 100 * 10 ** np.arange(groups)
    wl.W = rng.permutation(np.tile(np.repeat(window, gaps_each), caps)).astype(np.int32)
    wl.C = rng.permutation(np.repeat(np.arange(40000, 40000 + caps), groups * gaps_each)).astype(np.int32)
    scale = 1 + rng.permutation(jobs) / (2.0 * jobs)
    dur = np.empty((jobs, groups), dtype=np.int64)
    for k in range(groups):
        own = np.where(rng.random(jobs) < mixed, 1 + rng.random(jobs) / 2, scale)
        dur[:, k] = np.floor(window[k] * own / 2)
    wl.dur = np.diff(np.concatenate([np.zeros((jobs, 1), dtype=np.int64), dur], axis=1), axis=1).reshape(-1).astype(np.int32)
    wl.mem = np.repeat(rng.integers(20000, 20100, size=jobs), groups).astype(np.int32)
    wl.seg_off = (groups * np.arange(jobs + 1)).astype(np.int64)
    wl.safe = np.ones(jobs * groups, dtype=np.uint8)
    wl.progress = np.zeros(jobs, dtype=np.int32)
    wl.wait = rng.integers(0, 50, size=jobs).astype(np.int32)
    wl.sla_class = rng.integers(0, 3, size=jobs).astype(np.uint8)
    wl.max_rounds = max_rounds
    return wl


@pytest.mark.parametrize("caps,groups,gaps_each,jobs", [
    (1, 1, 300, 700),           # one list block's worth of windows, one set: its lowest gaps run out
    (1, 3, 70, 900), (5, 2, 40, 900), (3, 3, 65, 333),          # the last: fewer jobs than gaps
    (30, 2, 5, 1500), (64, 2, 3, 1500),                         # up to 64 sets, and 128
    (64, 3, 2, 900), (43, 3, 3, 600), (64, 4, 2, 1500)])        # more than 128 list blocks; up to 256 sets
@pytest.mark.parametrize("mixed", [0.0, 0.15])
def test_calm_rounds(engine, oracle, caps, groups, gaps_each, jobs, mixed):
    full_tick_check(engine, oracle, _calm(caps, groups, gaps_each, jobs, mixed), policies=[0, 3], resolve_modes=(0,))


@pytest.mark.parametrize("caps,groups,gaps_each,jobs", [
    (1, 1, 600, 1500), (2, 1, 300, 400),                        # batches as long as a set's jobs and gaps at hand allow
    (16, 1, 40, 1200), (17, 1, 40, 1200), (32, 1, 20, 1200), (33, 1, 20, 1200), (64, 1, 10, 1200), (33, 2, 8, 900),
    (40, 2, 6, 900), (41, 2, 6, 900),                           # one launch, and launches in turn
    (43, 3, 2, 100), (43, 3, 2, 40)])                           # fewer jobs listed for a piece than elsewhere, or no room for any
def test_jobs_at_hand(engine, oracle, caps, groups, gaps_each, jobs):
    full_tick_check(engine, oracle, _calm(caps, groups, gaps_each, jobs, 0.05, seed=3), policies=[0, 3], resolve_modes=(0,))


# launches in turn whose sets pass many jobs a round, by which they come to have more at hand; one launch begun in vain
@pytest.mark.parametrize("caps,groups,gaps_each,jobs", [(43, 3, 6, 2500), (60, 2, 5, 2000), (20, 2, 20, 1500)])
@pytest.mark.parametrize("mixed", [0.0, 0.5, 1.0])
def test_sets_that_take_each_others_jobs(engine, oracle, caps, groups, gaps_each, jobs, mixed):
    full_tick_check(engine, oracle, _calm(caps, groups, gaps_each, jobs, mixed, seed=5), policies=[0, 3], resolve_modes=(0,))


def _runs_dry(long_gaps, short_gaps, long_jobs, short_jobs):
    """Gaps with long windows, and behind them gaps with short ones; jobs for either.  The short jobs run out in the middle of
    a batch of rounds; then the last long gap is served, at which the batch pauses (the class's further gaps are far away)."""
    rng = np.random.default_rng(long_gaps)
    wl = make_workload("tiny", 0, n_gaps=8, n_jobs=8)
    wl.n_gaps, wl.n_jobs = long_gaps + short_gaps, long_jobs + short_jobs
    wl.W = np.repeat([100000, 100], [long_gaps, short_gaps]).astype(np.int32)
    wl.C = np.full(wl.n_gaps, 40960, dtype=np.int32)
    wl.dur = rng.permutation(np.concatenate([50000 + rng.permutation(long_jobs), 10 + rng.permutation(short_jobs) % 90])).astype(np.int32)
    wl.mem = rng.integers(20000, 20100, size=wl.n_jobs).astype(np.int32)
    wl.seg_off = np.arange(wl.n_jobs + 1, dtype=np.int64)
    wl.safe, wl.progress = np.ones(wl.n_jobs, dtype=np.uint8), np.zeros(wl.n_jobs, dtype=np.int32)
    wl.wait = rng.integers(0, 50, size=wl.n_jobs).astype(np.int32)
    wl.sla_class = np.zeros(wl.n_jobs, dtype=np.uint8)
    wl.max_rounds = 0
    return wl


# a set that found no job left in one batch does not count for a round of the next; one launch, and launches in turn
@pytest.mark.parametrize("long_gaps,short_gaps,long_jobs,short_jobs", [(160, 1300, 300, 90), (200, 1500, 260, 70), (150, 2000, 149, 80),
                                                                       (200, 7000, 400, 110), (250, 6500, 260, 90)])
def test_jobs_run_out_for_some(engine, oracle, long_gaps, short_gaps, long_jobs, short_jobs):
    full_tick_check(engine, oracle, _runs_dry(long_gaps, short_gaps, long_jobs, short_jobs), policies=[0, 1], resolve_modes=(0,))


@pytest.mark.parametrize("max_rounds", [41, 56, 57, 80, 119, 120, 121])
@pytest.mark.parametrize("caps,groups,gaps_each", [(1, 1, 120), (43, 3, 2)])
def test_caps_within_a_batch(engine, oracle, caps, groups, gaps_each, max_rounds):
    full_tick_check(engine, oracle, _calm(caps, groups, gaps_each, 500, max_rounds=max_rounds), policies=[1], resolve_modes=(0,))


@pytest.mark.parametrize("caps,groups", [(2, 3), (43, 3)])
def test_equal_keys(engine, oracle, caps, groups):
    # with weight 0 every cut of every job has the same key: a shorter window's record comes before a longer one's
    wl = _calm(caps, groups, 300 // (caps * groups) + 1, 400)
    wl.sla_weight, wl.class0_override = (0, 0, 0), 0
    full_tick_check(engine, oracle, wl, policies=[2], resolve_modes=(0,))


@pytest.mark.parametrize("name,gaps,jobs,policy", [("medium", 2048, 3000, 0), ("stress", 1500, 2500, 3), ("large", 3000, 2000, 1), ("stress", 9000, 1500, 3)])
def test_against_the_scanning_rounds(engine, name, gaps, jobs, policy):
    # sizes beyond the oracle's reach in a test; the matrix-scanning rounds are checked against it elsewhere
    import paper_2509_19086_amd as P
    wl = make_workload(name, 3, n_gaps=gaps, n_jobs=jobs)
    t = P.DeviceTick(engine, wl)
    t.prepare(); t.fit()
    par = P.Params.make(policy)
    got = []
    try:
        for mode in (1, 0):
            engine.sja_set_resolve_mode(mode)
            t.resolve(par)
            got.append([x.cpu().numpy().copy() for x in (t.grant_job, t.grant_cut, t.grant_score, t.job_gap, t.rounds)])
    finally:
        engine.sja_set_resolve_mode(0)
    for a, b in zip(*got):
        np.testing.assert_array_equal(a, b)
