"""Conflict rounds run by one thread block: what its rule takes and what it leaves to the launched
rounds, round caps on both sides of the hand-over, equal keys, lists that run dry, and keys that fall
along a job's atoms, against the oracle (small batches in the mode that leaves them to these kernels
too, see full_tick_check)."""
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


@pytest.mark.parametrize("max_rounds", [1, 4, 5, 19, 20, 21, 33, 0])
def test_caps_around_the_hand_over(engine, oracle, max_rounds):
    wl = make_workload("medium", 3, n_gaps=513, n_jobs=900)
    wl.max_rounds = max_rounds
    full_tick_check(engine, oracle, wl, policies=[0, 3], resolve_modes=(0,))


@pytest.mark.parametrize("name,gaps,jobs", [("stress", 900, 700), ("stress", 700, 1500), ("stress", 130, 3000), ("large", 70, 5000), ("large", 1025, 513), ("small", 65, 4000),
                                            ("medium", 1400, 40), ("tiny", 3, 700),
                                            ("stress", 5001, 300), ("medium", 5003, 700)])
def test_many_pieces_and_lists_that_run_dry(engine, oracle, name, gaps, jobs):
    # (the last two have more list blocks than those whose gap orders are kept in LDS)
    wl = make_workload(name, gaps + jobs, n_gaps=gaps, n_jobs=jobs)
    full_tick_check(engine, oracle, wl, policies=[0, 1, 2, 3], resolve_modes=(0,))


@pytest.mark.parametrize("weights", [(0, 0, 0), (1, 0, 0)])
def test_equal_keys(engine, oracle, weights):
    # with weight 0 every cut of every job has the same key: the job id decides, and a lower
    # window's record of the same job comes before a higher one's
    wl = make_workload("stress", 11, n_gaps=600, n_jobs=800)
    wl.sla_weight = weights
    wl.class0_override = 0
    full_tick_check(engine, oracle, wl, policies=[2], resolve_modes=(0,))


@pytest.mark.parametrize("caps,gain", [((36864, 73728, 110592), 36864), ((36864, 73728, 110592), 50000), ((36864, 40000, 147456), 4000)])
def test_hysteresis_keys_that_fall(engine, oracle, caps, gain):
    # with a gain above the distance of two capacities a longer fit can end in a shorter cut
    import paper_2509_19086_amd as P
    wl = make_workload("stress", 5, n_gaps=500, n_jobs=700)
    engine.sja_set_hysteresis(list(caps), gain)
    try:
        t = P.DeviceTick(engine, wl)
        t.prepare()
        want = None
        for fitted, mode in ((0, 1), (0, 0), (2, 0)):       # the matrix-scanning rounds are checked against the oracle elsewhere
            engine.sja_set_resolve_mode(fitted)
            t.fit()
            engine.sja_set_resolve_mode(mode)
            t.resolve(P.Params.make(3))
            got = [x.cpu().numpy().copy() for x in (t.grant_job, t.grant_cut, t.grant_score, t.job_gap, t.rounds)]
            want = want or got
            for a, b in zip(got, want):
                np.testing.assert_array_equal(a, b)
    finally:
        engine.sja_set_resolve_mode(0)
        engine.sja_set_hysteresis([], 1)


@pytest.mark.parametrize("gaps,jobs", [(600, 4500), (3001, 4500)])
def test_jobs_that_meet_in_a_claim_slot(engine, oracle, gaps, jobs):
    # ranked so that the jobs of consecutive rounds share a slot of the claim table (ids 2048 apart), with list
    # blocks in every wave; few list blocks, and more than those whose gap orders are kept in LDS
    wl = make_workload("stress", 3, n_gaps=gaps, n_jobs=jobs)
    rng = np.random.default_rng(gaps)
    wl.W = np.floor(10 * 10.0 ** (4 * rng.random(gaps))).astype(np.int32)
    order = np.argsort(np.arange(jobs) % 2048, kind="stable")          # 0, 2048, 4096, 1, 2049, ...
    wl.seg_off = np.arange(jobs + 1, dtype=np.int64)
    wl.dur = np.full(jobs, 9, dtype=np.int32)
    wl.mem = np.empty(jobs, dtype=np.int32)
    wl.mem[order] = 30000 - np.arange(jobs)
    wl.safe = np.ones(jobs, dtype=np.uint8)
    wl.progress = np.zeros(jobs, dtype=np.int32)
    wl.max_rounds = 90
    full_tick_check(engine, oracle, wl, policies=[0], resolve_modes=(0,))


def _by_windows(caps, windows, jobs_each, gaps_per_window=1, common=0, misfits=0, first=0):
    """Every capacity holds every job; each capacity has gaps of the same windows, and a window's best job
    is one as long as the window: a round serves one capacity, in as many pieces as there are windows.
    `first` jobs fit every gap and come before those, `common` ones after them; `misfits` fit none (they only
    lift the bound on the rounds)."""
    wl = make_workload("tiny", 0, n_gaps=8, n_jobs=8)
    wl.n_gaps, wl.n_jobs = caps * windows * gaps_per_window, windows * jobs_each + common + first + misfits
    wl.W = np.tile(np.repeat(np.arange(1000, 1000 + windows, dtype=np.int32), gaps_per_window), caps)
    wl.C = np.repeat(np.arange(10000, 10000 + caps, dtype=np.int32), windows * gaps_per_window)
    wl.seg_off = np.arange(wl.n_jobs + 1, dtype=np.int64)
    lengths = [np.repeat(np.arange(1000, 1000 + windows), jobs_each), np.full(common, 500), np.full(first + misfits, 1000)]
    wl.dur = np.concatenate(lengths).astype(np.int32)
    wl.mem = np.full(wl.n_jobs, 5000, dtype=np.int32)
    wl.mem[wl.n_jobs - misfits - first:] = 6000
    wl.mem[wl.n_jobs - misfits:] = 90000
    wl.safe = np.ones(wl.n_jobs, dtype=np.uint8)
    wl.progress = np.zeros(wl.n_jobs, dtype=np.int32)
    wl.wait = np.zeros(wl.n_jobs, dtype=np.int32)
    wl.sla_class = np.ones(wl.n_jobs, dtype=np.uint8)
    wl.max_rounds = 0
    return wl


@pytest.mark.parametrize("windows,first,caps", [(w, 10, c) for w in (24, 28, 32) for c in (4, 5, 6, 7, 8)] +
                         [(64, f, c) for f in (0, 10) for c in (3, 7, 8, 9, 28)])
def test_last_round_in_many_pieces(engine, oracle, windows, first, caps):
    # a round serves one capacity in as many pieces as it has windows, and the rounds add up to the block's
    # patience: it stops there, and with some number of capacities that is the very round that serves the last
    # gap (5 capacities of 28 or 32 windows, 7 of 24).  `first` jobs come before, one a round, so that the
    # block has taken over by then
    wl = _by_windows(caps, windows, caps, first=first)
    t = full_tick_check(engine, oracle, wl, policies=[0], resolve_modes=(0,))
    assert t.rounds.cpu().tolist() == [first + caps, 1]


@pytest.mark.parametrize("caps,windows,jobs_each,gaps_per_window,common",
                         [(1, 1, 3, 64, 0), (1, 1, 4, 64, 0), (1, 1, 5, 64, 0), (3, 1, 4, 30, 0)] +
                         [(28, 64, 10, 1, c) for c in (9, 10, 11, 13, 14, 15)] + [(28, 64, 20, 1, 0)])
def test_lists_that_end_where_the_block_takes_over(engine, oracle, caps, windows, jobs_each, gaps_per_window, common):
    # the jobs are used up one round before, with and one round after the last launched round (4, or 24 where
    # the rounds before are in too many pieces); gaps are left, so one more round finds nothing
    wl = _by_windows(caps, windows, jobs_each, gaps_per_window, common, misfits=64)
    t = full_tick_check(engine, oracle, wl, policies=[0], resolve_modes=(0,))
    assert t.rounds.cpu().tolist() == [jobs_each + common + 1, 1]


def test_launched_rounds_in_several_batches(engine):
    # more jobs than the one block's bitmaps hold: hundreds of launched rounds, in batches of 64, 128 and 256,
    # caps inside a batch and at the edges of one, against the matrix rounds (checked against the oracle elsewhere)
    import paper_2509_19086_amd as P
    jobs, gaps = 140001, 470
    wl = make_workload("tiny", 4, n_gaps=gaps, n_jobs=8)
    rng = np.random.default_rng(4)
    wl.n_jobs = jobs
    wl.seg_off = np.arange(jobs + 1, dtype=np.int64)
    wl.dur = rng.integers(1, 700, size=jobs).astype(np.int32)
    wl.mem = rng.integers(256, 41000, size=jobs).astype(np.int32)
    wl.safe, wl.progress = np.ones(jobs, dtype=np.uint8), np.zeros(jobs, dtype=np.int32)
    wl.wait, wl.sla_class = np.zeros(jobs, dtype=np.int32), np.ones(jobs, dtype=np.uint8)
    wl.W, wl.C = np.full(gaps, 1500, dtype=np.int32), np.full(gaps, 40960, dtype=np.int32)
    t = P.DeviceTick(engine, wl, want_cut=False)
    t.prepare()
    try:
        for cap in (0, 64, 65, 191, 192, 193, 447):
            par = P.Params.make(0, max_rounds=cap)
            t.fit_select(par)
            got = []
            for mode in (1, 0):
                engine.sja_set_resolve_mode(mode)
                t.resolve(par)
                got.append([x.cpu().numpy().copy() for x in (t.grant_job, t.grant_cut, t.grant_score, t.job_gap, t.rounds)])
            for a, b in zip(*got):
                np.testing.assert_array_equal(a, b)
            assert got[1][4].tolist() == [cap or gaps, int(cap == 0)]
    finally:
        engine.sja_set_resolve_mode(0)
