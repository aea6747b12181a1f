"""What the grants are built from, at the edges of its forms, against the oracle: list records (four bytes
while job ids fit 19 bits, eight beyond), the order of gaps and atoms, list entries, searched rounds, and
selection with gaps switched off."""
import numpy as np
import pytest

from gen import make_workload
from helpers import forms, in_mode
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
    t = full_tick_check(engine, oracle, wl, policies=[1], resolve_modes=(0,))
    jobs = t.grant_job.cpu().numpy()
    assert (jobs > n_jobs - 50).any() and (jobs < 50).any()


@pytest.mark.parametrize("classes,all_safe", [(64, True), (40, True), (1, False)])
def test_entries_by_groups_of_classes(engine, oracle, classes, all_safe):
    # an atom has a range of positions, and with it entries, in every class whose capacity holds it: one, many and
    # as many classes as the tables hold, every boundary safe or not
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


@pytest.mark.parametrize("caps,n_gaps,n_jobs,max_rounds", [(65, 65, 255, 0), (90, 301, 257, 0), (90, 301, 257, 3), (65, 1200, 300, 9),
                                                           (200, 203, 1, 0), (120, 121, 513, 5)])
def test_rounds_that_search(engine, oracle, caps, n_gaps, n_jobs, max_rounds):
    # more capacities than the class tables hold, after the fused call: pairs are searched one by one where a
    # capacity has few positions, stepped through where it has many; batches of rounds cut off by the cap
    import oracle as O
    import paper_2509_19086_amd as P
    wl = make_workload("stress", caps, n_gaps=n_gaps, n_jobs=n_jobs)
    rng = np.random.default_rng(n_gaps)
    pool = np.sort(rng.choice(np.arange(2000, 150000), size=caps, replace=False)).astype(np.int32)
    wl.C = pool[np.concatenate([np.arange(caps), rng.integers(0, caps, size=n_gaps - caps)])]
    wl.wait[: n_jobs // 3] = 7                      # equal scores
    t = P.DeviceTick(engine, wl)
    t.prepare()
    pd, pp, _ = O.prepare(wl.seg_off, wl.dur, wl.mem, wl.safe, wl.progress)
    cut, _ = O.fit(wl.seg_off, wl.dur, wl.mem, wl.safe, wl.progress, wl.W, wl.C)
    for policy in (0, 1, 3):
        par = P.Params.make(policy, max_rounds=max_rounds)
        opar = O.Params.make(policy, max_rounds=max_rounds)
        gj, gc, gs, jg, rounds, stable = O.resolve(cut, wl.seg_off, pd, pp, opar, wl.wait, wl.sla_class)
        for form in forms(wl):
            with in_mode(engine, form):
                t.fit_select(par)
                t.resolve(par)
            for got, want in ((t.grant_job, gj), (t.grant_cut, gc), (t.grant_score, gs), (t.job_gap, jg)):
                np.testing.assert_array_equal(got.cpu().numpy(), want)
            assert t.rounds.cpu().tolist() == [rounds, stable]


@pytest.mark.parametrize("n_gaps", [1, 15, 16, 17, 63, 65])
def test_select_with_gaps_switched_off(engine, oracle, n_gaps, form):
    # the masked pass and the reduction at the edges of a chunk of positions and of a block's gaps
    import torch
    import paper_2509_19086_amd as P
    wl = make_workload("medium", n_gaps, n_gaps=n_gaps, n_jobs=700)
    t = P.DeviceTick(engine, wl)
    t.prepare()
    t.fit()
    cut = t.cut.cpu().numpy()
    rng = np.random.default_rng(n_gaps)
    active = (rng.random(n_gaps) < 0.6).astype(np.uint8)
    held = np.where(rng.random(700) < 0.3, 0, -1).astype(np.int32)
    masked = np.where((held < 0)[None, :] & (active != 0)[:, None], cut, -1)
    pd, pp, _ = oracle.prepare(wl.seg_off, wl.dur, wl.mem, wl.safe, wl.progress)
    for policy in (0, 1, 2, 3):
        want = oracle.select(masked, wl.seg_off, pd, pp, oracle.Params.make(policy), wl.wait, wl.sla_class)
        engine.sja_select(P.Params.make(policy), t.wait, t.sla_class,
                          torch.from_numpy(held).cuda(), torch.from_numpy(active).cuda(), t.cand_job, t.cand_cut, t.cand_score)
        for got, w in zip((t.cand_job, t.cand_cut, t.cand_score), want):
            np.testing.assert_array_equal(got.cpu().numpy(), w)


@pytest.mark.parametrize("jobs_per_run", [2, 16, 33, 150])
def test_equal_scores_ordered_by_the_second_key(engine, oracle, jobs_per_run):
    # MIXED: jobs whose F x multiplier is equal while F is not, in runs shorter and longer than those put in
    # order in place, the smaller F first; enough other atoms that the sort is not one block's
    wl = make_workload("small", jobs_per_run, n_gaps=150, n_jobs=1200)
    wl.safe[:] = 1
    wl.sla_class[:] = 1
    wl.progress[:] = 0
    n = jobs_per_run
    L = int(wl.seg_off[1])
    for j in range(n):
        a = int(wl.seg_off[j])
        wl.dur[a:a + L], wl.mem[a:a + L] = 1, 512 if j % 2 == 0 else 1024        # key 512 * 2000 == 1024 * 1000 per tick
        wl.wait[j] = 1000 if j % 2 == 0 else 0
    full_tick_check(engine, oracle, wl, policies=[3], resolve_modes=(0,))


@pytest.mark.parametrize("n_gaps", [4 * 32768, 4 * 32768 + 1, 270001])
def test_rounds_that_search_over_more_gaps_than_a_launch_takes(engine, oracle, n_gaps):
    # four positions per row of blocks: on both sides of a launch's rows, and beyond what any one launch takes
    import paper_2509_19086_amd as P
    wl = make_workload("tiny", 9, n_gaps=n_gaps, n_jobs=7)
    rng = np.random.default_rng(n_gaps)
    wl.W = rng.integers(10, 20, size=n_gaps).astype(np.int32)                  # too short for any job,
    wl.W[-40:] = rng.integers(50, 4000, size=40)                               # but for a few at the end of the order
    wl.C = (20000 + np.arange(n_gaps) // 8).astype(np.int32)                   # eight gaps per capacity
    wl.dur = np.maximum(wl.dur, 25).astype(np.int32)
    t = P.DeviceTick(engine, wl)
    t.prepare()
    pd, pp, _ = oracle.prepare(wl.seg_off, wl.dur, wl.mem, wl.safe, wl.progress)
    cut, _ = oracle.fit(wl.seg_off, wl.dur, wl.mem, wl.safe, wl.progress, wl.W, wl.C)
    for policy in (0, 3):
        t.fit_select(P.Params.make(policy))
        t.resolve(P.Params.make(policy))
        gj, gc, gs, jg, rounds, stable = oracle.resolve(cut, wl.seg_off, pd, pp, oracle.Params.make(policy), wl.wait, wl.sla_class)
        assert (gj[-40:] >= 0).any()
        for got, want in ((t.grant_job, gj), (t.grant_cut, gc), (t.grant_score, gs), (t.job_gap, jg)):
            np.testing.assert_array_equal(got.cpu().numpy(), want)
        assert t.rounds.cpu().tolist() == [rounds, stable]


@pytest.mark.parametrize("name,n_gaps,n_jobs,classes,log_windows",
                         [("medium", 32769, 131, 5, False), ("stress", 40001, 900, 8, False), ("stress", 12000, 70, 64, True),
                          ("stress", 30001, 3, 64, True), ("tiny", 140003, 33, 3, True)])
def test_entries_of_large_batches(engine, oracle, name, n_gaps, n_jobs, classes, log_windows):
    # more gaps, or more list blocks, than those whose windows and first positions fit LDS; few and many atoms
    # to a wave's turn
    wl = make_workload(name, n_gaps, n_gaps=n_gaps, n_jobs=n_jobs)
    rng = np.random.default_rng(n_gaps)
    caps = np.sort(rng.choice(np.arange(2000, 150000), size=classes, replace=False)).astype(np.int32)
    wl.C = caps[rng.integers(0, classes, size=n_gaps)]
    if log_windows:
        wl.W = np.floor(10 * 10.0 ** (4 * rng.random(n_gaps))).astype(np.int32)
    wl.max_rounds = 6
    full_tick_check(engine, oracle, wl, policies=[0, 3], resolve_modes=(0,))


@pytest.mark.parametrize("n_jobs,longest", [(16383, 40), (16385, 40), (16386, 600), (20001, 1100)])
def test_select_from_many_jobs(engine, oracle, n_jobs, longest):
    # one, four, two and one job to a wave, some without anything left, the last wave without its full number
    wl = make_workload("tiny", 5, n_gaps=40, n_jobs=8)
    rng = np.random.default_rng(n_jobs)
    lens = rng.integers(1, longest + 1, size=n_jobs)
    lens[::3] = longest
    wl.n_jobs = n_jobs
    wl.seg_off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    S = int(wl.seg_off[-1])
    wl.dur, wl.mem = rng.integers(1, 30, size=S).astype(np.int32), rng.integers(256, 9000, size=S).astype(np.int32)
    wl.safe = (rng.random(S) < np.repeat(rng.choice([0.05, 0.3, 1.0], size=n_jobs), lens)).astype(np.uint8)
    wl.progress = np.where(rng.random(n_jobs) < 0.1, lens, (rng.random(n_jobs) * lens)).astype(np.int32)
    wl.wait, wl.sla_class = rng.integers(0, 100, size=n_jobs).astype(np.int32), rng.integers(0, 3, size=n_jobs).astype(np.uint8)
    full_tick_check(engine, oracle, wl, policies=[1, 3], check_resolve=False)


@pytest.mark.parametrize("how", ["plain", "area", "hysteresis", "limits"])
def test_select_from_jobs_of_few_and_of_many_cuts(engine, oracle, how):
    # the keys go along a job's atoms or along all its prefixes by how many of those are atoms: shares on both sides of the
    # line, and jobs with every boundary safe or only the end
    from test_gpu_area import area_tick_check
    from test_gpu_hysteresis import hysteresis_tick_check
    from test_gpu_limits import limited_tick_check
    wl = make_workload("medium", 17, n_gaps=1100, n_jobs=700)
    rng = np.random.default_rng(3)
    lens = np.diff(wl.seg_off)
    share = rng.choice([0.0, 0.1, 0.3, 0.36, 0.375, 0.39, 0.6, 0.9, 0.953, 0.98, 1.0], size=700)
    wl.safe = (rng.random(int(wl.seg_off[-1])) < np.repeat(share, lens)).astype(np.uint8)
    wl.progress = np.where(rng.random(700) < 0.3, lens - rng.integers(0, 3, size=700), wl.progress).astype(np.int32)
    if how == "plain":
        full_tick_check(engine, oracle, wl, policies=[0, 3], resolve_modes=(1,))
    elif how == "area":
        area_tick_check(engine, oracle, wl, [1, 3], False)
    elif how == "limits":
        limited_tick_check(engine, oracle, wl, "all", policy=3)
    else:
        hysteresis_tick_check(engine, oracle, wl, "gap_capacities", [2, 3], False)
        hysteresis_tick_check(engine, oracle, wl, "gap_capacities_big_gain", [0], False)
