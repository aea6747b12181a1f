"""sja_select: along the matrix up to 2^27 pairs, at the edges of blocks of jobs and of classes, with equal keys and masks,
each select after a resolve of the one before, against the oracle; larger batches along the chunks of the plan of the fit
(k_range_select), fit -> select likewise (tests/test_gpu_floor.py has the form of the largest)."""
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


def check(engine, oracle, wl, policies, held=None, act=None):
    import torch
    import paper_2509_19086_amd as P
    t = P.DeviceTick(engine, wl)
    t.prepare()
    t.fit()
    pd, pp, _ = oracle.prepare(wl.seg_off, wl.dur, wl.mem, wl.safe, wl.progress)
    cut, _ = oracle.fit(wl.seg_off, wl.dur, wl.mem, wl.safe, wl.progress, wl.W, wl.C, False)
    dev = lambda x: None if x is None else torch.from_numpy(x).cuda()
    d_held, d_act = dev(held), dev(act)
    for policy in policies:
        args = (policy, wl.wait_scale, wl.sla_weight, wl.class0_override, 2)
        par, opar = P.Params.make(*args), oracle.Params.make(*args)
        engine.sja_select(par, t.wait, t.sla_class, d_held, d_act, t.cand_job, t.cand_cut, t.cand_score)
        want = oracle.select(cut, wl.seg_off, pd, pp, opar, wl.wait, wl.sla_class, held, act)
        for got, x in zip((t.cand_job, t.cand_cut, t.cand_score), want):
            np.testing.assert_array_equal(got.cpu().numpy(), x)
        t.resolve(par)          # writes what the select before it left, and the next one works all the same


@pytest.mark.parametrize("name,gaps,jobs", [("stress", 1300, 14000), ("large", 1025, 16385), ("medium", 21000, 2049), ("small", 300, 56000),
                                            ("tiny", 80, 220001), ("large", 9000, 1900)])
def test_shapes(engine, oracle, name, gaps, jobs):
    check(engine, oracle, make_workload(name, gaps, n_gaps=gaps, n_jobs=jobs), (0, 1, 2, 3))


@pytest.mark.parametrize("caps", [1, 64, 65])
def test_classes(engine, oracle, caps):
    wl = make_workload("medium", 2, n_gaps=1500, n_jobs=14500)
    wl.C = np.linspace(2000, 90000, caps).astype(np.int32)[np.arange(1500) % caps]
    check(engine, oracle, wl, (0, 3))


@pytest.mark.parametrize("kind", ["weights", "memory", "profile"])
def test_equal_keys(engine, oracle, kind):
    # every key of a tier the same; every F 0; every job of the same profile, some with equal waits
    wl = make_workload("medium", 5, n_gaps=1500, n_jobs=14500)
    if kind == "weights":
        wl.sla_weight, wl.class0_override = (0, 0, 0), 0
    elif kind == "memory":
        wl.mem[:] = 0
    else:
        n = wl.n_jobs
        wl.dur, wl.mem, wl.safe = (np.tile(x[:512], n) for x in (wl.dur, wl.mem, wl.safe))
        wl.progress[:] = 0
        wl.wait = np.random.default_rng(1).integers(10**6, 10**6 + 5000, size=n).astype(np.int32)
    check(engine, oracle, wl, (0, 2, 3))


@pytest.mark.parametrize("held_share,on_share", [(0.5, 0.5), (1.0, 1.0)])
def test_masks(engine, oracle, held_share, on_share):
    wl = make_workload("large", 3, n_gaps=1500, n_jobs=13000)
    rng = np.random.default_rng(4)
    held = np.where(rng.random(wl.n_jobs) < held_share, 0, -1).astype(np.int32)
    check(engine, oracle, wl, (1, 3), held, (rng.random(wl.n_gaps) < on_share).astype(np.uint8))


# about 2^27 pairs, from which on a select goes along the chunks, some gaps of each against the oracle: a gap's best reply does
# not depend on the other gaps
@pytest.mark.parametrize("name,gaps,jobs,caps", [("stress", 2100, 65600, 0), ("large", 22000, 6144, 0), ("large", 22000, 6143, 0),
                                                 ("medium", 8300, 16400, 1), ("medium", 8300, 16400, 64), ("medium", 8300, 16400, 65)])
def test_large(engine, oracle, name, gaps, jobs, caps):
    import paper_2509_19086_amd as P
    wl = make_workload(name, 7, n_gaps=gaps, n_jobs=jobs)
    if caps:
        wl.C = np.linspace(2000, 90000, caps).astype(np.int32)[np.arange(gaps) % caps]
    t = P.DeviceTick(engine, wl)
    t.prepare()
    rows = np.unique(np.linspace(0, gaps - 1, 67).astype(np.int64))
    pd, pp, _ = oracle.prepare(wl.seg_off, wl.dur, wl.mem, wl.safe, wl.progress)
    cut, _ = oracle.fit(wl.seg_off, wl.dur, wl.mem, wl.safe, wl.progress, wl.W[rows], wl.C[rows], False)
    for policy in (0, 3):
        args = (policy, wl.wait_scale, wl.sla_weight, wl.class0_override, wl.max_rounds)
        want = oracle.select(cut, wl.seg_off, pd, pp, oracle.Params.make(*args), wl.wait, wl.sla_class)
        par = P.Params.make(*args)
        for call in (lambda: t.fit_select(par), lambda: (t.fit(), t.select(par))):
            call()
            for got, x in zip((t.cand_job, t.cand_cut, t.cand_score), want):
                np.testing.assert_array_equal(got.cpu().numpy()[rows], x)
