"""The best reply per gap by atoms (k_range_select): chunks of one and of many positions, windows that repeat or lie far
apart, jobs that end inside a chunk, sizes around its tiles, equal keys in one and in several jobs, held jobs and gaps
that are off, the area score, and batches that are left to the stepping form, against the oracle."""
import numpy as np
import pytest

from gen import make_workload
from test_gpu_area import area_tick_check
from test_gpu_parity import fused_check

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def engine():
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    import paper_2509_19086_amd as P
    eng = P.Engine(0)
    yield eng
    eng.sja_set_score(0)


@pytest.mark.parametrize("name,gaps,jobs", [("stress", 1025, 255), ("stress", 1300, 4097), ("large", 3000, 1111), ("medium", 2048, 2049),
                                            ("stress", 9000, 700), ("stress", 70, 33000), ("medium", 5000, 33), ("large", 1100, 1)])
def test_shapes(engine, oracle, name, gaps, jobs):
    fused_check(engine, oracle, make_workload(name, gaps, n_gaps=gaps, n_jobs=jobs), policies=[1, 3], resolve=False)


@pytest.mark.parametrize("windows", ["equal", "far", "negative", "huge"])
def test_windows(engine, oracle, windows):
    wl = make_workload("medium", 3, n_gaps=2500, n_jobs=900)
    rng = np.random.default_rng(1)
    if windows == "equal":
        wl.W[:] = 700
    elif windows == "far":
        wl.W[:] = (2.0 ** (31 * rng.random(len(wl.W)))).astype(np.int64) - 1
    elif windows == "negative":
        wl.W[:1200] = rng.integers(-2**31, 0, size=1200)
        wl.C[::7] = -5
    else:
        wl.W[:] = 2**31 - 1
        wl.W[::3] = -2**31
    fused_check(engine, oracle, wl, policies=[0, 2, 3], resolve=False)


@pytest.mark.parametrize("jobs", [300, 2600])
@pytest.mark.parametrize("kind", ["weights", "memory", "twins"])
def test_equal_keys(engine, oracle, jobs, kind):
    # weight 0: every reply of a tier has the same key; no memory: every F is 0; twins: pairs of equal (score, F), and
    # under MIXED equal scores of different F
    wl = make_workload("medium", 5, n_gaps=1500, n_jobs=jobs)
    if kind == "weights":
        wl.sla_weight, wl.class0_override = (0, 0, 0), 0
    elif kind == "memory":
        wl.mem[:] = 0
    else:
        half = jobs // 2
        n, lens = int(wl.seg_off[half]), np.diff(wl.seg_off[:half + 1])
        wl.n_jobs = 2 * half
        wl.seg_off = np.concatenate([[0], np.cumsum(np.tile(lens, 2))]).astype(np.int64)
        wl.dur, wl.safe = np.tile(wl.dur[:n], 2), np.tile(wl.safe[:n], 2)
        wl.mem = np.concatenate([wl.mem[:n], 2 * wl.mem[:n]]).astype(np.int32)
        wl.C[:] = int(wl.mem.max()) + 1
        wl.progress = np.tile(wl.progress[:half], 2)
        wl.sla_class = np.ones(2 * half, dtype=np.uint8)
        # the weight scale + wait is half as large where the memory is twice as large
        wl.wait = np.repeat([wl.wait_scale + 14, 7], half).astype(np.int32)
    fused_check(engine, oracle, wl, policies=[0, 2, 3], resolve=False)


@pytest.mark.parametrize("held_share,on_share", [(0.3, 0.6), (1.0, 1.0), (0.0, 0.0)])
def test_masks(engine, oracle, held_share, on_share):
    wl = make_workload("stress", 6, n_gaps=2100, n_jobs=1500)
    rng = np.random.default_rng(2)
    held = np.where(rng.random(wl.n_jobs) < held_share, 3, -1).astype(np.int32)
    act = (rng.random(wl.n_gaps) < on_share).astype(np.uint8)
    fused_check(engine, oracle, wl, policies=[0, 3], held=held, act=act)


def test_area_score(engine, oracle):
    area_tick_check(engine, oracle, make_workload("medium", 8, n_gaps=2100, n_jobs=1300), policies=[0, 3], fused=True)


def test_too_many_capacities(engine, oracle):
    wl = make_workload("medium", 9, n_gaps=2500, n_jobs=1200)
    wl.C = np.linspace(3000, 90000, 65).astype(np.int32)[np.arange(2500) % 65]
    fused_check(engine, oracle, wl, policies=[0, 3], resolve=False)


@pytest.mark.parametrize("max_rounds", [1, 6])
def test_scanning_rounds_without_a_matrix(engine, oracle, max_rounds):
    import paper_2509_19086_amd as P
    wl = make_workload("medium", 4, n_gaps=1100, n_jobs=2100)
    t = P.DeviceTick(engine, wl, want_cut=False)
    t.prepare()
    par, opar = (m.Params.make(3, wl.wait_scale, wl.sla_weight, wl.class0_override, max_rounds) for m in (P, oracle))
    t.fit_select(par)
    pd, pp, _ = oracle.prepare(wl.seg_off, wl.dur, wl.mem, wl.safe, wl.progress)
    cut, _ = oracle.fit(wl.seg_off, wl.dur, wl.mem, wl.safe, wl.progress, wl.W, wl.C, False)
    want = oracle.resolve(cut, wl.seg_off, pd, pp, opar, wl.wait, wl.sla_class)
    try:
        engine.sja_set_resolve_mode(1)
        t.resolve(par)
    finally:
        engine.sja_set_resolve_mode(0)
    for x, y in zip((t.grant_job, t.grant_cut, t.grant_score, t.job_gap), want[:4]):
        np.testing.assert_array_equal(x.cpu().numpy(), y)
    assert t.rounds.cpu().tolist() == [want[4], want[5]]
