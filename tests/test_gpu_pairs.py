"""Small batches, served pair by pair (k_pairs.h): the smallest and the largest of its range and sizes just beyond,
edges of waves, bit words and sort lengths, bounded rounds, equal keys, masks, and the ordered
forms on the same batches (mode 2 plans them after all), against the oracle."""
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


SHAPES = [(1, 1), (3, 2), (5, 65), (63, 64), (64, 63), (65, 33), (128, 257), (1024, 1), (1024, 256), (1023, 250), (256, 1024), (257, 1020),
          (255, 1025), (64, 4096), (1, 4096), (300, 900), (700, 2990), (1024, 2048), (512, 4096), (1025, 64), (63, 4097), (1024, 2049)]


@pytest.mark.parametrize("gaps,jobs", SHAPES)
@pytest.mark.parametrize("name", ["small", "stress"])
def test_shapes(engine, oracle, name, gaps, jobs):
    wl = make_workload(name, gaps + jobs, n_gaps=gaps, n_jobs=jobs)
    full_tick_check(engine, oracle, wl, policies=[0, 3], resolve_modes=(0, 1, 2))


@pytest.mark.parametrize("max_rounds", [1, 2, 3, 50])
@pytest.mark.parametrize("gaps,jobs", [(40, 30), (257, 700), (200, 900)])
def test_bounded_rounds(engine, oracle, gaps, jobs, max_rounds):
    wl = make_workload("medium", max_rounds, n_gaps=gaps, n_jobs=jobs)
    wl.max_rounds = max_rounds
    full_tick_check(engine, oracle, wl, policies=[1, 2], resolve_modes=(0, 2))


@pytest.mark.parametrize("gaps,jobs", [(100, 90), (300, 250)])
def test_all_want_the_same_jobs(engine, oracle, gaps, jobs):
    # equal gaps and equal keys: a grant per round, in the order of the jobs
    wl = make_workload("medium", 4, n_gaps=gaps, n_jobs=jobs)
    wl.W[:] = wl.W.max()
    wl.C[:] = wl.C.max()
    wl.sla_weight, wl.class0_override = (0, 0, 0), 0
    full_tick_check(engine, oracle, wl, policies=[2, 3], resolve_modes=(0, 2))


def test_nothing_fits(engine, oracle):
    wl = make_workload("small", 4, n_gaps=70, n_jobs=70)
    wl.W[:35] = -1
    wl.C[35:] = -1
    full_tick_check(engine, oracle, wl, policies=[0], resolve_modes=(0, 1, 2))


@pytest.mark.parametrize("gaps,jobs", [(7, 40), (64, 4096), (1000, 200)])
@pytest.mark.parametrize("policy", [0, 1, 2, 3])
def test_one_pass_and_masks(engine, oracle, gaps, jobs, policy):
    import torch
    import paper_2509_19086_amd as P
    wl = make_workload("medium", policy, n_gaps=gaps, n_jobs=jobs)
    rng = np.random.default_rng(gaps)
    held = np.where(rng.random(jobs) < 0.3, 0, -1).astype(np.int32)
    active = (rng.random(gaps) < 0.7).astype(np.uint8)
    t = P.DeviceTick(engine, wl)
    t.prepare()
    par = P.Params.make(policy, wl.wait_scale, wl.sla_weight, wl.class0_override, 0)
    opar = oracle.Params.make(policy, wl.wait_scale, wl.sla_weight, wl.class0_override, 0)
    pd, pp, _ = oracle.prepare(wl.seg_off, wl.dur, wl.mem, wl.safe, wl.progress)
    cut, _ = oracle.fit(wl.seg_off, wl.dur, wl.mem, wl.safe, wl.progress, wl.W, wl.C)
    want = oracle.select(cut, wl.seg_off, pd, pp, opar, wl.wait, wl.sla_class, held, active)
    masks = torch.from_numpy(held).cuda(), torch.from_numpy(active).cuda()
    t.fit()
    for call in (t.select, t.fit_select):
        for x in (t.cand_job, t.cand_cut, t.cand_score):
            x.fill_(-9)
        call(par, *masks)
        for x, y in zip((t.cand_job, t.cand_cut, t.cand_score), want):
            np.testing.assert_array_equal(x.cpu().numpy(), y)
    # the rounds after the one pass, also those that evaluate the pairs again
    want = oracle.resolve(cut, wl.seg_off, pd, pp, opar, wl.wait, wl.sla_class)
    try:
        for mode in (0, 1, 2):
            engine.sja_set_resolve_mode(mode)
            t.resolve(par)
            for x, y in zip((t.grant_job, t.grant_cut, t.grant_score, t.job_gap), want[:4]):
                np.testing.assert_array_equal(x.cpu().numpy(), y, err_msg=f"mode {mode}")
            assert t.rounds.cpu().tolist() == [want[4], want[5]]
    finally:
        engine.sja_set_resolve_mode(0)
