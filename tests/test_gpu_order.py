"""The gaps' orders of small batches (k_order_pairs): after sja_fit from its matrix, after sja_fit_select by searching or
from the atoms of k_pair_atoms, with and without a histogram that cuts the order off, at the edges of its rooms, with
keys that are equal and with keys whose digests are, against the oracle."""
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


def check(engine, oracle, wl, policies):
    import paper_2509_19086_amd as P
    t = P.DeviceTick(engine, wl)
    t.prepare()
    pd, pp, _ = oracle.prepare(wl.seg_off, wl.dur, wl.mem, wl.safe, wl.progress)
    cut, _ = oracle.fit(wl.seg_off, wl.dur, wl.mem, wl.safe, wl.progress, wl.W, wl.C, False)
    for policy in policies:
        args = (policy, wl.wait_scale, wl.sla_weight, wl.class0_override, wl.max_rounds)
        par, opar = P.Params.make(*args), oracle.Params.make(*args)
        want = oracle.resolve(cut, wl.seg_off, pd, pp, opar, wl.wait, wl.sla_class)
        best = oracle.select(cut, wl.seg_off, pd, pp, opar, wl.wait, wl.sla_class)
        for first in (t.fit, lambda: t.fit_select(par)):
            first()
            if first != t.fit:
                for got, x in zip((t.cand_job, t.cand_cut, t.cand_score), best):
                    np.testing.assert_array_equal(got.cpu().numpy(), x)
            t.resolve(par)
            for got, x in zip((t.grant_job, t.grant_cut, t.grant_score, t.job_gap), want[:4]):
                np.testing.assert_array_equal(got.cpu().numpy(), x)
            assert t.rounds.cpu().tolist() == [want[4], want[5]]


@pytest.mark.parametrize("name,gaps,jobs", [("stress", 512, 4096), ("stress", 257, 2049), ("medium", 700, 2048), ("large", 513, 1024),
                                            ("small", 300, 1023), ("medium", 130, 512), ("tiny", 3, 128), ("stress", 1024, 513)])
def test_rooms(engine, oracle, name, gaps, jobs):
    check(engine, oracle, make_workload(name, jobs, n_gaps=gaps, n_jobs=jobs), (0, 2, 3))


@pytest.mark.parametrize("gaps,jobs", [(150, 4000), (600, 1500), (20, 100)])
def test_equal_digests(engine, oracle, gaps, jobs):
    # score 2^45 + 3 * 2^22 of the even jobs, one more of the odd ones: alike in 44 bits behind the leading one
    wl = make_workload("tiny", 1, n_gaps=gaps, n_jobs=jobs)
    odd = np.arange(jobs) % 2 == 1
    wl.seg_off = np.arange(jobs + 1, dtype=np.int64)
    wl.dur = np.ones(jobs, dtype=np.int32)
    wl.mem = np.where(odd, 2**22 + 1, 2**22).astype(np.int32)
    wl.safe = np.ones(jobs, dtype=np.uint8)
    wl.progress = np.zeros(jobs, dtype=np.int32)
    wl.wait = (np.where(odd, 2**23 + 1, 2**23 + 3) - wl.wait_scale).astype(np.int32)
    wl.sla_class = (np.arange(jobs) // 2 % 3).astype(np.uint8)
    wl.W[:] = 5
    wl.C[:] = 2**22 + np.arange(gaps) % 2
    check(engine, oracle, wl, (1, 3))
    wl.wait[:] = 7          # and all keys of a tier the same
    wl.mem[:] = 2**20
    check(engine, oracle, wl, (1, 3))


# scores that differ by less than the bits behind a digest's would tell, just inside and just outside of what it holds whole:
# 0 to 2 (which share a leading digit, or have none), and 2^44 + 2^24 + 0, 3 and 4, half of that, twice that
@pytest.mark.parametrize("gaps,jobs", [(150, 4000), (20, 100)])
@pytest.mark.parametrize("e", [0, 1, 43, 44, 45])
def test_scores_at_the_digests_edges(engine, oracle, gaps, jobs, e):
    wl = make_workload("tiny", 1, n_gaps=gaps, n_jobs=jobs)
    rng = np.random.default_rng(e)
    wl.seg_off = np.arange(jobs + 1, dtype=np.int64)
    wl.dur = np.ones(jobs, dtype=np.int32)
    wl.safe = np.ones(jobs, dtype=np.uint8)
    wl.progress = np.zeros(jobs, dtype=np.int32)
    if e < 2:
        wl.mem = rng.integers(0, 2 + 2 * e, size=jobs).astype(np.int32)
        mult = np.where(rng.random(jobs) < 0.5, 1, 2)
    else:
        at = rng.integers(0, 3, size=jobs)
        wl.mem = (2**22 + at).astype(np.int32)
        mult = 2**(e - 22) + ((4 - at) << (e - 44) if e > 44 else (4 - at) >> (44 - e))
    wl.wait_scale, wl.wait = 1, (mult - 1).astype(np.int32)
    wl.sla_class = rng.integers(0, 3, size=jobs).astype(np.uint8)
    wl.W[:] = 5
    wl.C[:] = 2**22 + np.arange(gaps) % 3
    check(engine, oracle, wl, (0, 1, 3))


# one list for all gaps, so that every round passes an entry of each: less than the 16 that are read ahead, one, two and many
# times 16 and 64 of them
@pytest.mark.parametrize("gaps,jobs", [(1, 5), (63, 64), (65, 65), (72, 300), (128, 127), (136, 700), (256, 1024), (257, 1024), (333, 90), (1000, 70), (1024, 64)])
@pytest.mark.parametrize("max_rounds", [0, 60])
def test_rounds_along_one_list(engine, oracle, gaps, jobs, max_rounds):
    wl = make_workload("tiny", 3, n_gaps=gaps, n_jobs=jobs)
    rng = np.random.default_rng(gaps)
    wl.seg_off = np.arange(jobs + 1, dtype=np.int64)
    wl.dur = np.ones(jobs, dtype=np.int32)
    wl.mem = rng.integers(1000, 2000, size=jobs).astype(np.int32)
    wl.safe = np.ones(jobs, dtype=np.uint8)
    wl.progress = np.zeros(jobs, dtype=np.int32)
    wl.wait = rng.integers(0, 1000, size=jobs).astype(np.int32)
    wl.sla_class = rng.integers(0, 3, size=jobs).astype(np.uint8)
    wl.W[:] = 5
    wl.C = rng.choice(np.array([2000, 1990], np.int32), size=gaps)
    wl.max_rounds = max_rounds
    check(engine, oracle, wl, (1, 3))
