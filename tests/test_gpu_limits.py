"""GPU parity under admission limits (power trace under a cap, per-job
deadline, minimum / maximum subjob duration) and for the covering-capacity
mapping, against the CPU oracle.  Integer work: bit-exact."""
import numpy as np
import pytest

from gen import make_channels, make_gaps, make_workload
from helpers import forms, in_mode

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def engine():
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    import paper_2509_19086_amd as P
    eng = P.Engine(0)
    yield eng
    eng.sja_set_limits(None)


def _limit_sets(wl, power):
    p80 = int(np.percentile(power, 80))
    w_hi = int(wl.W.max())
    return {
        "tau_min": (dict(tau_min=max(1, w_hi // 10)), False, False),
        "tau_max": (dict(tau_max=w_hi // 2), False, False),
        "power": (dict(power_cap=p80), True, False),
        "deadline": (dict(now=5), False, True),
        "all": (dict(tau_min=max(1, w_hi // 14), tau_max=(2 * w_hi) // 3, power_cap=int(np.percentile(power, 85)),
                     now=7), True, True),
        "nothing_passes": (dict(tau_max=0), True, True),
        "limits_that_never_bind": (dict(), True, False),
    }


def limited_tick_check(engine, oracle, wl, which, policy=None, fused=False):
    import torch
    import paper_2509_19086_amd as P
    power, deadline = make_channels(wl, wl.seed)
    kw, use_pow, use_dl = _limit_sets(wl, power)[which]
    if which == "limits_that_never_bind":
        kw = dict(power_cap=int(power.max()))
    policy = wl.policy if policy is None else policy
    t = P.DeviceTick(engine, wl, want_bits=not fused, want_cut=not fused)
    d_power = torch.from_numpy(power).cuda() if use_pow else None
    d_deadline = torch.from_numpy(deadline).cuda() if use_dl else None
    engine.sja_set_limits(P.Limits.make(**kw), d_power, d_deadline)
    olim = oracle.Limits.make(**kw)
    try:
        t.prepare()
        par = P.Params.make(policy, wl.wait_scale, wl.sla_weight, wl.class0_override, 0)
        opar = oracle.Params.make(policy, wl.wait_scale, wl.sla_weight, wl.class0_override, 0)
        pd, pp, ps = oracle.prepare(wl.seg_off, wl.dur, wl.mem, wl.safe, wl.progress)
        cut, bits = oracle.fit_limited(wl.seg_off, wl.dur, wl.mem, wl.safe, wl.progress, wl.W, wl.C, olim,
                                       power if use_pow else None, deadline if use_dl else None, True)
        best = oracle.select(cut, wl.seg_off, pd, pp, opar, wl.wait, wl.sla_class)
        grants = oracle.resolve(cut, wl.seg_off, pd, pp, opar, wl.wait, wl.sla_class)
        for form in forms(wl):
            for out in (t.cand_job, t.cand_cut, t.cand_score, t.grant_job, t.grant_cut, t.grant_score, t.job_gap):
                out.fill_(-5)
            with in_mode(engine, form):
                if fused:
                    t.fit_select(par)
                else:
                    t.fit()
                    t.select(par)
                t.resolve(par)
            torch.cuda.synchronize()
            # the caller-visible running tables do not depend on the limits
            np.testing.assert_array_equal(t.pre_dur.cpu().numpy().astype(np.int64), pd)
            np.testing.assert_array_equal(t.pre_peak.cpu().numpy().astype(np.int64), pp)
            np.testing.assert_array_equal(t.prev_safe.cpu().numpy(), ps)
            if not fused:
                np.testing.assert_array_equal(t.cut.cpu().numpy(), cut)
                np.testing.assert_array_equal(t.bits.cpu().numpy().view(np.uint32), bits)
            for got, want in zip((t.cand_job, t.cand_cut, t.cand_score, t.grant_job, t.grant_cut, t.grant_score, t.job_gap), best + grants[:4]):
                np.testing.assert_array_equal(got.cpu().numpy(), want, err_msg=f"form {form}")
            assert t.rounds.cpu().tolist() == list(grants[4:])
        return (cut >= 0).mean()
    finally:
        engine.sja_set_limits(None)


WHICH = ["tau_min", "tau_max", "power", "deadline", "all", "nothing_passes", "limits_that_never_bind"]


@pytest.mark.parametrize("which", WHICH)
def test_tiny_limits(engine, oracle, which):
    for policy in (0, 3):
        limited_tick_check(engine, oracle, make_workload("tiny", 2), which, policy)


@pytest.mark.parametrize("which", WHICH)
@pytest.mark.parametrize("fused", [False, True])
def test_small_limits(engine, oracle, which, fused):
    density = limited_tick_check(engine, oracle, make_workload("small", 1), which, fused=fused)
    if which == "nothing_passes":
        assert density == 0.0
    else:
        assert density > 0.02


def test_medium_all_limits(engine, oracle):
    limited_tick_check(engine, oracle, make_workload("medium", 0), "all")


def test_ragged_all_limits(engine, oracle):
    limited_tick_check(engine, oracle, make_workload("stress", 7, n_gaps=333, n_jobs=1111), "all", fused=True)
    limited_tick_check(engine, oracle, make_workload("large", 7, n_gaps=130, n_jobs=70), "all")


def test_limits_differ_from_the_plain_fit_and_clear_again(engine, oracle):
    import torch
    import paper_2509_19086_amd as P
    wl = make_workload("small", 3)
    power, deadline = make_channels(wl, 3)
    t = P.DeviceTick(engine, wl, want_bits=False)
    plain, _ = oracle.fit(wl.seg_off, wl.dur, wl.mem, wl.safe, wl.progress, wl.W, wl.C, False)
    engine.sja_set_limits(P.Limits.make(tau_max=500), None, None)
    t.prepare(); t.fit(); torch.cuda.synchronize()
    assert (t.cut.cpu().numpy() != plain).mean() > 0.05
    engine.sja_set_limits(None)
    t.fit(); torch.cuda.synchronize()                          # takes effect at the next prepare only
    assert (t.cut.cpu().numpy() != plain).mean() > 0.05
    t.prepare(); t.fit(); torch.cuda.synchronize()
    np.testing.assert_array_equal(t.cut.cpu().numpy(), plain)
    with pytest.raises(RuntimeError):
        engine.sja_set_limits(P.Limits.make(tau_min=-1))
    with pytest.raises(RuntimeError):
        engine.sja_set_limits(P.Limits.make(tau_max=-2))


def test_chain_of_ticks_under_limits(engine, oracle, form):
    """sja_advance rebuilds the moved jobs under the limits their prepare used."""
    import torch
    import paper_2509_19086_amd as P
    wl = make_workload("small", 6)
    power, deadline = make_channels(wl, 6)
    kw = dict(tau_min=60, tau_max=1500, power_cap=int(np.percentile(power, 90)), now=3)
    d_power, d_deadline = torch.from_numpy(power).cuda(), torch.from_numpy(deadline).cuda()
    par = P.Params.make(3, wl.wait_scale, wl.sla_weight, wl.class0_override, 0)
    opar = oracle.Params.make(3, wl.wait_scale, wl.sla_weight, wl.class0_override, 0)
    olim = oracle.Limits.make(**kw)
    t = P.DeviceTick(engine, wl, want_bits=False, want_cut=False)
    engine.sja_set_limits(P.Limits.make(**kw), d_power, d_deadline)
    try:
        t.prepare()
        engine.sja_set_limits(None)                            # the chain keeps the limits of its prepare
        progress, wait = wl.progress.copy(), wl.wait.copy()
        moved = 0
        for tick in range(5):
            W, C = (wl.W, wl.C) if tick == 0 else make_gaps("small", 6, tick)
            t.set_gaps(W, C)
            t.fit_select(par); t.resolve(par)
            pd, pp, _ = oracle.prepare(wl.seg_off, wl.dur, wl.mem, wl.safe, progress)
            cut, _ = oracle.fit_limited(wl.seg_off, wl.dur, wl.mem, wl.safe, progress, W, C, olim, power, deadline)
            gj, gc, gs, jg, rounds, stable = oracle.resolve(cut, wl.seg_off, pd, pp, opar, wait, wl.sla_class)
            np.testing.assert_array_equal(t.grant_job.cpu().numpy(), gj, err_msg=f"tick {tick}")
            np.testing.assert_array_equal(t.grant_cut.cpu().numpy(), gc, err_msg=f"tick {tick}")
            np.testing.assert_array_equal(t.grant_score.cpu().numpy(), gs, err_msg=f"tick {tick}")
            t.advance(1000)
            torch.cuda.synchronize()
            p2, w2, m = oracle.advance(wl.seg_off, pd, pp, W, C, gj, gc, jg, progress, wait, 1000)
            np.testing.assert_array_equal(t.progress.cpu().numpy(), p2)
            assert t.metrics.cpu().tolist() == m.tolist()
            moved += int(m[2])
            progress, wait = p2, w2
        assert moved > 100
    finally:
        engine.sja_set_limits(None)


@pytest.mark.parametrize("name,seed", [("tiny", 0), ("small", 2), ("medium", 1)])
def test_cover(engine, oracle, name, seed):
    import torch
    import paper_2509_19086_amd as P
    wl = make_workload(name, seed)
    t = P.DeviceTick(engine, wl, want_bits=False, want_cut=False)
    par = P.Params.make(wl.policy, wl.wait_scale, wl.sla_weight, wl.class0_override, 0)
    t.prepare(); t.fit_select(par); t.resolve(par)
    gj, gc = t.grant_job.cpu().numpy(), t.grant_cut.cpu().numpy()
    assert (gj >= 0).any()
    _, pp, _ = oracle.prepare(wl.seg_off, wl.dur, wl.mem, wl.safe, wl.progress)
    i32 = dict(dtype=torch.int32, device="cuda:0")
    cover, slack = torch.full((wl.n_gaps,), -9, **i32), torch.full((wl.n_gaps,), -9, **i32)
    sets = [np.unique(wl.C), np.array([1024, 4096, 16384], np.int32), np.zeros(0, np.int32),
            np.array([5], np.int32), np.unique(np.concatenate([wl.C // 2, wl.C, [2**30]]))]
    for cap_set in sets:
        cap_set = np.ascontiguousarray(cap_set, dtype=np.int32)
        engine.sja_cover(t.C, t.grant_job, t.grant_cut, torch.from_numpy(cap_set).cuda(), cover, slack)
        torch.cuda.synchronize()
        want_c, want_s = oracle.cover(wl.seg_off, pp, wl.C, gj, gc, cap_set)
        np.testing.assert_array_equal(cover.cpu().numpy(), want_c)
        np.testing.assert_array_equal(slack.cpu().numpy(), want_s)
    # with the gaps' own capacities in the set, every grant is covered and no slack is negative
    engine.sja_cover(t.C, t.grant_job, t.grant_cut, torch.from_numpy(np.unique(wl.C)).cuda(), cover, slack)
    c, s = cover.cpu().numpy(), slack.cpu().numpy()
    assert (c[gj >= 0] > 0).all() and (s >= 0).all() and (c[gj < 0] == -1).all()
    # entries out of range count as ungranted
    bad_j = t.grant_job.clone(); bad_c = t.grant_cut.clone()
    g0 = int(np.nonzero(gj >= 0)[0][0])
    bad_j[g0] = wl.n_jobs + 1
    engine.sja_cover(t.C, bad_j, bad_c, torch.from_numpy(np.unique(wl.C)).cuda(), cover, slack)
    assert cover[g0].item() == -1 and slack[g0].item() == 0
