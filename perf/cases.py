"""What a scheduler has this library do, as cases that can be timed and compared.

A case is one pass through the public entry points (paper_2509_19086_amd.Engine)
on synthetic profiles made on the GPU from a seed.  The sizes and distributions
are those of the named workloads of this repository (tiny, small, medium, large,
stress) and of its tests (ragged sizes, more capacities than the class tables
hold, every admission option).

Paths:
  tick        prepare, fit (matrix and interest rows), select, resolve: one
              scheduling tick as a caller runs it that wants the replies
  chain       prepare once, then per tick fit_select, resolve, advance with fresh
              gaps: a scheduler that runs on
  prepare, fit, fit_select, select
              one call of it on a job table that is already there
"""
import math

import torch

import paper_2509_19086_amd as sja

EFFICIENCY, FAIRNESS, SLA, MIXED = 0, 1, 2, 3
WAIT_SCALE, SLA_WEIGHT, WAIT_STEP = 1000, (4, 2, 1), 1000

# Per profile kind: segment durations, probability of a safe cut, gap windows, slice capacities.
PROFILES = {
    "loguniform": dict(dur=(1, 100), safe=0.25, window=(50, 2000), caps=(5120, 10240, 20480, 40960)),
    "bimodal": dict(dur=(1, 100), safe=0.25, window=(100, 20000), caps=(9216, 18432, 36864, 73728, 147456)),
    "pareto": dict(dur=None, safe=0.1, window=(50, 2000), caps=(5120, 10240, 20480, 40960)),
    "walk": dict(dur=(1, 100), safe=0.25, window=(10, 100000), caps=tuple(36864 * u for u in range(1, 9))),
}

_CASE = dict(name="", path="tick", gaps=8, jobs=16, len_lo=64, len_hi=64, profile="loguniform", policy=EFFICIENCY,
             max_rounds=0, ticks=1, caps=0, options="plain")


def _case(**kw):
    return dict(_CASE, **kw)


def listed():
    return [
        # a handful of gaps and jobs: what a small cluster's scheduler does many times a second; launches and latency count
        _case(name="tick_tiny", gaps=8, jobs=16),
        # an ordinary tick of one node group, fairness by waiting time
        _case(name="tick_small", gaps=256, jobs=1024, len_lo=256, len_hi=256, policy=FAIRNESS),
        # a busy cluster, service classes with the urgent class first, two-peaked memory
        _case(name="tick_medium", gaps=2048, jobs=8192, len_lo=512, len_hi=512, profile="bimodal", policy=SLA),
        # a large cluster that bounds its tick: at most eight rounds of grants, heavy-tailed durations
        _case(name="tick_large", gaps=8192, jobs=32768, len_lo=1024, len_hi=1024, profile="pareto", max_rounds=8),
        # the largest batch of this repository's benchmark, grants until stable
        _case(name="tick_stress", path="tick", gaps=32768, jobs=65536, len_lo=16, len_hi=2048, profile="walk", policy=MIXED),
        # a scheduler that runs on at ordinary size: three ticks without the matrix, jobs move on between them
        _case(name="chain_medium", path="chain", gaps=2048, jobs=8192, len_lo=512, len_hi=512, profile="bimodal", policy=MIXED, ticks=3),
        # the same with every admission option on (limits, hysteresis, area score) at sizes that divide by nothing
        _case(name="chain_options", path="chain", gaps=1777, jobs=6151, len_lo=16, len_hi=700, profile="walk", policy=FAIRNESS, ticks=2,
              options="all"),
        # more capacities than the class tables hold (slices cut to measure): the searching forms, rounds bounded
        _case(name="chain_many_caps", path="chain", gaps=700, jobs=2501, len_lo=16, len_hi=500, profile="walk", policy=MIXED, max_rounds=8,
              caps=300),
        # the job table rebuilt at full size: what a scheduler pays when profiles were re-estimated
        _case(name="prepare_stress", path="prepare", gaps=8, jobs=65536, len_lo=16, len_hi=2048, profile="walk"),
        # all replies of a full-size batch as matrix and bits: the pair evaluation by itself
        _case(name="fit_stress", path="fit", gaps=32768, jobs=65536, len_lo=16, len_hi=2048, profile="walk"),
        # the best reply per gap without the matrix at full size, some jobs held and some gaps switched off
        _case(name="fit_select_stress", path="fit_select", gaps=32768, jobs=65536, len_lo=16, len_hi=2048, profile="walk", policy=MIXED),
        # another policy over replies that are already there, some jobs held and some gaps switched off
        _case(name="select_large", path="select", gaps=8192, jobs=32768, len_lo=1024, len_hi=1024, profile="pareto", policy=SLA),
    ]


def draw(rng):
    """One more case of these ranges: sizes spread over their logarithm, any path, profile, policy and option.

    Grants until stable stay at 8192 gaps, the searching forms at a few thousand: there the rounds, not the sizes,
    are the cost, and a drawn case shall not cost more than the largest listed one."""
    def spread(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    path = rng.choice(("tick", "tick", "chain", "chain", "prepare", "fit", "fit_select", "select"))
    grants = path in ("tick", "chain")
    many = grants and rng.random() < 0.2
    max_rounds = 8 if many or (grants and rng.random() < 0.25) else 0
    ticks = rng.randint(1, 3) if path == "chain" and not many else 1
    gaps = spread(8, 2048 if many else 8192 // ticks if grants else 32768)
    jobs = spread(16, 8192 if many else 65536)
    len_lo = spread(16, 512)
    len_hi = rng.choice((len_lo, min(4 * len_lo, 2048)))
    return _case(path=path, gaps=gaps, jobs=jobs, len_lo=len_lo, len_hi=len_hi, profile=rng.choice(sorted(PROFILES)),
                 policy=rng.randrange(4), max_rounds=max_rounds, ticks=ticks, caps=rng.randint(70, 400) if many else 0,
                 options=rng.choice(("plain", "plain", "area", "limits", "hysteresis", "all")))


# ---------------------------------------------------------------- inputs

def _uniform(gen, lo, hi, n):
    return torch.randint(lo, hi + 1, (n,), generator=gen, device="cuda", dtype=torch.int32)


def _loguniform(gen, lo, hi, n):
    u = torch.rand(n, generator=gen, device="cuda", dtype=torch.float64)
    return (lo * torch.pow(hi / lo, u)).floor().clamp(lo, hi).to(torch.int32)


def _memory(gen, profile, lens, job, k, n):
    """MiB per segment: log-uniform, two peaks, or a walk in steps of a tenth between 256 and 147456."""
    if profile == "bimodal":
        low = torch.rand(n, generator=gen, device="cuda") < 0.7
        return torch.where(low, _loguniform(gen, 256, 8192, n), _loguniform(gen, 16384, 81920, n))
    if profile != "walk":
        return _loguniform(gen, 256, 40960, n)
    jobs, longest = lens.numel(), int(lens.max())
    cur = _loguniform(gen, 256, 147456, jobs)
    sign = torch.randint(0, 2, (longest, jobs), generator=gen, device="cuda", dtype=torch.int8).mul_(2).sub_(1)
    rows = torch.empty((longest, jobs), device="cuda", dtype=torch.int32)
    rows[0] = cur
    for step in range(1, longest):
        cur = (cur + sign[step] * torch.div(cur, 10, rounding_mode="floor")).clamp_(256, 147456)
        rows[step] = cur
    return rows[k, job]


def _gaps(gen, case):
    p = PROFILES[case["profile"]]
    G = case["gaps"]
    W = _uniform(gen, p["window"][0], p["window"][1], G)
    if case["caps"]:
        caps = torch.sort(_uniform(gen, min(p["caps"]), max(p["caps"]), case["caps"])).values
    else:
        caps = torch.tensor(p["caps"], device="cuda", dtype=torch.int32)
    return W, caps[torch.randint(0, caps.numel(), (G,), generator=gen, device="cuda")].contiguous()


def _inputs(case, seed):
    """The job table, the preferences, the gaps of every tick and the masks of held jobs and active gaps."""
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    p, G, J = PROFILES[case["profile"]], case["gaps"], case["jobs"]
    # profile lengths spread evenly over their range, in an order of the seed's: every seed has as many segments
    lens = case["len_lo"] + torch.randperm(J, generator=gen, device="cuda") * (case["len_hi"] - case["len_lo"] + 1) // J
    seg_off = torch.zeros(J + 1, device="cuda", dtype=torch.int64)
    torch.cumsum(lens, 0, out=seg_off[1:])
    S = int(seg_off[-1])
    job = torch.repeat_interleave(torch.arange(J, device="cuda"), lens)
    k = torch.arange(S, device="cuda") - seg_off[job]
    if p["dur"]:
        dur = _uniform(gen, p["dur"][0], p["dur"][1], S)
    else:       # heavy-tailed
        u = torch.rand(S, generator=gen, device="cuda", dtype=torch.float64)
        dur = torch.pow(1 - u, -1 / 1.5).floor().clamp(1, 100000).to(torch.int32)
    mem = _memory(gen, case["profile"], lens, job, k, S)
    safe = (torch.rand(S, generator=gen, device="cuda") < p["safe"]).to(torch.uint8)
    last = seg_off[1:] - 1
    safe[last] = 1
    # progress: the start or one of the flagged boundaries inside the job, each as likely
    inner = safe.to(torch.int64)
    inner[last] = 0
    counts = torch.cumsum(inner, 0)
    before = torch.cat((torch.zeros(1, device="cuda", dtype=torch.int64), counts))[seg_off]
    n_inner = before[1:] - before[:-1]
    pick = torch.minimum((torch.rand(J, generator=gen, device="cuda", dtype=torch.float64) * (n_inner + 1)).to(torch.int64), n_inner)
    at = torch.searchsorted(counts, before[:-1] + pick)
    progress = torch.where(pick == 0, 0, at - seg_off[:-1] + 1).to(torch.int32)
    d = dict(seg_off=seg_off, dur=dur, mem=mem, safe=safe, progress=progress)
    d["wait"] = _uniform(gen, 0, 10**6, J)
    d["sla_class"] = _uniform(gen, 0, 2, J).to(torch.uint8)
    d["gaps"] = [_gaps(gen, case) for _ in range(case["ticks"])]
    if case["options"] in ("limits", "all"):
        d["power"] = (100 + 900 * (mem.double() / 147456 * (0.5 + torch.rand(S, generator=gen, device="cuda"))).clamp(0, 1.1)).to(torch.int32)
        d["deadline"] = (0.01 * p["window"][1] * torch.pow(400.0, torch.rand(J, generator=gen, device="cuda", dtype=torch.float64))).to(torch.int32)
    masked = case["path"] in ("select", "fit_select")
    d["held"] = torch.where(torch.rand(J, generator=gen, device="cuda") < 0.1, 0, -1).to(torch.int32) if masked else None
    d["active"] = (torch.rand(G, generator=gen, device="cuda") < 0.9).to(torch.uint8) if masked else None
    return d


def _set_options(engine, case, d):
    p, options = PROFILES[case["profile"]], case["options"]
    engine.sja_set_score(1 if options in ("area", "all") else 0)
    if options in ("limits", "all"):
        w = p["window"][1]
        engine.sja_set_limits(sja.Limits.make(tau_min=w // 50, tau_max=2 * w // 3, power_cap=900, now=w // 100), d["power"], d["deadline"])
    if options in ("hysteresis", "all"):
        engine.sja_set_hysteresis(list(p["caps"]), p["caps"][0])


def prepare(case, seed):
    d = _inputs(case, seed)
    G, J, S = case["gaps"], case["jobs"], d["dur"].numel()
    engine = sja.Engine(0)
    engine.ensure_workspace(G, J, S)
    _set_options(engine, case, d)
    i32, i64 = dict(device="cuda", dtype=torch.int32), dict(device="cuda", dtype=torch.int64)
    d.update(engine=engine, case=case, params=sja.Params.make(case["policy"], WAIT_SCALE, SLA_WEIGHT, 1, case["max_rounds"]))
    d["tables"] = [torch.zeros(S, **i32) for _ in range(3)]
    path, T = case["path"], case["ticks"]
    if path in ("tick", "fit", "select"):
        d["cut"] = torch.zeros((G, J), **i32)
        d["bits"] = torch.zeros((G, (J + 31) // 32), **i32)
    if path in ("tick", "fit_select", "select"):
        d["cand"] = [torch.zeros(G, **i32), torch.zeros(G, **i32), torch.zeros(G, **i64)]
    if path == "chain":
        d["cand"] = [torch.zeros(G, **i32), torch.zeros(G, **i32), torch.zeros(G, **i64)]
        d["now_progress"], d["now_wait"] = d["progress"].clone(), d["wait"].clone()
        d["metrics"] = [torch.zeros(4, **i64) for _ in range(T)]
    if path in ("tick", "chain"):
        d["grants"] = [[torch.zeros(G, **i32), torch.zeros(G, **i32), torch.zeros(G, **i64), torch.zeros(J, **i32), torch.zeros(2, **i32)]
                       for _ in range(T)]
    if path in ("fit", "fit_select", "select"):     # the job table that these calls work on
        engine.sja_prepare_profiles(d["seg_off"], d["dur"], d["mem"], d["safe"], d["progress"], *d["tables"])
    if path == "select":
        engine.sja_fit(*d["gaps"][0], d["cut"], d["bits"])
    return d


def run(d):
    engine, path, params, wait, cls = d["engine"], d["case"]["path"], d["params"], d["wait"], d["sla_class"]
    profile = (d["seg_off"], d["dur"], d["mem"], d["safe"])
    W, C = d["gaps"][0]
    if path == "prepare":
        engine.sja_prepare_profiles(*profile, d["progress"], *d["tables"])
        return d["tables"]
    if path == "fit":
        engine.sja_fit(W, C, d["cut"], d["bits"])
        return [d["cut"], d["bits"]]
    if path == "fit_select":
        engine.sja_fit_select(W, C, params, wait, cls, d["held"], d["active"], *d["cand"])
        return d["cand"]
    if path == "select":
        engine.sja_select(params, wait, cls, d["held"], d["active"], *d["cand"])
        return d["cand"]
    if path == "tick":
        engine.sja_prepare_profiles(*profile, d["progress"], *d["tables"])
        engine.sja_fit(W, C, d["cut"], d["bits"])
        engine.sja_select(params, wait, cls, None, None, *d["cand"])
        engine.sja_resolve(params, wait, cls, *d["grants"][0])
        return [d["tables"], d["cut"], d["bits"], d["cand"], d["grants"][0]]
    progress, wait = d["now_progress"].copy_(d["progress"]), d["now_wait"].copy_(wait)
    engine.sja_prepare_profiles(*profile, progress, *d["tables"])
    for (W, C), grants, metrics in zip(d["gaps"], d["grants"], d["metrics"]):
        engine.sja_fit_select(W, C, params, wait, cls, None, None, *d["cand"])
        engine.sja_resolve(params, wait, cls, *grants)
        engine.sja_advance(W, C, grants[0], grants[1], grants[3], progress, wait, WAIT_STEP, metrics)
    return [d["grants"], d["metrics"], progress, wait, d["cand"], d["tables"]]


def work(case):
    """Bytes: every input read once, every output written once (the profiles only after the progress point, half of
    them on average); whole-number work has no rate to be held against, so flops counts none."""
    G, J, T = case["gaps"], case["jobs"], case["ticks"]
    S = J * (case["len_lo"] + case["len_hi"]) // 2
    table = (9 + 12) * S // 2 + 12 * J
    matrix = 4 * G * J + G * ((J + 31) // 32) * 4
    cand, grants = 16 * G, 16 * G + 4 * J
    atoms = int(S // 2 * PROFILES[case["profile"]]["safe"]) * 8
    b = {
        "prepare": table,
        "fit": 8 * G + atoms + matrix,
        "fit_select": 9 * G + atoms + 9 * J + cand,
        "select": 4 * G * J + G + 9 * J + cand,
        "tick": table + 8 * G + matrix + 5 * J + cand + grants,
        "chain": table + T * (8 * G + atoms + 13 * J + cand + grants),
    }[case["path"]]
    return {"bytes": float(b), "flops": 0.0}


def tolerance(case):
    return "exact"          # whole numbers throughout


# ---------------------------------------------------------------- the same in plain torch

def _tables(d, progress, before=None):
    """Per job a row of its boundaries 1..L (padded): running duration, running peak, flag, and the tables prepare writes
    (entries before the progress point keep what was there: `before`, or nothing yet)."""
    seg_off = d["seg_off"]
    lens = seg_off[1:] - seg_off[:-1]
    J, L = lens.numel(), int(lens.max())
    k = torch.arange(L, device="cuda").expand(J, L)
    inside = k < lens[:, None]
    at = (seg_off[:-1, None] + k)[inside]
    def rows(x):
        out = torch.zeros((J, L), device="cuda", dtype=torch.int64)
        out[inside] = x[at].to(torch.int64)
        return out
    left = inside & (k >= progress[:, None])
    D = torch.cumsum(rows(d["dur"]) * left, 1)
    P = torch.cummax(torch.where(left, rows(d["mem"]), -1), 1).values
    flag = left & ((rows(d["safe"]) != 0) | (k == lens[:, None] - 1))
    last = torch.cummax(torch.where(flag, k + 1, -1), 1).values
    flat = [torch.where(left, x, 0)[inside].to(torch.int32) for x in (D, P, last)]
    if before is not None:
        flat = [torch.where(left[inside], new, old) for new, old in zip(flat, before)]
    return D, P, flag, flat


def _replies(D, P, flag, W, C):
    J, L = D.shape
    cut = torch.empty((W.numel(), J), device="cuda", dtype=torch.int64)
    b = torch.arange(1, L + 1, device="cuda")
    for g in range(W.numel()):
        cut[g] = torch.where(flag & (D <= W[g]) & (P <= C[g]), b, -1).max(1).values
    return cut


def _keys(case, F, cut, wait, cls):
    """(tier, score, second) per pair; score 0 and tier -1 where declined."""
    f = torch.gather(F.expand(cut.shape[0], -1, -1), 2, cut.clamp(min=1)[:, :, None] - 1)[:, :, 0]
    cls, wait, policy = cls.to(torch.int64), wait.to(torch.int64), case["policy"]
    tier, mult = torch.zeros_like(cls), torch.ones_like(wait)
    if policy in (FAIRNESS, MIXED):
        mult = WAIT_SCALE + wait
    if policy == SLA:
        mult, tier = torch.tensor(SLA_WEIGHT, device="cuda")[cls], (cls == 0).to(torch.int64)
    if policy == MIXED:
        tier = 2 - cls
    return torch.where(cut >= 0, tier, -1), f * mult, f if policy == MIXED else torch.zeros_like(f)


def _best(keys, allowed):
    """Per gap the first job with the largest key among those allowed, and whether there is one."""
    on = allowed & (keys[0] >= 0)
    some = on.any(1)
    for x in keys:
        top = torch.where(on, x, -1).max(1, keepdim=True).values
        on = on & (x == top)
    return on.to(torch.int8).argmax(1), some


def _pick(keys, cut, allowed):
    j, some = _best(keys, allowed)
    at = (torch.arange(cut.shape[0], device="cuda"), j)
    return [torch.where(some, j, -1).to(torch.int32), torch.where(some, cut[at], -1).to(torch.int32), torch.where(some, keys[1][at], 0)]


def _grants(case, keys, cut):
    G, J = cut.shape
    job = torch.full((G,), -1, device="cuda", dtype=torch.int64)
    gap = torch.full((J,), -1, device="cuda", dtype=torch.int64)
    g = torch.arange(G, device="cuda")
    rounds = stable = 0
    while case["max_rounds"] == 0 or rounds < case["max_rounds"]:
        rounds += 1
        j, some = _best(keys, (gap < 0)[None] & (job < 0)[:, None])
        if not bool(some.any()):
            stable = 1
            break
        lowest = torch.full((J,), G, device="cuda", dtype=torch.int64).scatter_reduce(0, j[some], g[some], "amin")
        won = some & (lowest[j] == g)
        job[won] = j[won]
        gap[j[won]] = g[won]
        if bool((won == some).all()):
            stable = 1
            break
    held = job >= 0
    at = (g, job.clamp(min=0))
    return [job.to(torch.int32), torch.where(held, cut[at], -1).to(torch.int32), torch.where(held, keys[1][at], 0), gap.to(torch.int32),
            torch.tensor([rounds, stable], device="cuda", dtype=torch.int32)]


def exact(case, seed):
    """What run() returns, for the plain option at sizes where dense tables of every pair's boundaries are quick."""
    if case["options"] != "plain" or case["gaps"] * case["jobs"] * case["len_hi"] > 2**27:
        return None
    d = _inputs(case, seed)
    progress, wait, cls, path = d["progress"].to(torch.int64), d["wait"], d["sla_class"], case["path"]
    D, P, flag, flat = _tables(d, progress)
    if path == "prepare":
        return flat
    W, C = d["gaps"][0]
    if path != "chain":
        cut = _replies(D, P, flag, W, C)
        J = case["jobs"]
        words = torch.zeros((case["gaps"], (J + 31) // 32 * 32), device="cuda", dtype=torch.int64)
        words[:, :J] = cut >= 0
        bits = (words.view(case["gaps"], -1, 32) << torch.arange(32, device="cuda")).sum(2).to(torch.int32)
        if path == "fit":
            return [cut.to(torch.int32), bits]
        keys = _keys(case, D * P, cut, wait, cls)
        allowed = torch.ones_like(cut, dtype=torch.bool)
        if path != "tick":
            return _pick(keys, cut, (d["held"] < 0)[None] & (d["active"] != 0)[:, None])
        return [flat, cut.to(torch.int32), bits, _pick(keys, cut, allowed), _grants(case, keys, cut)]
    lens = d["seg_off"][1:] - d["seg_off"][:-1]
    wait, all_grants, all_metrics, cand = wait.to(torch.int64), [], [], None
    for W, C in d["gaps"]:
        D, P, flag, flat = _tables(d, progress, flat)
        cut = _replies(D, P, flag, W, C)
        keys = _keys(case, D * P, cut, wait, cls)
        cand = _pick(keys, cut, torch.ones_like(cut, dtype=torch.bool))
        grants = _grants(case, keys, cut)
        all_grants.append(grants)
        gap, job, boundary = grants[3], grants[0].to(torch.int64), grants[1].to(torch.int64)
        held = job >= 0
        filled = int((D * P)[job[held], boundary[held] - 1].sum())
        offered = int((W.to(torch.int64) * C.to(torch.int64)).sum())
        granted = gap >= 0
        progress = torch.where(granted, boundary[gap.clamp(min=0).to(torch.int64)], progress)
        wait = torch.where(granted, 0, torch.where(progress < lens, (wait + WAIT_STEP).clamp(max=2**31 - 1), wait))
        all_metrics.append(torch.tensor([filled, offered, int(held.sum()), int((progress >= lens).sum())], device="cuda"))
    flat = _tables(d, progress, flat)[-1]
    return [all_grants, all_metrics, progress.to(torch.int32), wait.to(torch.int32), cand, flat]
