// Fused fit -> select: the per-gap policy arg-max straight from the atom
// tables, without a (gap, job) matrix in between (Sec. 3.5: a subjob only
// comes into being at its grant, so all a gap needs from the jobs' replies is
// the best one).
//
// The stepping is that of the pair-evaluation kernel: lanes run along jobs,
// waves step through sorted gap positions of one capacity class, each lane
// advances a merge pointer through its job's atoms (staged in an LDS window
// that is topped up once per period).  Instead of storing the cut, a lane that
// passes an atom recomputes its key F * weight from the atom's (duration,
// peak).  Along the sorted positions of a class a job's key decreases only
// where the hysteresis rule lets a longer fit end in a shorter cut, so the
// wave's arg-max is a running one: a key that changed and reaches the wave's
// best can move it, and a best that falls itself, after which all lanes are
// compared again.  After every period the waves of a block
// combine their bests per position and the block leaves one partial per (job
// tile, gap); k_fused_reduce finishes the arg-max and turns the winning atom
// into its boundary.
#pragma once

#include "k_fit.h"
#include "k_grant.h"

namespace sja {

constexpr int kFusedBlock = kSelBlock;     // the partials are laid out per tile of kSelBlock jobs
constexpr int kFusedWindow = 8;
constexpr int kFusedPeriod = 32;

__device__ __forceinline__ bool fused_better(unsigned long long hi_a, unsigned long long lo_a, int j_a,
                                             unsigned long long hi_b, unsigned long long lo_b, int j_b)
{
    if (hi_a != hi_b) return hi_a > hi_b;
    if (lo_a != lo_b) return lo_a > lo_b;
    return j_a < j_b;
}

__device__ __forceinline__ unsigned long long fused_readlane_u64(unsigned long long v, int l)
{
    const unsigned int lo = __builtin_amdgcn_readlane(int(uint32_t(v)), l);
    const unsigned int hi = __builtin_amdgcn_readlane(int(uint32_t(v >> 32)), l);
    return (static_cast<unsigned long long>(hi) << 32) | lo;
}

// Eight waves per SIMD (64 registers, a few spilled) beat the 94 registers the
// compiler takes by itself: the stepping loop is bound by latency (1.5 against 2.1 ms).
// AREA: the key's F is the atom's area under the envelope (a second window of
// 64-bit values beside the (duration, peak) one) instead of duration x peak.
// keys_fall: a job's key may fall along the positions (the host's keys_rise); else k_range_select serves the batch
// if its classes have tables.
template <int BLOCK, int CAP, int PERIOD, bool MIXED, bool AREA>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(8, 8))) void k_fit_select(
    int n_jobs, int n_gaps, int chunk_bound, int keys_fall, PolicyDev pol, const int64_t *__restrict__ seg_off,
    const int2 *__restrict__ atom_dp, const long long *__restrict__ atom_area,
    const int32_t *__restrict__ n_atoms,
    const int32_t *__restrict__ plan, const int32_t *__restrict__ chunk_begin,
    const int32_t *__restrict__ chunk_end, const int32_t *__restrict__ chunk_class,
    const int32_t *__restrict__ chunk_sub, const int32_t *__restrict__ start_tab,
    const int32_t *__restrict__ ncap_tab, const int32_t *__restrict__ gap_w,
    const int32_t *__restrict__ gap_c, const int32_t *__restrict__ gap_order,
    const int32_t *__restrict__ gap_run_end, const int32_t *__restrict__ wait,
    const uint8_t *__restrict__ sla_class,
    const int32_t *__restrict__ job_held, const uint8_t *__restrict__ gap_active,
    SelPartial *__restrict__ part)
{
    static_assert((CAP & (CAP - 1)) == 0 && BLOCK % kWave == 0 && PERIOD <= 64, "tile shape");
    constexpr int WAVES = BLOCK / kWave;
    __shared__ int2 win[CAP][BLOCK];
    __shared__ long long win_area[AREA ? CAP : 1][AREA ? BLOCK : 1];
    // per wave and period: the steps at which its running best changed, with the new best
    __shared__ unsigned long long e_hi[WAVES][PERIOD + 1];
    __shared__ unsigned long long e_lo[WAVES][PERIOD + 1];
    __shared__ int e_lane[WAVES][PERIOD + 1];
    __shared__ int e_atoms[WAVES][PERIOD + 1];
    __shared__ int e_step[WAVES][PERIOD + 1];
    __shared__ int e_count[WAVES];

    const int xcd = blockIdx.x & 7;
    const int k = blockIdx.x >> 3;
    const int job_tile = (k / chunk_bound) * 8 + xcd;
    const int chunk = k % chunk_bound;
    if (job_tile * BLOCK >= n_jobs || chunk >= plan[kPlanChunks]) return;
    const bool tabled = plan[kPlanTabled] != 0;
    if (tabled && !keys_fall) return;
    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1), wave = tid / kWave;
    const int j_raw = job_tile * BLOCK + tid;
    const bool live = j_raw < n_jobs;
    const int j = live ? j_raw : n_jobs - 1;
    const bool usable = live && !(job_held && job_held[j] >= 0);
    const int64_t base = seg_off[j];
    const int n = usable ? n_atoms[j] : 0;
    const int2 *dp = atom_dp + base;
    const long long *da = atom_area + base;        // read with AREA only
    unsigned long long mult = 1, tier = 0;
    job_policy(pol, wait, sla_class, j, mult, tier);
    const int s_begin = chunk_begin[chunk], s_end = chunk_end[chunk];

    int n_cap = 0;   // atoms the current capacity class can reach
    int a = 0;       // atoms whose running duration fits the current window
    int hi = 0;      // atoms [a, hi) are staged in the LDS window
    int nd = 0, np = 0;      // atom a     (meaningful while a < hi)
    int nd2 = 0, np2 = 0;    // atom a + 1 (meaningful while a + 1 < hi)
    unsigned long long key_hi = 0, key_lo = 0;   // key of atom a - 1, 0 while a == 0
    int c_cur = 0;
    unsigned long long dry_mask = 0;
    // the wave's running best, the same values in every lane
    unsigned long long best_hi = 0, best_lo = 0;
    int best_lane = kWave, best_atoms = 0;
    int q_now = 0;       // step of the current period (for the change list)
    int n_events = 0;    // entries of this wave's change list (the same in every lane)
    int q_noted = -1;    // step of the list's last entry
    auto uniform64 = [](unsigned long long v) {
        const unsigned int lo = __builtin_amdgcn_readfirstlane(int(uint32_t(v)));
        const unsigned int hi = __builtin_amdgcn_readfirstlane(int(uint32_t(v >> 32)));
        return (static_cast<unsigned long long>(hi) << 32) | lo;
    };
    auto note = [&]() {
        // at most one entry per step: a second change in the same step overwrites the first
        if (n_events > 0 && q_noted == q_now) --n_events;
        q_noted = q_now;
        if (lane == 0) {
            e_step[wave][n_events] = q_now;
            e_hi[wave][n_events] = best_hi;
            e_lo[wave][n_events] = best_lo;
            e_lane[wave][n_events] = best_lane;
            e_atoms[wave][n_events] = best_atoms;
        }
        ++n_events;
    };

    auto key_from = [&](unsigned long long F) {
        key_hi = ((tier << 62) | times_mult(F, mult)) + 1ull;
        key_lo = MIXED ? F : 0ull;
    };
    // key of the atom just passed: a - 1, whose window slot is still intact (a top-up writes at most
    // up to atom a + CAP - 1)
    auto key_of = [&](int d, int p) {
        if (AREA) key_from((unsigned long long)win_area[(a - 1) & (CAP - 1)][tid]);
        else key_from(rect_of(d, p));
    };
    // a key changed in the lanes of `ch` (those that can matter): move the running best
    auto challenge = [&](bool in) {
        unsigned long long ch = __ballot(in);
        if (!ch) return;
        if (__popcll(ch) > 4) {
            unsigned long long bh = in ? key_hi : 0ull, bl = in ? key_lo : 0ull;
            int bj = in ? lane : kWave;
#pragma unroll
            for (int d = 1; d < kWave; d <<= 1) {
                const unsigned long long oh = (unsigned long long)__shfl_xor((long long)bh, d, kWave);
                const unsigned long long ol = (unsigned long long)__shfl_xor((long long)bl, d, kWave);
                const int oj = __shfl_xor(bj, d, kWave);
                if (fused_better(oh, ol, oj, bh, bl, bj)) { bh = oh; bl = ol; bj = oj; }
            }
            // the best of the changed keys replaces the running best if it beats it, or if it is the
            // best lane's own new key; a best lane that changed without being this maximum is beaten by it
            const bool own = (ch >> (best_lane & (kWave - 1))) & 1ull && best_lane < kWave;
            if (own || fused_better(bh, bl, bj, best_hi, best_lo, best_lane)) {
                best_hi = uniform64(bh); best_lo = uniform64(bl); best_lane = __builtin_amdgcn_readfirstlane(bj);
                best_atoms = __builtin_amdgcn_readlane(a, best_lane & (kWave - 1));
                note();
            }
        } else {
            bool moved = false;
            while (ch) {
                const int l = __ffsll((long long)ch) - 1;
                ch &= ch - 1;
                const unsigned long long kh = fused_readlane_u64(key_hi, l);
                const unsigned long long kl = MIXED ? fused_readlane_u64(key_lo, l) : 0ull;
                if (l == best_lane || fused_better(kh, kl, l, best_hi, best_lo, best_lane)) {
                    best_hi = kh; best_lo = kl; best_lane = l;
                    best_atoms = __builtin_amdgcn_readlane(a, l);
                    moved = true;
                }
            }
            if (moved) note();
        }
    };
    auto init = [&](int s) {
        c_cur = gap_c[s];
        if (!usable) {
            n_cap = 0; a = 0;
        } else if (tabled) {
            a = start_tab[int64_t(chunk) * n_jobs + j];
            n_cap = ncap_tab[int64_t(chunk_class[chunk]) * n_jobs + j];
        } else {
            n_cap = upper_bound_peak(dp, n, c_cur);
            a = upper_bound_dur(dp, n_cap, gap_w[s]);
        }
        key_hi = 0; key_lo = 0;
        if (a > 0) {
            if (AREA) {
                key_from((unsigned long long)da[a - 1]);
            } else {
                const int2 v = dp[a - 1];
                key_from(rect_of(v.x, v.y));
            }
        }
        hi = a;
        best_hi = 0; best_lo = 0; best_lane = kWave; best_atoms = 0;
        note();
        challenge(a > 0);
    };
    auto reload = [&]() {
        const int2 x = win[a & (CAP - 1)][tid]; nd = x.x; np = x.y;
        const int2 y = win[(a + 1) & (CAP - 1)][tid]; nd2 = y.x; np2 = y.y;
    };
    auto topup = [&]() {
        const int want = min(a + CAP, n_cap);
        int2 v[CAP];
#pragma unroll
        for (int t = 0; t < CAP; ++t)
            if (hi + t < want) v[t] = dp[hi + t];
#pragma unroll
        for (int t = 0; t < CAP; ++t)
            if (hi + t < want) win[(hi + t) & (CAP - 1)][tid] = v[t];
        if (AREA) {
            for (int idx = hi; idx < want; ++idx) win_area[idx & (CAP - 1)][tid] = da[idx];
        }
        hi = max(hi, want);
        reload();
    };
    // One step: move every lane past the atoms that window w has reached and keep the
    // running best (q = step within the period).
    auto step = [&](int w, int q) {
        bool adv = a < hi && nd <= w;
        if (__any(adv)) {
            bool changed = false;
            int ld = 0, lp = 0;                  // (duration, peak) of the last atom passed
            do {
                if (adv) { ld = nd; lp = np; ++a; nd = nd2; np = np2; changed = true; }
                {
                    const int2 y = win[(a + 1) & (CAP - 1)][tid];
                    nd2 = y.x; np2 = y.y;
                }
                if (__ballot(a == hi) & dry_mask) {
                    // a window ran dry inside a period: refill at once (rare)
                    if (a == hi && hi < n_cap) {
                        // with AREA one slot stays back: atom a - 1 shares its slot with atom a + CAP - 1
                        const int want = min(a + CAP - (AREA ? 1 : 0), n_cap);
                        for (int idx = hi; idx < want; ++idx) {
                            win[idx & (CAP - 1)][tid] = dp[idx];
                            if (AREA) win_area[idx & (CAP - 1)][tid] = da[idx];
                        }
                        hi = want;
                        reload();
                    }
                    dry_mask = __ballot(hi < n_cap);
                }
                adv = a < hi && nd <= w;
            } while (__any(adv));
            q_now = q;
            if (changed) key_of(ld, lp);         // once per step, for the last atom passed
            bool in = changed && key_hi >= best_hi;
            // the best lane's key fell: any lane may lead now
            if (keys_fall && __ballot(changed && lane == best_lane && fused_better(best_hi, best_lo, 0, key_hi, key_lo, 0))) {
                best_hi = best_lo = 0;
                best_lane = kWave;
                in = a > 0;
            }
            challenge(in);
        }
    };

    for (int s0 = s_begin; s0 < s_end; s0 += PERIOD) {
        const int s1 = min(s_end, s0 + PERIOD);
        n_events = 0;
        q_now = 0;
        q_noted = -1;
        if (s0 == s_begin || gap_c[s0] != c_cur) init(s0); else note();     // the list starts with the best so far
        topup();
        dry_mask = __ballot(hi < n_cap);
        if (s1 - s0 == PERIOD && gap_run_end[s0] >= s1) {
#pragma unroll
            for (int u4 = 0; u4 < PERIOD; u4 += 4) {
                const int wv[4] = {gap_w[s0 + u4], gap_w[s0 + u4 + 1], gap_w[s0 + u4 + 2], gap_w[s0 + u4 + 3]};
#pragma unroll
                for (int u = 0; u < 4; ++u) step(wv[u], u4 + u);
            }
        } else {
            for (int s = s0; s < s1; ++s) {
                q_now = s - s0;
                if (gap_c[s] != c_cur) { init(s); topup(); dry_mask = __ballot(hi < n_cap); }
                step(gap_w[s], s - s0);
            }
        }
        if (lane == 0) e_count[wave] = n_events;
        __syncthreads();
        // one partial per position of this period: the best of the block's waves at that step
        for (int q = tid; q < s1 - s0; q += BLOCK) {
            const int g = gap_order[s0 + q];
            const bool on = !gap_active || gap_active[g];
            unsigned long long bh = 0, bl = 0;
            int bj = INT32_MAX, ba = 0;
#pragma unroll
            for (int w = 0; w < WAVES; ++w) {
                const int ne = e_count[w];
                int e = 0;                                   // the last change at or before step q
                for (int i = 1; i < ne && e_step[w][i] <= q; ++i) e = i;
                const unsigned long long oh = on ? e_hi[w][e] : 0ull, ol = e_lo[w][e];
                const int oj = oh ? job_tile * BLOCK + w * kWave + e_lane[w][e] : INT32_MAX;
                if (fused_better(oh, ol, oj, bh, bl, bj)) { bh = oh; bl = ol; bj = oj; ba = e_atoms[w][e]; }
            }
            SelPartial out;
            out.hi = bh; out.lo = bl; out.job = bh ? bj : -1; out.cut = bh ? ba : -1; out.pad = 0;
            part[int64_t(job_tile) * n_gaps + g] = out;
        }
        __syncthreads();
    }
}

// One gap position and one job at a time, for batches with so many capacities that the stepping form would
// begin anew (two searches and a window) every few positions: a thread per job finds the pair's atom by one
// search on both conditions, kSearchGaps positions side by side so that their loads overlap, and the block
// leaves the same partial per (job tile, gap).  Gaps that are switched off cost nothing, and rounds switch
// more and more of them off.  700 gaps of 300 capacities x 2501 jobs: 165 us a round stepping, 47 us so.
constexpr int kSearchGaps = 4;
constexpr int kSearchRows = 32768;      // groups of positions per launch, a row of blocks each (a launch takes fewer than 65536 rows)

// The largest value over the lanes up to this one; over all 64, the same in every lane.
__device__ __forceinline__ uint32_t wave_scan_max_u32(uint32_t v) { return uint32_t(wave_scan_max_dpp(int(v ^ 0x80000000u))) ^ 0x80000000u; }
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v)
{
    return uint32_t(__builtin_amdgcn_readlane(int(wave_scan_max_u32(v)), kWave - 1));
}

// Positions per capacity, on average, below which it is used.  A searched round takes the same time whatever the
// capacities, a stepped one less the longer their runs: at 2048 gaps x 8192 jobs 180 us searched against 430 stepped
// with runs of 16 and 340 with 20; at 8192 x 16384 and the MIXED policy 2.5 ms against 2.6 with runs of 14 and 1.7
// with 27.
constexpr int kShortRun = 16;

template <bool MIXED, bool AREA>
__global__ __launch_bounds__(kFusedBlock) void k_search_select(
    int n_jobs, int n_gaps, int first_row, PolicyDev pol, const int64_t *__restrict__ seg_off, const int2 *__restrict__ atom_dp,
    const long long *__restrict__ atom_area, const int32_t *__restrict__ n_atoms, const int32_t *__restrict__ gap_w,
    const int32_t *__restrict__ gap_c, const int32_t *__restrict__ gap_order, const int32_t *__restrict__ wait,
    const uint8_t *__restrict__ sla_class, const int32_t *__restrict__ job_held, const uint8_t *__restrict__ gap_active,
    SelPartial *__restrict__ part)
{
    constexpr int WAVES = kFusedBlock / kWave, Q = kSearchGaps;
    __shared__ unsigned long long s_hi[Q][WAVES], s_lo[Q][WAVES];
    __shared__ int s_job[Q][WAVES], s_atoms[Q][WAVES];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const int s0 = (first_row + int(blockIdx.y)) * Q, j = blockIdx.x * kFusedBlock + threadIdx.x;
    int g[Q], w[Q], c[Q];
    bool on[Q], any = false;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int s = min(s0 + q, n_gaps - 1);
        g[q] = gap_order[s];
        w[q] = gap_w[s];
        c[q] = gap_c[s];
        on[q] = s0 + q < n_gaps && (!gap_active || gap_active[g[q]]);
        any = any || on[q];
    }
    const bool usable = any && j < n_jobs && !(job_held && job_held[j] >= 0);
    const int64_t base = usable ? seg_off[j] : 0;
    const int n = usable ? n_atoms[j] : 0;
    const int2 *dp = atom_dp + base;
    unsigned long long mult = 1, tier = 0;
    if (usable) job_policy(pol, wait, sla_class, j, mult, tier);
    int lo[Q], hi[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) { lo[q] = 0; hi[q] = on[q] ? n : 0; }
    for (int left = n; left > 0; left >>= 1) {          // atoms that fit are a prefix: durations and peaks ascend
        int2 v[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q)
            if (lo[q] < hi[q]) v[q] = dp[(lo[q] + hi[q]) >> 1];
#pragma unroll
        for (int q = 0; q < Q; ++q)
            if (lo[q] < hi[q]) {
                const int mid = (lo[q] + hi[q]) >> 1;
                if (v[q].x <= w[q] && v[q].y <= c[q]) lo[q] = mid + 1; else hi[q] = mid;
            }
    }
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        unsigned long long bh = 0, bl = 0;
        if (lo[q] > 0) {
            unsigned long long F;
            if (AREA) {
                F = (unsigned long long)atom_area[base + lo[q] - 1];
            } else {
                const int2 v = dp[lo[q] - 1];
                F = rect_of(v.x, v.y);
            }
            bh = ((tier << 62) | times_mult(F, mult)) + 1ull;
            bl = MIXED ? F : 0ull;
        }
        // the wave's best: the largest high word, among those the largest low word (and secondary key), the lowest lane
        unsigned long long best = __ballot(bh != 0);
        if (best) {
            auto keep = [&](uint32_t x) {
                const uint32_t top = wave_max_u32((best >> lane) & 1ull ? x : 0u);
                best &= __ballot(x == top);
            };
            keep(uint32_t(bh >> 32));
            if (best & (best - 1)) keep(uint32_t(bh));
            if (MIXED && (best & (best - 1))) keep(uint32_t(bl >> 32));
            if (MIXED && (best & (best - 1))) keep(uint32_t(bl));
        }
        const int src = best ? __ffsll((long long)best) - 1 : 0;
        bh = best ? fused_readlane_u64(bh, src) : 0ull;
        bl = MIXED && best ? fused_readlane_u64(bl, src) : 0ull;
        const int bj = best ? __builtin_amdgcn_readlane(j, src) : INT32_MAX, ba = __builtin_amdgcn_readlane(lo[q], src);
        if (lane == 0) { s_hi[q][wave] = bh; s_lo[q][wave] = bl; s_job[q][wave] = bj; s_atoms[q][wave] = ba; }
    }
    __syncthreads();
    const int q = threadIdx.x;
    if (q >= Q || s0 + q >= n_gaps) return;
    unsigned long long bh = s_hi[q][0], bl = s_lo[q][0];
    int bj = s_job[q][0], ba = s_atoms[q][0];
    for (int v = 1; v < WAVES; ++v)
        if (fused_better(s_hi[q][v], s_lo[q][v], s_job[q][v], bh, bl, bj)) {
            bh = s_hi[q][v]; bl = s_lo[q][v]; bj = s_job[q][v]; ba = s_atoms[q][v];
        }
    SelPartial out;
    out.hi = bh; out.lo = bl; out.job = bh ? bj : -1; out.cut = bh ? ba : -1; out.pad = 0;
    part[int64_t(blockIdx.x) * n_gaps + gap_order[s0 + q]] = out;
}

// The arg-max over the job tiles for kReduceGaps gaps by a block of 256: a group of threads shares a gap's
// tiles, the groups' bests meet in LDS.  (A thread per gap walked all tiles alone: 66 us for 8192 gaps and
// 128 tiles, 150 us at Stress, by 32 and 128 blocks.)  Returns true in the one thread that holds gap g's best.
constexpr int kReduceGaps = 16, kReduceGroups = 256 / kReduceGaps;

__device__ __forceinline__ bool reduce_tiles(int n_gaps, int n_job_tiles, const SelPartial *__restrict__ part, int &g,
                                             unsigned long long &bh, int &bj, int &bc)
{
    __shared__ unsigned long long s_hi[kReduceGroups][kReduceGaps], s_lo[kReduceGroups][kReduceGaps];
    __shared__ int s_job[kReduceGroups][kReduceGaps], s_cut[kReduceGroups][kReduceGaps];
    const int at = threadIdx.x % kReduceGaps, group = threadIdx.x / kReduceGaps;
    g = blockIdx.x * kReduceGaps + at;
    unsigned long long bl = 0;
    bh = 0;
    bj = INT32_MAX;
    bc = -1;
    if (g < n_gaps) {
#pragma unroll 4
        for (int t = group; t < n_job_tiles; t += kReduceGroups) {
            const SelPartial p = part[int64_t(t) * n_gaps + g];
            const int pj = p.hi ? p.job : INT32_MAX;
            if (fused_better(p.hi, p.lo, pj, bh, bl, bj)) { bh = p.hi; bl = p.lo; bj = pj; bc = p.cut; }
        }
    }
    s_hi[group][at] = bh; s_lo[group][at] = bl; s_job[group][at] = bj; s_cut[group][at] = bc;
    __syncthreads();
    if (group > 0 || g >= n_gaps) return false;
    for (int k = 1; k < kReduceGroups; ++k)
        if (fused_better(s_hi[k][at], s_lo[k][at], s_job[k][at], bh, bl, bj)) {
            bh = s_hi[k][at]; bl = s_lo[k][at]; bj = s_job[k][at]; bc = s_cut[k][at];
        }
    return true;
}

// Final arg-max over the job tiles; the winner's atom count becomes its boundary.
__global__ __launch_bounds__(256) void k_fused_reduce(int n_gaps, int n_job_tiles, const SelPartial *__restrict__ part,
                                                      const int64_t *__restrict__ seg_off, const int2 *__restrict__ atom_db,
                                                      int32_t *__restrict__ cand_job, int32_t *__restrict__ cand_cut,
                                                      int64_t *__restrict__ cand_score)
{
    int g, bj, ba;
    unsigned long long bh;
    if (!reduce_tiles(n_gaps, n_job_tiles, part, g, bh, bj, ba)) return;
    cand_job[g] = bh ? bj : -1;
    cand_cut[g] = bh ? atom_db[seg_off[bj] + ba - 1].y : -1;
    cand_score[g] = bh ? int64_t((bh - 1ull) & ((1ull << 62) - 1ull)) : 0;
}

// The same without a step per position.  Along the sorted positions of a class a job's key never falls (the
// host sees to it where the hysteresis rule could undo that), so the best key at a position is the largest one
// that any job has reached by then: every atom is an event at the first position whose window reaches its
// duration, and the answer a running maximum over the positions.  A block takes a chunk of positions and
// `batches` x 256 jobs.  Most jobs end the chunk below what the best one began it with: a thread per job looks at its
// last atom there and at its first one; of the others sixteen lanes read the atoms side by side, find their
// positions by a table in LDS and raise the largest key there.  Then those jobs are looked through again for the keys that
// are exactly the largest, the lowest of them counts (under MIXED the one with the largest F: a third time, if a
// position has several).  Work per atom of few jobs instead of per pair: what is left are the tables of the plan and the
// trips for the jobs' ends.  2048 gaps x 8192 jobs 80 -> 21 us, 1777 x 6151 with the area score 102 -> 59; 32768 x 65536
// 1607 -> 293 us (with every atom looked at 856), where k_floor.h has come in its place since.
constexpr int kRangeThreads = 256, kRangeLanes = 16, kRangeGroups = kRangeThreads / kRangeLanes;
constexpr int kRangeBatches = 8;            // batches of kRangeThreads jobs per block, at most,
constexpr int kRangeBlocks = 2048;          // as long as there are so many blocks
constexpr int kRangeTable = 512;
constexpr int kRangeTogether = 4;           // jobs whose atoms a group asks for together

template <bool MIXED, bool AREA>
__global__ __launch_bounds__(kRangeThreads) void k_range_select(
    int n_jobs, int n_gaps, int chunk_bound, int batches, int most_classes, PolicyDev pol, const int64_t *__restrict__ seg_off,
    const int2 *__restrict__ atom_dp, const long long *__restrict__ atom_area, const int32_t *__restrict__ plan,
    const int32_t *__restrict__ chunk_begin, const int32_t *__restrict__ chunk_end, const int32_t *__restrict__ chunk_class,
    const int32_t *__restrict__ start_tab, const int32_t *__restrict__ ncap_tab, const int32_t *__restrict__ gap_w,
    const int32_t *__restrict__ gap_order, const int32_t *__restrict__ wait, const uint8_t *__restrict__ sla_class,
    const int32_t *__restrict__ job_held, const uint8_t *__restrict__ gap_active, SelPartial *__restrict__ part)
{
    __shared__ unsigned long long s_best[kFitMaxChunk], s_second[MIXED ? kFitMaxChunk : 1];
    __shared__ int s_who[kFitMaxChunk], s_w[kFitMaxChunk];
    __shared__ uint16_t s_tab[kRangeTable + 1];
    __shared__ long long s_base[kRangeThreads];
    __shared__ unsigned long long s_mult[kRangeThreads];
    __shared__ int s_from[kRangeThreads], s_to[kRangeThreads], s_id[kRangeThreads];
    __shared__ uint8_t s_tier[kRangeThreads];
    __shared__ uint16_t s_near[kRangeBatches * kRangeThreads];      // jobs of the tile that came near the best
    __shared__ int s_count, s_n_near, s_several;
    const int k = blockIdx.x >> 3, job_tile = (k / chunk_bound) * 8 + (blockIdx.x & 7), chunk = k % chunk_bound;
    const int tile_jobs = batches * kRangeThreads, job0 = job_tile * tile_jobs;
    if (!serves(plan, most_classes) || job0 >= n_jobs || chunk >= plan[kPlanChunks]) return;
    const int tid = threadIdx.x, sub = tid & (kRangeLanes - 1), group = tid / kRangeLanes;
    const int begin = chunk_begin[chunk], n = chunk_end[chunk] - begin, cls = chunk_class[chunk];
    const bool last_of_class = chunk + 1 >= plan[kPlanChunks] || chunk_class[chunk + 1] != cls;
    const int32_t *from_row = start_tab + int64_t(chunk) * n_jobs;
    const int32_t *to_row = last_of_class ? ncap_tab + int64_t(cls) * n_jobs : from_row + n_jobs;
    for (int i = tid; i < n; i += kRangeThreads) {
        s_w[i] = gap_w[begin + i];
        s_best[i] = 0;
        if (MIXED) s_second[MIXED ? i : 0] = 0;
        s_who[i] = INT32_MAX;
    }
    if (tid == 0) s_count = s_n_near = s_several = 0;
    __syncthreads();
    const int w_first = s_w[0], w_last = s_w[n - 1];
    int shift = 0;
    while (((uint32_t(w_last) - uint32_t(w_first)) >> shift) >= uint32_t(kRangeTable - 1)) ++shift;
    // entry t: the first position whose window reaches w_first + (t << shift)
    for (int t = tid; t <= kRangeTable; t += kRangeThreads) {
        const long long d = (long long)w_first + ((long long)t << shift);
        int lo = 0, hi = n;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (s_w[mid] < d) lo = mid + 1; else hi = mid;
        }
        s_tab[t] = uint16_t(lo);
    }
    auto position = [&](int d) {            // of a duration up to w_last
        if (d <= w_first) return 0;
        const uint32_t t = (uint32_t(d) - uint32_t(w_first)) >> shift;
        int lo = s_tab[t], hi = s_tab[t + 1];
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (s_w[mid] < d) lo = mid + 1; else hi = mid;
        }
        return lo;
    };
    auto key_of = [](unsigned long long F, unsigned long long mult, unsigned long long tier) { return ((tier << 62) | times_mult(F, mult)) + 1ull; };
    auto area = [&](int64_t at) { return AREA ? (unsigned long long)atom_area[at] : 0ull; };
    auto size_of = [](const int2 &v, unsigned long long area_of) { return AREA ? area_of : rect_of(v.x, v.y); };
    // Calls on(duration, key, F, job) for the atoms that the jobs near the best have in the chunk: of the tile's jobs, or of
    // those that were near it before.
    auto walk = [&](bool again, auto on) {
        const int n_jobs_here = again ? s_n_near : min(tile_jobs, n_jobs - job0);
        for (int b = 0; b < n_jobs_here; b += kRangeThreads) {
            int job = -1;
            if (b + tid < n_jobs_here) job = job0 + (again ? int(s_near[b + tid]) : b + tid);
            if (!again && job >= 0 && job_held && job_held[job] >= 0) job = -1;
            int from = 0, to = 0;
            int64_t base = 0;
            unsigned long long mult = 1, tier = 0, last = 0, first = 0;
            if (job >= 0) {
                from = max(from_row[job] - 1, 0);
                to = to_row[job];
                base = seg_off[job];
                job_policy(pol, wait, sla_class, job, mult, tier);
            }
            if (from < to) {
                const int2 v = atom_dp[base + to - 1], u = atom_dp[base + from];
                const unsigned long long last_area = area(base + to - 1), first_area = area(base + from);
                last = key_of(size_of(v, last_area), mult, tier);
                if (!again && u.x <= w_first) first = key_of(size_of(u, first_area), mult, tier);
            }
            if (!again) {
#pragma unroll
                for (int d = 1; d < kWave; d <<= 1) {
                    const unsigned long long o = (unsigned long long)__shfl_xor((long long)first, d, kWave);
                    first = o > first ? o : first;
                }
                if ((tid & (kWave - 1)) == 0 && first) atomicMax(&s_best[0], first);
                __syncthreads();
            }
            const bool near = from < to && last >= s_best[0];
            if (near) {
                const int to_slot = atomicAdd(&s_count, 1);
                s_base[to_slot] = base; s_mult[to_slot] = mult; s_tier[to_slot] = uint8_t(tier);
                s_from[to_slot] = from; s_to[to_slot] = to; s_id[to_slot] = job;
                if (!again) s_near[atomicAdd(&s_n_near, 1)] = uint16_t(job - job0);
            }
            __syncthreads();
            const int count = s_count;
            for (int i0 = group; i0 < count; i0 += kRangeTogether * kRangeGroups) {
                int2 v[kRangeTogether];
                unsigned long long f[kRangeTogether];
                int a[kRangeTogether], end[kRangeTogether];
#pragma unroll
                for (int q = 0; q < kRangeTogether; ++q) {
                    const int i = i0 + q * kRangeGroups;
                    a[q] = i < count ? s_from[i] + sub : 0;
                    end[q] = i < count ? s_to[i] : 0;
                    if (a[q] < end[q]) { v[q] = atom_dp[s_base[i] + a[q]]; f[q] = area(s_base[i] + a[q]); }
                }
#pragma unroll
                for (int q = 0; q < kRangeTogether; ++q) {
                    const int i = min(i0 + q * kRangeGroups, count - 1);
                    while (a[q] < end[q] && v[q].x <= w_last) {
                        const int64_t at = s_base[i] + a[q];
                        const unsigned long long F = size_of(v[q], f[q]);
                        on(v[q].x, key_of(F, s_mult[i], s_tier[i]), F, s_id[i]);
                        a[q] += kRangeLanes;
                        if (a[q] < end[q]) { v[q] = atom_dp[at + kRangeLanes]; f[q] = area(at + kRangeLanes); }
                    }
                }
            }
            __syncthreads();
            if (tid == 0) s_count = 0;
            __syncthreads();
        }
    };
    // the running best over the positions: keys, then F, then the lowest job
    auto running = [&]() {
        constexpr int PER = kFitMaxChunk / kRangeThreads;
        for (int d = 1; d < n; d <<= 1) {
            unsigned long long hi[PER], lo[PER];
            int job[PER];
            __syncthreads();
#pragma unroll
            for (int q = 0; q < PER; ++q) {
                const int i = tid + q * kRangeThreads;
                if (i >= n) continue;
                hi[q] = s_best[i]; lo[q] = MIXED ? s_second[MIXED ? i : 0] : 0ull; job[q] = s_who[i];
                if (i < d) continue;
                const unsigned long long oh = s_best[i - d], ol = MIXED ? s_second[MIXED ? i - d : 0] : 0ull;
                const int oj = s_who[i - d];
                if (fused_better(oh, ol, oj, hi[q], lo[q], job[q])) { hi[q] = oh; lo[q] = ol; job[q] = oj; }
            }
            __syncthreads();
#pragma unroll
            for (int q = 0; q < PER; ++q) {
                const int i = tid + q * kRangeThreads;
                if (i >= n) continue;
                s_best[i] = hi[q];
                if (MIXED) s_second[MIXED ? i : 0] = lo[q];
                s_who[i] = job[q];
            }
        }
        __syncthreads();
    };
    __syncthreads();
    walk(false, [&](int d, unsigned long long key, unsigned long long, int) {
        if (key >= *static_cast<volatile unsigned long long *>(&s_best[0])) atomicMax(&s_best[position(d)], key);      // else below the best everywhere
    });
    running();
    walk(true, [&](int d, unsigned long long key, unsigned long long F, int job) {
        if (key < s_best[0]) return;
        const int p = position(d);
        if (key != s_best[p]) return;
        if (MIXED) atomicMax(&s_second[MIXED ? p : 0], F);
        const int other = atomicMin(&s_who[p], job);
        if (MIXED && other != INT32_MAX && other != job) s_several = 1;
    });
    const bool several = MIXED && s_several;
    running();
    if (several) {
        for (int i = tid; i < n; i += kRangeThreads) s_who[i] = INT32_MAX;
        __syncthreads();
        walk(true, [&](int d, unsigned long long key, unsigned long long F, int job) {
            if (key < s_best[0]) return;
            const int p = position(d);
            if (key == s_best[p] && F == s_second[MIXED ? p : 0]) atomicMin(&s_who[p], job);
        });
        running();
    }
    for (int i = tid; i < n; i += kRangeThreads) {
        const int g = gap_order[begin + i];
        const unsigned long long best = !gap_active || gap_active[g] ? s_best[i] : 0ull;
        SelPartial out;
        out.hi = best; out.lo = MIXED ? s_second[MIXED ? i : 0] : 0ull; out.job = best ? s_who[i] : -1; out.cut = begin + i; out.pad = 0;
        part[int64_t(job_tile) * n_gaps + g] = out;
    }
}

// Final arg-max over the job tiles of either form: where there were steps, the winner's atom count becomes its
// boundary (from_matrix: the partial has the boundary itself), else its atom is searched.
__global__ __launch_bounds__(256) void k_range_reduce(int n_gaps, int step_tiles, int range_tiles, int most_classes, int from_matrix, const SelPartial *__restrict__ part,
                                                      const int32_t *__restrict__ plan, const int32_t *__restrict__ gap_w,
                                                      const int32_t *__restrict__ gap_c, const int64_t *__restrict__ seg_off,
                                                      const int2 *__restrict__ atom_dp, const int2 *__restrict__ atom_db,
                                                      const int32_t *__restrict__ n_atoms, int32_t *__restrict__ cand_job,
                                                      int32_t *__restrict__ cand_cut, int64_t *__restrict__ cand_score)
{
    const bool ranges = serves(plan, most_classes);
    int g, bj, ba;
    unsigned long long bh;
    if (!reduce_tiles(n_gaps, ranges ? range_tiles : step_tiles, part, g, bh, bj, ba)) return;
    if (bh && ranges) {
        const int w = gap_w[ba], c = gap_c[ba];         // (the partial has the gap's position)
        const int2 *dp = atom_dp + seg_off[bj];
        int lo = 0, hi = n_atoms[bj];
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            const int2 v = dp[mid];
            if (v.x <= w && v.y <= c) lo = mid + 1; else hi = mid;
        }
        ba = lo;
    }
    cand_job[g] = bh ? bj : -1;
    cand_cut[g] = !bh ? -1 : !ranges && from_matrix ? ba : atom_db[seg_off[bj] + ba - 1].y;
    cand_score[g] = bh ? int64_t((bh - 1ull) & ((1ull << 62) - 1ull)) : 0;
}

}  // namespace sja
