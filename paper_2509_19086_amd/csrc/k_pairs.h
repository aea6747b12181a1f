// Small batches, pair by pair.
//
// A tick of a few hundred gaps and jobs has next to no work in it: what it
// costs are the launches of the ordered forms (nine for a fit, three for a
// select, some thirty for the lists and the rounds of a resolve) and three looks
// of the host at what came out.  Up to kPairsMost pairs nothing is ordered ahead:
//   * k_fit_pairs, k_best_pairs: a thread per pair finds its atom by one search
//     on both conditions;
//   * k_select_pairs: a thread block per gap reads the gap's row of replies;
//   * k_order_pairs, k_rounds_pairs: a thread block per gap puts the jobs that
//     fit in the order of their keys, and one block plays all rounds, a thread per gap.
// A whole tick is five launches and one look (six after sja_fit_select with many pairs).  Gaps x jobs, 256 segments each, us a tick
// (fairness), ordered forms and so: 8 x 16 300 / 57, 256 x 1024 547 / 91, 1024 x 512 578 / 182,
// 256 x 4096 537 / 179, 1024 x 1024 with 784 rounds 1306 / 707, 1024 x 2048 with 221 rounds 796 / 415.
#pragma once

#include "k_fused.h"

namespace sja {

constexpr int kPairsGaps = 1024;            // a thread per gap in k_rounds_pairs
constexpr int kPairsJobs = 4096;            // a gap's keys are put in order in LDS
// Pairs up to which all of it is faster.  fit -> select by itself decides: 51 us at 1024 x 2048 against 54 in the
// ordered form, 77 against 54 at 1024 x 4096 (a fit takes 20 against 67 and 38 against 69, a tick as above and 607
// against 767).  Where all gaps are alike the ordered form has next to nothing to do: 512 equal gaps x 4096 jobs 41 us
// against 65 so, but the rounds that follow, a grant each, 1005 against 385.
constexpr int64_t kPairsMost = 1 << 21;
constexpr int kPairsQ = 4;                  // pairs a thread searches side by side: their loads overlap
constexpr int kPairsThreads = 256;           // of a block of k_fit_pairs;
constexpr int kPairsMostThreads = 1024;     // the others have as many as they have work for
constexpr int kPairsSlots = 4;              // list entries are read four at a time (16 bits each)

// Of pair q the atoms that fit, a prefix: durations and peaks ascend.  The first atom of pair q is dp[q], there are
// n[q] of them.
template <int Q>
__device__ __forceinline__ void search_pairs(const int2 *const (&dp)[Q], const int (&n)[Q], const int (&w)[Q], const int (&c)[Q], int (&lo)[Q])
{
    int hi[Q], most = 0;
#pragma unroll
    for (int q = 0; q < Q; ++q) { lo[q] = 0; hi[q] = n[q]; most = max(most, n[q]); }
    for (; most > 0; most >>= 1) {
        int2 v[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q)
            if (lo[q] < hi[q]) v[q] = dp[q][(lo[q] + hi[q]) >> 1];
#pragma unroll
        for (int q = 0; q < Q; ++q)
            if (lo[q] < hi[q]) {
                const int mid = (lo[q] + hi[q]) >> 1;
                if (v[q].x <= w[q] && v[q].y <= c[q]) lo[q] = mid + 1; else hi[q] = mid;
            }
    }
}

// The same where the atoms of some pairs are known already: n is 0 for them.
template <int Q>
__device__ __forceinline__ void pair_atoms_or_search(const int2 *const (&dp)[Q], const int (&n)[Q], const int (&w)[Q], const int (&c)[Q], int (&at)[Q])
{
    int any = 0, lo[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) any |= n[q];
    if (any == 0) return;
    search_pairs<Q>(dp, n, w, c, lo);
#pragma unroll
    for (int q = 0; q < Q; ++q)
        if (n[q] > 0) at[q] = lo[q];
}

// The gaps as they came, for the calls that follow.
struct PairGaps {
    int32_t *w, *c, *order;
};
__device__ __forceinline__ void keep_gap(const PairGaps &keep, int g, int w, int c)
{
    keep.w[g] = w;
    keep.c[g] = c;
    keep.order[g] = g;
}

// A block per 256 jobs and kPairsQ gaps.
__global__ __launch_bounds__(kPairsThreads) void k_fit_pairs(int n_gaps, int n_jobs, const int32_t *__restrict__ W, const int32_t *__restrict__ C,
                                                             const int64_t *__restrict__ seg_off, const int2 *__restrict__ atom_dp,
                                                             const int2 *__restrict__ atom_db, const int32_t *__restrict__ n_atoms,
                                                             PairGaps keep, int32_t *__restrict__ cut, uint32_t *__restrict__ bits)
{
    constexpr int Q = kPairsQ;
    const int j = blockIdx.x * kPairsThreads + threadIdx.x, g0 = blockIdx.y * Q, words = (n_jobs + 31) / 32;
    const int64_t base = j < n_jobs ? seg_off[j] : 0;
    const int atoms = j < n_jobs ? n_atoms[j] : 0;
    const int2 *dp[Q];
    int n[Q], w[Q], c[Q], lo[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int g = min(g0 + q, n_gaps - 1);
        dp[q] = atom_dp + base;
        n[q] = g0 + q < n_gaps ? atoms : 0;
        w[q] = W[g];
        c[q] = C[g];
    }
    if (blockIdx.x == 0 && threadIdx.x < Q && g0 + int(threadIdx.x) < n_gaps)
        keep_gap(keep, g0 + threadIdx.x, W[g0 + threadIdx.x], C[g0 + threadIdx.x]);
    search_pairs<Q>(dp, n, w, c, lo);
    int b[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) b[q] = lo[q] > 0 ? atom_db[base + lo[q] - 1].y : -1;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        if (g0 + q >= n_gaps) break;
        if (j < n_jobs) cut[int64_t(g0 + q) * n_jobs + j] = b[q];
        if (!bits) continue;
        const unsigned long long on = __ballot(b[q] >= 0);
        const int lane = threadIdx.x & (kWave - 1), word = (j - lane) / 32 + (lane >> 5);
        if ((lane & 31) == 0 && word < words) bits[int64_t(g0 + q) * words + word] = lane ? uint32_t(on >> 32) : uint32_t(on);
    }
}

// The best of a block's keys (hi 0: none), in every thread of its first wave.
template <bool MIXED>
__device__ __forceinline__ void best_of_block(unsigned long long &bh, unsigned long long &bl, int &bj, int &ba)
{
    constexpr int kMostWaves = kPairsMostThreads / kWave;
    __shared__ unsigned long long s_hi[kMostWaves], s_lo[kMostWaves];
    __shared__ int s_job[kMostWaves], s_atoms[kMostWaves];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    auto wave_best = [&]() {
#pragma unroll
        for (int d = 1; d < kWave; d <<= 1) {
            const unsigned long long oh = (unsigned long long)__shfl_xor((long long)bh, d, kWave);
            const unsigned long long ol = MIXED ? (unsigned long long)__shfl_xor((long long)bl, d, kWave) : 0ull;
            const int oj = __shfl_xor(bj, d, kWave), oa = __shfl_xor(ba, d, kWave);
            if (fused_better(oh, ol, oj, bh, bl, bj)) { bh = oh; bl = ol; bj = oj; ba = oa; }
        }
    };
    wave_best();
    if (lane == 0) { s_hi[wave] = bh; s_lo[wave] = bl; s_job[wave] = bj; s_atoms[wave] = ba; }
    __syncthreads();
    if (wave > 0) return;
    const bool there = lane < int(blockDim.x) / kWave;
    const int at = there ? lane : 0;
    bh = there ? s_hi[at] : 0ull; bl = there ? s_lo[at] : 0ull; bj = there ? s_job[at] : INT32_MAX; ba = s_atoms[at];
    wave_best();
}

// Key of a job's reply: (tier : F * multiplier) + 1, and F for the MIXED policy's ties.
template <bool MIXED>
__device__ __forceinline__ void pair_key(unsigned long long F, unsigned long long mult, unsigned long long tier, unsigned long long &hi, unsigned long long &lo)
{
    hi = ((tier << 62) | times_mult(F, mult)) + 1ull;
    lo = MIXED ? F : 0ull;
}

// Where the replies of a gap come from: the matrix of sja_fit; the atoms that k_pair_atoms has left; or neither, each is
// searched.
struct PairReplies {
    const int32_t *cut, *pre_dur, *pre_peak;        // [gap][job], and the running tables
    const long long *pre_area;
    const uint16_t *atoms;                          // [gap][job]: atoms that fit (kManyAtoms: so many or more)
};
constexpr int kManyAtoms = 0xffff;

// The atoms of every pair, job by job: a block keeps 64 jobs' atoms in LDS and goes through a share of the gaps, four at a
// time a wave, a lane per job.  (From memory each step of a search is a trip to the caches: the best replies of 700 gaps x
// 2501 jobs took 48 us, so 15 and 22.)
constexpr int kAtomsThreads = 256, kAtomsJobs = kWave, kAtomsRoom = 4096, kAtomsQ = 4;
constexpr int kAtomsGaps = 32;              // gaps of a share
__global__ __launch_bounds__(kAtomsThreads) void k_pair_atoms(int n_gaps, int n_jobs, const int32_t *__restrict__ gap_w, const int32_t *__restrict__ gap_c,
                                                              const int64_t *__restrict__ seg_off, const int2 *__restrict__ atom_dp,
                                                              const int32_t *__restrict__ n_atoms, uint16_t *__restrict__ atoms)
{
    constexpr int WAVES = kAtomsThreads / kWave, Q = kAtomsQ;
    __shared__ int2 s_atom[kAtomsRoom];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int j = blockIdx.x * kAtomsJobs + lane;
    const int n = j < n_jobs ? n_atoms[j] : 0;
    const int64_t base = j < n_jobs ? seg_off[j] : 0;
    const int off = min(wave_scan_add(n) - n, kAtomsRoom), kept = min(n, kAtomsRoom - off);
    for (int l = wave; l < kWave; l += WAVES) {
        const int to = lane_value(off, l), m = lane_value(kept, l);
        const int2 *src = atom_dp + int64_t(lane_value64((unsigned long long)base, l));
        for (int a = lane; a < m; a += kWave) s_atom[to + a] = src[a];
    }
    __syncthreads();
    const int2 *dp = atom_dp + base;
    const bool whole = __all(kept == n);        // (the same in every wave)
    const int g1 = min((int(blockIdx.y) + 1) * kAtomsGaps, n_gaps);
    for (int g0 = int(blockIdx.y) * kAtomsGaps + wave * Q; g0 < g1; g0 += WAVES * Q) {
        int w[Q], c[Q], lo[Q], hi[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int g = min(g0 + q, g1 - 1);
            w[q] = gap_w[g];
            c[q] = gap_c[g];
            lo[q] = 0;
            hi[q] = n;
        }
        auto search = [&](auto atom) {
            for (int most = n; most > 0; most >>= 1) {
                int2 v[Q];
#pragma unroll
                for (int q = 0; q < Q; ++q) v[q] = atom(min((lo[q] + hi[q]) >> 1, n - 1));
#pragma unroll
                for (int q = 0; q < Q; ++q) {
                    const int mid = (lo[q] + hi[q]) >> 1;
                    const bool in = (v[q].x <= w[q]) & (v[q].y <= c[q]), open = lo[q] < hi[q];
                    lo[q] = open & in ? mid + 1 : lo[q];
                    hi[q] = open & !in ? mid : hi[q];
                }
            }
        };
        if (whole) search([&](int a) { return s_atom[off + a]; });
        else search([&](int a) { return dp[a]; });
#pragma unroll
        for (int q = 0; q < Q; ++q)
            if (g0 + q < g1 && j < n_jobs) atoms[int64_t(g0 + q) * n_jobs + j] = uint16_t(min(lo[q], kManyAtoms));
    }
}

// The best reply to a gap, a block per gap.
template <bool MIXED, bool ATOMS>
__global__ __launch_bounds__(kPairsMostThreads) void k_best_pairs(int n_jobs, PolicyDev pol, const int32_t *__restrict__ W, const int32_t *__restrict__ C,
                                                              const int64_t *__restrict__ seg_off, const int2 *__restrict__ atom_dp,
                                                              const int2 *__restrict__ atom_db, const long long *__restrict__ atom_area,
                                                              const int32_t *__restrict__ n_atoms, const int32_t *__restrict__ wait,
                                                              const uint8_t *__restrict__ sla_class, const int32_t *__restrict__ job_held,
                                                              const uint8_t *__restrict__ gap_active, PairGaps keep, const uint16_t *__restrict__ atoms,
                                                              int32_t *__restrict__ cand_job, int32_t *__restrict__ cand_cut,
                                                              int64_t *__restrict__ cand_score)
{
    constexpr int Q = kPairsQ;
    const int g = blockIdx.x, tid = threadIdx.x;
    const int gw = W[g], gc = C[g];
    const bool on = !gap_active || gap_active[g];
    if (tid == 0) keep_gap(keep, g, gw, gc);
    unsigned long long bh = 0, bl = 0;
    int bj = INT32_MAX, ba = 0;
    for (int j0 = tid; on && j0 < n_jobs; j0 += Q * int(blockDim.x)) {
        const int2 *dp[Q];
        int n[Q], w[Q], c[Q], lo[Q];
        int64_t base[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int j = j0 + q * int(blockDim.x);
            const bool usable = j < n_jobs && !(job_held && job_held[j] >= 0);
            base[q] = usable ? seg_off[j] : 0;
            if (ATOMS) lo[q] = usable ? int(atoms[int64_t(g) * n_jobs + j]) : 0;
            n[q] = usable && (!ATOMS || lo[q] == kManyAtoms) ? n_atoms[j] : 0;
            dp[q] = atom_dp + base[q];
            w[q] = gw;
            c[q] = gc;
        }
        if (ATOMS) pair_atoms_or_search<Q>(dp, n, w, c, lo);
        else search_pairs<Q>(dp, n, w, c, lo);
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            if (lo[q] == 0) continue;
            const int j = j0 + q * int(blockDim.x);
            unsigned long long mult, tier, kh, kl;
            job_policy(pol, wait, sla_class, j, mult, tier);
            const int2 v = dp[q][lo[q] - 1];
            pair_key<MIXED>(atom_area ? (unsigned long long)atom_area[base[q] + lo[q] - 1] : rect_of(v.x, v.y), mult, tier, kh, kl);
            if (fused_better(kh, kl, j, bh, bl, bj)) { bh = kh; bl = kl; bj = j; ba = lo[q]; }
        }
    }
    best_of_block<MIXED>(bh, bl, bj, ba);
    if (tid == 0) {
        cand_job[g] = bh ? bj : -1;
        cand_cut[g] = bh ? atom_db[seg_off[bj] + ba - 1].y : -1;
        cand_score[g] = bh ? int64_t((bh - 1ull) & ((1ull << 62) - 1ull)) : 0;
    }
}

// The same from the replies that sja_fit left: the gap's row of the matrix.
template <bool MIXED>
__global__ __launch_bounds__(kPairsMostThreads) void k_select_pairs(int n_jobs, PolicyDev pol, const int64_t *__restrict__ seg_off,
                                                                const int32_t *__restrict__ pre_dur, const int32_t *__restrict__ pre_peak,
                                                                const long long *__restrict__ pre_area, const int32_t *__restrict__ cut,
                                                                const int32_t *__restrict__ wait, const uint8_t *__restrict__ sla_class,
                                                                const int32_t *__restrict__ job_held, const uint8_t *__restrict__ gap_active,
                                                                int32_t *__restrict__ cand_job, int32_t *__restrict__ cand_cut,
                                                                int64_t *__restrict__ cand_score)
{
    const int g = blockIdx.x, tid = threadIdx.x;
    const bool on = !gap_active || gap_active[g];
    unsigned long long bh = 0, bl = 0;
    int bj = INT32_MAX, bc = -1;
#pragma unroll 4
    for (int j = tid; on && j < n_jobs; j += int(blockDim.x)) {
        const int b = cut[int64_t(g) * n_jobs + j];
        if (b < 0 || (job_held && job_held[j] >= 0)) continue;
        const int64_t at = seg_off[j] + b - 1;
        unsigned long long mult, tier, kh, kl;
        job_policy(pol, wait, sla_class, j, mult, tier);
        pair_key<MIXED>(pre_area ? (unsigned long long)pre_area[at] : rect_of(pre_dur[at], pre_peak[at]), mult, tier, kh, kl);
        if (fused_better(kh, kl, j, bh, bl, bj)) { bh = kh; bl = kl; bj = j; bc = b; }
    }
    best_of_block<MIXED>(bh, bl, bj, bc);
    if (tid == 0) {
        cand_job[g] = bh ? bj : -1;
        cand_cut[g] = bh ? bc : -1;
        cand_score[g] = bh ? int64_t((bh - 1ull) & ((1ull << 62) - 1ull)) : 0;
    }
}

// Where entry k of gap g's list is: four entries side by side, those of neighbouring gaps next to each other.
__host__ __device__ constexpr size_t pair_list_words(int n_gaps, int most) { return size_t((most + kPairsSlots - 1) / kPairsSlots) * n_gaps; }

// A key as 52 bits that order nearly as it does: tier, exponent and 44 bits of the score.
__device__ __forceinline__ unsigned long long pair_digest(unsigned long long hi)
{
    const unsigned long long key = hi - 1ull, score = key & ((1ull << 62) - 1ull);
    const int e = score ? 63 - __clzll((long long)score) : 0;
    const unsigned long long mantissa = e ? score << (64 - e) : 0ull;
    return (key >> 62) << 50 | (unsigned long long)e << 44 | mantissa >> 20;
}
// Whether two keys of this digest are the same: a score from 2 up to 2^45 - 1 is in it whole.
__device__ __forceinline__ bool pair_digest_is_key(unsigned long long digest)
{
    const uint32_t e = uint32_t(digest >> 44) & 63u;
    return e - 1u < 44u;
}

// The jobs that fit gap blockIdx.x in the order of their keys, as many as the rounds can ask for: a gap passes
// only jobs that other gaps hold, so it needs no more of them than there are gaps (`most`).  A job is one word, its key's
// digest and its number.  Where fewer jobs are needed than fit, a histogram of the digests' leading bits says down to
// which of them to go; what is left is sorted in LDS by a bitonic network (steps within the 128 entries that a wave's
// threads exchange need no barrier).  Neighbours of the same digest are compared by their keys, and if one pair is out of
// order the gap's jobs are sorted anew, by all of the key.  ROOM: a power of two, at least the number of jobs.
// 700 gaps x 2501 jobs, 700 of them each, MIXED: 60 us and 15 for k_pair_atoms, where all jobs searched and sorted by keys
// of 128 bits took 243; 256 x 1024 from the matrix, all words sorted, 16 us where that took 26.
// Two blocks of 1024 threads to a compute unit (that is, up to 78 scalar registers): with one, 283 blocks took two turns, 283 gaps
// x 1542 jobs 29 us where this takes 22, a resolve of eight rounds of 1005 x 1174 111 and 89.
constexpr int kOrderBins = 4096, kOrderBinShift = 40;
constexpr int kOrderBinsLeast = 1024;       // room from which on a histogram pays
static_assert(kPairsJobs <= 4096, "12 bits for a job");
template <bool MIXED, int ROOM, int THREADS>
__global__ __launch_bounds__(THREADS) __attribute__((amdgpu_waves_per_eu(THREADS == 1024 ? 8 : 1, 8))) void k_order_pairs(int n_gaps, int n_jobs, int most, PolicyDev pol, PairReplies from, const int32_t *__restrict__ gap_w,
                                                         const int32_t *__restrict__ gap_c, const int64_t *__restrict__ seg_off,
                                                         const int2 *__restrict__ atom_dp, const long long *__restrict__ atom_area,
                                                         const int32_t *__restrict__ n_atoms, const int32_t *__restrict__ wait,
                                                         const uint8_t *__restrict__ sla_class, int32_t *__restrict__ list_len,
                                                         unsigned long long *__restrict__ list)
{
    constexpr int Q = (ROOM + THREADS - 1) / THREADS, WAVES = THREADS / kWave;
    // the words, before them the histogram; or the keys of all jobs
    constexpr bool BINS = ROOM >= kOrderBinsLeast;
    constexpr int bytes = BINS && kOrderBins * 4 > ROOM * (MIXED ? 18 : 10) ? kOrderBins * 4 : ROOM * (MIXED ? 18 : 10);
    __shared__ alignas(8) unsigned char s_room[bytes];
    __shared__ int s_n, s_kept, s_all, s_bin, s_upto, s_bad, s_wave[WAVES];
    unsigned long long *const s_item = reinterpret_cast<unsigned long long *>(s_room);
    int *const s_hist = reinterpret_cast<int *>(s_room);
    unsigned long long *const s_hi = s_item, *const s_lo = s_item + (MIXED ? ROOM : 0);
    uint16_t *const s_job = reinterpret_cast<uint16_t *>(s_lo + ROOM);
    const int g = blockIdx.x, tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const int gw = gap_w[g], gc = gap_c[g];
    // the keys of N jobs; hi 0: it does not fit
    auto keys = [&](auto many, const int *job, unsigned long long *hi, unsigned long long *lo) {
        constexpr int N = decltype(many)::value;
        unsigned long long F[N];
        bool fits[N];
        if (from.cut) {
            int b[N];
#pragma unroll
            for (int q = 0; q < N; ++q) b[q] = job[q] < n_jobs ? from.cut[int64_t(g) * n_jobs + job[q]] : -1;
#pragma unroll
            for (int q = 0; q < N; ++q) {
                fits[q] = b[q] > 0;
                const int64_t at = fits[q] ? seg_off[job[q]] + b[q] - 1 : 0;
                F[q] = !fits[q] ? 0ull : from.pre_area ? (unsigned long long)from.pre_area[at] : rect_of(from.pre_dur[at], from.pre_peak[at]);
            }
        } else {
            const int2 *dp[N];
            int n[N], w[N], c[N], at[N];
            int64_t base[N];
#pragma unroll
            for (int q = 0; q < N; ++q) {
                base[q] = job[q] < n_jobs ? seg_off[job[q]] : 0;
                dp[q] = atom_dp + base[q];
                at[q] = from.atoms && job[q] < n_jobs ? int(from.atoms[int64_t(g) * n_jobs + job[q]]) : 0;
                n[q] = job[q] < n_jobs && (!from.atoms || at[q] == kManyAtoms) ? n_atoms[job[q]] : 0;
                w[q] = gw;
                c[q] = gc;
            }
            pair_atoms_or_search<N>(dp, n, w, c, at);
#pragma unroll
            for (int q = 0; q < N; ++q) {
                fits[q] = at[q] > 0;
                F[q] = 0;
                if (!fits[q]) continue;
                if (atom_area) {
                    F[q] = (unsigned long long)atom_area[base[q] + at[q] - 1];
                } else {
                    const int2 v = dp[q][at[q] - 1];
                    F[q] = rect_of(v.x, v.y);
                }
            }
        }
#pragma unroll
        for (int q = 0; q < N; ++q) {
            hi[q] = lo[q] = 0;
            if (!fits[q]) continue;
            unsigned long long mult, tier;
            job_policy(pol, wait, sla_class, job[q], mult, tier);
            pair_key<MIXED>(F[q], mult, tier, hi[q], lo[q]);
        }
    };
    // a bitonic network over n entries, a power of two: swap(a, b) if entry b is to come before a
    auto network = [&](int n, auto exchange) {
        __syncthreads();
        for (int k = 2; k <= n; k <<= 1) {
            for (int d = k >> 1; d > 0; d >>= 1) {
                for (int t = tid; t < n / 2; t += THREADS) {
                    const int a = 2 * t - (t & (d - 1));
                    exchange(a, a + d, (a & k) == 0);
                }
                // what the next step reads was written by the same wave while it stays within 128 entries
                const int next = d > 1 ? d >> 1 : k;
                if (max(d, next) > kWave) __syncthreads(); else asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            }
        }
        __syncthreads();
    };
    const bool cut_off = BINS && most + most / 8 < n_jobs;
    if (tid == 0) { s_n = s_kept = s_all = s_bad = 0; s_bin = kOrderBins; }
    if (cut_off)
        for (int i = tid; i < kOrderBins; i += THREADS) s_hist[i] = 0;
    __syncthreads();
    unsigned long long item[Q];
    unsigned fits = 0;                  // which of them are
    int fit = 0;                        // of this wave's jobs
    {
        int job[Q];
        unsigned long long hi[Q], lo[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) job[q] = tid + q * THREADS;
        keys(std::integral_constant<int, Q>{}, job, hi, lo);
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            item[q] = hi[q] ? (~pair_digest(hi[q]) << 12) | uint32_t(job[q]) : ~0ull;
            fits |= unsigned(hi[q] != 0) << q;
            fit += __popcll(__ballot(hi[q] != 0));
            if (cut_off && hi[q]) atomicAdd(&s_hist[item[q] >> (kOrderBinShift + 12)], 1);
        }
    }
    if (lane == 0) atomicAdd(&s_n, fit);
    __syncthreads();
    const int n_fit = s_n;
    int n = n_fit;                      // entries to be put in order
    if (BINS && cut_off && n_fit > most) {
        // the first bin by whose end there are enough
        constexpr int each = kOrderBins / THREADS;
        int mine = 0;
#pragma unroll 4
        for (int i = 0; i < each; ++i) mine += s_hist[tid * each + i];
        const int upto = wave_scan_add(mine);
        if (lane == kWave - 1) s_wave[wave] = upto;
        __syncthreads();
        int before = upto - mine;
        for (int w = 0; w < wave; ++w) before += s_wave[w];
        if (before < most && before + mine >= most) {
            int b = tid * each, sum = before;
            while ((sum += s_hist[b]) < most) ++b;
            s_bin = b;
            s_upto = sum;
        }
        __syncthreads();
        n = s_upto;
    }
    const int last_bin = s_bin;
    __syncthreads();                    // (the words take the histogram's place)
    int room = kPairsSlots;
    while (room < n) room <<= 1;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const bool in = (fits >> q & 1u) && int(item[q] >> (kOrderBinShift + 12)) <= last_bin;
        const unsigned long long some = __ballot(in);
        if (!some) continue;
        int at = 0;
        if (lane == 0) at = atomicAdd(&s_kept, __popcll(some));
        at = __builtin_amdgcn_readfirstlane(at) + __popcll(some & ((1ull << lane) - 1ull));
        if (in) s_item[at] = item[q];
    }
    for (int i = n + tid; i < room; i += THREADS) s_item[i] = ~0ull;
    network(room, [&](int a, int b, bool up) {
        const unsigned long long x = s_item[a], y = s_item[b];
        if ((y < x) == up) { s_item[a] = y; s_item[b] = x; }
    });
    const int len = min(n_fit, most);
    // neighbours of one digest: the jobs are in order, the keys may not be
    for (int i = tid; i + 1 < n; i += THREADS) {
        if (s_item[i] >> 12 != s_item[i + 1] >> 12) continue;
        if (!MIXED && pair_digest_is_key(~(s_item[i] >> 12))) continue;
        const int job[2] = {int(s_item[i] & 0xfffu), int(s_item[i + 1] & 0xfffu)};
        unsigned long long hi[2], lo[2];
        keys(std::integral_constant<int, 2>{}, job, hi, lo);
        if (hi[1] > hi[0] || (hi[1] == hi[0] && lo[1] > lo[0])) s_bad = 1;
    }
    __syncthreads();
    const int words = (min(room, most) + kPairsSlots - 1) / kPairsSlots;
    if (tid == 0) list_len[g] = len;
    if (!s_bad) {
        for (int k = tid; k < words; k += THREADS) {
            unsigned long long out = 0;
#pragma unroll
            for (int q = 0; q < kPairsSlots; ++q) {
                const int i = kPairsSlots * k + q;
                out |= (unsigned long long)(i < n ? uint32_t(s_item[i]) & 0xfffu : uint32_t(n_jobs)) << (16 * q);
            }
            list[size_t(k) * n_gaps + g] = out;
        }
        return;
    }
    // all jobs that fit, by all of their keys
    __syncthreads();
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const bool in = fits >> q & 1u;
        const unsigned long long some = __ballot(in);
        if (!some) continue;
        int at = 0;
        if (lane == 0) at = atomicAdd(&s_all, __popcll(some));
        at = __builtin_amdgcn_readfirstlane(at) + __popcll(some & ((1ull << lane) - 1ull));
        if (!in) continue;
        const int job[1] = {int(item[q] & 0xfffu)};
        unsigned long long hi[1], lo[1];
        keys(std::integral_constant<int, 1>{}, job, hi, lo);
        s_hi[at] = hi[0];
        if (MIXED) s_lo[at] = lo[0];
        s_job[at] = uint16_t(job[0]);
    }
    room = kPairsSlots;
    while (room < n_fit) room <<= 1;
    for (int i = n_fit + tid; i < room; i += THREADS) {
        s_hi[i] = 0;
        if (MIXED) s_lo[i] = 0;
        s_job[i] = uint16_t(n_jobs);            // nobody
    }
    network(room, [&](int a, int b, bool up) {
        const unsigned long long ha = s_hi[a], hb = s_hi[b];
        const unsigned long long la = MIXED ? s_lo[a] : 0ull, lb = MIXED ? s_lo[b] : 0ull;
        const uint16_t ja = s_job[a], jb = s_job[b];
        if (fused_better(hb, lb, jb, ha, la, ja) == up) {
            s_hi[a] = hb; s_hi[b] = ha;
            if (MIXED) { s_lo[a] = lb; s_lo[b] = la; }
            s_job[a] = jb; s_job[b] = ja;
        }
    });
    for (int k = tid; k < (min(room, most) + kPairsSlots - 1) / kPairsSlots; k += THREADS)
        list[size_t(k) * n_gaps + g] = *reinterpret_cast<const unsigned long long *>(s_job + kPairsSlots * k);
}

// All rounds by one block, a thread per gap.  A job's word is the smallest of its claims, round (22 bits) : gap
// (10 bits), all ones before; a job is named in one round only, so its word also says whether it is held: if it is
// smaller than any of the present round.  Behind a round's barrier one trip to LDS tells who won and which of the next
// four jobs on the list are free in the next round: claims that others have made there already look free, too.
// So a round is that trip, some 50 instructions and the barrier.
// list holds `most` entries for each gap, rounded up.

// Where the rounds leave what they found, and what a grant's cut is found by.
struct RoundsOut {
    PolicyDev pol;
    const int32_t *gap_w, *gap_c;
    const int64_t *seg_off;
    const int32_t *n_atoms;
    const int2 *atom_dp, *atom_db;
    const long long *atom_area;
    const int32_t *wait;
    const uint8_t *sla_class;
    int32_t *grant_job, *grant_cut;
    int64_t *grant_score;
    int32_t *job_gap, *rounds_and_stable;
};

// The outcome of the rounds: gap g won job `won`, or none.
__device__ __forceinline__ void rounds_out(int n_gaps, int n_jobs, int g, int threads, int won, int rounds, int stable, const uint32_t *s_word, const RoundsOut &out)
{
    for (int j = g; j < n_jobs; j += threads) out.job_gap[j] = s_word[j] == ~0u ? -1 : int(s_word[j] & (kPairsGaps - 1));
    if (g == 0) { out.rounds_and_stable[0] = rounds; out.rounds_and_stable[1] = stable; }
    if (g >= n_gaps) return;
    out.grant_job[g] = won;
    int b = -1;
    long long score = 0;
    if (won >= 0) {
        const int64_t base = out.seg_off[won];
        const int2 *dp[1] = {out.atom_dp + base};
        const int n[1] = {out.n_atoms[won]}, w[1] = {out.gap_w[g]}, c[1] = {out.gap_c[g]};
        int lo[1];
        search_pairs<1>(dp, n, w, c, lo);
        const int2 v = dp[0][lo[0] - 1];
        unsigned long long mult, tier;
        job_policy(out.pol, out.wait, out.sla_class, won, mult, tier);
        b = out.atom_db[base + lo[0] - 1].y;
        score = int64_t(times_mult(out.atom_area ? (unsigned long long)out.atom_area[base + lo[0] - 1] : rect_of(v.x, v.y), mult));
    }
    out.grant_cut[g] = b;
    out.grant_score[g] = score;
}

// A thread reads 16 entries of its list ahead, from memory.  With the lists in LDS (64 entries at a time, the next four jobs
// shifted in from eight) a round was no shorter: 330 resolves of up to 1024 gaps took 1.6 % longer on average, 0.86 to 1.06
// times as long this way, the most where all gaps pass the same jobs (263 gaps x 657 jobs of one capacity, 81 rounds:
// 83 us so and 71) or fill more than four waves; 256 x 1024 the same.
__global__ __launch_bounds__(kPairsGaps) void k_rounds_pairs(int n_gaps, int n_jobs, int most, int cap, const int32_t *__restrict__ list_len,
                                                             const unsigned long long *__restrict__ list, RoundsOut out)
{
    __shared__ uint32_t s_word[kPairsJobs + 1];         // the one behind the last job's: nobody, never free
    __shared__ int s_claims, s_lost;                    // the last round in which somebody claimed; the last one had losers
    const int g = threadIdx.x, threads = blockDim.x, lane = g & (kWave - 1);
    for (int i = g; i <= n_jobs; i += threads) s_word[i] = i < n_jobs ? ~0u : 0u;
    if (g == 0) s_claims = s_lost = 0;
    const int words = (most + kPairsSlots - 1) / kPairsSlots;
    int left = g < n_gaps ? (list_len[g] + kPairsSlots - 1) / kPairsSlots : 0;      // words of the list not yet read
    constexpr int kAhead = 4;
    unsigned long long ahead[kAhead];           // what the list has next
    uint32_t c[4], w[4];            // the next four jobs (byte offsets of their words), and their words
    int at = 0, in_hand = 0;
    auto ask = [&]() {
        if (in_hand > 0) return;
#pragma unroll
        for (int k = 0; k < kAhead; ++k) {
            const size_t to = size_t(min(at + k, words - 1)) * n_gaps + g;
            ahead[k] = list[to];
        }
        at += kAhead;
        in_hand = kAhead;
    };
    auto take = [&]() {
        const uint32_t a = uint32_t(ahead[0]), b = uint32_t(ahead[0] >> 32);
        c[0] = (a & 0xffffu) * 4; c[1] = (a >> 16) * 4; c[2] = (b & 0xffffu) * 4; c[3] = (b >> 16) * 4;
#pragma unroll
        for (int k = 1; k < kAhead; ++k) ahead[k - 1] = ahead[k];
        --in_hand;
        --left;
    };
    auto word = [&](uint32_t off) -> uint32_t & { return *reinterpret_cast<uint32_t *>(reinterpret_cast<char *>(s_word) + off); };
    const uint32_t nobody = uint32_t(n_jobs) * 4;
    __syncthreads();
    bool open = left > 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) { c[k] = nobody; w[k] = 0; }
    if (open) {
        ask();
        take();
        ask();
#pragma unroll
        for (int k = 0; k < 4; ++k) w[k] = word(c[k]);
    }
    int won = -1, lost_in = 0, rounds = 0, stable = 0;
    for (int round = 1;; ++round) {
        const uint32_t now = uint32_t(round) << 10;
        // (a job that was passed is held, and stays so)
        while (open && max(max(w[0], w[1]), max(w[2], w[3])) < now) {
            if (left == 0) { open = false; break; }
            take();
            ask();
#pragma unroll
            for (int k = 0; k < 4; ++k) w[k] = word(c[k]);
        }
        uint32_t job = w[0] >= now ? c[0] : w[1] >= now ? c[1] : w[2] >= now ? c[2] : c[3];
        job = open ? job : nobody;
        // the job of a wave's lowest gap is claimed once for all of its gaps that want it
        const unsigned long long claims = __ballot(open);
        if (claims) {
            const int first = __ffsll((long long)claims) - 1;
            const bool same = job == uint32_t(__builtin_amdgcn_readlane(int(job), first));
            if (open && (!same || lane == first)) atomicMin(&word(job), now | uint32_t(g));
            if (lane == first) s_claims = round;
        }
        __syncthreads();
        const uint32_t outcome = word(job);
#pragma unroll
        for (int k = 0; k < 4; ++k) w[k] = word(c[k]);
        const int claimed = *static_cast<volatile int *>(&s_claims);
        if (claimed < round || round == cap) {
            // nobody is left that could claim anything, or it is to end: were there losers in the last round played?
            const bool lost = claimed < round ? round > 1 && lost_in == round - 1 : open && outcome != (now | uint32_t(g));
            if (claimed >= round && open && !lost) won = int(job >> 2);
            if (lost) s_lost = 1;
            __syncthreads();
            rounds = claimed >= round || round == 1 || s_lost ? round : round - 1;
            stable = claimed < round || !s_lost;
            break;
        }
        if (open) {
            if (outcome == (now | uint32_t(g))) { won = int(job >> 2); open = false; }
            else lost_in = round;
        }
    }
    rounds_out(n_gaps, n_jobs, g, threads, won, rounds, stable, s_word, out);
}

}  // namespace sja
