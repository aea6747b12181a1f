// K4, list-driven: conflict rounds without re-scanning the pair matrix.
//
// The rounds are inherently sequential (a round's selections depend on the
// grants of the round before) and a large batch needs thousands of them, so a
// round must cost next to nothing.  What a gap needs in a round is "my best job
// that no gap holds yet".  Every gap ranks jobs by the same per-atom policy key
// (an atom is a safe cut of a job; the key depends on the job and on the cut,
// not on the gap), and in sorted gap order an atom is the answer of a job for
// one contiguous range of positions.  So:
//   1. all reachable atoms are ranked once by policy key (stable radix passes:
//      key descending, job id ascending);
//   2. along the ranked atoms, for every list block (<= 64 sorted gap positions of one capacity class
//      whose windows are of similar length) the atoms some position of it would
//      get are listed in rank order, each with the range of lanes (positions)
//      it applies to;
//   3. a round is one small kernel: a wave per list block, a lane per gap; a
//      lane that lost walks on through its block's list to the next entry that
//      covers it and whose job is not held, and claims that job with an
//      atomicMax of (round, ~gap index), the claims of a thread block merged
//      first; the next round's kernel first checks who won.  Claims carry the
//      round number, so nothing is ever reset and a claim made in the current
//      round is not mistaken for a hold.  Where lanes pass hundreds of
//      records of jobs that were just taken, the waves also keep the held
//      jobs as a bitmap (see grant_step).  Round 1 of long lists has a kernel
//      of its own (k_grant_first), and most rounds run in one thread block
//      (k_grant_solo).
#pragma once

#include "k_policy.h"
#include "k_sort.h"

namespace sja {

// A list entry as it is sorted: list block (27 bits) : job (24) : lane range hi (7) : lo (6).
// With places: list block (18 bits) : place of the atom's first position (16) : job (17) : hi : lo; a place is
// the list block and lane of a position (up to kPlacedBlocks list blocks and kPlacedJobs jobs).
constexpr int kEntryJobShift = 13, kEntryBlockShift = 37, kEntryPlaceShift = 30, kEntryPlacedBlockShift = 46;
constexpr int kPlacedBlocks = 1 << (kEntryPlacedBlockShift - kEntryPlaceShift - 6), kPlacedJobs = 1 << (kEntryPlaceShift - kEntryJobShift);
static_assert(SJA_MAX_JOBS <= 1 << (kEntryBlockShift - kEntryJobShift), "job ids fit an entry");

// reach[j] = atoms of job j that some capacity class can reach; reach[n_jobs] = 0.  all_classes: ncap_tab already has
// that in its first row.
__global__ void k_reach(int n_jobs, const int32_t *__restrict__ plan, const int32_t *__restrict__ ncap_tab, int all_classes,
                        int32_t *__restrict__ reach)
{
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j > n_jobs) return;
    int r = 0;
    if (j < n_jobs && plan[kPlanTabled]) {
        const int n_classes = all_classes ? 1 : plan[kPlanClasses];
        for (int c = 0; c < n_classes; ++c) r = max(r, ncap_tab[int64_t(c) * n_jobs + j]);
    }
    reach[j] = r;
}

// Whether digests tell atoms apart depends on the keys: many jobs of one profile, their waits a thousandth apart, have
// hundreds of atoms of different keys behind each 24 bits.  kAlikeLeast to twice as many atoms, by a hash of their ids,
// are compared with the last one before them in a slot of `seen` (zeros at the start): alike counts those whose keys
// differ and whose leading 24 bits (lower half) or 32 bits (upper half) do not.
constexpr int kAlikeSlots = 4096, kAlikeLeast = 2048;
__host__ __device__ inline int alike_shift(uint32_t n_atoms)          // one atom in 2^shift is looked at
{
    int s = 0;
    while ((n_atoms >> s) >= 2u * kAlikeLeast) ++s;
    return s;
}
__device__ __forceinline__ void note_alike(const PolicyDev &pol, unsigned long long key, uint32_t digest, unsigned long long *seen, int32_t *alike)
{
    const unsigned long long was = atomicExch(&seen[((digest >> 8) * 2654435761u) >> 20], key + 1);
    if (was == 0 || was == key + 1) return;
    const uint32_t other = key_digest(pol, (was - 1) >> 62, (was - 1) & ((1ull << 62) - 1));
    if (other >> 8 == digest >> 8) atomicAdd(alike, other == digest ? 0x10001 : 1);
}
static_assert(kAlikeSlots == 1 << 12 && 2 * kAlikeLeast < 1 << 15, "slots by 12 bits of the product; the counts fit");

// One wave per job: inverted policy keys of its reachable atoms (ascending sort
// of the inverted key = descending key) and the identity permutation, and both as one word: inverted digest : atom.
// seen may be null.
__global__ __launch_bounds__(256) void k_atom_keys(
    int n_jobs, PolicyDev pol, const int64_t *__restrict__ seg_off, const int2 *__restrict__ atom_dp,
    const long long *__restrict__ atom_area, const int32_t *__restrict__ abase, const int32_t *__restrict__ wait,
    const uint8_t *__restrict__ sla_class, unsigned long long *__restrict__ key_hi,
    unsigned long long *__restrict__ key_lo, uint32_t *__restrict__ perm, int4 *__restrict__ info, unsigned long long *__restrict__ digest,
    unsigned long long *bits, unsigned long long *seen, int32_t *alike)
{
    __shared__ unsigned long long s_bits[2][256 / kWave];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const bool mixed = pol.policy == SJA_POLICY_MIXED;
    unsigned long long any_hi = 0, any_lo = 0;
    const uint32_t total = seen ? uint32_t(abase[n_jobs]) : 0u;
    const uint32_t sampled = total > uint32_t(kKeyTile) ? uint32_t((1ull << 32) >> alike_shift(total)) : 0u;      // (a hash below it)
    for (int j = blockIdx.x * (256 / kWave) + wave; j < n_jobs; j += gridDim.x * (256 / kWave)) {
        const int a0 = abase[j], n = abase[j + 1] - a0;
        const int64_t base = seg_off[j];
        const int2 *dp = atom_dp + base;
        unsigned long long mult, tier;
        job_policy(pol, wait, sla_class, j, mult, tier);
        for (int a = lane; a < n; a += kWave) {
            const int2 v = dp[a];
            const unsigned long long F = atom_area ? (unsigned long long)atom_area[base + a]
                                                   : (unsigned long long)v.x * (unsigned long long)v.y;
            const unsigned long long k = (tier << 62) | (F * mult);
            key_hi[a0 + a] = ~k;
            const uint32_t lead = key_digest(pol, tier, F * mult);
            digest[a0 + a] = (static_cast<unsigned long long>(~lead) << 32) | uint32_t(a0 + a);
            if (uint32_t(a0 + a) * 2654435761u < sampled) note_alike(pol, k, lead, seen, alike);
            any_hi |= k;
            if (mixed) {
                key_lo[a0 + a] = ~F;
                any_lo |= F;
            }
            perm[a0 + a] = uint32_t(a0 + a);
            info[a0 + a] = make_int4(j, v.x, v.y, 0);
        }
    }
    // bits that are set in some key: a byte without any is the same in all (inverted) keys
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        any_hi |= (unsigned long long)__shfl_xor((long long)any_hi, d, kWave);
        any_lo |= (unsigned long long)__shfl_xor((long long)any_lo, d, kWave);
    }
    if (lane == 0) { s_bits[0][wave] = any_hi; s_bits[1][wave] = any_lo; }
    __syncthreads();
    if (threadIdx.x < 2) {
        const unsigned long long v = s_bits[threadIdx.x][0] | s_bits[threadIdx.x][1] | s_bits[threadIdx.x][2] | s_bits[threadIdx.x][3];
        // after the first few blocks there is nothing left to add
        if (v & ~__hip_atomic_load(&bits[threadIdx.x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicOr(&bits[threadIdx.x], v);
    }
}

// Grant-list blocks.  A list serves its gaps well when most of its records
// cover most of its lanes; a sub-block that starts at a very small window and
// ends at a much larger one is therefore cut into pieces, each ending before
// the first window beyond 1.5 * (its first window) + 64.
__device__ __forceinline__ int list_piece_end(const int32_t *__restrict__ gap_w, int b, int e)
{
    const int64_t w0 = max(gap_w[b], 0);
    const int64_t limit = w0 + (w0 >> 1) + 64;
    int p = b + 1;
    while (p < e && int64_t(gap_w[p]) <= limit) ++p;
    return p;
}

// Pieces per sub-block (an exclusive scan turns them into lb_off).
__global__ void k_list_blocks_count(int n_slots, const int32_t *__restrict__ plan,
                                    const int32_t *__restrict__ sub_begin, const int32_t *__restrict__ sub_end,
                                    const int32_t *__restrict__ gap_w, int32_t *lb_off)
{
    const int u = blockIdx.x * blockDim.x + threadIdx.x;
    if (u >= n_slots) return;
    int cnt = 0;
    if (plan[kPlanTabled] && u < plan[kPlanSubBlocks]) {
        const int e = sub_end[u];
        for (int b = sub_begin[u]; b < e; b = list_piece_end(gap_w, b, e)) ++cnt;
    }
    lb_off[u] = cnt;
}

// Writes the pieces, the list block of every position, and per class a table of positions by duration:
// entry k of a class's pos_entries / n_classes entries is the first position whose window reaches k << shift
// (the class's end from the last window on), so that a search for a duration only has a few positions left.
constexpr int kEntryWinBig = 32768, kEntryWinSmall = 8192;     // batches whose windows k_list_entries keeps in LDS
constexpr int kPosTable = 2048, kPosTableMany = 16384;          // entries for such batches, and for larger ones

__device__ __forceinline__ int pos_shift(int longest, int entries)
{
    int s = 0;
    while (s < 31 && (max(longest, 0) >> s) > entries - 2) ++s;
    return s;
}

__device__ __forceinline__ void pos_table_entry(int i, int pos_entries, int n_gaps, const int32_t *__restrict__ plan,
                                                const int32_t *__restrict__ class_begin,
                                                const int32_t *__restrict__ gap_w, int32_t *pos_tab)
{
    if (i >= pos_entries) return;
    const int n_classes = plan[kPlanClasses], entries = pos_entries / n_classes;
    const int c = i / entries;
    if (c >= n_classes) return;
    const int k = i - c * entries;
    const int begin = class_begin[c], end = c + 1 < n_classes ? class_begin[c + 1] : n_gaps;
    const int64_t d = int64_t(k) << pos_shift(gap_w[end - 1], entries);
    int lo = begin, hi = end;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (gap_w[mid] < d) lo = mid + 1; else hi = mid;
    }
    pos_tab[i] = k == entries - 1 ? end : lo;
}

__global__ void k_list_blocks_write(int lb_cap, int n_gaps, int pos_entries, const int32_t *__restrict__ plan, const int32_t *__restrict__ class_begin,
                                    const int32_t *__restrict__ sub_begin, const int32_t *__restrict__ sub_end,
                                    const int32_t *__restrict__ gap_w, const int32_t *__restrict__ lb_off,
                                    int32_t *lb_begin, int32_t *lb_end, int32_t *pos_block, int32_t *pos_tab)
{
    const int u = blockIdx.x * blockDim.x + threadIdx.x;
    if (!plan[kPlanTabled]) return;
    if (u < plan[kPlanSubBlocks]) {
        int v = lb_off[u];
        const int e = sub_end[u];
        for (int b = sub_begin[u]; b < e && v < lb_cap; ++v) {
            const int p = list_piece_end(gap_w, b, e);
            lb_begin[v] = b;
            lb_end[v] = p;
            for (int i = b; i < p; ++i) pos_block[i] = v;
            b = p;
        }
    }
    pos_table_entry(u, pos_entries, n_gaps, plan, class_begin, gap_w, pos_tab);
}

// All of it in one launch while the sub-blocks are few: block 0 cuts them into pieces (a wave per sub-block,
// a lane per position: a piece ends at the first lane beyond its limit), the other blocks make the table.
// The serial walk of one thread per sub-block above takes 60 us at Stress, with its scan.
constexpr int kListBlocksOne = 2048;

__global__ __launch_bounds__(1024) void k_list_blocks(int lb_cap, int n_gaps, int pos_entries, int32_t *plan, const int32_t *__restrict__ class_begin,
                                                      const int32_t *__restrict__ sub_begin, const int32_t *__restrict__ sub_end,
                                                      const int32_t *__restrict__ gap_w, int32_t *lb_begin, int32_t *lb_end,
                                                      int32_t *pos_block, int32_t *pos_tab)
{
    __shared__ unsigned long long s_start[kListBlocksOne];     // lanes that start a piece
    __shared__ int s_off[kListBlocksOne];
    __shared__ int s_sum[1024 / kWave];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const bool tabled = plan[kPlanTabled] != 0;
    if (blockIdx.x > 0) {
        const int i = (int(blockIdx.x) - 1) * 1024 + tid;
        if (tabled) pos_table_entry(i, pos_entries, n_gaps, plan, class_begin, gap_w, pos_tab);
        return;
    }
    const int n_subs = tabled ? min(plan[kPlanSubBlocks], kListBlocksOne) : 0;
    for (int u = wave; u < n_subs; u += 1024 / kWave) {
        const int b = sub_begin[u], len = sub_end[u] - b;
        const int w = gap_w[b + min(lane, len - 1)];
        unsigned long long starts = 0;
        for (int s = 0; s < len;) {
            starts |= 1ull << s;
            const int64_t w0 = max(__builtin_amdgcn_readlane(w, s), 0);
            const unsigned long long beyond = __ballot(lane > s && lane < len && int64_t(w) > w0 + (w0 >> 1) + 64);
            s = beyond ? __ffsll((long long)beyond) - 1 : len;
        }
        if (lane == 0) s_start[u] = starts;
    }
    __syncthreads();
    int mine[kListBlocksOne / 1024], sum = 0;
#pragma unroll
    for (int k = 0; k < kListBlocksOne / 1024; ++k) {
        const int u = tid * (kListBlocksOne / 1024) + k;
        mine[k] = u < n_subs ? __popcll(s_start[u]) : 0;
        sum += mine[k];
    }
    const int upto = wave_scan_add(sum);
    if (lane == kWave - 1) s_sum[wave] = upto;
    __syncthreads();
    int off = upto - sum, all = 0;
    for (int v = 0; v < 1024 / kWave; ++v) {
        if (v < wave) off += s_sum[v];
        all += s_sum[v];
    }
#pragma unroll
    for (int k = 0; k < kListBlocksOne / 1024; ++k) {
        const int u = tid * (kListBlocksOne / 1024) + k;
        if (u < n_subs) s_off[u] = off;
        off += mine[k];
    }
    if (tid == 0) plan[kPlanListBlocks] = all;
    __syncthreads();
    for (int u = wave; u < n_subs; u += 1024 / kWave) {
        const int b = sub_begin[u], len = sub_end[u] - b;
        const unsigned long long starts = s_start[u], upto_me = starts & (~0ull >> (kWave - 1 - lane));
        const int v = s_off[u] + __popcll(upto_me) - 1;
        if (lane < len && v < lb_cap) {
            pos_block[b + lane] = v;
            if ((starts >> lane) & 1ull) {
                const unsigned long long later = starts & ~upto_me;
                lb_begin[v] = b + lane;
                lb_end[v] = later ? b + __ffsll((long long)later) - 1 : b + len;
            }
        }
    }
}

// Entries of the lists, in rank order.  An atom is the answer of its job for the positions from the first
// window that reaches its duration up to the first that reaches the next atom's: in every capacity class one
// range of positions, an entry for each list block it touches.  Lanes walk along the atoms as they are ranked,
// so that the entries leave in rank order and only their list block is left to sort by.  Two passes: counts per
// chunk of per_chunk atoms and per list block (EMIT false; chunk_at receives the counts), then the entries
// (chunk_at holds their exclusive sums).  The chunks go to the waves in turn: ranks far down, where many an
// atom answers for a whole class, hold most of the entries.
// Ranked atoms lie anywhere, so every load of a step is 64 lines for a wave: with the windows in global
// memory the count took 1.25 ms at Stress (8.5 million atoms, 8 classes), all of it those lines.  WIN > 0:
// the windows of all positions are kept in LDS (up to WIN of them, and up to kEntryBlocks list blocks).
// WIN = 0: their space goes to a finer table of positions, which leaves one or two steps of a search, and to
// the list blocks.  The counts per list block are added up in LDS in either form (an addition to global memory
// per entry, to a few hundred words, took 4.2 ms for 40000 gaps x 8192 jobs).
constexpr int kEntryThreads = 1024;
constexpr int kEntryBlocks = 1024;        // list blocks whose first positions a thread block keeps in LDS
constexpr int kEntryGrid = 512;           // most thread blocks: two per compute unit
constexpr int kEntryLeastAtoms = 8;       // atoms per wave's turn, at least
constexpr int kEntryFewWide = 2;          // ranges of three or more list blocks among a wave's that are served one by one
constexpr int kEntryMostBlocks = 19456;   // list blocks that the largest batch can have

template <bool EMIT, int WIN>
__global__ __launch_bounds__(kEntryThreads) void k_list_entries(
    int n_atoms, int per_chunk, int n_lb, int n_gaps, int pos_entries, const int32_t *__restrict__ plan, const int32_t *__restrict__ class_begin,
    const int32_t *__restrict__ lb_begin, const int32_t *__restrict__ pos_block, const int32_t *__restrict__ pos_tab,
    const int32_t *__restrict__ gap_w, const int32_t *__restrict__ gap_c, const uint32_t *__restrict__ perm,
    const int4 *__restrict__ info, int32_t *chunk_at, int32_t *list_count, unsigned long long *total,
    unsigned long long *__restrict__ ekey, int placed)
{
    constexpr bool kLds = WIN > 0;
    __shared__ int s_w[kLds ? WIN : 1];
    __shared__ int s_pos[kLds ? kPosTable : kPosTableMany];
    constexpr bool kBegins = kLds || EMIT;
    __shared__ int s_begin[kBegins ? (kLds ? kEntryBlocks : kEntryMostBlocks) + 1 : 1];      // first positions of the list blocks
    __shared__ int s_hint[kLds ? WIN / kWave : 1];             // list block of every 64th position
    __shared__ int s_diff[EMIT ? 1 : (kLds ? kEntryBlocks : kEntryMostBlocks) + 1];
    __shared__ int s_cap[kMaxClasses], s_end[kMaxClasses], s_shift[kMaxClasses], s_lb[kMaxClasses + 1];
    __shared__ long long s_all[kEntryThreads / kWave];
    __shared__ int s_src[EMIT ? kEntryThreads / kWave : 1][kWave];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
    const int n_classes = min(plan[kPlanClasses], kMaxClasses), entries = pos_entries / n_classes;
    for (int i = tid; i < entries * n_classes; i += kEntryThreads) s_pos[i] = pos_tab[i];
    for (int c = tid; c < n_classes; c += kEntryThreads) {
        const int end = c + 1 < n_classes ? class_begin[c + 1] : n_gaps;
        s_cap[c] = gap_c[end - 1];
        s_end[c] = end;
        s_shift[c] = pos_shift(gap_w[end - 1], entries);
        s_lb[c + 1] = end < n_gaps ? pos_block[end] : n_lb;       // list blocks of class c: [s_lb[c], s_lb[c + 1])
    }
    if (tid == 0) s_lb[0] = 0;
    if (kLds) {
        for (int i = tid; i < n_gaps; i += kEntryThreads) {
            s_w[kLds ? i : 0] = gap_w[i];
            if ((i & (kWave - 1)) == 0) s_hint[kLds ? i / kWave : 0] = pos_block[i];
        }
    }
    if (kBegins)
        for (int k = tid; k <= n_lb; k += kEntryThreads) s_begin[kBegins ? k : 0] = k < n_lb ? lb_begin[k] : n_gaps;
    if (!EMIT)
        for (int k = tid; k <= n_lb; k += kEntryThreads) s_diff[EMIT ? 0 : k] = 0;
    __syncthreads();
    auto window = [&](int p) { return kLds ? s_w[kLds ? p : 0] : gap_w[p]; };
    auto begin_of = [&](int k) { return s_begin[kBegins ? k : 0]; };
    auto block_of = [&](int p) {
        if (!kLds) return pos_block[p];
        int k = s_hint[kLds ? p / kWave : 0];
        while (begin_of(k + 1) <= p) ++k;
        return k;
    };

    const int n_chunks = int((int64_t(n_atoms) + per_chunk - 1) / per_chunk), n_waves = int(gridDim.x) * (kEntryThreads / kWave);
    long long count_all = 0;
    for (int chunk = blockIdx.x * (kEntryThreads / kWave) + wave; chunk < n_chunks; chunk += n_waves) {
        const int64_t i = int64_t(chunk) * per_chunk + lane;
        const bool valid = lane < per_chunk && i < n_atoms;
        int64_t at = EMIT ? chunk_at[chunk] : 0;
        int count = 0;
        const int a = valid ? int(perm[i]) : 0;
        const int4 x = info[a], y = info[min(a + 1, n_atoms - 1)];
        const bool more = a + 1 < n_atoms && y.x == x.x;           // the job's next atom
        for (int c = 0; c < n_classes; ++c) {
            int n = 0, k_lo = 0, p1 = 0, p2 = 0;
            if (valid && x.z <= s_cap[c]) {
                const int *tab = s_pos + c * entries;
                const int shift = s_shift[c];
                const int t1 = min(x.y >> shift, entries - 1);
                p1 = tab[t1];
                int q1 = tab[min(t1 + 1, entries - 1)];
                p2 = s_end[c];
                int q2 = p2;
                if (more && y.z <= s_cap[c]) {
                    const int t2 = min(y.y >> shift, entries - 1);
                    p2 = tab[t2];
                    q2 = tab[min(t2 + 1, entries - 1)];
                }
                if (p1 < q2) {          // else no position is left between the two
                    while (p1 < q1) {
                        const int m = (p1 + q1) >> 1;
                        if (window(m) < x.y) p1 = m + 1; else q1 = m;
                    }
                    while (p2 < q2) {
                        const int m = (p2 + q2) >> 1;
                        if (window(m) < y.y) p2 = m + 1; else q2 = m;
                    }
                    if (p1 < p2) {
                        k_lo = block_of(p1);
                        n = block_of(p2 - 1) - k_lo + 1;
                    }
                }
            }
            if (EMIT) {
                if (!__ballot(n > 0)) continue;
                const int upto = wave_scan_add(n);
                const int64_t out = at + (upto - n);
                const int block_shift = placed ? kEntryPlacedBlockShift : kEntryBlockShift;
                auto put = [&](int64_t to, int k, int job, int lo, int hi, int place) {
                    ekey[to] = (static_cast<unsigned long long>(uint32_t(k)) << block_shift) |
                               (static_cast<unsigned long long>(uint32_t(place)) << kEntryPlaceShift) |
                               (static_cast<unsigned long long>(uint32_t(job)) << kEntryJobShift) | uint32_t((hi << 6) | lo);
                };
                const int place = placed && n > 0 ? (k_lo << 6) + p1 - begin_of(k_lo) : 0;
                unsigned long long wide = __ballot(n > 2);
                if (__popcll(wide) > kEntryFewWide) {
                    // many ranges over several list blocks: a lane per entry (its range is the last one that starts
                    // at or before it)
                    const int total_n = __builtin_amdgcn_readlane(upto, kWave - 1), start = upto - n;
                    volatile int *src = s_src[EMIT ? wave : 0];
                    int carry = -1;
                    for (int e0 = 0; e0 < total_n; e0 += kWave) {
                        src[lane] = -1;
                        __builtin_amdgcn_wave_barrier();
                        if (n > 0 && start >= e0 && start < e0 + kWave) src[start - e0] = lane;
                        __builtin_amdgcn_wave_barrier();
                        const int mark = src[lane];
                        const int from_lane = wave_scan_max_dpp(lane == 0 ? max(mark, carry) : mark);
                        carry = __builtin_amdgcn_readlane(from_lane, kWave - 1);
                        const int fl = max(from_lane, 0);
                        const int k = e0 + lane - __shfl(start, fl, kWave), fn = __shfl(n, fl, kWave), fk = __shfl(k_lo, fl, kWave) + k;
                        const int f1 = __shfl(p1, fl, kWave), f2 = __shfl(p2, fl, kWave), fj = __shfl(x.x, fl, kWave),
                                  fp = placed ? __shfl(place, fl, kWave) : 0;
                        if (e0 + lane < total_n) {
                            const int b = begin_of(fk);
                            put(at + e0 + lane, fk, fj, k == 0 ? f1 - b : 0, (k == fn - 1 ? f2 : begin_of(fk + 1)) - b, fp);
                        }
                    }
                } else {
                    // most ranges lie in one list block or reach over one border: the first and the last part by the
                    // atom's lane, the whole list blocks between them, if any, by the wave together
                    if (n > 0) {
                        const int b = begin_of(k_lo);
                        put(out, k_lo, x.x, p1 - b, (n == 1 ? p2 : begin_of(k_lo + 1)) - b, place);
                    }
                    if (n > 1) put(out + n - 1, k_lo + n - 1, x.x, 0, p2 - begin_of(k_lo + n - 1), place);
                    for (; wide; wide &= wide - 1) {
                        const int t = __ffsll((long long)wide) - 1;
                        const int tn = lane_value(n, t), tk = lane_value(k_lo, t), tj = lane_value(x.x, t), tp = lane_value(place, t);
                        const int64_t to = at + lane_value(upto, t) - tn;
                        for (int k = lane + 1; k < tn - 1; k += kWave) put(to + k, tk + k, tj, 0, begin_of(tk + k + 1) - begin_of(tk + k), tp);
                    }
                }
                at += __builtin_amdgcn_readlane(upto, kWave - 1);
            } else if (n > 0) {
                count += n;
                atomicAdd(&s_diff[EMIT ? 0 : k_lo], 1);
                // (nothing to take back behind the class: the sums start anew there)
                if (k_lo + n < s_lb[c + 1]) atomicAdd(&s_diff[EMIT ? 0 : k_lo + n], -1);
            }
        }
        if (!EMIT) {
            const int all = __builtin_amdgcn_readlane(wave_scan_add(count), kWave - 1);
            if (lane == 0) chunk_at[chunk] = all;
            count_all += all;
        }
    }
    if (EMIT) return;
    if (lane == 0) s_all[wave] = count_all;
    __syncthreads();
    if (tid == 0) {         // (an addition per wave, thousands to one word, took 80 us)
        unsigned long long t = 0;
        for (int v = 0; v < kEntryThreads / kWave; ++v) t += (unsigned long long)s_all[v];
        if (t) atomicAdd(total, t);
    }
    // the list blocks' counts are the running sums of a class's differences
    for (int c = wave; c < n_classes; c += kEntryThreads / kWave) {
        const int lb0 = s_lb[c], lb1 = s_lb[c + 1];
        int run = 0;
        for (int k0 = lb0; k0 < lb1; k0 += kWave) {
            const int k = k0 + lane;
            const int upto = run + wave_scan_add(k < lb1 ? s_diff[EMIT ? 0 : k] : 0);
            if (k < lb1 && upto) atomicAdd(&list_count[k], upto);
            run = __builtin_amdgcn_readlane(upto, kWave - 1);
        }
    }
}

__device__ __forceinline__ unsigned long long claim_of(int round, int g)
{
    return (static_cast<unsigned long long>(round) << 32) | (0xffffffffu - uint32_t(g));
}

// One round for one list block (one wave, one lane per gap position).  First
// the outcome of round k-1: a gap whose candidate job carries the gap's own
// claim word has won (the grant is final), otherwise it lost.  Then, if
// `propose`, every lane that still needs a job walks on from its own pointer to
// the first entry that covers it and whose job is not held, and claims it.
// st = (pointer, candidate job, unused, flag) with flag 0 = active,
// 1 = granted, 2 = no candidate left (in memory the flag shares its word with
// the gap index).
//
// The lanes of a wave walk together: per round trip the wave reads kSweep chunks
// of 64 records, starting at the chunk of its lowest pointer still looking, and
// the claim words of those that cover a lane still looking.  A lane passes the
// records of its block that cover other lanes only (a job's other cuts), so
// most rounds some lane of most waves has more than one record to look at; a
// first look at the lane's own next record alone, with the joint walk behind it
// when that was not the one, made nine rounds in ten two trips longer.  The
// first chunks are asked for before the wave knows who won round k-1 (nearly
// every open lane lost), so they travel beside that check's claim word.
constexpr int kSweep = 2;        // chunks of 64 records the wave reads per trip (3: 1.7 ms slower per Stress resolve, 4: 3.7 ms)
constexpr int kSweepHeld = 8;  // the same with the held bitmap: no claim words to fetch, so a wider trip costs little
constexpr int kRoundBlock = 256; // threads per block of the round kernel
constexpr int kBlockClaims = 256; // claims a block merges in LDS per round
constexpr int kClaimTurns = 4;    // jobs whose claims a wave merges over its lanes before the rest are sent singly

constexpr int kHeldMaxWords = 4096;   // words of the held-job bitmap a block keeps in LDS (jobs / 32)
constexpr int kEffortWindow = 8;      // a window of kSweepHeld chunks in pieces (a block reads them chunk by chunk)
constexpr int kHeldRounds = 512;      // rounds that keep and read the bitmap

__device__ __forceinline__ bool held_bit(const uint32_t *s_held, uint32_t job)
{
    return (s_held[job >> 5] >> (job & 31u)) & 1u;
}

// HELD (the early rounds, where lanes pass hundreds of records of jobs that were
// just taken): the wave asks a bitmap in LDS which jobs were held before this
// round, instead of fetching a claim word per record, so a trip is one memory
// trip, not two; only the record a lane settles on has its claim word fetched.
// Two bitmaps alternate: a round reads one and writes only the other
// (held_next), so nothing it reads changes under it.  A job named in round k is
// held from round k+1 on, whoever wins it: the gaps naming it set its bit in the
// bitmap round k+1 reads, and its winner, when it learns in round k+1 that it
// won, sets it in the other one, after which both carry it.
// `pieces` and `windows`: how many jobs the lanes named, beyond one, and how many windows of records they took,
// beyond one: what the round would cost a single thread block.
template <bool HELD, typename REC>
__device__ __forceinline__ void grant_step(int round, bool propose, int lane, int g, int list_begin, int list_end,
                                           const REC *__restrict__ rec, unsigned long long *claim, int4 &st,
                                           bool &lost, bool &cand, int *s_n, int *s_job,
                                           unsigned long long *s_word, const uint32_t *s_held,
                                           uint32_t *held_next, int &pieces, int &windows)
{
    pieces = windows = -1;
    constexpr int SW = HELD ? kSweepHeld : kSweep;
    lost = false;
    cand = false;
    // the first chunks, for every lane that is open now
    const bool open_now = st.w == 0 && propose && st.x < list_end;
    int e0 = wave_min_dpp(open_now ? st.x : 0x7fffffff);
    bool ahead = e0 != 0x7fffffff;                 // rr holds the chunks from c0 on
    int c0 = ahead ? list_begin + ((e0 - list_begin) & ~(kWave - 1)) : 0;
    REC rr[SW];
    if (ahead) {
#pragma unroll
        for (int k = 0; k < SW; ++k) rr[k] = rec[min(c0 + k * kWave + lane, list_end - 1)];
    }
    if (st.w == 0 && st.y >= 0) {
        if (claim[st.y] == claim_of(round - 1, g)) {               // won: final
            st.w = 1;
            if (HELD) atomicOr(&held_next[uint32_t(st.y) >> 5], 1u << (uint32_t(st.y) & 31u));
        } else {
            lost = true;
        }
    }
    int cand_job = -1;
    unsigned long long cand_word = 0;      // the candidate job's claim word as the walk saw it
    const bool walking = st.w == 0 && propose;
    int e = st.x, found = -1, found_j = -1;
    bool by_bitmap = false;                // found with HELD: the claim word is still to fetch
    bool looking = walking && e < list_end;
    // HELD: the chunks behind the ones being looked at are asked for before the look starts (a wave
    // whose lanes' pointers lie thousands of records apart takes window after window, and a lane
    // that finds nothing goes on exactly there), so their trip overlaps the look.  Always issued,
    // at clamped addresses: a load that may be skipped makes every later wait a wait for all.
    REC rn[HELD ? SW : 1];
    int c_next = -1;
    for (;;) {
        const unsigned long long need = __ballot(looking);
        if (!need) break;
        ++windows;
        if (!ahead) {
            e0 = wave_min_dpp(looking ? e : 0x7fffffff);    // the wave's lowest pointer still looking
            c0 = list_begin + ((e0 - list_begin) & ~(kWave - 1));
            if (HELD && c0 == c_next) {
#pragma unroll
                for (int k = 0; k < SW; ++k) rr[k] = rn[k];
            } else {
#pragma unroll
                for (int k = 0; k < SW; ++k) rr[k] = rec[min(c0 + k * kWave + lane, list_end - 1)];
            }
        }
        ahead = false;
        if (HELD) {
            c_next = c0 + SW * kWave;
#pragma unroll
            for (int k = 0; k < SW; ++k) rn[k] = rec[min(c_next + k * kWave + lane, list_end - 1)];
        }
        // claim words only of records that cover some lane still looking
        const int all_lo = __ffsll((long long)need) - 1, all_hi = 63 - __clzll((long long)need);
        unsigned long long cw[HELD ? 1 : SW];      // the claim words; HELD asks the bitmap instead
        bool open_job[HELD ? SW : 1];
        if (HELD) {
#pragma unroll
            for (int k = 0; k < SW; ++k) open_job[k] = !held_bit(s_held, rr[k].job());
        } else {
            // every lane loads (the others word 0, one request per wave) so that the loads of all
            // chunks are issued back to back: a load that may be skipped makes the next one wait for it
            bool worth[SW];
#pragma unroll
            for (int k = 0; k < SW; ++k) worth[k] = rr[k].lo() <= all_hi && rr[k].hi() > all_lo;
#pragma unroll
            for (int k = 0; k < SW; ++k) cw[k] = claim[worth[k] ? rr[k].job() : 0u];
#pragma unroll
            for (int k = 0; k < SW; ++k) cw[k] = worth[k] ? cw[k] : ~0ull;
        }
        const bool here = looking && e < c0 + SW * kWave;
        int hit = -1, hj = 0;
        unsigned int hw_lo = 0, hw_hi = 0;
#pragma unroll
        for (int k = 0; k < SW; ++k) {
            // lanes this chunk can serve: still looking, and standing before its end (the pointers of
            // a wave of the early rounds lie thousands of records apart: most lanes `here` only
            // start in a later chunk of the window, and nothing in this one is for them)
            const bool elig = here && hit < 0 && e < c0 + (k + 1) * kWave;
            const unsigned long long still = __ballot(elig);
            if (!still) continue;
            // records worth a look: free, and covering some lane that can take one here
            const int need_lo = __ffsll((long long)still) - 1;
            const int need_hi = 63 - __clzll((long long)still);
            const uint32_t stamp = HELD ? 0u : uint32_t(cw[HELD ? 0 : k] >> 32);
            const bool not_held = HELD ? open_job[HELD ? k : 0] : (stamp == 0 || (stamp >= uint32_t(round) && stamp != 0xffffffffu));
            const bool free_rec = c0 + k * kWave + lane < list_end && not_held &&
                                  rr[k].lo() <= need_hi && rr[k].hi() > need_lo;
            unsigned long long fm = __ballot(free_rec);
            int hk = -1;
            while (fm) {
                const int t = __ffsll((long long)fm) - 1;
                fm &= fm - 1;
                const REC rt = rr[k].of_lane(t);
                const bool h = elig && hk < 0 && c0 + k * kWave + t >= e && lane >= rt.lo() && lane < rt.hi();
                if (__any(h)) {
                    // record t's job and claim word straight from lane t's registers
                    const int tj = int(rt.job());
                    // (with HELD the claim word of the record a lane settles on is fetched afterwards)
                    const unsigned int t_lo = HELD ? 0u : __builtin_amdgcn_readlane(int(uint32_t(cw[HELD ? 0 : k])), t);
                    const unsigned int t_hi = HELD ? 0u : __builtin_amdgcn_readlane(int(uint32_t(cw[HELD ? 0 : k] >> 32)), t);
                    if (h) { hk = t; hit = k * kWave + t; hj = tj; hw_lo = t_lo; hw_hi = t_hi; }
                }
                if (!__any(elig && hk < 0)) break;
            }
        }
        if (here) {
            if (hit >= 0) {
                found = c0 + hit; found_j = hj;
                cand_word = (static_cast<unsigned long long>(hw_hi) << 32) | hw_lo;
                by_bitmap = HELD;
                looking = false;
            } else {
                e = c0 + SW * kWave;
                looking = e < list_end;
            }
        }
    }
    if (HELD && by_bitmap) cand_word = claim[found_j];      // what this round's earlier claims left there
    if (walking) {
        if (found >= 0) {
            st = make_int4(found + 1, found_j, 0, 0);
            cand = true;
            cand_job = found_j;
        } else {
            st = make_int4(list_end, -1, -1, 2);
        }
    }
    // Claims.  Most gaps of a batch name the same few jobs in a round, so the
    // lanes of a wave that name one job first agree on their lowest gap index,
    // and a claim that the job's word (as the walk read it) already beats is not
    // made.  The wave's claims go to the block's list (s_n, s_job, s_word); the
    // block merges them before anything is sent (a claim that finds the list
    // full is sent at once).
    unsigned long long todo = __ballot(cand);
    for (int turn = 0; todo; ++turn) {
        ++pieces;
        if (turn == kClaimTurns) {
            pieces += __popcll(todo) - 1;
            // a wave of the early rounds, whose lanes name dozens of different jobs: one turn of
            // this loop per job costs more than the claims it merges, so the rest go out as they are
            if ((todo >> lane) & 1ull) {
                const unsigned long long word = claim_of(round, g);
                if (cand_word < word) {
                    atomicMax(&claim[cand_job], word);
                    if (HELD) atomicOr(&held_next[uint32_t(cand_job) >> 5], 1u << (uint32_t(cand_job) & 31u));
                }
            }
            break;
        }
        const int leader = __ffsll((long long)todo) - 1;
        const int job = __builtin_amdgcn_readlane(cand_job, leader);
        const bool mine = cand && cand_job == job;
        const unsigned int best = 0xffffffffu - uint32_t(wave_min_dpp(mine ? g : 0x7fffffff));   // larger = lower gap index
        if (lane == leader) {
            const unsigned long long word = (static_cast<unsigned long long>(round) << 32) | best;
            if (cand_word < word) {
                const int slot = atomicAdd(s_n, 1);
                if (slot < kBlockClaims) {
                    s_job[slot] = job;
                    s_word[slot] = word;
                } else {
                    atomicMax(&claim[job], word);
                    if (HELD) atomicOr(&held_next[uint32_t(job) >> 5], 1u << (uint32_t(job) & 31u));
                }
            }
        }
        todo &= ~__ballot(mine);
    }
}

// One round per launch, several list blocks per thread block.  Hundreds of
// waves name the same few jobs in a round and atomics on one word are served
// one after the other, so the waves of a block first merge their claims in LDS
// and the block sends one atomicMax per job.  A round leaves two flags: somebody
// lost (round k-1), somebody selected (round k); the host only asks those two
// questions.
// n_lb, the number of list blocks, comes as an argument (the host has read it
// back to size its launches): the state and the block's list bounds are all a
// wave has to wait for before it can ask for its records and its claim word.
// effort (may be null): two words by turns of the rounds, what the round would have cost one thread block beyond
// the least; k_grant_solo looks at it.
// The arguments a wave needs first come first: the library is built so that
// the leading 16 dwords of a kernel's arguments are in scalar registers when
// the wave starts, and the state load does not wait for an argument load.
template <bool HELD, typename REC>
__global__ __launch_bounds__(kRoundBlock) void k_grant_round(
    int4 *state, const int32_t *__restrict__ list_off, const REC *__restrict__ rec, unsigned long long *claim,
    int round, int propose, int n_lb, int held_words, uint32_t *held, const int32_t *__restrict__ lb_begin,
    const int32_t *__restrict__ lb_end, const int32_t *__restrict__ gap_order, int32_t *cnt_lost, int32_t *cnt_cand, int32_t *effort)
{
    __shared__ int s_n, s_effort;
    __shared__ int s_job[kBlockClaims];
    __shared__ unsigned long long s_word[kBlockClaims];
    __shared__ uint4 s_held4[HELD ? kHeldMaxWords / 4 : 1];
    const uint32_t *s_held = reinterpret_cast<const uint32_t *>(s_held4);
    uint32_t *held_next = nullptr;
    const int u = blockIdx.x * (kRoundBlock / kWave) + (threadIdx.x / kWave);
    const int lane = threadIdx.x & (kWave - 1);
    // The state of a gap lives at (list block, lane) and carries the gap's index, so
    // that its load needs none of the block tables and travels together with them.
    const int slot = u * kWave + lane;
    int4 raw = make_int4(0, -1, -1, 2);
    int list_begin = 0, list_end = 0;
    if (u < n_lb) {
        raw = state[slot];               // round 1 reads what an earlier resolve left and replaces it below
        list_begin = list_off[u];
        list_end = list_off[u + 1];
    }
    if (HELD) {
        // the bitmap travels together with the state; held_words is a multiple of 4 and at most
        // kHeldMaxWords, and the two bitmaps lie back to back
        const uint4 *src = reinterpret_cast<const uint4 *>(held + size_t(round & 1) * held_words);
        for (int i = threadIdx.x; i < held_words / 4; i += kRoundBlock) s_held4[i] = src[i];
        held_next = held + size_t((round + 1) & 1) * held_words;
    }
    if (threadIdx.x == 0) s_n = s_effort = 0;
    __syncthreads();
    if (u < n_lb) {
        if (round == 1) {
            const int b0 = lb_begin[u];
            const bool valid = lane < lb_end[u] - b0;
            raw = make_int4(list_begin, -1, -1, valid ? (gap_order[b0 + lane] << 2) : 2);
        }
        const int g = raw.w >> 2;
        int4 st = make_int4(raw.x, raw.y, raw.z, raw.w & 3);
        const int4 before = st;
        bool lost, cand;
        int pieces, windows;
        grant_step<HELD, REC>(round, propose != 0, lane, g, list_begin, list_end, rec, claim, st, lost, cand, &s_n, s_job,
                         s_word, s_held, held_next, pieces, windows);
        const int mine = max(pieces, 0) + kEffortWindow * max(windows, 0);
        if (HELD && mine > 0 && lane == 0) atomicAdd(&s_effort, mine);
        if (st.x != before.x || st.w != before.w || round == 1) state[slot] = make_int4(st.x, st.y, st.z, st.w | (g << 2));
        if (__ballot(lost) && lane == 0) cnt_lost[round - 1] = 1;
        if (__ballot(cand) && lane == 0) cnt_cand[round] = 1;
    }
    __syncthreads();
    if (HELD && effort && threadIdx.x == kRoundBlock - 1) {        // (not the wave that merges the claims)
        if (s_effort > 0) atomicAdd(&effort[round & 1], s_effort);
        if (blockIdx.x == 0) effort[(round + 1) & 1] = 0;
    }
    const int n = min(s_n, kBlockClaims);
    if (n <= kWave) {
        // the usual case, a handful of claims: one lane of the first wave per claim, the others'
        // claims read from their lanes (a loop over the list in LDS pays two dependent LDS trips
        // per entry, at the very end of every round)
        if (threadIdx.x < kWave) {
            const bool valid = lane < n;
            const int job = valid ? s_job[lane] : -1;
            const unsigned long long word = valid ? s_word[lane] : 0ull;
            unsigned long long best = word;
            bool first = valid;
            for (int k = 0; k < n; ++k) {
                const int jk = __builtin_amdgcn_readlane(job, k);
                const unsigned long long wk =
                    (static_cast<unsigned long long>(uint32_t(__builtin_amdgcn_readlane(int(uint32_t(word >> 32)), k))) << 32) |
                    uint32_t(__builtin_amdgcn_readlane(int(uint32_t(word)), k));
                if (jk == job) {
                    best = max(best, wk);
                    first = first && k >= lane;
                }
            }
            if (first) {
                atomicMax(&claim[job], best);
                if (HELD) atomicOr(&held_next[uint32_t(job) >> 5], 1u << (uint32_t(job) & 31u));
            }
        }
        return;
    }
    for (int i = threadIdx.x; i < n; i += kRoundBlock) {
        const int job = s_job[i];
        unsigned long long word = s_word[i];
        bool first = true;
        for (int k = 0; k < n; ++k) {
            if (s_job[k] == job) {
                word = max(word, s_word[k]);
                first = first && k >= i;
            }
        }
        if (first) {
            atomicMax(&claim[job], word);
            if (HELD) atomicOr(&held_next[uint32_t(job) >> 5], 1u << (uint32_t(job) & 31u));
        }
    }
}

// One round per launch while rounds are much work, with the held-job bitmap: a thread block per list block, a
// wave per gap.  In the first rounds of a batch the gaps of a list block stand thousands of records apart and
// each of them has a few dozen to pass: a wave that walks for all of them (k_grant_round) sweeps everything
// between in window after window, 10 to 40 us a round.  Here every gap still looking is a wave's, which reads 256
// records a step from the gap's own place on (its waves take up to four gaps each, and ask for the first step
// of all four before they look at one).  What the gaps found is merged by the first wave, as there.
// Waves per list block: sixteen while two such thread blocks per compute unit hold all list blocks, else eight.
constexpr int kWideWaves = 16, kWideFewWaves = 8, kWideManyBlocks = 512;
constexpr int kWideChunk = 4 * kWave;    // records a wave reads at a time, four a lane
// Large (8192 gaps x 32768 jobs) 36 -> 6.2 us a round, the first rounds of Medium 12 -> 7; where the gaps of a list
// block stand together k_grant_round's one wave is quicker (Stress, 566 list blocks, from some hundred rounds on:
// 5.5 against 8.7).
constexpr int kWideBlocks = 1024;        // list blocks: beyond that the waves come in several turns
// Gaps stand the further apart the earlier the round.  A resolve with the first 64, 128, 256 and 512 rounds so: Stress 41.0,
// 41.0, 40.7 and 41.9 ms (MIXED), 4096 gaps x 16384 jobs 4.75, 4.25, 4.25 and 4.26, 8192 x 8192 9.38, 8.45, 8.41 and 8.54
// (FAIRNESS); Medium and 8192 x 32768 within 3 %.
constexpr int kWideRounds = 256;

template <int WAVES>
__global__ __launch_bounds__(WAVES * kWave) void k_grant_wide(
    int4 *state, const int32_t *__restrict__ list_off, const Rec32 *__restrict__ rec, unsigned long long *claim, int round, int held_words,
    uint32_t *held, const int32_t *__restrict__ lb_begin, const int32_t *__restrict__ lb_end, const int32_t *__restrict__ gap_order,
    int32_t *cnt_lost, int32_t *cnt_cand, int32_t *effort)
{
    __shared__ uint4 s_held4[kHeldMaxWords / 4];
    __shared__ int s_found[kWave], s_job[kWave];
    constexpr int kTurns = kWave / WAVES;
    const uint32_t *s_held = reinterpret_cast<const uint32_t *>(s_held4);
    const int u = blockIdx.x, lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    int4 st = state[u * kWave + lane];
    const int begin = list_off[u], end = list_off[u + 1], last4 = (end - 1) >> 2;
    const uint4 *now = reinterpret_cast<const uint4 *>(held + size_t(round & 1) * held_words);
    uint32_t *held_next = held + size_t((round + 1) & 1) * held_words;
    for (int i = threadIdx.x; i < held_words / 4; i += WAVES * kWave) s_held4[i] = now[i];
    if (round == 1) {
        const int b0 = lb_begin[u];
        st = make_int4(begin, -1, 0, lane < lb_end[u] - b0 ? (gap_order[b0 + lane] << 2) : 2);
    }
    const int g = st.w >> 2, flag = st.w & 3;
    const bool waiting = flag == 0 && st.y >= 0;
    const bool won = waiting && claim[max(st.y, 0)] == claim_of(round - 1, g), lost = waiting && !won;
    const bool open = flag == 0 && !won, looking = open && st.x < end;
    const unsigned long long look = __ballot(looking);
    const int rank = __popcll(look & ((1ull << lane) - 1ull));
    int at[kTurns], of[kTurns];
    uint4 ahead[kTurns];
#pragma unroll
    for (int t = 0; t < kTurns; ++t) {
        const unsigned long long mine = __ballot(looking && rank == t * WAVES + wave);
        of[t] = mine ? __ffsll((long long)mine) - 1 : -1;
        at[t] = __builtin_amdgcn_readlane(st.x, max(of[t], 0));
        if (mine) ahead[t] = reinterpret_cast<const uint4 *>(rec)[min((at[t] >> 2) + lane, last4)];
    }
    __syncthreads();
#pragma unroll
    for (int t = 0; t < kTurns; ++t) {
        const int l = of[t];
        if (l < 0) continue;
        uint4 r4 = ahead[t];
        int found = -1, job = 0;
        for (int base = at[t] & ~3;;) {
            const uint32_t r[4] = {r4.x, r4.y, r4.z, r4.w};
            unsigned ok = 0;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const Rec32 x{r[k]};
                const int i = base + 4 * lane + k;
                const bool covers = (i >= at[t]) & (i < end) & (uint32_t(l - x.lo()) < uint32_t(x.hi() - x.lo()));
                ok |= unsigned(covers && !held_bit(s_held, x.job())) << k;
            }
            const unsigned long long some = __ballot(ok != 0);
            if (some) {
                const int s = __ffsll((long long)some) - 1, k = __ffs(__builtin_amdgcn_readlane(int(ok), s)) - 1;
                const uint32_t v = k & 2 ? (k & 1 ? r4.w : r4.z) : (k & 1 ? r4.y : r4.x);
                found = base + 4 * s + k;
                job = int(Rec32{v}.of_lane(s).job());
                break;
            }
            base += kWideChunk;
            if (base >= end) break;
            r4 = reinterpret_cast<const uint4 *>(rec)[min((base >> 2) + lane, last4)];
        }
        if (lane == 0) { s_found[l] = found; s_job[l] = job; }
    }
    __syncthreads();
    if (wave > 0) return;
    const bool cand = looking && s_found[lane] >= 0;
    const int job = cand ? s_job[lane] : -1;
    if (won) {
        atomicOr(&held_next[uint32_t(st.y) >> 5], 1u << (uint32_t(st.y) & 31u));
        state[u * kWave + lane].w = st.w | 1;
    } else if (cand) {
        state[u * kWave + lane] = make_int4(s_found[lane] + 1, job, 0, g << 2);
    } else if (open || round == 1) {
        state[u * kWave + lane] = make_int4(end, -1, 0, (g << 2) | 2);
    }
    if (__ballot(lost) && lane == 0) cnt_lost[round - 1] = 1;
    if (__ballot(cand) && lane == 0) cnt_cand[round] = 1;
    // the claims: the gaps that name one job agree on the lowest of them; one that the job's word already beats is not made
    const unsigned long long word_was = cand ? claim[job] : ~0ull;
    auto send = [&](int low) {
        const unsigned long long word = claim_of(round, low);
        if (word_was >= word) return;
        atomicMax(&claim[job], word);
        atomicOr(&held_next[uint32_t(job) >> 5], 1u << (uint32_t(job) & 31u));
    };
    int pieces = -1;
    unsigned long long todo = __ballot(cand);
    for (int turn = 0; todo; ++turn) {
        ++pieces;
        if (turn == kClaimTurns) {
            pieces += __popcll(todo) - 1;
            if ((todo >> lane) & 1ull) send(g);
            break;
        }
        const int leader = __ffsll((long long)todo) - 1;
        const bool same = cand && job == __builtin_amdgcn_readlane(job, leader);
        const int low = wave_min_dpp(same ? g : 0x7fffffff);
        if (lane == leader) send(low);
        todo &= ~__ballot(same);
    }
    const int nearest = wave_min_dpp(looking ? st.x : INT32_MAX), furthest = -wave_min_dpp(cand ? -s_found[lane] : 0);
    if (effort && lane == 0) {
        // (a wave of k_grant_round would have swept all records between the first and the last of them)
        const int mine = max(pieces, 0) + kEffortWindow * max((furthest - nearest) / (kSweepHeld * kWave), 0);
        if (mine > 0) atomicAdd(&effort[round & 1], mine);
        if (u == 0) effort[(round + 1) & 1] = 0;
    }
}

// Round 1 where the lists are long.  No job is held yet, so a lane's candidate is the first record that covers
// it, but the lowest lanes' lie tens of thousands of records down (a Large list block: 25 thousand records,
// 200 us for one wave in k_grant_round).  A thread block per list block: its waves take stretches of
// kFirstStretch records in turn and note the lowest record per lane; a wave stops once every lane has one
// before its next stretch.  Leaves state and claims as k_grant_round does for round 1.
constexpr int kFirstThreads = 1024, kFirstStretch = 4 * kWave;
constexpr int kFirstLong = 1024;         // records per list, on average, from which it pays (4 us launched)

template <typename REC>
__global__ __launch_bounds__(kFirstThreads) void k_grant_first(
    int4 *state, const int32_t *__restrict__ list_off, const REC *__restrict__ rec, unsigned long long *claim, uint32_t *held_next,
    const int32_t *__restrict__ lb_begin, const int32_t *__restrict__ lb_end, const int32_t *__restrict__ gap_order,
    int32_t *cnt_cand)
{
    __shared__ int s_first[kWave];
    const int u = blockIdx.x, lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const int begin = list_off[u], end = list_off[u + 1], b0 = lb_begin[u], len = lb_end[u] - b0;
    if (threadIdx.x < kWave) s_first[lane] = lane < len ? INT32_MAX : -1;
    __syncthreads();
    for (int64_t c64 = int64_t(begin) + wave * kFirstStretch; c64 < end; c64 += kFirstThreads / kWave * kFirstStretch) {
        const int c = int(c64);
        unsigned long long without = __ballot(s_first[lane] > c);       // lanes with no record before this stretch
        if (!without) break;
        REC r[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) r[k] = rec[min(c64 + k * kWave + lane, int64_t(end) - 1)];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int width = r[k].hi() - r[k].lo();
            const unsigned long long mine = width > 0 ? (~0ull >> (kWave - width)) << r[k].lo() : 0ull;
            unsigned long long hits = __ballot(c64 + k * kWave + lane < end && (mine & without) != 0);
            while (hits) {
                const int t = __ffsll((long long)hits) - 1;
                hits &= hits - 1;
                const REC x = r[k].of_lane(t);
                const bool takes = ((without >> lane) & 1ull) && lane >= x.lo() && lane < x.hi();
                if (takes) atomicMin(&s_first[lane], c + k * kWave + t);
                without &= ~__ballot(takes);
            }
        }
    }
    __syncthreads();
    if (wave > 0) return;
    const int first = s_first[lane];
    const bool valid = lane < len, cand = valid && first != INT32_MAX;
    const int g = valid ? gap_order[b0 + lane] : 0;
    const int job = cand ? int(rec[first].job()) : -1;
    state[u * kWave + lane] = cand ? make_int4(first + 1, job, 0, g << 2) : make_int4(end, -1, 0, (g << 2) | 2);
    if (__ballot(cand) && lane == 0) cnt_cand[1] = 1;
    auto send = [&](int j, int low) {
        atomicMax(&claim[j], claim_of(1, low));
        if (held_next) atomicOr(&held_next[uint32_t(j) >> 5], 1u << (uint32_t(j) & 31u));
    };
    unsigned long long todo = __ballot(cand);
    for (int turn = 0; todo; ++turn) {
        if (turn == kClaimTurns) {
            if ((todo >> lane) & 1ull) send(job, g);
            break;
        }
        const int leader = __ffsll((long long)todo) - 1;
        const bool same = cand && job == __builtin_amdgcn_readlane(job, leader);
        const int low = wave_min_dpp(same ? g : 0x7fffffff);
        if (lane == leader) send(job, low);
        todo &= ~__ballot(same);
    }
}

// Gap positions that are neither granted nor out of candidates.  Every round that
// does not end the process grants at least one of them, so this bounds the rounds
// that can still follow; the host sizes its next batch of launches with it.
// out: how many, then the counters of n rounds, lost and cand.
__global__ __launch_bounds__(1024) void k_count_open(int lb_cap, const int32_t *__restrict__ plan, const int4 *__restrict__ state,
                                                     const int32_t *__restrict__ lost, const int32_t *__restrict__ cand, int n_rounds, int32_t *out)
{
    for (int i = threadIdx.x; i < n_rounds; i += 1024) {
        out[1 + i] = lost[i];
        out[1 + n_rounds + i] = cand[i];
    }
    __shared__ int s_sum[1024 / kWave];
    const int n = min(plan[kPlanListBlocks], lb_cap) * kWave;
    int c = 0;
    for (int i = threadIdx.x; i < n; i += 1024) c += (state[i].w & 3) == 0;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) c += __shfl_xor(c, d, kWave);
    if ((threadIdx.x & (kWave - 1)) == 0) s_sum[threadIdx.x / kWave] = c;
    __syncthreads();
    if (threadIdx.x == 0) {
        int t = 0;
        for (int i = 0; i < 1024 / kWave; ++i) t += s_sum[i];
        out[0] = t;
    }
}

// After the last round: the grants themselves.  A granted position still holds
// its winning job in its state; which of the job's atoms it got is what the fit
// says for that pair, min(#{D <= W}, #{P <= C}) - 1.
__global__ void k_grant_finish(int lb_cap, PolicyDev pol, const int32_t *__restrict__ plan,
                               const int4 *__restrict__ state, const int32_t *__restrict__ lb_begin,
                               const int32_t *__restrict__ gap_w, const int32_t *__restrict__ gap_c,
                               const int64_t *__restrict__ seg_off, const int32_t *__restrict__ n_atoms,
                               const int2 *__restrict__ atom_dp, const int2 *__restrict__ atom_db,
                               const long long *__restrict__ atom_area,
                               const int32_t *__restrict__ wait, const uint8_t *__restrict__ sla_class,
                               int32_t *grant_job, int32_t *grant_cut, int64_t *grant_score,
                               int32_t *job_gap, int rounds, int stable, int32_t *rounds_and_stable)
{
    const int slot = blockIdx.x * blockDim.x + threadIdx.x;
    if (slot == 0) { rounds_and_stable[0] = rounds; rounds_and_stable[1] = stable; }
    if (slot >= min(plan[kPlanListBlocks], lb_cap) * kWave) return;
    const int4 st = state[slot];
    if ((st.w & 3) != 1) return;
    const int g = st.w >> 2, j = st.y;
    const int pos = lb_begin[slot / kWave] + (slot & (kWave - 1));
    const int w = gap_w[pos], c = gap_c[pos];
    const int64_t base = seg_off[j];
    int atom = 0, hi = n_atoms[j];              // atoms that fit (a prefix: durations and peaks ascend)
    while (atom < hi) {
        const int mid = (atom + hi) >> 1;
        const int2 v = atom_dp[base + mid];
        if (v.x <= w && v.y <= c) atom = mid + 1; else hi = mid;
    }
    --atom;                                     // the job was a candidate of this gap: at least one fits
    const int2 v = atom_dp[base + atom];
    unsigned long long mult, tier;
    job_policy(pol, wait, sla_class, j, mult, tier);
    grant_job[g] = j;
    grant_cut[g] = atom_db[base + atom].y;
    const unsigned long long F = atom_area ? (unsigned long long)atom_area[base + atom]
                                           : (unsigned long long)v.x * (unsigned long long)v.y;
    grant_score[g] = int64_t(F * mult);
    job_gap[j] = g;
}

}  // namespace sja
