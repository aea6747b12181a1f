// The best job per gap by atoms, without the (gap, job) replies and without stepping along the gaps.
//
// Along the windows of one capacity a job's key never falls (the host sees to it where the hysteresis rule could
// undo that), so the best key at a window w and a capacity c is the largest one of all atoms of duration <= w and
// peak <= c: every atom is an event at the first position whose window reaches its duration, and the answer a running
// maximum over the positions.  Nearly all atoms lie far below it, so it is made twice:
//   * k_floor_first, k_floor_merge: roughly.  An atom counts for the smallest capacity class that admits it and for
//     the first bucket boundary at or behind its duration; the running maximum over both, classes and buckets, is what
//     any window of a bucket has at least (of stand-ins for the keys: 32 bits each, a few thousand buckets in LDS);
//   * k_floor_filter: the atoms whose key reaches that, some ten thousand of 8 million at 32768 gaps x 65536 jobs (an
//     atom below it in the smallest class that admits it is below it in every larger one).  They raise the key at
//     their position of every class that admits them;
//   * k_floor_ties: who has that key, under MIXED with the largest F; k_floor_reduce: the running maximum.
// What is left is reading all atoms once and those of every fourth job twice, bound by some fifty instructions for an
// atom (filter, 32768 gaps x 65536 jobs of 130 atoms: 56 us; with keys of 64 bits throughout, 83), and 40 us of short
// kernels.  At that size fit -> select takes 171 us where k_range_select takes 398, at 8192 x 32768 a select 66 us where
// reading the matrix takes 320.  sja.hip says where the line lies (by_floor).
#pragma once

#include "k_fused.h"

namespace sja {

constexpr int kFloorThreads = 1024, kFloorLanes = 16, kFloorGroups = kFloorThreads / kFloorLanes;      // sixteen lanes take a job
constexpr int kFloorBlocks = 512;           // blocks that share the jobs, at most: two per compute unit,
constexpr int kFloorLeastJobs = 64;         // with a job per group at least
constexpr int kFloorFirstBlocks = 256;      // of k_floor_first,
constexpr int kFloorStep = 4;               // which looks at every second or fourth job only where there are many: any jobs
                                            // give a floor, a quarter of them leaves three times as many atoms (12 of 4 thousand)
constexpr int kFloorBuckets = 8192;         // of all classes together
constexpr int kFloorAhead = 4;              // atoms a lane asks for together
constexpr int kFloorThinFrom = 1024;        // atoms that a block keeps from which on it looks for equal ones among them
constexpr int kFloorMergeThreads = 256, kFloorMergeEntries = 32;

inline int floor_blocks_of(int n_jobs, int most)
{
    const int b = (n_jobs + kFloorLeastJobs - 1) / kFloorLeastJobs;
    return b < most ? b : most;
}
inline int floor_step_of(int n_jobs)
{
    int step = 1;
    while (step < kFloorStep && n_jobs > step * kFloorFirstBlocks * kFloorLeastJobs) step *= 2;
    return step;
}

// Buckets of durations: exact below 2^(bits + 1), then 2^bits to an octave.
__device__ __forceinline__ int bucket_of(int d, int bits)
{
    const int e = max(31 - __clz(d) - bits, 0);
    return (e << bits) + (d >> e);
}
__device__ __forceinline__ int bucket_behind(int d, int bits)          // the first that begins at or behind it
{
    const int e = max(31 - __clz(d) - bits, 0);
    return (e << bits) + (d >> e) + int((d & ((1 << e) - 1)) != 0);
}
__device__ __forceinline__ int bucket_begin(int b, int bits)
{
    const int e = max((b >> bits) - 1, 0);
    return (b - (e << bits)) << e;
}
struct FloorBuckets {
    int bits, per_class;        // per_class: 0 if there is no room for any
    int base, low;

    __device__ __forceinline__ int of(int d) const { return bucket_of(max(d, low), bits) - base; }
    __device__ __forceinline__ int behind(int d) const { return d <= low ? 0 : bucket_behind(d, bits) - base; }     // the first that begins at or behind it
    __device__ __forceinline__ int begin(int k) const { return k == 0 ? low : bucket_begin(k + base, bits); }
};
// The buckets of a batch: from its smallest window on, which stands for all durations below, up to its longest one; as fine
// as there is room for.
__device__ __forceinline__ FloorBuckets floor_buckets(int n_classes, int low, int longest, int room)
{
    low = max(low, 1);
    longest = max(longest, low);
    for (int bits = 12; bits >= 0; --bits) {
        const int base = bucket_of(low, bits), n = bucket_of(longest, bits) - base + 2;
        if (int64_t(n) * n_classes <= room) return {bits, n, base, low};
    }
    return {0, 0, 0, 1};
}

// What the kernels share: the tables of the plan, and where the intermediate results are.
struct FloorArgs {
    PolicyDev pol;
    int n_jobs, n_gaps, room;                   // room: buckets that there is space for
    int most_classes;                           // of the batches that are served
    const int64_t *seg_off;
    const int2 *atom_dp;
    const long long *atom_area;                 // F of an atom, null: duration x peak
    const int32_t *n_atoms;
    const int32_t *plan, *class_begin, *gap_w, *gap_c;
    const int32_t *wait;
    const uint8_t *sla_class;
    const int32_t *job_held;
    uint32_t *floors;                           // [kFloorFirstBlocks][room]: a block's maxima
    uint32_t *floor;                            // [room]: of all blocks
    uint32_t *running;                          // [room]: the running maximum of these
    int32_t *bucket_pos;                        // [room]: per class and bucket the first position whose window reaches it
    ulonglong2 *near;                           // atoms that are left: key, (duration, peak); a block's begin at its first job's segment
    ulonglong2 *near_job;                       // their F, job
    int32_t *n_near;                            // [kFloorBlocks], and whether a position has several jobs of its largest key
    unsigned long long *best, *second;          // per sorted position: the largest key that begins there, under MIXED its F,
    int32_t *who;                               // and its job
    int32_t *reach;                             // [n_jobs] atoms that some class can reach, may be null
};

constexpr int kPeakBits = 3, kPeakBuckets = 256, kPeakLast = ((31 - kPeakBits) << kPeakBits) + (1 << kPeakBits) - 1;
static_assert(kPeakLast < kPeakBuckets, "the bucket of 2^31 - 1");
struct FloorClasses {
    int cap[kMaxClasses + 1], longest[kMaxClasses + 1];     // capacity; the largest window of this class and those of larger capacities
    int begin[kMaxClasses + 1];                             // the first position
    int low;                                                // the smallest window
    uint8_t below[kPeakBuckets];                            // classes whose capacity is below a bucket of peaks
};

__device__ __forceinline__ FloorBuckets floor_classes(const FloorArgs &A, FloorClasses &S)
{
    const int tid = threadIdx.x, n_classes = A.plan[kPlanClasses];
    if (tid < kWave) {
        const int begin = A.class_begin[tid], end = A.class_begin[tid + 1];         // (asked for together with the plan)
        const bool there = tid < n_classes;
        int w = there ? A.gap_w[end - 1] : INT32_MIN, low = there ? A.gap_w[begin] : INT32_MAX;
        S.cap[tid] = there ? A.gap_c[begin] : INT32_MAX;
        S.begin[tid] = begin;
        if (tid == kWave - 1) S.begin[kMaxClasses] = end;
#pragma unroll
        for (int d = 1; d < kWave; d <<= 1) {
            const int o = __shfl_down(w, d, kWave);
            if (tid + d < kWave) w = max(w, o);
            low = min(low, __shfl_xor(low, d, kWave));
        }
        S.longest[tid] = w;
        if (tid == 0) { S.cap[kMaxClasses] = INT32_MAX; S.longest[kMaxClasses] = INT32_MIN; S.low = low; }
    }
    __syncthreads();
    if (tid < kPeakBuckets) {            // (blocks have as many threads)
        int c = 0;
        const int peak = tid <= kPeakLast ? bucket_begin(tid, kPeakBits) : INT32_MAX;
        while (c < n_classes && S.cap[c] < peak) ++c;
        S.below[tid] = uint8_t(c);
    }
    __syncthreads();
    return floor_buckets(n_classes, __builtin_amdgcn_readfirstlane(S.low), __builtin_amdgcn_readfirstlane(S.longest[0]), A.room);
}

// A stand-in for a key that grows with it, but for kDigestSlack: tier, and the score rounded to 24 bits (five roundings
// of at most half a unit in the last of them, on either side of a comparison).
constexpr uint32_t kDigestSlack = 16;
__device__ __forceinline__ uint32_t floor_digest(uint32_t tier, float score)
{
    constexpr uint32_t least = 0x3f000000u;         // 0.5: scores are whole numbers below 2^62
    return (tier << 30) + max(__float_as_uint(score), least) - least;
}

// The atoms of every step-th of the block's jobs.  The next ones are on their way while a trip's are looked at, those of
// the next job behind a job's last ones; the first ones from begin() on.
template <bool AREA>
struct FloorAtoms {
    static constexpr int Q = kFloorAhead, TRIP = Q * kFloorLanes;
    struct Job {
        int64_t base;
        int n, tier;            // tier: -1 if it is held
        uint32_t mult;
    };
    struct Trip {
        int2 v[Q];
        long long f[AREA ? Q : 1];
    };
    int j, j1, stride;
    Job x, next;
    Trip now;

    __device__ __forceinline__ Job ask(const FloorArgs &A, int job) const
    {
        Job y{0, 0, 0, 0};
        if (job >= j1) return y;
        unsigned long long mult, tier;
        y.base = A.seg_off[job];
        y.n = A.n_atoms[job];
        job_policy(A.pol, A.wait, A.sla_class, job, mult, tier);
        y.mult = uint32_t(mult);
        y.tier = A.job_held && A.job_held[job] >= 0 ? -1 : int(tier);
        return y;
    }
    __device__ __forceinline__ void load(const FloorArgs &A, const Job &y, int a0, Trip &t) const
    {
        const int sub = threadIdx.x & (kFloorLanes - 1), last = y.n - 1 - a0 - sub;
        const int64_t at = y.base + a0 + sub;
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            if (q * kFloorLanes <= last) {
                t.v[q] = A.atom_dp[at + q * kFloorLanes];
                if (AREA) t.f[AREA ? q : 0] = A.atom_area[at + q * kFloorLanes];
            }
        }
    }
    __device__ __forceinline__ void begin(const FloorArgs &A, int step)
    {
        const int each = (A.n_jobs + int(gridDim.x) - 1) / int(gridDim.x);
        stride = kFloorGroups * step;
        j = int(blockIdx.x) * each + int(threadIdx.x) / kFloorLanes * step;
        j1 = min((int(blockIdx.x) + 1) * each, A.n_jobs);
        x = ask(A, j);
        next = ask(A, j + stride);
        load(A, x, 0, now);
    }
    // Calls on(job, atom, F with AREA, class, digest) for every atom that some gap's window
    // and capacity reach (held jobs are left out), and done(job, how many of them this lane met) for every job.
    struct Atom {
        int2 v;                 // duration, peak
        int64_t at;
        int tier;
        uint32_t mult;
        bool first;             // of its job
    };
    template <typename On, typename Done>
    __device__ __forceinline__ void walk(const FloorArgs &A, const FloorClasses &S, On on, Done done)
    {
        const int sub = threadIdx.x & (kFloorLanes - 1), first_lane = threadIdx.x & (kWave - 1) & ~(kFloorLanes - 1);
        int a0 = 0, reached = 0;
        Trip behind;
        while (j < j1) {
            const bool more = a0 + TRIP < x.n;
            load(A, more ? x : next, more ? a0 + TRIP : 0, behind);
            int c[Q];                               // the smallest class that admits it
#pragma unroll
            for (int q = 0; q < Q; ++q) c[q] = S.below[bucket_of(now.v[q].y, kPeakBits) & (kPeakBuckets - 1)];
            for (bool below = true; below;) {
                below = false;
#pragma unroll
                for (int q = 0; q < Q; ++q)
                    if (S.cap[c[q]] < now.v[q].y) { ++c[q]; below = true; }
            }
            bool any = false;
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                if (a0 + sub + q * kFloorLanes >= x.n || now.v[q].x > S.longest[c[q]]) continue;
                ++reached;
                any = true;
                if (x.tier < 0) continue;
                const unsigned long long area = AREA ? (unsigned long long)now.f[AREA ? q : 0] : 0ull;
                const float F = AREA ? float(area) : float(now.v[q].x) * float(now.v[q].y);
                const int a = a0 + sub + q * kFloorLanes;
                on(j, Atom{now.v[q], x.base + a, x.tier, x.mult, a == 0}, area, c[q], floor_digest(uint32_t(x.tier), F * float(x.mult)));
            }
            // (behind atoms that nothing reaches there are no others)
            const unsigned long long met = __ballot(any);
            const uint32_t half = first_lane & 32 ? uint32_t(met >> 32) : uint32_t(met);
            if (more && (half >> (first_lane & 31) & ((1u << kFloorLanes) - 1u)) != 0) {
                a0 += TRIP;
                now = behind;
                continue;
            }
            done(j, reached);
            j += stride;
            x = next;
            next = ask(A, j + stride);
            a0 = reached = 0;
            if (more) load(A, x, 0, now); else now = behind;
        }
    }
};

template <bool AREA>
__global__ __launch_bounds__(kFloorThreads) __attribute__((amdgpu_waves_per_eu(AREA ? 4 : 8, 8))) void k_floor_first(FloorArgs A, int step)
{
    __shared__ uint32_t s_table[kFloorBuckets];
    __shared__ FloorClasses S;
    if (!serves(A.plan, A.most_classes)) return;
    FloorAtoms<AREA> atoms;
    atoms.begin(A, step);
    const FloorBuckets B = floor_classes(A, S);
    const int entries = B.per_class * A.plan[kPlanClasses];
    for (int i = threadIdx.x; i < entries; i += kFloorThreads) s_table[i] = 0;
    // (what the later kernels start from)
    for (int p = blockIdx.x * kFloorThreads + threadIdx.x; p < A.n_gaps; p += gridDim.x * kFloorThreads) {
        A.best[p] = 0;
        A.second[p] = 0;
        A.who[p] = INT32_MAX;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) A.n_near[kFloorBlocks] = 0;
    __syncthreads();
    if (B.per_class > 0)
        atoms.walk(A, S,
                   [&](int, const typename FloorAtoms<AREA>::Atom &x, unsigned long long, int c, uint32_t digest) {
                       uint32_t &at = s_table[c * B.per_class + B.behind(x.v.x)];
                       if (digest > *static_cast<volatile uint32_t *>(&at)) atomicMax(&at, digest);
                   },
                   [](int, int) {});
    __syncthreads();
    for (int i = threadIdx.x; i < entries; i += kFloorThreads) A.floors[int64_t(blockIdx.x) * A.room + i] = s_table[i];
}

// The maximum over the blocks, and the positions of the buckets.
__global__ __launch_bounds__(kFloorMergeThreads) void k_floor_merge(FloorArgs A, int n_blocks)
{
    constexpr int GROUPS = kFloorMergeThreads / kFloorMergeEntries;
    __shared__ uint32_t s_top[GROUPS][kFloorMergeEntries];
    __shared__ FloorClasses S;
    static_assert(kFloorMergeThreads >= kPeakBuckets && kFloorThreads >= kPeakBuckets, "a thread per bucket of peaks");
    if (!serves(A.plan, A.most_classes)) return;
    const FloorBuckets B = floor_classes(A, S);
    const int at = threadIdx.x % kFloorMergeEntries, group = threadIdx.x / kFloorMergeEntries, i = blockIdx.x * kFloorMergeEntries + at;
    const bool there = i < B.per_class * A.plan[kPlanClasses];
    uint32_t top = 0;
    if (there) {
#pragma unroll 8
        for (int b = group; b < n_blocks; b += GROUPS) top = max(top, A.floors[int64_t(b) * A.room + i]);
    }
    s_top[group][at] = top;
    __syncthreads();
    if (!there) return;
    if (group == 1) {
        const int c = i / B.per_class, k = i - c * B.per_class, w = B.begin(k);
        int lo = A.class_begin[c], hi = A.class_begin[c + 1];
        if (k == B.per_class - 1) lo = hi;          // (begins behind every window, be it beyond 31 bits)
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (A.gap_w[mid] < w) lo = mid + 1; else hi = mid;
        }
        A.bucket_pos[i] = lo;
    }
    if (group > 0) return;
#pragma unroll
    for (int g = 1; g < GROUPS; ++g) top = max(top, s_top[g][at]);
    A.floor[i] = top;
}

// Calls on(position, key, place, largest key there so far) for the first position that each of n atoms from `first` on reaches
// in every class that admits it, unless it is below the running maximum there already; as that does not fall along the
// classes, an atom is done with at the first one where it is.  Several atoms side by side: each is a chain of trips to memory.
// Where many atoms are near the best that is what counts, and how fine the buckets are (fit -> select of 32768 gaps of 64
// capacities x 65536 jobs of 128 segments, EFFICIENCY: 1190 us with a lane for each of 64 classes and buckets from duration
// 1 on, 746 so; of one profile 489 and 318).
constexpr int kEventsLanes = 16;
template <int Q, typename On>
__device__ __forceinline__ void floor_events(const FloorArgs &A, const FloorClasses &S, const FloorBuckets &B, const uint32_t *running, int64_t first,
                                             int n, int threads, On on)
{
    const int n_classes = A.plan[kPlanClasses];
    int lanes = 1;                              // to an atom: one to a class,
    while (lanes < n_classes && lanes < kEventsLanes) lanes <<= 1;      // of many classes they take the next ones after these
    const int c0 = threadIdx.x & (lanes - 1), step = threads / lanes;
    for (int i = threadIdx.x / lanes; i < n; i += Q * step) {
        ulonglong2 x[Q];
        int k[Q];
        uint32_t digest[Q];
        unsigned live = 0;
#pragma unroll
        for (int q = 0; q < Q; ++q) x[q] = A.near[first + min(i + q * step, n - 1)];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const unsigned long long score = (x[q].x - 1ull) & ((1ull << 62) - 1ull);
            digest[q] = floor_digest(uint32_t((x[q].x - 1ull) >> 62), float(score)) + kDigestSlack;
            k[q] = B.of(int(x[q].y >> 32));
            live |= unsigned(i + q * step < n && (B.per_class == 0 || k[q] < B.per_class - 1)) << q;        // (not longer than every window)
        }
#pragma unroll 1
        for (int c = c0; c < n_classes && live; c += lanes) {
            const int cap = S.cap[c], begin = S.begin[c], end = S.begin[c + 1];
            int lo[Q], hi[Q];
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                lo[q] = hi[q] = end;
                if (!(live >> q & 1u) || int(uint32_t(x[q].y)) > cap) continue;
                if (B.per_class == 0) {
                    lo[q] = begin;
                } else if (digest[q] < running[c * B.per_class + k[q]]) {
                    live &= ~(1u << q);
                } else {
                    lo[q] = A.bucket_pos[c * B.per_class + k[q]];
                    hi[q] = A.bucket_pos[c * B.per_class + k[q] + 1];
                }
            }
            for (bool more = true; more;) {
                int w[Q];
                more = false;
#pragma unroll
                for (int q = 0; q < Q; ++q)
                    if (lo[q] < hi[q]) w[q] = A.gap_w[(lo[q] + hi[q]) >> 1];
#pragma unroll
                for (int q = 0; q < Q; ++q) {
                    if (lo[q] >= hi[q]) continue;
                    const int mid = (lo[q] + hi[q]) >> 1;
                    if (w[q] < int(x[q].y >> 32)) lo[q] = mid + 1; else hi[q] = mid;
                    more |= lo[q] < hi[q];
                }
            }
            unsigned long long best[Q];
#pragma unroll
            for (int q = 0; q < Q; ++q)
                if (lo[q] < end) best[q] = __hip_atomic_load(&A.best[lo[q]], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
            for (int q = 0; q < Q; ++q)
                if (lo[q] < end) on(lo[q], x[q].x, first + i + q * step, best[q]);
        }
    }
}

// Jobs of one profile and equal preferences have nothing but equal keys, and every atom that leads is there once for each of
// them.  Of a block's atoms of one duration and peak only the one that a position can want is kept: the largest key, of equal
// ones the largest F, of these the lowest job.  In place; returns how many are left.
template <bool AREA>
struct FloorSlots {
    static constexpr int N = AREA ? 1024 : 2048, TRIES = 4;         // (with the table of floors, half of a compute unit's LDS)
    unsigned long long at[N], key[N], second[AREA ? N : 1];         // duration and peak, 0: free
    int job[N];
    int n;

    __device__ __forceinline__ static int slot_of(unsigned long long x, int k)
    {
        return int(((uint32_t(x) * 2654435761u ^ uint32_t(x >> 32)) * 2246822519u >> 16) + k) & (N - 1);
    }
    __device__ __forceinline__ int find(unsigned long long x) const         // -1: all of its slots are others'
    {
        for (int k = 0; k < TRIES; ++k)
            if (at[slot_of(x, k)] == x) return slot_of(x, k);
        return -1;
    }
};
template <bool AREA>
__device__ __forceinline__ int floor_thin(const FloorArgs &A, FloorSlots<AREA> &T, int64_t first, int n)
{
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const bool by_second = AREA && A.pol.policy == SJA_POLICY_MIXED;        // (else F follows from the key, or does not matter)
    for (int i = tid; i < FloorSlots<AREA>::N; i += kFloorThreads) {
        T.at[i] = T.key[i] = 0;
        if (AREA) T.second[AREA ? i : 0] = 0;
        T.job[i] = INT32_MAX;
    }
    if (tid == 0) T.n = 0;
    __syncthreads();
#pragma unroll 1
    for (int i = tid; i < n; i += kFloorThreads) {
        const ulonglong2 x = A.near[first + i];
        for (int k = 0; k < FloorSlots<AREA>::TRIES; ++k) {
            const int to = T.slot_of(x.y, k);
            unsigned long long was = *static_cast<volatile unsigned long long *>(&T.at[to]);
            if (was == 0) was = atomicCAS(&T.at[to], 0ull, x.y);
            if (was != 0 && was != x.y) continue;
            if (x.x > *static_cast<volatile unsigned long long *>(&T.key[to])) atomicMax(&T.key[to], x.x);
            break;
        }
    }
    __syncthreads();
    if (by_second) {
    #pragma unroll 1
    for (int i = tid; i < n; i += kFloorThreads) {
            const ulonglong2 x = A.near[first + i];
            const int to = T.find(x.y);
            if (to >= 0 && x.x == T.key[to]) atomicMax(&T.second[AREA ? to : 0], A.near_job[first + i].x);
        }
        __syncthreads();
    }
    auto leads = [&](int to, const ulonglong2 &x, const ulonglong2 &y) { return x.x == T.key[to] && (!by_second || y.x == T.second[AREA ? to : 0]); };
#pragma unroll 1
    for (int i = tid; i < n; i += kFloorThreads) {
        const ulonglong2 x = A.near[first + i], y = A.near_job[first + i];
        const int to = T.find(x.y), job = int(y.y);
        if (to >= 0 && leads(to, x, y) && job < *static_cast<volatile int *>(&T.job[to])) atomicMin(&T.job[to], job);
    }
    __syncthreads();
    for (int i0 = 0; i0 < n; i0 += kFloorThreads) {
        const int i = i0 + tid;
        ulonglong2 x{}, y{};
        bool stays = false;
        if (i < n) {
            x = A.near[first + i];
            y = A.near_job[first + i];
            const int to = T.find(x.y);
            stays = to < 0 || (leads(to, x, y) && int(y.y) == T.job[to]);
        }
        __syncthreads();            // (these have been read: what is left takes no more places than there were)
        const unsigned long long some = __ballot(stays);
        if (!some) continue;
        int to = 0;
        if (lane == 0) to = atomicAdd(&T.n, __popcll(some));
        to = __builtin_amdgcn_readfirstlane(to) + __popcll(some & ((1ull << lane) - 1ull));
        if (stays) {
            A.near[first + to] = x;
            A.near_job[first + to] = y;
        }
    }
    __syncthreads();
    return T.n;
}

template <bool AREA>
__global__ __launch_bounds__(kFloorThreads) __attribute__((amdgpu_waves_per_eu(AREA ? 4 : 8, 8))) void k_floor_filter(FloorArgs A)
{
    __shared__ uint32_t s_table[kFloorBuckets];
    __shared__ FloorClasses S;
    __shared__ FloorSlots<AREA> s_slots;
    __shared__ int s_n;
    if (!serves(A.plan, A.most_classes)) return;
    FloorAtoms<AREA> atoms;
    atoms.begin(A, 1);
    const FloorBuckets B = floor_classes(A, S);
    const int n_classes = A.plan[kPlanClasses], entries = B.per_class * n_classes;
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    for (int i = tid; i < entries; i += kFloorThreads) s_table[i] = A.floor[i];
    if (tid == 0) s_n = 0;
    __syncthreads();
    // the running maximum: over the classes, then over the buckets, a class a wave
    for (int i = tid; i < B.per_class; i += kFloorThreads) {
        uint32_t top = 0;
        for (int c = 0; c < n_classes; ++c) s_table[c * B.per_class + i] = top = max(top, s_table[c * B.per_class + i]);
    }
    __syncthreads();
    for (int c = tid / kWave; c < n_classes; c += kFloorThreads / kWave) {
        uint32_t before = 0;
        for (int b0 = 0; b0 < B.per_class; b0 += kWave) {
            const int b = c * B.per_class + min(b0 + lane, B.per_class - 1);
            const uint32_t top = max(wave_scan_max_u32(s_table[b]), before);
            if (b0 + lane < B.per_class) s_table[b] = top;
            before = uint32_t(__builtin_amdgcn_readlane(int(top), kWave - 1));
        }
    }
    __syncthreads();
    if (blockIdx.x == 0)
        for (int i = tid; i < entries; i += kFloorThreads) A.running[i] = s_table[i];
    const int each = (A.n_jobs + int(gridDim.x) - 1) / int(gridDim.x), j0 = int(blockIdx.x) * each;
    const int64_t first = j0 < A.n_jobs ? A.seg_off[j0] : 0;
    atoms.walk(A, S,
               [&](int j, const typename FloorAtoms<AREA>::Atom &x, unsigned long long area, int c, uint32_t digest) {
                   if (B.per_class && digest + kDigestSlack < s_table[c * B.per_class + B.of(x.v.x)]) return;
                   const unsigned long long F = AREA ? area : rect_of(x.v.x, x.v.y), score = times_mult(F, x.mult);
                   if (!x.first) {              // a key that the atom before it had already says nothing new
                       const int2 u = A.atom_dp[x.at - 1];
                       if (times_mult(AREA ? (unsigned long long)A.atom_area[x.at - 1] : rect_of(u.x, u.y), x.mult) == score) return;
                   }
                   const int64_t to = first + atomicAdd(&s_n, 1);
                   A.near[to] = make_ulonglong2((((unsigned long long)x.tier << 62) | score) + 1ull, (unsigned long long)uint32_t(x.v.x) << 32 | uint32_t(x.v.y));
                   A.near_job[to] = make_ulonglong2(F, (unsigned long long)j);
               },
               [&](int j, int reached) {
                   if (!A.reach) return;
#pragma unroll
                   for (int d = 1; d < kFloorLanes; d <<= 1) reached += __shfl_xor(reached, d, kFloorLanes);
                   if ((tid & (kFloorLanes - 1)) == 0) A.reach[j] = reached;
               });
    __syncthreads();
    int n = s_n;
    if (n > kFloorThinFrom) n = floor_thin<AREA>(A, s_slots, first, n);
    if (tid == 0) A.n_near[blockIdx.x] = n;
    floor_events<4>(A, S, B, s_table, first, n, kFloorThreads, [&](int p, unsigned long long key, int64_t, unsigned long long best) {
        if (key > best) atomicMax(&A.best[p], key);
    });
}

// Who has the largest key of a position: the lowest job, under MIXED of those with the largest F.  Where a position has
// several jobs of its largest key that takes a second pass (again); the jobs of the first one are marked, so that any of
// the second one's is lower.
constexpr int kTiesThreads = 1024;           // an atom and class each in one go (with 256 the first pass took 33 us, 18 so)
constexpr int kTiesMark = 1 << 30;
static_assert(SJA_MAX_JOBS <= kTiesMark, "job ids below the mark");
template <bool MIXED>
__global__ __launch_bounds__(kTiesThreads) void k_floor_ties(FloorArgs A, int again)
{
    __shared__ FloorClasses S;
    if (!serves(A.plan, A.most_classes)) return;
    int32_t *several = A.n_near + kFloorBlocks;
    if (again && !*several) return;
    const int n = A.n_near[blockIdx.x];
    if (n == 0) return;
    const int each = (A.n_jobs + int(gridDim.x) - 1) / int(gridDim.x), j0 = int(blockIdx.x) * each;
    const int64_t first = j0 < A.n_jobs ? A.seg_off[j0] : 0;
    const FloorBuckets B = floor_classes(A, S);
    // (atomics on one word are served one after the other: most need none)
    auto now = [](auto &x) { return __hip_atomic_load(&x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
    floor_events<2>(A, S, B, A.running, first, n, kTiesThreads, [&](int p, unsigned long long key, int64_t place, unsigned long long best) {
        if (key != best) return;
        const ulonglong2 y = A.near_job[place];
        const int job = int(y.y);
        if (again) {
            if (y.x == A.second[p] && job < now(A.who[p])) atomicMin(&A.who[p], job);
            return;
        }
        if (MIXED) {
            if (y.x > now(A.second[p])) atomicMax(&A.second[p], y.x);
            // (of a job only the first atom of a key is here: two jobs)
            if ((now(A.who[p]) != INT32_MAX || atomicExch(&A.who[p], job | kTiesMark) != INT32_MAX) && !now(*several)) atomicMax(several, 1);
        } else if (job < now(A.who[p])) {
            atomicMin(&A.who[p], job);
        }
    });
}

// The running maximum over the positions of a class, by blocks of `tile` positions that first look at those before them;
// and the winner's atom.  Where another form has served the batch the best over its job tiles: the winner's
// atom count becomes its boundary (from_matrix: the partial has the boundary itself).
constexpr int kFloorTile = 256;
inline int floor_tile(int n_gaps) { return kFloorTile * ((n_gaps + 65535) / 65536); }

template <bool MIXED>
__global__ __launch_bounds__(256) void k_floor_reduce(FloorArgs A, int tile, int step_tiles, int from_matrix, const SelPartial *__restrict__ part,
                                                      const int32_t *__restrict__ gap_cls, const int32_t *__restrict__ gap_order,
                                                      const uint8_t *__restrict__ gap_active, const int2 *__restrict__ atom_db,
                                                      int32_t *__restrict__ cand_job, int32_t *__restrict__ cand_cut, int64_t *__restrict__ cand_score)
{
    if (!serves(A.plan, A.most_classes)) {
        int g, bj, ba;
        unsigned long long bh;
        if (!reduce_tiles(A.n_gaps, step_tiles, part, g, bh, bj, ba)) return;
        cand_job[g] = bh ? bj : -1;
        cand_cut[g] = !bh ? -1 : from_matrix ? ba : atom_db[A.seg_off[bj] + ba - 1].y;
        cand_score[g] = bh ? int64_t((bh - 1ull) & ((1ull << 62) - 1ull)) : 0;
        return;
    }
    constexpr int WAVES = kFloorTile / kWave;
    __shared__ unsigned long long s_hi[WAVES + 1], s_lo[WAVES + 1];
    __shared__ int s_job[WAVES + 1], s_cls[WAVES + 1];          // of each wave's last position; behind them what came before the block
    const int p0 = blockIdx.x * tile, p1 = min(p0 + tile, A.n_gaps);
    if (p0 >= A.n_gaps) return;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    struct Best {
        unsigned long long hi, lo;
        int job;
    };
    auto merge = [&](Best &b, unsigned long long oh, unsigned long long ol, int oj) {
        if (fused_better(oh, ol, oj, b.hi, b.lo, b.job)) b = {oh, ol, oj};
    };
    const int first_class = gap_cls[p0];
    Best b{0, 0, INT32_MAX};
    for (int p = A.class_begin[first_class] + tid; p < p0; p += kFloorTile) merge(b, A.best[p], MIXED ? A.second[p] : 0ull, A.who[p]);
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1)
        merge(b, (unsigned long long)__shfl_xor((long long)b.hi, d, kWave), MIXED ? (unsigned long long)__shfl_xor((long long)b.lo, d, kWave) : 0ull,
              __shfl_xor(b.job, d, kWave));
    if (lane == 0) { s_hi[wave] = b.hi; s_lo[wave] = b.lo; s_job[wave] = b.job; }
    __syncthreads();
    if (tid == 0) {
        for (int w = 1; w < WAVES; ++w) merge(b, s_hi[w], s_lo[w], s_job[w]);
        s_hi[WAVES] = b.hi; s_lo[WAVES] = b.lo; s_job[WAVES] = b.job; s_cls[WAVES] = first_class;
    }
    for (int q0 = p0; q0 < p1; q0 += kFloorTile) {
        const int p = min(q0 + tid, p1 - 1), cls = gap_cls[p];
        b = {A.best[p], MIXED ? A.second[p] : 0ull, A.who[p]};
#pragma unroll
        for (int d = 1; d < kWave; d <<= 1) {
            const unsigned long long oh = (unsigned long long)__shfl_up((long long)b.hi, d, kWave);
            const unsigned long long ol = MIXED ? (unsigned long long)__shfl_up((long long)b.lo, d, kWave) : 0ull;
            const int oj = __shfl_up(b.job, d, kWave), oc = __shfl_up(cls, d, kWave);
            if (lane >= d && oc == cls) merge(b, oh, ol, oj);
        }
        __syncthreads();
        if (lane == kWave - 1) { s_hi[wave] = b.hi; s_lo[wave] = b.lo; s_job[wave] = b.job; s_cls[wave] = cls; }
        __syncthreads();
        for (int w = 0; w < wave; ++w)
            if (s_cls[w] == cls) merge(b, s_hi[w], s_lo[w], s_job[w]);
        if (s_cls[WAVES] == cls) merge(b, s_hi[WAVES], s_lo[WAVES], s_job[WAVES]);
        __syncthreads();
        if (tid == kFloorTile - 1) { s_hi[WAVES] = b.hi; s_lo[WAVES] = b.lo; s_job[WAVES] = b.job; s_cls[WAVES] = cls; }
        if (q0 + tid >= p1) continue;
        const int g = gap_order[p];
        int cut = -1;
        if (gap_active && !gap_active[g]) b.hi = 0;
        b.job &= kTiesMark - 1;
        if (b.hi) {
            const int w = A.gap_w[p], c = A.gap_c[p];
            const int64_t base = A.seg_off[b.job];
            const int2 *dp = A.atom_dp + base;
            int lo = 0, hi = A.n_atoms[b.job];
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                const int2 v = dp[mid];
                if (v.x <= w && v.y <= c) lo = mid + 1; else hi = mid;
            }
            cut = atom_db[base + lo - 1].y;
        }
        cand_job[g] = b.hi ? b.job : -1;
        cand_cut[g] = cut;
        cand_score[g] = b.hi ? int64_t((b.hi - 1ull) & ((1ull << 62) - 1ull)) : 0;
    }
}

}  // namespace sja
