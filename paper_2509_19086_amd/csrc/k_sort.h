// Device-wide building blocks used by the grant path: an exclusive scan and a
// stable least-significant-digit radix pass (8-bit digits), each of three
// kernels, or of one or two where the items are few; sizes here are tens of
// millions of items at most.
#pragma once

#include <type_traits>

#include "sja_internal.h"

namespace sja {

// --------------------------------------------------------------------------
// Exclusive scan of int32, in place, any length: per-block scan of 2048
// items, one block scans the block sums, a third kernel adds them back.
// --------------------------------------------------------------------------
constexpr int kScanTile = 2048;

__global__ __launch_bounds__(256) void k_scan_tiles(int32_t *data, int64_t n, int32_t *tile_sums)
{
    __shared__ int s_part[256];
    const int64_t base = int64_t(blockIdx.x) * kScanTile + threadIdx.x * 8;
    int v[8];
    int sum = 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        v[i] = (base + i < n) ? data[base + i] : 0;
        sum += v[i];
    }
    s_part[threadIdx.x] = sum;
    __syncthreads();
    for (int d = 1; d < 256; d <<= 1) {
        const int add = threadIdx.x >= d ? s_part[threadIdx.x - d] : 0;
        __syncthreads();
        s_part[threadIdx.x] += add;
        __syncthreads();
    }
    int run = s_part[threadIdx.x] - sum;           // exclusive prefix of this thread
    if (threadIdx.x == 255) tile_sums[blockIdx.x] = s_part[255];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        if (base + i < n) data[base + i] = run;
        run += v[i];
    }
}

__global__ __launch_bounds__(1024) void k_scan_sums(int32_t *sums, int n_tiles, int32_t *total)
{
    __shared__ int s_part[1024];
    __shared__ int s_carry;
    if (threadIdx.x == 0) s_carry = 0;
    __syncthreads();
    for (int b0 = 0; b0 < n_tiles; b0 += 1024) {
        const int i = b0 + threadIdx.x;
        const int mine = i < n_tiles ? sums[i] : 0;
        s_part[threadIdx.x] = mine;
        __syncthreads();
        for (int d = 1; d < 1024; d <<= 1) {
            const int add = threadIdx.x >= d ? s_part[threadIdx.x - d] : 0;
            __syncthreads();
            s_part[threadIdx.x] += add;
            __syncthreads();
        }
        const int carry = s_carry;
        if (i < n_tiles) sums[i] = carry + s_part[threadIdx.x] - mine;
        __syncthreads();
        if (threadIdx.x == 1023) s_carry = carry + s_part[1023];
        __syncthreads();
    }
    if (threadIdx.x == 0 && total) *total = s_carry;
}

__global__ __launch_bounds__(256) void k_scan_add(int32_t *data, int64_t n, const int32_t *tile_sums)
{
    const int add = tile_sums[blockIdx.x];
    const int64_t base = int64_t(blockIdx.x) * kScanTile + threadIdx.x * 8;
#pragma unroll
    for (int i = 0; i < 8; ++i)
        if (base + i < n) data[base + i] += add;
}

// The same by one thread block, for scans whose three launches cost more than the work: a wave takes up to
// kScanOneRows rows of 64 items a turn, all of them asked for together (32 consecutive items a thread, every
// load of it 64 lines for a wave: 19 us for 32768 items, so 8; a tick with three of them 1443 -> 1404).
constexpr int kScanOneRows = 32, kScanOneMost = 2 * 1024 * kScanOneRows;

__global__ __launch_bounds__(1024) void k_scan_one(int32_t *data, int n, int32_t *total)
{
    __shared__ int s_sum[1024 / kWave];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    int carry = 0;
    for (int b0 = 0; b0 < n; b0 += 1024 * kScanOneRows) {
        const int rows = min(kScanOneRows, (n - b0 + 1023) / 1024);
        const int base = b0 + wave * rows * kWave + lane;
        int v[kScanOneRows];
#pragma unroll
        for (int i = 0; i < kScanOneRows; ++i) v[i] = i < rows && base + i * kWave < n ? data[base + i * kWave] : 0;
        int sum = 0;
#pragma unroll
        for (int i = 0; i < kScanOneRows; ++i) {
            if (i >= rows) continue;
            const int upto = wave_scan_add(v[i]);
            v[i] = sum + upto - v[i];
            sum += __builtin_amdgcn_readlane(upto, kWave - 1);
        }
        if (lane == 0) s_sum[wave] = sum;
        __syncthreads();
        int run = carry;
        for (int w = 0; w < 1024 / kWave; ++w) {
            if (w < wave) run += s_sum[w];
            carry += s_sum[w];
        }
#pragma unroll
        for (int i = 0; i < kScanOneRows; ++i)
            if (i < rows && base + i * kWave < n) data[base + i * kWave] = run + v[i];
        __syncthreads();
    }
    if (threadIdx.x == 0 && total) *total = carry;
}

// Enqueues an in-place exclusive scan; tile_sums needs ceil(n/2048) ints.
// total (device, may be null) receives the sum of all items.
inline hipError_t enqueue_scan(hipStream_t st, int32_t *data, int64_t n, int32_t *tile_sums, int32_t *total)
{
    if (n <= 0) return hipSuccess;
    if (n <= kScanOneMost) {
        hipLaunchKernelGGL(k_scan_one, dim3(1), dim3(1024), 0, st, data, int(n), total);
        return hipGetLastError();
    }
    const int n_tiles = int((n + kScanTile - 1) / kScanTile);
    hipLaunchKernelGGL(k_scan_tiles, dim3(n_tiles), dim3(256), 0, st, data, n, tile_sums);
    hipLaunchKernelGGL(k_scan_sums, dim3(1), dim3(1024), 0, st, tile_sums, n_tiles, total);
    hipLaunchKernelGGL(k_scan_add, dim3(n_tiles), dim3(256), 0, st, data, n, tile_sums);
    return hipGetLastError();
}

// --------------------------------------------------------------------------
// Stable radix pass over bare 64-bit keys (the grant-list entries), tiles of
// kKeyTile items.  A tile is ranked per wave (each wave owns a contiguous
// part, walked in order so the pass stays stable), put in digit order in
// LDS and written out from there, so that items of one digit leave as one
// contiguous run.  hist is digit-major ([256][n_tiles]) so that one exclusive
// scan over it yields every (digit, tile) output offset; up to kKeyFewTiles tiles
// (FEW) it is tile-major, with the sums of every kKeyGroup tiles beside it, and every
// tile of the scatter adds its column up itself, which saves the scan's
// launches.  n lives in device memory (it is produced by earlier kernels).
//
// A pass of some hundred thousand items is a chain of waits (a tile's columns, its
// keys, a ballot chain and two trips to LDS for every 64 of a wave's items), so
// a tile has sixteen waves, of four times 64 items each, and four threads a column:
// 124 tiles 17 us a scatter with four waves and a thread that reads all rows of hist,
// 9.8 so, the counts 6.8 and 4.0; 387 tiles with payloads 16 and three launches less.
// --------------------------------------------------------------------------
constexpr int kKeyTile = 4096;
constexpr int kKeyThreads = 1024, kKeyWaves = kKeyThreads / kWave;
constexpr int kKeyPerWave = kKeyTile / kKeyWaves;
constexpr int kKeyChunks = kKeyPerWave / kWave;

// Lanes of the wave (among `valid`) holding the same 8-bit digit as this lane.
__device__ __forceinline__ unsigned long long digit_peers(unsigned d, bool valid)
{
    unsigned long long peers = __ballot(valid);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
        const unsigned long long m = __ballot((d >> b) & 1u);
        peers &= ((d >> b) & 1u) ? m : ~m;
    }
    return peers;
}

constexpr int kKeyGroup = 16;
constexpr int kKeyFewTiles = 1024;       // (the scan takes three launches, 12 us and more; a column's sums of so many tiles 20 rows a thread)
constexpr int kKeyGroupSums = kKeyFewTiles / kKeyGroup * 256;

template <bool FEW>
__global__ __launch_bounds__(kKeyThreads) void k_keys_hist(const unsigned long long *__restrict__ keys,
                                                           const int32_t *n_ptr, int shift, unsigned digit_mask, int32_t *hist,
                                                           int n_tiles, int32_t *group_sums)
{
    __shared__ int s_h[256];
    const int64_t n = *n_ptr;
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    if (tid < 256) s_h[tid] = 0;
    __syncthreads();
    const int64_t base = int64_t(blockIdx.x) * kKeyTile;
#pragma unroll
    for (int r = 0; r < kKeyTile / kKeyThreads; ++r) {
        const int64_t i = base + r * kKeyThreads + tid;
        const bool valid = i < n;
        const unsigned d = valid ? unsigned(keys[i] >> shift) & digit_mask : 0u;
        // counting needs no order: a wave whose keys all carry one digit (the block digits, and
        // any digit of keys that the earlier passes have brought together) adds its count once,
        // any other wave lets every lane add its own one (finding each lane's peers first, as
        // the scatter has to, made this kernel bound by the instructions of that search)
        const unsigned long long live = __ballot(valid);
        if (live == 0) continue;
        const unsigned d0 = unsigned(__builtin_amdgcn_readlane(int(d), __ffsll((long long)live) - 1));
        if (__ballot(valid && d != d0) == 0) {
            if (lane == 0) atomicAdd(&s_h[d0], __popcll(live));
        } else if (valid) {
            atomicAdd(&s_h[d], 1);
        }
    }
    __syncthreads();
    if (tid >= 256) return;
    const int h = s_h[tid];
    hist[FEW ? int64_t(blockIdx.x) * 256 + tid : int64_t(tid) * n_tiles + blockIdx.x] = h;
    if (FEW && h) atomicAdd(&group_sums[int(blockIdx.x) / kKeyGroup * 256 + tid], h);
}

// A list record: a job and the lane range [lo, hi) of its list block that one of the job's atoms
// serves.  Four bytes while job ids fit 19 bits (the rounds are bound by the records they sweep:
// 16-byte records with the atom's rank in them cost the early rounds four times the bytes), eight
// beyond.  Which atom it is need not be kept: job and gap determine it.
constexpr int kRec32JobBits = 19;
struct Rec32 {
    uint32_t v;
    __device__ static Rec32 make(uint32_t job, uint32_t lo, uint32_t hi) { return {job | (lo << kRec32JobBits) | (hi << (kRec32JobBits + 6))}; }
    __device__ uint32_t job() const { return v & ((1u << kRec32JobBits) - 1u); }
    __device__ int lo() const { return int((v >> kRec32JobBits) & 63u); }
    __device__ int hi() const { return int(v >> (kRec32JobBits + 6)); }
    __device__ Rec32 of_lane(int t) const { return {uint32_t(__builtin_amdgcn_readlane(int(v), t))}; }
};
struct Rec64 {
    uint32_t j, z;
    __device__ static Rec64 make(uint32_t job, uint32_t lo, uint32_t hi) { return {job, lo | (hi << 8)}; }
    __device__ uint32_t job() const { return j; }
    __device__ int lo() const { return int(z & 255u); }
    __device__ int hi() const { return int(z >> 8); }
    __device__ Rec64 of_lane(int t) const
    {
        return {uint32_t(__builtin_amdgcn_readlane(int(j), t)), uint32_t(__builtin_amdgcn_readlane(int(z), t))};
    }
};
struct NoRec {};
struct Rec32Placed {};          // Rec32, and the entries' places beside them

// What the last pass over list entries writes instead of the keys themselves: the record of an entry
// job : hi (7 bits) : lo (6 bits), whatever bits (the list block) lie above the job's 24.
template <typename REC>
__device__ __forceinline__ REC key_record(unsigned long long v)
{
    return REC::make(uint32_t(v >> 13) & 0xffffffu, unsigned(v) & 63u, unsigned(v >> 6) & 127u);
}

// PAY: every key carries a 32-bit payload that moves with it.  REC other than NoRec: the sorted keys
// are not written at all, their records are (the pass that finishes the order of the list entries).
template <bool FEW, bool PAY, typename REC = NoRec>
__global__ __launch_bounds__(kKeyThreads) void k_keys_scatter(const unsigned long long *__restrict__ src,
                                                              unsigned long long *__restrict__ dst,
                                                              const uint32_t *__restrict__ pay_src,
                                                              uint32_t *__restrict__ pay_dst, const int32_t *n_ptr,
                                                              int shift, unsigned digit_mask, const int32_t *__restrict__ hist,
                                                              int n_tiles, const int32_t *__restrict__ group_sums, int32_t *next_sums,
                                                              void *rec, uint16_t *rec_from)
{
    __shared__ unsigned long long s_key[kKeyTile];
    __shared__ uint32_t s_pay[PAY ? kKeyTile : 1];
    __shared__ int s_cnt[kKeyWaves][256];       // per wave and digit: running count, later the offset inside the digit
    __shared__ int s_start[256];        // first tile-local slot of a digit
    __shared__ int s_goff[256];         // where the tile's items of a digit go
    __shared__ int s_wsum[4];
    const int64_t n = *n_ptr;
    const int64_t base = int64_t(blockIdx.x) * kKeyTile;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
    if (FEW)        // the sums of the next pass start at zero
        for (int i = int(blockIdx.x) * kKeyThreads + tid; i < kKeyGroupSums; i += int(gridDim.x) * kKeyThreads) next_sums[i] = 0;
    if (base >= n) return;
    unsigned long long key[kKeyChunks];
    uint32_t pay[PAY ? kKeyChunks : 1];
    int pos[kKeyChunks];
    const int64_t wbase = base + wave * kKeyPerWave + lane;
#pragma unroll
    for (int c = 0; c < kKeyChunks; ++c) {
        key[c] = wbase + c * kWave < n ? src[wbase + c * kWave] : ~0ull;
        if (PAY) pay[c] = wbase + c * kWave < n ? pay_src[wbase + c * kWave] : 0u;
    }
#pragma unroll
    for (int i = 0; i < kKeyWaves * 256; i += kKeyThreads) s_cnt[0][i + tid] = 0;
    if (FEW) {
        // digit d: its items in all tiles and in those before this one, a share of them by each of four threads
        constexpr int kShares = kKeyThreads / 256;
        int (*const s_part)[256] = reinterpret_cast<int (*)[256]>(s_key);
        const int d = tid & 255, share = tid >> 8, own = int(blockIdx.x) / kKeyGroup, groups = (n_tiles + kKeyGroup - 1) / kKeyGroup;
        int all = 0, before = 0;
#pragma unroll 8
        for (int g = share; g < groups; g += kShares) {
            const int h = group_sums[g * 256 + d];
            all += h;
            before += g < own ? h : 0;
        }
#pragma unroll
        for (int k = 0; k < kKeyGroup; k += kShares) {
            const int t = own * kKeyGroup + k + share;
            if (t < int(blockIdx.x)) before += hist[t * 256 + d];
        }
        s_part[share][d] = all;
        s_part[kShares + share][d] = before;
        __syncthreads();
        if (tid < 256) {
            all = before = 0;
#pragma unroll
            for (int k = 0; k < kShares; ++k) { all += s_part[k][d]; before += s_part[kShares + k][d]; }
            const int upto = wave_scan_add(all);
            if (lane == kWave - 1) s_wsum[wave] = upto;
            s_goff[d] = upto - all + before;
        }
        __syncthreads();
        if (tid < 256)
            for (int w = 0; w < wave; ++w) s_goff[d] += s_wsum[w];
    } else if (tid < 256) {
        s_goff[tid] = hist[int64_t(tid) * n_tiles + blockIdx.x];
    }
    __syncthreads();

    volatile int *cnt = &s_cnt[wave][0];
#pragma unroll
    for (int c = 0; c < kKeyChunks; ++c) {
        const bool valid = wbase + c * kWave < n;
        const unsigned d = unsigned(key[c] >> shift) & digit_mask;
        const unsigned long long peers = digit_peers(d, valid);
        const int before = __popcll(peers & ((1ull << lane) - 1ull));
        const int prev = cnt[d];
        pos[c] = prev + before;
        __builtin_amdgcn_wave_barrier();
        if (valid && before == 0) cnt[d] = prev + __popcll(peers);
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();

    // digit tid: offsets of the waves inside the digit, then the digits' starts
    int total = 0, upto = 0;
    if (tid < 256) {
        int h[kKeyWaves];
#pragma unroll
        for (int w = 0; w < kKeyWaves; ++w) h[w] = s_cnt[w][tid];
#pragma unroll
        for (int w = 0; w < kKeyWaves; ++w) { s_cnt[w][tid] = total; total += h[w]; }
        upto = wave_scan_add(total);
        if (lane == kWave - 1) s_wsum[wave] = upto;
    }
    __syncthreads();
    if (tid < 256) {
        int off = upto - total;
        for (int w = 0; w < wave; ++w) off += s_wsum[w];
        s_start[tid] = off;
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < kKeyChunks; ++c) {
        if (wbase + c * kWave < n) {
            const unsigned d = unsigned(key[c] >> shift) & digit_mask;
            const int slot = s_start[d] + s_cnt[wave][d] + pos[c];
            s_key[slot] = key[c];
            if (PAY) s_pay[slot] = pay[c];
        }
    }
    __syncthreads();
    const int count = int(n - base < kKeyTile ? n - base : kKeyTile);
    for (int k = tid; k < count; k += kKeyThreads) {
        const unsigned long long v = s_key[k];
        const unsigned d = unsigned(v >> shift) & digit_mask;
        const int64_t o = int64_t(s_goff[d]) + (k - s_start[d]);
        if constexpr (std::is_same<REC, Rec32Placed>::value) {
            static_cast<Rec32 *>(rec)[o] = Rec32::make(uint32_t(v >> 13) & 0x1ffffu, unsigned(v) & 63u, unsigned(v >> 6) & 127u);
            rec_from[o] = uint16_t(v >> 30);
        } else if constexpr (!std::is_same<REC, NoRec>::value) {
            static_cast<REC *>(rec)[o] = key_record<REC>(v);
        } else {
            dst[o] = v;
        }
        if (PAY) pay_dst[o] = s_pay[k];
    }
}

// The whole sort of up to kKeyTile keys with their payloads by one thread block: by the bytes of `mask_lo`
// of the secondary keys (if any), then by those of `mask_hi` of the primary ones, lowest byte first.  A few
// thousand keys are a few microseconds a pass here, and a launch or three a pass as a chain of kernels.
constexpr int kSortOneThreads = 1024;

__global__ __launch_bounds__(kSortOneThreads) void k_sort_one(int n, const unsigned long long *__restrict__ key_lo, unsigned mask_lo,
                                                              const unsigned long long *__restrict__ key_hi, unsigned mask_hi,
                                                              uint32_t *__restrict__ perm)
{
    constexpr int WAVES = kSortOneThreads / kWave, PER = kKeyTile / kSortOneThreads;
    __shared__ unsigned long long s_key[kKeyTile];
    __shared__ uint32_t s_pay[kKeyTile];
    __shared__ int s_cnt[WAVES][256];
    __shared__ int s_start[256], s_wsum[4];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const int first = wave * PER * kWave + lane;
    unsigned long long key[PER];
    uint32_t pay[PER];
#pragma unroll
    for (int c = 0; c < PER; ++c) pay[c] = uint32_t(first + c * kWave);
    for (int half = 0; half < 2; ++half) {
        const unsigned mask = half ? mask_hi : mask_lo;
        const unsigned long long *src = half ? key_hi : key_lo;
        if (!mask) continue;
#pragma unroll
        for (int c = 0; c < PER; ++c) key[c] = first + c * kWave < n ? src[pay[c]] : ~0ull;
        for (int b = 0; b < 8; ++b) {
            if (!((mask >> b) & 1u)) continue;
            for (int i = tid; i < WAVES * 256; i += kSortOneThreads) s_cnt[0][i] = 0;
            __syncthreads();
            volatile int *cnt = &s_cnt[wave][0];
            int pos[PER];
#pragma unroll
            for (int c = 0; c < PER; ++c) {
                const bool valid = first + c * kWave < n;
                const unsigned d = unsigned(key[c] >> (8 * b)) & 255u;
                const unsigned long long peers = digit_peers(d, valid);
                const int before = __popcll(peers & ((1ull << lane) - 1ull));
                const int prev = cnt[d];
                pos[c] = prev + before;
                __builtin_amdgcn_wave_barrier();
                if (valid && before == 0) cnt[d] = prev + __popcll(peers);
                __builtin_amdgcn_wave_barrier();
            }
            __syncthreads();
            int total = 0, upto = 0;
            if (tid < 256) {            // digit tid: the waves' offsets inside the digit, then the digits' starts
                for (int w = 0; w < WAVES; ++w) {
                    const int h = s_cnt[w][tid];
                    s_cnt[w][tid] = total;
                    total += h;
                }
                upto = wave_scan_add(total);
                if (lane == kWave - 1) s_wsum[wave] = upto;
            }
            __syncthreads();
            if (tid < 256) {
                int off = upto - total;
                for (int w = 0; w < wave; ++w) off += s_wsum[w];
                s_start[tid] = off;
            }
            __syncthreads();
#pragma unroll
            for (int c = 0; c < PER; ++c) {
                if (first + c * kWave < n) {
                    const unsigned d = unsigned(key[c] >> (8 * b)) & 255u;
                    const int slot = s_start[d] + s_cnt[wave][d] + pos[c];
                    s_key[slot] = key[c];
                    s_pay[slot] = pay[c];
                }
            }
            __syncthreads();
#pragma unroll
            for (int c = 0; c < PER; ++c) {
                if (first + c * kWave < n) { key[c] = s_key[first + c * kWave]; pay[c] = s_pay[first + c * kWave]; }
            }
        }
    }
#pragma unroll
    for (int c = 0; c < PER; ++c)
        if (first + c * kWave < n) perm[first + c * kWave] = pay[c];
}

// Two keys per item, sorted by the first only: puts the items whose first keys are equal in the order of their
// second keys (stable).  Equal first keys are rare accidents (two jobs' products) where there is a second key at
// all, so this replaces five or six passes over it; a run of more than kTieRun that is out of order sets *flag,
// and the caller sorts by both keys after all.
constexpr int kTieRun = 32;

__global__ __launch_bounds__(256) void k_fix_ties(const int32_t *n_ptr, const unsigned long long *__restrict__ keys,
                                                  const unsigned long long *__restrict__ second, uint32_t *perm, int32_t *flag)
{
    const int64_t n = *n_ptr, i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const unsigned long long key = keys[i];
    const bool tied = i > 0 && keys[i - 1] == key;
    if (tied) {
        // beyond the part of a long run that its first item's thread looks at (such a run is never reordered here)
        if (i > kTieRun && keys[i - kTieRun - 1] == key && second[perm[i - 1]] > second[perm[i]]) *flag = 1;
        return;
    }
    if (i + 1 >= n || keys[i + 1] != key) return;
    int64_t e = i + 1;
    while (e < n && e - i <= kTieRun && keys[e] == key) ++e;
    bool ordered = true;
    for (int64_t k = i + 1; k < e; ++k) ordered = ordered && second[perm[k - 1]] <= second[perm[k]];
    if (ordered) return;
    if (e - i > kTieRun) { *flag = 1; return; }
    for (int64_t k = i + 1; k < e; ++k) {
        const uint32_t a = perm[k];
        const unsigned long long v = second[a];
        int64_t at = k;
        for (; at > i && second[perm[at - 1]] > v; --at) perm[at] = perm[at - 1];
        perm[at] = a;
    }
}

// Items in the order of their digests (the upper bits of `items`, from `shift` on; their ids in the lower 32): puts
// those of equal digests in the order of their keys, then second keys (MIXED), then as they stand, and writes
// the ids.  The first one's thread serves a run, all of its keys asked for together if they are at most kRunNear;
// a run of more than kTieRun that is out of order sets *flag: kRunsByKey if keys are, kRunsBySecond if second keys of
// equal ones are.
constexpr int kRunNear = 8;
enum { kRunsByKey = 1, kRunsBySecond = 2 };

template <bool MIXED>
__global__ __launch_bounds__(256) void k_fix_runs(const int32_t *n_ptr, const unsigned long long *__restrict__ items, int shift,
                                                  const unsigned long long *__restrict__ keys, const unsigned long long *__restrict__ second,
                                                  uint32_t *perm, int32_t *flag)
{
    const int64_t n = *n_ptr, i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const unsigned long long digest = items[i] >> shift;
    const uint32_t id = uint32_t(items[i]);
    auto same = [&](int64_t k) { return items[k] >> shift == digest; };
    auto less = [&](unsigned long long ka, unsigned long long sa, unsigned long long kb, unsigned long long sb) { return ka < kb || (MIXED && ka == kb && sa < sb); };
    auto before = [&](uint32_t a, uint32_t b) { return less(keys[a], MIXED ? second[a] : 0ull, keys[b], MIXED ? second[b] : 0ull); };
    if (i > 0 && same(i - 1)) {
        if (i > kTieRun && same(i - kTieRun - 1)) {             // beyond the part that the first one's thread looks at
            perm[i] = id;
            const uint32_t a = uint32_t(items[i - 1]);
            if (before(id, a)) atomicOr(flag, keys[id] < keys[a] ? kRunsByKey : kRunsBySecond);
        }
        return;
    }
    if (i + 1 >= n || !same(i + 1)) { perm[i] = id; return; }
    uint32_t ids[kRunNear];
    int run = 1;
#pragma unroll
    for (int k = 0; k < kRunNear; ++k) {
        const unsigned long long v = items[i + k < n ? i + k : n - 1];
        ids[k] = uint32_t(v);
        if (run == k && i + k < n && v >> shift == digest) ++run;
    }
    if (run < kRunNear || i + run >= n || !same(i + run)) {
        unsigned long long key[kRunNear], sec[kRunNear];
#pragma unroll
        for (int k = 0; k < kRunNear; ++k) {
            key[k] = k < run ? keys[ids[k]] : ~0ull;
            sec[k] = MIXED && k < run ? second[ids[k]] : ~0ull;
        }
#pragma unroll
        for (int k = 0; k < kRunNear; ++k) {
            int rank = 0;
#pragma unroll
            for (int l = 0; l < kRunNear; ++l) {
                if (l < k) rank += l < run && !less(key[k], sec[k], key[l], sec[l]);
                if (l > k) rank += l < run && less(key[l], sec[l], key[k], sec[k]);
            }
            if (k < run) perm[i + rank] = ids[k];
        }
        return;
    }
    int64_t e = i;
    int found = 0;
    for (; e < n && e - i <= kTieRun && same(e); ++e) {
        const uint32_t a = uint32_t(items[e]), b = uint32_t(items[e > i ? e - 1 : e]);
        perm[e] = a;
        if (before(a, b)) found |= keys[a] < keys[b] ? kRunsByKey : kRunsBySecond;
    }
    if (!found) return;
    if (e - i > kTieRun) { atomicOr(flag, found); return; }
    for (int64_t k = i + 1; k < e; ++k) {
        const uint32_t a = perm[k];
        int64_t at = k;
        for (; at > i && before(a, perm[at - 1]); --at) perm[at] = perm[at - 1];
        perm[at] = a;
    }
}

// out[i] = keys[idx[i]]: the keys of a permutation, laid out in its order.
__global__ void k_gather_keys(const int32_t *n_ptr, const unsigned long long *__restrict__ keys,
                              const uint32_t *__restrict__ idx, unsigned long long *__restrict__ out)
{
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < *n_ptr) out[i] = keys[idx[i]];
}

}  // namespace sja
