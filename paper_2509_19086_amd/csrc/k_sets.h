// K4, the calm part of the conflict rounds: many rounds between two looks at the lists.
//
// After the first hundreds of rounds nearly all open gaps want the same few
// jobs: at Stress (32768 gaps x 65536 jobs) most of 9400 rounds name one to
// three jobs, each by thousands of gaps.  k_grant_solo pays 1.7 to 3 us for such
// a round, most of it for looking at every list block's list and for its
// barrier.  Here the rounds are played in batches:
//   * a wave per list block searches its list for the next free jobs of its
//     highest open lane; the lanes below that share at least the first of them
//     are a piece, the rest form further ones (sets_form);
//   * neighbouring pieces of a capacity class whose gaps want the same jobs for
//     some rounds to come are joined to a set, a range of the class's sorted
//     positions (sets_join), and a set's jobs and lowest gaps are brought to LDS
//     (sets_fill);
//   * one wave plays round after round on what lies there, a lane for one to
//     four sets: the first of the set's jobs that no round has named yet, a claim
//     for the set's lowest open gap, the outcome (sets_play).  A round is one
//     trip to LDS and 55 instructions and needs no barrier: 0.21 us.
// A batch ends when some set has used up its jobs or the lowest gaps it has at
// hand: up to 252 rounds of a few sets, some 20 to 60 where there are many.  Up
// to kSetsOneBlocks list blocks one launch does all of it (k_sets_one); beyond
// that the lists are searched by many thread blocks, which also list the pieces'
// jobs, and the rounds played by one, in turn (k_sets_form, k_sets_play).
//
// Between two batches lie 17 us at 66 list blocks and 4 sets (searching 7, jobs
// and gaps 7, joining 2, writing down 1) and 35 to 45 with 40 sets, as much as 80
// to 150 rounds: hence as many jobs at hand as a lane's registers and LDS allow.
// 2048 gaps x 8192 jobs, 542 rounds: 10 batches of 54 in 345 us when a set had 63
// jobs at hand and a round took 0.40 us, now three batches in 160.
//
// Working the rounds of a batch out together (all waves, pass after pass over the
// claims until they stay) was slower: neighbouring sets want nearly the same jobs,
// so that a pass puts right only one to two rounds more.
//
// What the sets rely on: along the positions of a class a job's key never falls
// (F grows with the cut; the host sees to it where the hysteresis rule could
// undo that).  Take the next free jobs of an open gap, and a gap of the class
// with a shorter window that gets the same atoms of these jobs: it meets them in
// the same order and no other free job between them, whatever other gaps are
// granted meanwhile.  (Another job would come earlier for the longer window,
// too, but for equal keys; then it is one of these jobs by another atom.)  Every
// record says from which position on its atom is the job's answer.
//
// It takes over from k_grant_solo once the rounds are calm (few list blocks whose
// lanes want different jobs), and hands back when batches get short.
#pragma once

#include "k_solo.h"

namespace sja {

constexpr int kSetsWaves = 16, kSetsThreads = kSetsWaves * kWave;
constexpr int kSetsMaxBlocks = 768;     // list blocks
static_assert(kSetsMaxBlocks <= kPlacedBlocks, "a place is a list block and a lane");
// and up to which one thread block does it all, and begins early (k_solo.h).  With the line at 40 and at 60, resolves of 41
// to 80 list blocks took 1.0 to 1.47 times as long, 1.2 on average (107 of random sizes, profiles, capacities), those
// of up to 40 the same.  With 104 and 128, those of 81 to 128 took 0.74 to 1.32 times as long, 0.88 on average (126 of
// them): the longer ones are those of many sets.
constexpr int kSetsOneBlocks = 80;
constexpr int kSetsPieces = 6;          // pieces of a list block, at most
constexpr int kSetsMost = 256;          // sets, at most
constexpr int kSetsMostJobs = 252;      // jobs at hand of a set, at most,
constexpr int kSetsMostRounds = kSetsMostJobs + 1;      // and rounds of a batch: each passes a job of every set
constexpr int kSetsSeq = kSetsMost * 70;        // 16-bit words for the jobs at hand of all sets; a set's last four are nobody's job
constexpr int kSetsHeads = 6144;        // lowest gaps at hand of all sets
constexpr int kSetsGapsAhead = 8;       // chunks of 64 gaps a wave looks at together,
constexpr int kSetsFewGaps = 8, kSetsGapsFar = 512;     // and how far for more than a few gaps
constexpr int kSetsListed = 2 * kWave;  // jobs that are listed for a piece, at most,
constexpr int kSetsLeastListed = 16;    // and at least
constexpr int kSetsChunk = 4 * kWave;   // records a wave reads at a time, four a lane
constexpr int kSetsMostSteps = 64;      // chunks a wave reads for one piece before it gives up
// jobs that the gaps of a set have in common, at least: at first, and at most (k_sets_one, and with more list blocks,
// where more in common makes more sets: 32768 gaps x 65536 jobs 43.0 / 42.0 / 41.4 / 42.3 / 43.0 ms for 16 / 24 / 32 / 48 / 64)
constexpr int kSetsLeastFirst = 16, kSetsLeast = 64, kSetsLeastMany = 32;
// batches of so few rounds are short ones (a batch takes as long as so many by k_grant_solo, or in turn as so many launched
// ones); more of those than others by so many end it
constexpr int kSetsShort = 8, kSetsShortMany = 5, kSetsPatience = 3;
constexpr int kSetsState = 3;           // out[]: k_grant_solo's words, and this one between launches: jobs << 16 | least << 8 | strain
enum { kSetsRunning = 4, kSetsLeft = 5 };       // out[kSoloDone]: between launches; on with k_grant_solo
enum { kSetsPause = 0, kSetsNoClaim = 1, kSetsAtCap = 2 };          // why the rounds of a batch stopped

// The jobs at hand: slots of a hash table, so that a set needs two bytes for a job and a claim has a word of its
// own, which also says whether the job is held.  A job is named in one round only: its word is the smallest of
// that round's claims, round of the batch (12 bits) : gap (20 bits), all ones before.  Behind the last
// slot there are two claims more: nobody's job, never free, and one that always is and stays so.
constexpr int kSetsSlots = 4096;
constexpr uint32_t kSetsNoJob = ~0u;
constexpr int kSetsTries = 16;
struct SetsJobs {
    uint32_t job[kSetsSlots];
    uint32_t claim[kSetsSlots + 2];
};
constexpr uint32_t kSetsNobody = 4 * kSetsSlots, kSetsIdle = kSetsNobody + 4;       // byte offsets of the last two claims
constexpr uint32_t kSetsServed = 1u << 20, kSetsMoreGaps = kSetsServed + 1;            // behind a set's lowest gaps: it has no others, or has some
__device__ __forceinline__ void sets_clear(SetsJobs &t, int i)
{
    if (i < kSetsSlots) t.job[i] = kSetsNoJob;
    t.claim[i] = i == kSetsSlots ? 0u : i == kSetsSlots + 1 ? ~1u : ~0u;
}
// The job's slot, -1 if there is none within reach: the set has fewer jobs at hand then.
__device__ __forceinline__ int sets_slot(SetsJobs &t, uint32_t job)
{
    uint32_t h = (job * 2654435761u) >> 20;
#pragma unroll 1
    for (int k = 0; k < kSetsTries; ++k) {
        uint32_t was = t.job[h];
        if (was == kSetsNoJob) was = atomicCAS(&t.job[h], kSetsNoJob, job);
        if (was == job || was == kSetsNoJob) return int(h);
        h = (h + 1) & (kSetsSlots - 1);
    }
    return -1;
}
static_assert(kSetsSlots == 1 << 12, "slots by the upper 12 bits of the product");

__device__ __forceinline__ unsigned long long sets_readlane64(unsigned long long v, int l)
{
    return (static_cast<unsigned long long>(uint32_t(__builtin_amdgcn_readlane(int(uint32_t(v >> 32)), l))) << 32) |
           uint32_t(__builtin_amdgcn_readlane(int(uint32_t(v)), l));
}

// A gap's place is its list block and lane: block << 6 | lane, ascending along the positions of a class.
// The gaps of every class by index, for the lowest ones of a set: by_class[class_begin[c] ...] = (place, gap).
// 16 waves take a stretch of the gaps each: they count per class, then write behind the waves before them.
__device__ __forceinline__ void sets_by_class(int n_gaps, int n_classes, const int32_t *__restrict__ class_begin, const int *s_first,
                                              const int32_t *place_of, int2 *by_class, int (*s_count)[kMaxClasses])
{
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x >> 6;
    const int each = ((n_gaps + kSetsWaves - 1) / kSetsWaves + kWave - 1) / kWave * kWave;
    const int begin = wave * each, end = min(begin + each, n_gaps);
    s_count[wave][lane] = 0;
    auto class_of = [&](int place) {
        const int u = place >> 6;
        int lo = 0, hi = n_classes - 1;         // the last class that begins at or before the list block
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (s_first[mid] <= u) lo = mid; else hi = mid - 1;
        }
        return lo;
    };
    for (int g0 = begin; g0 < end; g0 += kWave)
        if (g0 + lane < end) atomicAdd(&s_count[wave][class_of(place_of[g0 + lane])], 1);
    __syncthreads();
    int at = lane < n_classes ? class_begin[lane] : 0;
    for (int w = 0; w < wave; ++w) at += s_count[w][lane];
    __syncthreads();
    s_count[wave][lane] = at;
    for (int g0 = begin; g0 < end; g0 += kWave) {
        const bool valid = g0 + lane < end;
        const int place = valid ? place_of[g0 + lane] : 0, c = class_of(place);
        const unsigned long long peers = digit_peers(unsigned(c), valid);
        const int rank = __popcll(peers & ((1ull << lane) - 1ull));
        const int to = s_count[wave][c];
        asm volatile("" ::: "memory");          // (the wave's lanes read before one of them writes)
        if (valid) by_class[to + rank] = make_int2(place, g0 + lane);
        if (valid && rank == 0) s_count[wave][c] = to + __popcll(peers);
        asm volatile("" ::: "memory");
    }
}

// Per list block what the last search found: its open lanes, where the search for the highest one's jobs goes on,
// and the pieces.
struct SetsPiece {
    uint16_t top, bottom;           // places of its highest and lowest lane
    uint16_t from_most;             // the highest place from which on one of the first jobs' atoms is the answer
    uint16_t jobs;                  // none is left for these lanes; else how many are listed, with kSetsAll if those are all
    int at;                         // where the first free job of its highest lane is
};
constexpr uint16_t kSetsAll = 0x8000;
struct SetsBlock {
    unsigned long long open;
    int at, pieces;                 // pieces: -1 if the block has more of them, -2 if the next job lies further on
    SetsPiece piece[kSetsPieces];
};
static_assert(sizeof(SetsBlock) == 88, "layout");

struct SetsArgs {
    int4 *state;
    const int32_t *list_off;
    const Rec32 *rec;
    const uint16_t *rec_from;       // per record the place from which on its atom is the job's answer
    unsigned long long *claim;
    uint32_t *held;
    const int32_t *plan, *class_begin, *gap_cls, *lb_begin, *lb_end, *gap_order;
    int32_t *place_of;              // [gaps]
    int2 *by_class;                 // [gaps]
    SetsBlock *block;               // [list blocks]
    uint32_t *list;                 // [list blocks][kSetsPieces][list_jobs] jobs of the pieces, and behind all of them
    uint16_t *list_from;            // the places from which on they are the answer (not for k_sets_one)
    int list_jobs;
    // between launches: per class where its lowest open gap lies among its gaps; its first list block and first position
    int32_t *low, *classes;
    int32_t *out;
    int cap, n_gaps, n_lb, held_words;
    int build;                      // place_of and by_class are to be made
};

// The open lanes of list block u, and where the search for the highest one's jobs starts.
__device__ __forceinline__ void sets_open(const SetsArgs &A, int u, int lane)
{
    const int b0 = A.lb_begin[u], len = A.lb_end[u] - b0, slot = u * kWave + lane;
    if (A.build && lane < len) A.place_of[A.gap_order[b0 + lane]] = slot;
    const int4 st = A.state[slot];
    const unsigned long long on = __ballot((st.w & 3) == 0);
    const int at = __builtin_amdgcn_readlane(st.x, on ? 63 - __clzll((long long)on) : 0);
    if (lane == 0) {
        A.block[u].open = on;
        A.block[u].at = at;
    }
}

// A list's records from i0 on that cover lane `top` and whose job is free, kSetsChunk at a time.
struct SetsSearch {
    const uint4 *rec4;
    const ushort4 *from4;
    const uint32_t *held;
    int i0, end, top, base;
    uint4 r0, r1;
    ushort4 f0, f1;

    __device__ __forceinline__ void ask(int i, int lane, uint4 &r, ushort4 &f) const
    {
        const int k = min((i >> 2) + lane, (end - 1) >> 2);
        r = rec4[k];
        f = from4[k];
    }
    __device__ __forceinline__ void start(const SetsArgs &A, const uint32_t *is_held, int at, int list_end, int for_lane, int lane)
    {
        rec4 = reinterpret_cast<const uint4 *>(A.rec);
        from4 = reinterpret_cast<const ushort4 *>(A.rec_from);
        held = is_held;
        i0 = at;
        end = list_end;
        top = for_lane;
        base = at & ~3;
        if (i0 < end) {
            ask(base, lane, r0, f0);
            ask(base + kSetsChunk, lane, r1, f1);
        }
    }
    __device__ __forceinline__ bool over() const { return i0 >= end || base >= end; }
    // Which of the lane's four records (r0, f0) are such ones.
    __device__ __forceinline__ unsigned look(int lane) const
    {
        const uint32_t r[4] = {r0.x, r0.y, r0.z, r0.w};
        unsigned ok = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const Rec32 x{r[k]};
            const int i = base + 4 * lane + k;
            const bool covers = (i >= i0) & (i < end) & (uint32_t(top - x.lo()) < uint32_t(x.hi() - x.lo()));
            ok |= unsigned(covers && !held_bit(held, x.job())) << k;
        }
        return ok;
    }
    __device__ __forceinline__ void next(int lane)
    {
        r0 = r1;
        f0 = f1;
        base += kSetsChunk;
        ask(base + kSetsChunk, lane, r1, f1);
    }
};

// The pieces of list block u.  A lane's records lie behind a higher lane's, but for 63 of equal keys.
// LISTS: with the jobs of each, twice as many as its lanes are to have in common, or `jobs` if those are more.
template <bool LISTS>
__device__ __forceinline__ void sets_form(const SetsArgs &A, int u, int lane, int least, int jobs, const uint32_t *s_held)
{
    SetsBlock &B = A.block[u];
    unsigned long long rest = B.open;
    int at = B.at, end = A.list_off[u + 1], n_pieces = 0;
    asm volatile("" : "+v"(rest), "+v"(at), "+v"(end));        // one trip to memory for all of them
    rest = sets_readlane64(rest, 0);
    at = __builtin_amdgcn_readfirstlane(at);
    end = __builtin_amdgcn_readfirstlane(end);
    if (!rest) return;
    int first_at = at;
    for (bool first = true; rest; first = false) {
    again:
        const int top = 63 - __clzll((long long)rest);
        const int bottom = __ffsll((long long)rest) - 1;
        SetsSearch find;
        find.start(A, s_held, first ? at : max(at - 63, __builtin_amdgcn_readfirstlane(A.state[u * kWave + top].x)), end, top, lane);
        const int room = LISTS ? A.list_jobs : 0, want = LISTS ? min(max(2 * least, jobs), room) : least;
        const size_t list = LISTS && n_pieces < kSetsPieces ? size_t(u * kSetsPieces + n_pieces) * room : 0;
        int n = 0, hit = -1, steps = 0, most = 0;       // most: of the first `least` jobs
        if (!find.over()) {
            for (;;) {
                const unsigned ok = find.look(lane);
                const unsigned long long some = __ballot(ok != 0);
                if (some) {
                    const int mine = __popc(ok), upto = wave_scan_add(mine);
                    const uint32_t r[4] = {find.r0.x, find.r0.y, find.r0.z, find.r0.w};
                    const uint16_t f[4] = {find.f0.x, find.f0.y, find.f0.z, find.f0.w};
                    int rank = n + upto - mine;
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        if (!(ok >> k & 1u)) continue;
                        if (rank < least) most = max(most, int(f[k]));
                        if (LISTS && rank < room && n_pieces < kSetsPieces) {
                            A.list[list + rank] = Rec32{r[k]}.job();
                            A.list_from[list + rank] = f[k];
                        }
                        ++rank;
                    }
                    if (n == 0) {
                        const int t = __ffsll((long long)some) - 1;
                        hit = find.base + 4 * t + __ffs(__builtin_amdgcn_readlane(int(ok), t)) - 1;
                    }
                    n += __builtin_amdgcn_readlane(upto, kWave - 1);
                }
                if (n >= want || find.base + kSetsChunk >= end || ++steps > kSetsMostSteps) break;
                find.next(lane);
            }
        }
        if (n == 0 && find.i0 < end && find.base + kSetsChunk < end) {              // from there on the next time
            if (lane == 0) { if (first) B.at = find.base + kSetsChunk; else A.state[u * kWave + top].x = find.base + kSetsChunk; }
            n_pieces = -2;
            break;
        }
        if (n_pieces == kSetsPieces) {
            if (least == 1) { n_pieces = -1; break; }
            // too many: once more, with fewer jobs in common
            least /= 2;
            rest = B.open;
            at = first_at;
            n_pieces = 0;
            first = true;
            goto again;
        }
        SetsPiece &P = B.piece[n_pieces++];
        // the lanes that share the first jobs
        const int most_of_all = -wave_min_dpp(-most);
        const bool parted = n > 0 && most_of_all > u * kWave + bottom;
        const unsigned long long set = parted ? rest & (~0ull << (most_of_all & 63)) : rest;
        if (lane == 0) {
            P.top = uint16_t(u * kWave + top);
            P.bottom = uint16_t(u * kWave + __ffsll((long long)set) - 1);
            P.from_most = uint16_t(most_of_all);
            P.jobs = uint16_t(LISTS ? min(n, room) | (n <= room && find.base + kSetsChunk >= end ? kSetsAll : 0) : n);
            if (n == 0) P.jobs = 0;
            P.at = hit;
            if (n > 0) { if (first) B.at = hit; else A.state[u * kWave + top].x = hit; }
        }
        if (n == 0) break;          // no job is left for the highest lane, and so for none below it
        if (first) first_at = hit;
        at = hit;
        rest &= ~set;
    }
    if (lane == 0) B.pieces = n_pieces;
}

template <int BLOCKS>
struct SetsShared {
    SetsJobs jobs;                                      // the jobs at hand and their claims
    alignas(16) uint16_t seq[kSetsSeq];                 // per set its jobs' slots in there
    alignas(8) uint16_t idle[kSetsMostRounds + 11];     // nobody's jobs that are always free, for those that have left
    uint32_t head[kSetsHeads + kSetsMost];              // its lowest open gaps
    unsigned long long open[BLOCKS];            // open lanes of the list blocks
    uint16_t piece[BLOCKS * kSetsPieces], ends[BLOCKS * kSetsPieces], from_most[BLOCKS * kSetsPieces];  // the pieces: number, highest lane << 8 | lowest lane
    uint8_t none[BLOCKS * kSetsPieces];                 // no job is left for its lanes
    int8_t pieces[BLOCKS];
    uint16_t lo[kSetsMost], hi[kSetsMost], source[kSetsMost], cls[kSetsMost];    // first and last place of a set, the piece whose jobs it has, its class
    uint32_t set[kSetsMost];                            // jobs at hand, bit 16: no more jobs
    uint8_t dry[kSetsMost];                             // the round of the batch in which it found no job left, 0: none
    int most, through;                                  // jobs that a set has at hand at most; one that had so many has passed them all
    int first[kMaxClasses + 1], gaps_at[kMaxClasses + 1];       // first list block of a class, its first position,
    int low[kMaxClasses];                               // and where its lowest open gap lies among its gaps
    uint32_t found[kSetsWaves][kWave];
    int n, over, closed, lost, end, why;
};

template <int BLOCKS>
__device__ __forceinline__ unsigned long long sets_lanes(const SetsShared<BLOCKS> &S, int u, int from, int to)      // open lanes of list block u between two places
{
    unsigned long long m = u >= from >> 6 && u <= to >> 6 ? S.open[u] : 0ull;
    if (u == from >> 6) m &= ~0ull << (from & 63);
    if (u == to >> 6) m &= ~0ull >> (63 - (to & 63));
    return m;
}

// The sets of class c: from the highest piece down, each takes the gaps that get the same atoms of its first jobs.
template <int BLOCKS>
__device__ __forceinline__ void sets_join(const SetsArgs &A, SetsShared<BLOCKS> &S, int c, int lane)
{
    // its pieces, the highest first
    const int u_first = S.first[c], u_last = S.first[c + 1] - 1, base = u_first * kSetsPieces;
    int n = 0;
    for (int k0 = 0; k0 < (u_last - u_first + 1) * kSetsPieces; k0 += kWave) {
        const int u = max(u_last - (k0 + lane) / kSetsPieces, u_first), i = (k0 + lane) % kSetsPieces;
        const bool there = k0 + lane < (u_last - u_first + 1) * kSetsPieces && i < S.pieces[u];
        const unsigned long long b = __ballot(there);
        if (there) {
            const int to = base + n + __popcll(b & ((1ull << lane) - 1ull));
            const SetsPiece P = A.block[u].piece[i];
            S.ends[to] = uint16_t((P.top & 63) << 8 | (P.bottom & 63));
            S.from_most[to] = P.from_most;
            S.piece[to] = uint16_t(u * kSetsPieces + i);
        }
        n += __popcll(b);
    }
    asm volatile("" ::: "memory");
    auto top_of = [&](int k) { return S.piece[base + k] / kSetsPieces * kWave + (S.ends[base + k] >> 8); };
    auto bottom_of = [&](int k) { return S.piece[base + k] / kSetsPieces * kWave + (S.ends[base + k] & 63); };
    int top = n ? top_of(0) : 0;        // the highest gap not yet in a set
    for (int k = 0; k < n;) {
        const int piece = __builtin_amdgcn_readfirstlane(int(S.piece[base + k])), most = S.from_most[base + k];
        top = __builtin_amdgcn_readfirstlane(top);
        // the first one behind it that reaches below the place from which on the first jobs' atoms are the answer
        int k1 = k + 1, next_top = 0, next_bottom = 0, its_piece = 0;
        for (; k1 < n; k1 += kWave) {
            const int at = min(k1 + lane, n - 1), t = top_of(at), bt = bottom_of(at), its = S.piece[base + at];
            const unsigned long long b = __ballot(k1 + lane < n && bt < most);
            if (!b) continue;
            const int l = __ffsll((long long)b) - 1;
            k1 += l;
            next_top = __builtin_amdgcn_readlane(t, l);
            next_bottom = __builtin_amdgcn_readlane(bt, l);
            its_piece = __builtin_amdgcn_readlane(its, l);
            break;
        }
        int lo = u_first * kWave;
        if (S.none[piece]) {                    // no job is left for these lanes
            k1 = k + 1;
            next_top = k1 < n ? top_of(k1) : 0;
            if (lane == 0) {
                S.open[piece / kSetsPieces] &= ~sets_lanes(S, piece / kSetsPieces, bottom_of(k), top);
                S.closed = 1;
            }
            asm volatile("" ::: "memory");
        } else {
            if (k1 < n) {
                lo = most;
                if (next_top < most) {
                    lo = next_top + 1;
                } else {            // the part of it below goes on
                    const int v = its_piece / kSetsPieces;
                    next_top = v * kWave + 63 - __clzll((long long)sets_lanes(S, v, next_bottom, most - 1));
                }
            }
            if (lane == 0) {
                const int id = atomicAdd(&S.n, 1);
                if (id < kSetsMost) {
                    S.lo[id] = uint16_t(lo);
                    S.hi[id] = uint16_t(top);
                    S.source[id] = uint16_t(piece);
                    S.cls[id] = uint16_t(c);
                }
            }
        }
        k = k1;
        top = next_top;
    }
}

// How the space is shared out among the sets of a batch: per set `room` words for up to `most` jobs (twice an odd
// number: banks), and up to `heads` lowest gaps, of which the r-th of set i is at i + r * width.
struct SetsShape { int room, most, width, heads; };
constexpr SetsShape sets_shape(int n_sets)
{
    if (n_sets <= 16) return {262, kSetsMostJobs, 16, 253};
    if (n_sets <= 32) return {262, kSetsMostJobs, 32, 191};
    if (n_sets <= kWave) return {262, kSetsMostJobs, 64, 95};
    if (n_sets <= 2 * kWave) return {138, 126, 128, 47};
    return {70, 58, kSetsMost, 23};
}
// (every round passes a job of each set: a batch ends by its jobs before it ends by its bound, and a round fits a claim's word and a byte)
static_assert(sets_shape(1).most < kSetsMostRounds && sets_shape(17).most < kSetsMostRounds && sets_shape(33).most < kSetsMostRounds &&
              sets_shape(kWave + 1).most < kSetsMostRounds && sets_shape(kSetsMost).most < kSetsMostRounds && kSetsMostRounds + 1 < 1 << 8, "rounds of a batch");
static_assert(kWave * 262 <= kSetsSeq && 2 * kWave * 138 <= kSetsSeq && kSetsMost * 70 <= kSetsSeq, "jobs at hand");
// (behind the last gap a word that says whether there are more, and one that is read and not looked at)
static_assert((253 + 2) * 16 <= kSetsHeads + kSetsMost && (191 + 2) * 32 <= kSetsHeads + kSetsMost && (95 + 2) * 64 <= kSetsHeads + kSetsMost &&
              (47 + 2) * 128 <= kSetsHeads + kSetsMost && (23 + 2) * kSetsMost <= kSetsHeads + kSetsMost, "gaps at hand");

// The jobs (up to `most`) and the lowest gaps of a set.  LISTS: its piece's jobs are listed.
template <bool LISTS, int BLOCKS>
__device__ __forceinline__ void sets_fill(const SetsArgs &A, SetsShared<BLOCKS> &S, int id, int lane, int wave, const SetsShape &shape, int most, const uint32_t *held)
{
    const int lo = __builtin_amdgcn_readfirstlane(int(S.lo[id])), hi = __builtin_amdgcn_readfirstlane(int(S.hi[id]));
    const int piece = __builtin_amdgcn_readfirstlane(int(S.source[id])), c = __builtin_amdgcn_readfirstlane(int(S.cls[id]));
    const int u = piece / kSetsPieces, H = shape.heads;
    const SetsPiece P = A.block[u].piece[piece % kSetsPieces];
    const int begin = S.gaps_at[c], count = S.gaps_at[c + 1] - begin;
    const int low = S.low[c];
    int2 ahead[kSetsGapsAhead];
#pragma unroll
    for (int k = 0; k < kSetsGapsAhead; ++k) ahead[k] = A.by_class[begin + min(low + k * kWave + lane, count - 1)];
    SetsSearch find;
    constexpr int kLane = kSetsListed / kWave;
    uint32_t listed[kLane];
    int listed_from[kLane];
    const int room = A.list_jobs;
    if (LISTS) {
#pragma unroll
        for (int m = 0; m < kLane; ++m) {
            const size_t at = size_t(piece) * room + min(m * kWave + lane, room - 1);
            listed[m] = A.list[at];
            listed_from[m] = A.list_from[at];
        }
    } else {
        find.start(A, held, __builtin_amdgcn_readfirstlane(P.at), A.list_off[u + 1], __builtin_amdgcn_readfirstlane(int(P.top & 63)), lane);
    }
    // its lowest place, and how many are open (a few, or more than a wave)
    int bottom = hi, n_open = 0;
    for (int v0 = hi >> 6; v0 >= lo >> 6; v0 -= kWave) {
        const unsigned long long m = sets_lanes(S, v0 - lane, lo, hi), some = __ballot(m != 0);
        if (some) {
            const int t = 63 - __clzll((long long)some);
            bottom = (v0 - t) * kWave + __ffsll((long long)sets_readlane64(m, t)) - 1;
            n_open += __builtin_amdgcn_readlane(wave_scan_add(__popcll(m)), kWave - 1);
        }
    }
    // its jobs, up to the first one whose atom is not the answer of all its gaps
    int n = 0, limit = most;
    if (LISTS) {
        n = min(__builtin_amdgcn_readfirstlane(int(P.jobs & ~kSetsAll)), limit + 1);
#pragma unroll
        for (int m = 0; m < kLane; ++m) {
            const int k = m * kWave + lane;
            const unsigned long long beyond = __ballot(k < n && listed_from[m] > bottom);
            if (beyond) limit = min(limit, m * kWave + __ffsll((long long)beyond) - 1);
            const bool in = k < min(n, limit);
            const int slot = in ? sets_slot(S.jobs, listed[m]) : -1;
            if (slot >= 0) S.seq[id * shape.room + k] = uint16_t(4 * slot);
            const unsigned long long none = __ballot(in && slot < 0);
            if (none) limit = min(limit, m * kWave + __ffsll((long long)none) - 1);
        }
    }
    for (int steps = 0; !LISTS;) {
        const unsigned ok = find.look(lane);
        if (__ballot(ok != 0)) {
            constexpr int none = 0x7fffffff;
            const int mine = __popc(ok), upto = wave_scan_add(mine);
            const uint32_t r[4] = {find.r0.x, find.r0.y, find.r0.z, find.r0.w};
            const uint16_t f[4] = {find.f0.x, find.f0.y, find.f0.z, find.f0.w};
            int rank = n + upto - mine, cut = none;
#pragma unroll
            for (int k = 3; k >= 0; --k)
                if ((ok >> k & 1u) && int(f[k]) > bottom) cut = rank + __popc(ok & ((1u << k) - 1u));
            limit = min(limit, wave_min_dpp(cut));
            cut = none;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                if (!(ok >> k & 1u)) continue;
                if (rank < limit) {
                    const int slot = sets_slot(S.jobs, Rec32{r[k]}.job());
                    if (slot < 0) cut = min(cut, rank);
                    else S.seq[id * shape.room + rank] = uint16_t(4 * slot);
                }
                ++rank;
            }
            if (__ballot(cut != none)) limit = min(limit, wave_min_dpp(cut));
            n += __builtin_amdgcn_readlane(upto, kWave - 1);
        }
        if (n >= limit || find.base + kSetsChunk >= find.end || ++steps > kSetsMostSteps) break;
        find.next(lane);
    }
    const bool last = n <= limit && (LISTS ? (P.jobs & kSetsAll) != 0 : find.base + kSetsChunk >= find.end);        // nothing behind these
    const int jobs = min(n, limit);
    if (jobs == 0 && lane == 0) S.over = 1;
    asm volatile("" ::: "memory");
    if (lane < 4) S.seq[id * shape.room + jobs + lane] = uint16_t(4 * kSetsSlots);
    // its lowest gaps: few open ones are put in order, of many the class's are looked through
    int gaps = 0;
    bool all_gaps;
    if (n_open <= kWave) {
        uint32_t *list = S.found[wave];
        for (int v0 = lo >> 6; v0 <= hi >> 6; v0 += kWave) {
            const unsigned long long m = sets_lanes(S, v0 + lane, lo, hi);
            for (unsigned long long some = __ballot(m != 0); some; some &= some - 1) {
                const int t = __ffsll((long long)some) - 1;
                const unsigned long long mt = sets_readlane64(m, t);
                if ((mt >> lane) & 1ull) list[gaps + __popcll(mt & ((1ull << lane) - 1ull))] = uint32_t((v0 + t) << 6 | lane);
                gaps += __popcll(mt);
            }
        }
        asm volatile("" ::: "memory");
        const int place = int(list[min(lane, gaps - 1)]);
        const int g = A.state[place].w >> 2;
        int rank = 0;
        for (int l = 0; l < gaps; ++l) rank += __builtin_amdgcn_readlane(g, l) < g;
        if (lane < gaps && rank < H) S.head[id + rank * shape.width] = uint32_t(g);
        all_gaps = gaps <= H;
    } else {
        int g0 = low;
        for (;;) {
#pragma unroll
            for (int k = 0; k < kSetsGapsAhead; ++k) {
                if (g0 >= count || gaps >= H) continue;
                const int2 x = ahead[k];
                const bool on = g0 + lane < count && ((S.open[x.x >> 6] >> (x.x & 63)) & 1ull);
                const bool in = on && x.x >= lo && x.x <= hi;
                const unsigned long long b = __ballot(in);
                const int rank = gaps + __popcll(b & ((1ull << lane) - 1ull));
                if (in && rank < H) S.head[id + rank * shape.width] = uint32_t(x.y);
                gaps += __popcll(b);
                if (g0 == low) {                        // the class's lowest open gap only moves up
                    const unsigned long long o = __ballot(on);
                    if (lane == 0) atomicMax(&S.low[c], o ? g0 + __ffsll((long long)o) - 1 : min(g0 + kWave, count - 1));
                }
                g0 += kWave;
            }
            if (g0 >= count || gaps >= H || (gaps >= kSetsFewGaps && g0 - low >= kSetsGapsFar)) break;
#pragma unroll
            for (int k = 0; k < kSetsGapsAhead; ++k) ahead[k] = A.by_class[begin + min(g0 + k * kWave + lane, count - 1)];
        }
        all_gaps = g0 >= count && gaps <= H;
    }
    if (lane == 0) {
        S.head[id + min(gaps, H) * shape.width] = all_gaps ? kSetsServed : kSetsMoreGaps;
        S.set[id] = uint32_t(jobs) | uint32_t(last) << 16;
        S.dry[id] = 0;
    }
}

// The rounds of a batch by one wave, N sets per lane.  Leaves why they stopped and at which round of the batch; who was
// granted what is read off the claims.
// A lane issues an instruction every five cycles or so, and so a round takes as long as its instructions and one trip to
// LDS.  What is seldom (a set without a job or a gap at hand) is looked for in one go and sorted out aside, the round
// then begun anew; the next jobs are shifted in from eight that are there, instead of being fetched once it is known
// how many were passed; a lane without a set goes on with words that change nothing.  0.40 -> 0.21 us a round of up
// to 64 sets.
template <bool LISTS, int N, int BLOCKS>
__device__ __forceinline__ void sets_play(SetsShared<BLOCKS> &S, int lane, int n_sets, const SetsShape &shape, int before, int cap)
{
    auto claim_at = [&](uint32_t off) -> uint32_t & { return *reinterpret_cast<uint32_t *>(reinterpret_cast<char *>(S.jobs.claim) + off); };
    uint2 c[N];                     // the slots of the next four jobs (byte offsets of their claims)
    uint32_t head[N];               // the lowest open gap
    const uint32_t *next[N];        // where the one after it is
    const uint16_t *at[N];          // where the slots are
    uint32_t cand[N], word[N];      // the claim of the round before
    uint32_t out[N];                // all ones: no gaps or no jobs are left
    auto four = [](const uint16_t *from) { uint2 x; __builtin_memcpy(&x, from, 8); return x; };
    auto leave = [&](int i) {
        at[i] = S.idle;
        c[i] = four(at[i]);
        head[i] = 0;
        out[i] = ~0u;
    };
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const int id = lane + i * kWave;
        at[i] = &S.seq[min(id, n_sets - 1) * shape.room];
        next[i] = &S.head[id + shape.width];
        head[i] = S.head[id];
        c[i] = four(at[i]);
        out[i] = 0;
        cand[i] = kSetsNobody;
        word[i] = ~0u;
        if (id >= n_sets) leave(i);
    }
    int why = kSetsPause;
    const int last = min(cap - before, kSetsMostRounds);
    int q = 1;
    for (;;) {
        const uint32_t now = uint32_t(q) << 20;
        uint32_t w[N][4], outcome[N], after[N];
        uint2 more[N];
#pragma unroll
        for (int i = 0; i < N; ++i) {
            w[i][0] = claim_at(c[i].x & 0xffffu); w[i][1] = claim_at(c[i].x >> 16);
            w[i][2] = claim_at(c[i].y & 0xffffu); w[i][3] = claim_at(c[i].y >> 16);
            outcome[i] = claim_at(cand[i]);
            more[i] = four(at[i] + 4);
            after[i] = *next[i];
        }
#pragma unroll
        for (int i = 0; i < N; ++i)     // all of them are on their way before the first is waited for
            asm volatile("" : "+v"(w[i][0]), "+v"(w[i][1]), "+v"(w[i][2]), "+v"(w[i][3]), "+v"(outcome[i]), "+v"(more[i].x), "+v"(more[i].y), "+v"(after[i]));
        bool rare = q > last;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const bool won = outcome[i] == word[i];
            head[i] = won ? after[i] : head[i];
            next[i] += won ? shape.width : 0;
            rare |= (max(max(w[i][0], w[i][1]), max(w[i][2], w[i][3])) < now) | (head[i] >= kSetsServed);
        }
        if (__builtin_expect(__ballot(rare) != 0, 0)) {
            bool none[N], go_on = false, lost = false;
#pragma unroll
            for (int i = 0; i < N; ++i) {
                if (head[i] == kSetsServed) leave(i);
                lost |= out[i] == 0;
                cand[i] = kSetsNobody;          // its outcome is known
                word[i] = ~0u;
                none[i] = out[i] == 0 && max(max(w[i][0], w[i][1]), max(w[i][2], w[i][3])) < now;
            }
            if (q > last) {
                if (q > cap - before) {
                    if (lost) S.lost = 1;
                    why = kSetsAtCap;
                }
                break;          // (at the batch's own bound it is a pause like any other)
            }
            bool cannot = false, dry = false, some = false, through = false;
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const int id = min(lane + i * kWave, n_sets - 1);
                const uint32_t info = S.set[id];
                if (none[i] && at[i] + 4 < &S.seq[id * shape.room + int(info & 255u)]) {       // there are more
                    at[i] += 4;
                    c[i] = four(at[i]);
                    none[i] = false;
                    go_on = true;
                }
                cannot |= none[i] ? !(info >> 16) : head[i] == kSetsMoreGaps;
                dry |= none[i];
                if (LISTS) through |= none[i] && !(info >> 16) && int(info & 255u) >= S.most;
            }
            if (__ballot(go_on)) continue;
            if (__ballot(cannot)) {              // round q cannot be played
                if (LISTS && __ballot(through)) S.through = 1;
                break;
            }
            if (__ballot(dry)) S.closed = q;
#pragma unroll
            for (int i = 0; i < N; ++i) {
                if (none[i]) {
                    S.dry[lane + i * kWave] = uint8_t(q);
                    leave(i);
                }
                some |= out[i] == 0;
            }
            if (!__ballot(some)) { why = kSetsNoClaim; break; }       // nobody claims anything in round q
            continue;
        }
#pragma unroll
        for (int i = 0; i < N; ++i) {
            // the first free one, and what is shifted in
            const bool f0 = w[i][0] >= now, f1 = w[i][1] >= now, f2 = w[i][2] >= now;
            const uint32_t s01 = f0 ? c[i].x & 0xffffu : c[i].x >> 16, s23 = f2 ? c[i].y & 0xffffu : c[i].y >> 16;
            const bool none_of_two = !(f0 | f1);
            cand[i] = none_of_two ? s23 : s01;
            word[i] = now | head[i] | out[i];
            atomicMin(&claim_at(cand[i]), word[i]);
            at[i] += none_of_two ? (f2 ? 3 : 4) : (f0 ? 1 : 2);
            const bool all = none_of_two & !f2;
            const uint32_t shift = f0 | (none_of_two & f2) ? 16u : 0u;
            const uint32_t d0 = all ? more[i].x : f0 ? c[i].x : c[i].y, d1 = all ? more[i].y : f0 ? c[i].y : more[i].x;
            const uint32_t d2 = f0 ? more[i].x : more[i].y;
            c[i].x = __builtin_amdgcn_alignbit(d1, d0, shift);
            c[i].y = __builtin_amdgcn_alignbit(d2, d1, shift);
        }
        ++q;
        asm volatile("" ::: "memory");
    }
    if (lane == 0) { S.end = q; S.why = why; }
}

template <int BLOCKS>
__device__ __forceinline__ void sets_empty(SetsShared<BLOCKS> &S)
{
    for (int i = threadIdx.x; i < kSetsSlots + 2; i += kSetsThreads) sets_clear(S.jobs, i);
    if (threadIdx.x < kSetsMostRounds + 11) S.idle[threadIdx.x] = uint16_t(kSetsIdle);
}

// The classes.
template <int BLOCKS>
__device__ __forceinline__ void sets_classes(const SetsArgs &A, SetsShared<BLOCKS> &S)
{
    const int tid = threadIdx.x, n_classes = A.plan[kPlanClasses];
    if (tid <= kMaxClasses) {
        S.first[tid] = A.n_lb;
        S.gaps_at[tid] = tid < n_classes ? A.class_begin[tid] : A.n_gaps;
    }
    __syncthreads();
    if (tid < A.n_lb) {
        const int c = A.gap_cls[A.lb_begin[tid]];
        if (tid == 0 || A.gap_cls[A.lb_begin[tid - 1]] != c) S.first[c] = tid;
    }
    sets_empty(S);
    if (tid < kMaxClasses) S.low[tid] = 0;
    __syncthreads();
}

// A batch: the pieces are joined, its rounds played, and the grants written down.  held: the bitmap that sets_form
// reads.  Returns whether the process has ended (out says how), how many rounds were played (-1: too much
// work, none was) and by how many sets.  LISTS: jobs is how many a set is to have at hand at least, and becomes that of
// the next batch.
template <bool LISTS, int BLOCKS>
__device__ __forceinline__ bool sets_batch(const SetsArgs &A, SetsShared<BLOCKS> &S, int done, int least, uint32_t *held, int &played, int &sets, int &jobs)
{
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n_classes = A.plan[kPlanClasses];
    if (tid == 0) S.n = S.over = S.closed = S.lost = S.through = 0;
    __syncthreads();
    for (int u = tid; u < A.n_lb; u += kSetsThreads) {
        const unsigned long long open = A.block[u].open;
        const int n = open ? A.block[u].pieces : 0;
        S.open[u] = open;
        S.pieces[u] = int8_t(max(n, 0));
        if (n < 0) atomicOr(&S.over, -n);
    }
    for (int k = tid; k < A.n_lb * kSetsPieces; k += kSetsThreads) S.none[k] = uint8_t(A.block[k / kSetsPieces].piece[k % kSetsPieces].jobs == 0);
    __syncthreads();
    played = S.over & 1 ? -1 : 0;
    if (S.over) return false;
    played = -1;
    for (int c = wave; c < n_classes; c += kSetsWaves) sets_join(A, S, c, lane);
    __syncthreads();
    const int n_sets = sets = S.n;
    if (n_sets > kSetsMost) return false;
    const SetsShape shape = sets_shape(n_sets);
    // Where there are many sets the batch ends by one of them that has hardly more jobs than they are to have in common.
    // Not where the sets take each other's jobs: a round passes as many as there are sets then, the batch ends by
    // the jobs at hand after a few, and the next one would have no more of them.  So twice as many if that was its end: 2379
    // gaps of 40 capacities x 3077 jobs 2430 -> 1700 us a resolve, 3446 of 64 x 3420 2570 -> 1890; 32768 x 65536 the same.
    const int most = n_sets <= kSetsWaves ? shape.most : min(shape.most, LISTS ? max(3 * least / 2, jobs) : 3 * least / 2);
    if (LISTS && tid == 0) S.most = min(most, min(max(2 * least, jobs), A.list_jobs));
    for (int id = wave; id < n_sets; id += kSetsWaves) sets_fill<LISTS>(A, S, id, lane, wave, shape, most, held);
    __syncthreads();
    const bool over = S.over != 0;
    if (!over && wave == 0) {
        if (n_sets == 0) {              // nobody claims anything
            if (lane == 0) { S.end = 1; S.why = done < A.cap ? kSetsNoClaim : kSetsAtCap; }
        } else if (n_sets <= kWave) sets_play<LISTS, 1>(S, lane, n_sets, shape, done, A.cap);
        else if (n_sets <= 2 * kWave) sets_play<LISTS, 2>(S, lane, n_sets, shape, done, A.cap);
        else sets_play<LISTS, 4>(S, lane, n_sets, shape, done, A.cap);
    }
    __syncthreads();
    // the rounds played: not one that could not be; one without any claim if it found out that a set has no job left
    const int why = S.why;
    if (LISTS) jobs = S.through ? min(2 * S.most, kSetsListed) : 3 * jobs / 4;
    played = over ? -1 : why == kSetsNoClaim && S.closed == S.end ? S.end : S.end - 1;
    for (int k = tid; k < kSetsSlots + 2; k += kSetsThreads) {
        const uint32_t j = k < kSetsSlots ? S.jobs.job[k] : kSetsNoJob, claim = S.jobs.claim[k];
        if (j != kSetsNoJob && int(claim >> 20) <= played) {        // named, and granted to the gap of the smallest claim
            const int gap = int(claim & 0xfffffu), place = A.place_of[gap];
            atomicOr(&held[j >> 5], 1u << (j & 31u));
            A.state[place].y = int(j);
            A.state[place].w = gap << 2 | 1;
            atomicAnd(&S.open[place >> 6], ~(1ull << (place & 63)));
        }
        sets_clear(S.jobs, k);
    }
    // the gaps of a set that found no job left in one of these rounds are done with: found again by the next batch they
    // would count for a round of that
    for (int id = wave; id < n_sets && !over; id += kSetsWaves) {
        const int dry = S.dry[id], lo = S.lo[id], hi = S.hi[id];
        if (dry == 0 || dry > played) continue;
        for (int u = (lo >> 6) + lane; u <= hi >> 6; u += kWave) {
            unsigned long long gone = ~0ull;
            if (u == lo >> 6) gone &= ~0ull << (lo & 63);
            if (u == hi >> 6) gone &= ~0ull >> (63 - (hi & 63));
            atomicAnd(&S.open[u], ~gone);
        }
    }
    __syncthreads();
    for (int u = tid; u < A.n_lb; u += kSetsThreads) A.block[u].open = S.open[u];
    if (over || why == kSetsPause) return false;
    if (tid == 0) {
        A.out[kSoloDone] = kSoloEnded; A.out[kSoloRounds] = done + played; A.out[kSoloStable] = why == kSetsNoClaim || S.lost == 0;
    }
    return true;
}

// After a batch of `played` rounds, a short one if they are up to `few`: the jobs the gaps of a set are to have in common in
// the next one, and whether to go on.
__device__ __forceinline__ bool sets_go_on(int played, int most, int few, int &least, int &strain)
{
    if (played < 0) return false;
    least = min(max(2 * played, kSetsLeastFirst), most);
    strain = max(strain + (played <= few ? 1 : -1), 0);
    return strain < kSetsPatience;
}

// Too much work: the state of list block u as a launched round leaves it, but for the outcome already known.
__device__ __forceinline__ void sets_hand_back(const SetsArgs &A, int u, int lane)
{
    const int slot = u * kWave + lane;
    const unsigned long long on = A.block[u].open;
    const int at = A.block[u].at;
    const int4 st = A.state[slot];
    const bool highest = on != 0 && lane == 63 - __clzll((long long)on);
    if ((on >> lane) & 1ull) A.state[slot].x = max(st.x, highest ? at : at - 63);
    else if ((st.w & 3) == 0) A.state[slot].w |= 2;
    else if ((st.w & 3) == 1) A.claim[st.y] = claim_of(1, st.w >> 2);       // any stamp of a past round says held
}

// The rounds behind those that k_grant_solo has left calm, up to round cap.  held: two copies of the bitmap, alike.
// out: whether the process has ended, the rounds done, whether they are stable.
__global__ __launch_bounds__(kSetsThreads) void k_sets_one(SetsArgs A)
{
    __shared__ SetsShared<kSetsOneBlocks> S;
    __shared__ uint32_t s_held[kHeldMaxWords];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (A.out[kSoloDone] != kSoloCalm) return;
    sets_classes(A, S);
    for (int i = tid; i < A.held_words; i += kSetsThreads) s_held[i] = A.held[i];
    for (int u = wave; u < A.n_lb; u += kSetsWaves) sets_open(A, u, lane);
    __syncthreads();
    if (A.build) sets_by_class(A.n_gaps, A.plan[kPlanClasses], A.class_begin, S.first, A.place_of, A.by_class, reinterpret_cast<int(*)[kMaxClasses]>(&S.found[0][0]));
    const int begun = A.out[kSoloRounds];
    int done = begun, least = kSetsLeastFirst, strain = 0, played = 0, sets = 0, jobs = 0;
    for (;;) {
        __syncthreads();
        for (int u = wave; u < A.n_lb; u += kSetsWaves) sets_form<false>(A, u, lane, least, 0, s_held);
        __syncthreads();
        const bool ended = sets_batch<false>(A, S, done, least, s_held, played, sets, jobs);
        const bool first = done == begun;
        done += max(played, 0);
        if (ended) return;
        // Begun in vain: many sets, whose batches take long, and which have no jobs for themselves (2328 gaps x 1074 jobs, 37
        // sets, four rounds a batch: 590 us a resolve with two more of them, 525 so, 480 with no batch at all)
        if (first && 6 * played < sets) break;
        if (!sets_go_on(played, kSetsLeast, kSetsShort, least, strain)) break;
    }
    if (tid == 0) {
        A.out[kSoloDone] = kSetsLeft; A.out[kSoloRounds] = done; A.out[kSoloStable] = 0;
    }
    __syncthreads();
    for (int i = tid; i < A.held_words; i += kSetsThreads) A.held[i] = A.held[A.held_words + i] = s_held[i];
    for (int u = wave; u < A.n_lb; u += kSetsWaves) sets_hand_back(A, u, lane);
}

// The same in several launches: the start; then searches and batches in turn, as long as out says that it is
// running; and what is left for launched rounds.
constexpr int kSetsFormThreads = 256;

__global__ __launch_bounds__(kSetsFormThreads) void k_sets_open(SetsArgs A)
{
    const int lane = threadIdx.x & (kWave - 1), u = blockIdx.x * (kSetsFormThreads / kWave) + (threadIdx.x >> 6);
    if (u < A.n_lb) sets_open(A, u, lane);
}

__global__ __launch_bounds__(kSetsThreads) void k_sets_begin(SetsArgs A)
{
    __shared__ SetsShared<kSetsMaxBlocks> S;
    sets_classes(A, S);
    if (threadIdx.x <= kMaxClasses) {
        A.classes[threadIdx.x] = S.first[threadIdx.x];
        A.classes[kMaxClasses + 1 + threadIdx.x] = S.gaps_at[threadIdx.x];
    }
    if (threadIdx.x < kMaxClasses) A.low[threadIdx.x] = 0;
    if (threadIdx.x == 0) { A.out[kSoloDone] = kSetsRunning; A.out[kSetsState] = kSetsLeastFirst << 8; }
    if (A.build)
        sets_by_class(A.n_gaps, A.plan[kPlanClasses], A.class_begin, S.first, A.place_of, A.by_class, reinterpret_cast<int(*)[kMaxClasses]>(&S.found[0][0]));
}

__global__ __launch_bounds__(kSetsFormThreads) void k_sets_form(SetsArgs A)
{
    __shared__ uint4 s_held[kHeldMaxWords / 4];
    int running = A.out[kSoloDone], state = A.out[kSetsState];
    const uint4 *held = reinterpret_cast<const uint4 *>(A.held);
    for (int i = threadIdx.x; i < A.held_words / 4; i += kSetsFormThreads) s_held[i] = held[i];
    asm volatile("" : "+v"(running), "+v"(state));
    __syncthreads();
    if (__builtin_amdgcn_readfirstlane(running) != kSetsRunning) return;
    const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int u = blockIdx.x * (kSetsFormThreads / kWave) + wave;
    state = __builtin_amdgcn_readfirstlane(state);
    if (u < A.n_lb) sets_form<true>(A, u, lane, state >> 8 & 255, state >> 16, reinterpret_cast<const uint32_t *>(s_held));
}

__global__ __launch_bounds__(kSetsThreads) void k_sets_play(SetsArgs A)
{
    __shared__ SetsShared<kSetsMaxBlocks> S;
    // one trip to memory for all that is known from the launch before
    const int tid = threadIdx.x, c = min(tid, kMaxClasses);
    int running = A.out[kSoloDone], done = A.out[kSoloRounds], state = A.out[kSetsState];
    int first = A.classes[c], gaps_at = A.classes[kMaxClasses + 1 + c], low = A.low[min(c, kMaxClasses - 1)];
    asm volatile("" : "+v"(running), "+v"(done), "+v"(state), "+v"(first), "+v"(gaps_at), "+v"(low));
    if (__builtin_amdgcn_readfirstlane(running) != kSetsRunning) return;
    done = __builtin_amdgcn_readfirstlane(done);
    if (tid <= kMaxClasses) { S.first[tid] = first; S.gaps_at[tid] = gaps_at; }
    if (tid < kMaxClasses) S.low[tid] = low;
    sets_empty(S);
    __syncthreads();
    state = __builtin_amdgcn_readfirstlane(state);
    int played = 0, sets = 0, jobs = state >> 16, least = state >> 8 & 255, strain = state & 255;
    if (sets_batch<true>(A, S, done, least, A.held, played, sets, jobs)) return;
    const bool go_on = sets_go_on(played, kSetsLeastMany, kSetsShortMany, least, strain);
    if (threadIdx.x < kMaxClasses) A.low[threadIdx.x] = S.low[threadIdx.x];
    if (threadIdx.x == 0) {
        A.out[kSoloRounds] = done + max(played, 0);
        A.out[kSetsState] = jobs << 16 | least << 8 | strain;
        if (!go_on) A.out[kSoloDone] = kSetsLeft;
    }
}

__global__ __launch_bounds__(kSetsFormThreads) void k_sets_hand_back(SetsArgs A)
{
    const int lane = threadIdx.x & (kWave - 1), u = blockIdx.x * (kSetsFormThreads / kWave) + (threadIdx.x >> 6);
    if (u < A.n_lb) sets_hand_back(A, u, lane);
    uint32_t *to = A.held + A.held_words;
    for (int i = blockIdx.x * kSetsFormThreads + threadIdx.x; i < A.held_words; i += gridDim.x * kSetsFormThreads) to[i] = A.held[i];
}

}  // namespace sja
