// K4, the long tail of the conflict rounds in one thread block.
//
// After the first rounds nearly all open gaps want the same job: at Stress
// (32768 gaps x 65536 jobs) all but the first 300 of 9400 rounds name one to
// three jobs, each by thousands of gaps.  Such a round has next to no work in
// it, and a launch per round paid 4.4 us for the memory trips of its chain
// (state, records, claim words) and 1.3 us more until the next launch.
// Here ONE block runs round after round: a thread per list block, which keeps
// its open lanes, its place in the list and its lowest open gap in registers;
// the held jobs (a bitmap) and the claims (two small hash tables, by turns of
// the rounds) live in LDS, and a round has a single barrier.  A round takes
// 1.7 us at Medium (66 list blocks) and 2.7 at Stress (566), by its
// instructions, LDS trips and the hand-overs between the scalar and the vector
// side: 440 instructions a wave.
// Medium tick 4586 -> 2220 us, Stress 62.8 -> 56.3 ms when it came.
//
// What a thread relies on: along the positions of a list block a job's key
// never falls (F grows with the cut; the host sees to it where the hysteresis
// rule could undo that), so the job of the highest open lane is the job of every open
// lane its record covers, and of no other records need be looked at for them.
// Lanes below that record form further pieces with jobs of their own; those
// (and a thread that has many records to pass) are served by the whole wave,
// 64 records a trip.
//
// When a round is much work (the first rounds of a large batch, or when a
// service class runs out and the next one's jobs begin) one block is the wrong
// place for it: it starts only when the last launched round was little work,
// and once the work adds up it stops and leaves the gaps' state as the round
// kernel expects it.
#pragma once

#include "k_claims.h"
#include "k_grant.h"

namespace sja {

constexpr int kSoloMaxWaves = 16;
constexpr int kSoloMinWaves = 8;        // list blocks in pieces are served by several waves side by side (4: 4 % slower, 16: 5 %)
constexpr int kSoloSmallBlocks = 128;   // list blocks whose gap orders are kept in LDS
constexpr int kSoloMaxBlocks = kSoloMaxWaves * kWave;
// launched rounds before the block may first take over: up to kSoloFewBlocks list blocks the fourth is little
// work, with more of them the eighth (Medium, 66: 20 us saved over a look after four)
constexpr int kSoloFirstFew = 4, kSoloFirstMany = 8, kSoloFewBlocks = 32;
constexpr int kSoloFewRounds = 16;      // rounds it takes over at least, if the caller bounds them,
constexpr int kSoloBlocksPerRound = 4;  // and one more for this many list blocks (it needs up to 3 us for each wave's next one to start)
constexpr int kSoloSteps = 3;           // steps of eight records before a lane still looking alone is served by its wave
// A wave's effort in a round: pieces it serves and steps of records it takes (0.5 us each; a round without any
// takes 1.7 us, a launched one 6).
constexpr int kSoloEasy = 7;            // effort per wave and round that costs no more than a launched round
constexpr int kSoloPatience = 96;       // effort beyond that, summed up, after which the block stops
constexpr int kSoloMostSteps = 48;      // steps after which it stops in the middle of a round
constexpr int kSoloStart = 3;           // effort per wave of the last launched round up to which it starts;
constexpr int kSoloStartFew = 16;       // with few list blocks, whose start and whose rounds in pieces cost little
enum { kSoloDone = 0, kSoloRounds = 1, kSoloStable = 2 };
// Rounds are calm if few pieces were served in the last ones of them (two to the power of the shift).  Where one launch
// plays them from there on (k_sets_one) it is worth to begin early, and to end after one batch if that was in vain: 2048 gaps x
// 8192 jobs 905 us a tick by the first line, 810 by the second; 118 list blocks, with launches in turn, 5.48 ms by the
// first, 6.1 with 512 pieces, and 5.26 and 5.71 by the two lines since the sets have more jobs at hand.
constexpr int kSoloCalmShift = 5, kSoloCalmPieces = 128;
constexpr int kSoloCalmShiftFew = 3, kSoloCalmPiecesFew = 8;
enum { kSoloHandedBack = 0, kSoloEnded = 1, kSoloPutOff = 2, kSoloCalm = 3 };      // what out[kSoloDone] says

__device__ __forceinline__ unsigned long long solo_readlane64(unsigned long long v, int l)
{
    return (static_cast<unsigned long long>(uint32_t(__builtin_amdgcn_readlane(int(uint32_t(v >> 32)), l))) << 32) |
           uint32_t(__builtin_amdgcn_readlane(int(uint32_t(v)), l));
}

// Rounds after + 1 .. at most cap, by blockDim.x / kWave waves (n_lb <= blockDim.x).  `after` rounds have
// been launched; cnt_lost / cnt_cand tell of those from first_check on whether one of them was already the
// last.  out: whether the process has ended, is to be taken up again by launched rounds, has not been taken
// over at all (the end of round `after` is then still open), or has become calm by round calm_from or later; the
// rounds done, whether they are stable.
//
// A wave has its SIMD to itself (or shares it with one or two others), so a round takes as long as its
// instructions: what a thread tests every round (eight records' held bits) is prepared when the records
// arrive or its highest open lane changes.  The held jobs are two bitmaps: a round reads one and marks the
// jobs it names in the other, and in the first one round later.
// SMALL: at most kSoloSmallBlocks list blocks, whose lanes' gap orders fit LDS (in global memory the next
// entry's load is waited for together with the records that were asked for last).
template <bool SMALL>
__global__ __launch_bounds__(kSoloMaxWaves * kWave) void k_grant_solo(
    int4 *state, const int32_t *__restrict__ list_off, const Rec32 *__restrict__ rec, unsigned long long *claim, int after,
    int first_check, int cap, int n_lb, int held_words, uint32_t *held, const int32_t *__restrict__ cnt_lost,
    const int32_t *__restrict__ cnt_cand, int calm_from, int calm_shift, int calm_pieces, int32_t *effort, int32_t *out)
{
    __shared__ uint32_t s_held[2][kHeldMaxWords + 4];           // the word behind the last job's is all ones: nobody's job
    __shared__ SoloTables s_tabs;       // the claims of this round and of the one before or after it
    __shared__ unsigned long long s_piece[kSoloMaxWaves][kWave];        // a wave's claims for pieces of list blocks
    __shared__ int s_at[kSoloMaxWaves][kWave];                  // whose they are: thread << 6 | lane
    __shared__ unsigned long long s_log[kSoloMaxWaves][kWave];  // grants not yet written to the state: slot << 32 | job
    // by round stamp: somebody claims, a wave gives up, (round << 8 | most effort of a wave), open lanes found nothing more
    __shared__ int4 s_ctl[2];
    __shared__ int s_flag;
    __shared__ int s_served[2];         // pieces served, by turns of as many rounds as have to be calm
    __shared__ int s_order[SMALL ? kSoloSmallBlocks * kWave : 1];      // per list block its open lanes, lowest gap first: gap << 6 | lane
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int threads = blockDim.x, waves = threads / kWave;
    // neighbouring list blocks split in the same rounds: they go to different waves
    const int u = lane * waves + wave;
    const uint32_t nobody = uint32_t(held_words) * 32u;

    if (effort[after & 1] > (n_lb <= kSoloFewBlocks ? kSoloStartFew : kSoloStart) * waves) {
        if (tid == 0) {
            out[kSoloDone] = kSoloPutOff; out[kSoloRounds] = after; out[kSoloStable] = 0;
            for (int r = first_check; r <= after; ++r)
                if (cnt_cand[r] == 0 || (r < after && cnt_lost[r] == 0)) {
                    out[kSoloDone] = kSoloEnded; out[kSoloRounds] = r; out[kSoloStable] = 1;
                    break;
                }
        }
        return;
    }
    for (int i = tid; i < held_words; i += threads) s_held[0][i] = s_held[1][i] = held[size_t((after + 1) & 1) * held_words + i];
    for (int i = tid; i < kSoloTable; i += threads) s_tabs.word[0][i] = s_tabs.word[1][i] = 0;
    if (tid < 2) { s_ctl[tid] = make_int4(0, 0, 0, 0); s_held[tid][held_words] = ~0u; s_served[tid] = 0; }
    if (tid == 0) s_flag = 0;
    __syncthreads();

    // the outcome of round `after`, the open lanes, and the lanes of every list block by gap index
    unsigned long long open = 0;        // open lanes of this thread's list block
    int e = 0, list_end = 0;            // its place in the list: what covers its highest open lane before it is held
    {
        bool any_lost = false;
        constexpr int Q = 4;            // list blocks whose state and claims are asked for together
        for (int i0 = 0; i0 * waves + wave < n_lb; i0 += Q) {
            int4 raw[Q];
            unsigned long long word[Q];
#pragma unroll
            for (int q = 0; q < Q; ++q) raw[q] = state[min((i0 + q) * waves + wave, n_lb - 1) * kWave + lane];
#pragma unroll
            for (int q = 0; q < Q; ++q) word[q] = claim[max(raw[q].y, 0)];
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const int i = i0 + q, slot0 = (i * waves + wave) * kWave;
                if (i * waves + wave >= n_lb) break;
                const int g = raw[q].w >> 2;
                if ((raw[q].w & 3) == 0 && raw[q].y >= 0) {
                    if (word[q] == claim_of(after, g)) {
                        state[slot0 + lane].w = raw[q].w |= 1;
                    } else {
                        state[slot0 + lane].y = -1;
                        any_lost = true;
                    }
                }
                const unsigned long long on = __ballot((raw[q].w & 3) == 0);
                int place = 0;
                for (unsigned long long m = on; m; m &= m - 1)
                    place += __builtin_amdgcn_readlane(g, __ffsll((long long)m) - 1) < g;
                if ((on >> lane) & 1ull) {
                    if (SMALL) s_order[SMALL ? slot0 + place : 0] = (g << 6) | lane;
                    else state[slot0 + place].z = (g << 6) | lane;
                }
                const int e_top = __builtin_amdgcn_readlane(raw[q].x, on ? 63 - __clzll((long long)on) : 0);
                if (lane == i) { open = on; e = e_top; }
            }
        }
        if (any_lost) s_flag = 1;
        if (u < n_lb) list_end = list_off[u + 1];
        if (e >= list_end) open = 0;
        __threadfence_block();
    }
    int top = 0, bottom = 0;            // its highest and lowest open lane
    int order = 0, next_low = 0, low_gap = -1, low_lane = 0;    // its lowest open gap, and the entry after it
    uint32_t w[8];                      // its records from w0 on (0 where there is none)
    uint32_t job_of[8];                 // and their jobs, `nobody` where the highest open lane is not covered
    int w0 = 0;
    uint4 behind = make_uint4(0, 0, 0, 0);      // the four records after them, asked for ahead
    const uint4 *rec4 = reinterpret_cast<const uint4 *>(rec);
    auto cover = [&](int q) {
        const Rec32 r{w[q]};
        job_of[q] = uint32_t(top - r.lo()) < uint32_t(r.hi() - r.lo()) ? r.job() : nobody;
    };
    auto ends = [&]() {
        top = 63 - __clzll((long long)open);
        bottom = __ffsll((long long)open) - 1;
    };
    // the half window from record i on; records before `from` and behind the list are none
    auto take = [&](int half, const uint4 &r, int i, int from) {
        w[4 * half] = r.x; w[4 * half + 1] = r.y; w[4 * half + 2] = r.z; w[4 * half + 3] = r.w;
        if (__builtin_expect(i < from || i + 4 > list_end, 0)) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (i + q < from || i + q >= list_end) w[4 * half + q] = 0u;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) cover(4 * half + q);
    };
    auto ask = [&](int i) { return rec4[min(i, (list_end - 1) & ~3) >> 2]; };
    auto window = [&]() {
        w0 = e & ~3;
        const uint4 r = ask(w0), r2 = ask(w0 + 4);
        behind = ask(w0 + 8);
        take(0, r, w0, e);
        take(1, r2, w0 + 4, e);
    };
    auto order_at = [&](int k) { return SMALL ? s_order[SMALL ? u * kWave + min(k, kWave - 1) : 0] : state[u * kWave + min(k, kWave - 1)].z; };
    auto closed = [&]() {       // lanes were closed: the ends, what covers the highest, the lowest gap
        const int was = top;
        if (!open) { low_gap = -1; return; }
        ends();
        if (top != was) {
#pragma unroll
            for (int q = 0; q < 8; ++q) cover(q);
        }
        while (!((open >> low_lane) & 1ull) && order <= kWave) {
            low_gap = next_low >> 6; low_lane = next_low & 63;
            ++order;
            next_low = order_at(order);
        }
    };
#pragma unroll
    for (int q = 0; q < 8; ++q) { w[q] = 0; job_of[q] = nobody; }
    if (open) {
        const int first = order_at(0);
        low_gap = first >> 6; low_lane = first & 63;
        order = 1;
        next_low = order_at(1);
        ends();
        window();
    }
    __syncthreads();
    const bool lost_before = s_flag != 0;
    __syncthreads();
    if (tid == 0) {
        // the process may have ended within the launched rounds
        s_flag = 0;
        for (int r = first_check; r <= after; ++r)
            if (cnt_cand[r] == 0 || (r < after ? cnt_lost[r] != 0 : lost_before) == false) {
                out[kSoloDone] = kSoloEnded; out[kSoloRounds] = r; out[kSoloStable] = 1;
                s_flag = 1;
                break;
            }
    }
    __syncthreads();
    if (s_flag) return;

    int n_log = 0;
    auto flush = [&]() {
        if (lane < n_log) {
            const unsigned long long x = s_log[wave][lane];
            const int slot = int(x >> 32);
            state[slot].y = int(uint32_t(x));
            state[slot].w |= 1;
        }
        n_log = 0;
    };
    int strain = 0;             // effort beyond what is easy, summed up
    int done = after;           // rounds finished
    int ended = 0, stable = 0;
    bool calm = false;
    uint32_t marked = nobody, marked_piece = nobody;    // the jobs this lane marked a round ago
    for (int round = after + 1;; ++round) {
        const int half = round & 1;
        const uint32_t *const is_held = s_held[half];
        uint32_t *const mark = s_held[half ^ 1];
        unsigned long long *const tab = solo_table(s_tabs, round);
        auto set_mark = [&](uint32_t j) { atomicOr(&mark[j >> 5], 1u << (j & 31u)); };
        bool looking = open != 0, found = false, have = false;
        const bool any_open = __ballot(looking) != 0;
        uint32_t job = 0;
        int lo = 0;
        // the job of the highest open lane: eight records a step
        int step = 0;
        for (;; ++step) {
            uint32_t b[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) b[q] = is_held[job_of[q] >> 5];
            uint32_t taken = 0;
#pragma unroll
            for (int q = 7; q >= 0; --q) taken = (taken << 1) | ((b[q] >> (job_of[q] & 31u)) & 1u);
            const int first = __ffs(int(~taken)) - 1;       // 8: none of them
            const bool in0 = first < 4;
            const uint32_t r01 = (first & 1) ? w[1] : w[0], r23 = (first & 1) ? w[3] : w[2];
            const uint32_t r45 = (first & 1) ? w[5] : w[4], r67 = (first & 1) ? w[7] : w[6];
            const uint32_t r03 = (first & 2) ? r23 : r01, r47 = (first & 2) ? r67 : r45;
            const uint32_t r = in0 ? r03 : r47;
            found = looking & (first < 8);
            if (found) {
                job = Rec32{r}.job();
                lo = Rec32{r}.lo();
                e = w0 + first;
            }
            if (looking & !in0) {       // the first half is used up
#pragma unroll
                for (int q = 0; q < 4; ++q) { w[q] = w[q + 4]; job_of[q] = job_of[q + 4]; }
                w0 += 4;
                take(1, behind, w0 + 4, 0);
                behind = ask(w0 + 8);
                if (!found) e = w0;
                if (w0 >= list_end) {   // no job is left for the highest lane, and so for none below it
                    open = 0;
                    low_gap = -1;
                    looking = false;
                }
            }
            have = have | found;
            looking = looking & !found;
            const unsigned long long look = __ballot(looking);
            if (!look || (step >= kSoloSteps && (look & (look - 1)) == 0) || step >= kSoloMostSteps) break;
        }
        found = have;
        const bool split = found & (lo > bottom);
        unsigned long long together = __ballot(looking | split);
        int n_pieces = 0;
        bool over = step >= kSoloMostSteps;     // a round for many thread blocks
        if (together && !over) {
            // list blocks the whole wave looks at: those still looking, and those in pieces
            const unsigned long long have_first = __ballot(found);
            while (together) {
                const int t = __ffsll((long long)together) - 1;
                together &= together - 1;
                const int slot0 = (t * waves + wave) * kWave;
                const int end = __builtin_amdgcn_readlane(list_end, t);
                int g = state[slot0 + lane].w >> 2;
                int from = state[slot0 + lane].x;               // where this lane's own search may start
                asm volatile("" : "+v"(g), "+v"(from));         // both have arrived: no load is left open over the rest of the round
                unsigned long long rest = solo_readlane64(open, t);
                int at = __builtin_amdgcn_readlane(e, t);
                int pj = __builtin_amdgcn_readlane(int(job), t), plo = __builtin_amdgcn_readlane(lo, t);
                bool have = (have_first >> t) & 1ull, first = true;
                const int e_was = at;
                int e_first = at;
                while (rest) {
                    const int p = 63 - __clzll((long long)rest);
                    if (!have) {
                        // a lower lane's record lies behind the higher lane's, but for records of that same
                        // job with an equal key (at most 63 of them, next to it)
                        int c = first ? at : max(at - 63, __builtin_amdgcn_readlane(from, p));
                        unsigned long long ok = 0;
                        Rec32 r{0};
                        for (; c < end; c += kWave) {
                            const int i = c + lane;
                            r = rec[min(i, end - 1)];
                            const uint32_t word = is_held[r.job() >> 5];
                            const bool free_job = ((word >> (r.job() & 31u)) & 1u) == 0;
                            ok = __ballot(i < end && r.lo() <= p && p < r.hi() && free_job);
                            if (ok) break;
                        }
                        if (!ok) break;             // none for lane p, nor for any below it
                        const int hit = __ffsll((long long)ok) - 1;
                        const Rec32 x = r.of_lane(hit);
                        at = c + hit; pj = int(x.job()); plo = x.lo();
                    }
                    if (n_pieces == kWave) { over = true; rest = 0; break; }
                    if (first) e_first = at;
                    else if (lane == p) state[slot0 + lane].x = at;
                    const unsigned long long piece = rest & ~((1ull << plo) - 1ull);
                    const bool in = (piece >> lane) & 1ull;
                    const int low = wave_min_dpp(in ? g : 0x7fffffff);
                    if (in && g == low) {
                        s_piece[wave][n_pieces] = solo_word(round, pj, low);
                        s_at[wave][n_pieces] = (t << 6) | lane;
                    }
                    ++n_pieces;
                    rest &= ~piece;
                    have = false;
                    first = false;
                }
                if (lane == t) {
                    found = false;
                    if (rest) { open &= ~rest; closed(); }
                    if (e_first != e_was) { e = e_first; window(); }
                }
            }
        }
        // claims: the list blocks that name the first one's job agree on their lowest gap, the rest go by themselves
        const bool whole = found & !split;
        const unsigned long long todo = __ballot(whole);
        if (marked != nobody) set_mark(marked);
        marked = nobody;
        if (todo) {
            const int leader = __ffsll((long long)todo) - 1;
            const bool same = whole & (job == uint32_t(__builtin_amdgcn_readlane(int(job), leader)));
            const int low = wave_min_dpp(same ? low_gap : 0x7fffffff);
            if (whole & (!same | (lane == leader))) {
                if (!solo_enter(tab, solo_word(round, int(job), same ? low : low_gap))) s_ctl[half].y = round;
                set_mark(job);
                marked = job;
            }
        }
        if (marked_piece != nobody) set_mark(marked_piece);
        marked_piece = nobody;
        if (n_pieces) {
            if (lane < n_pieces) {
                const unsigned long long v = s_piece[wave][lane];
                if (!solo_enter(tab, v)) s_ctl[half].y = round;
                marked_piece = uint32_t(v >> 20) & 0xfffffu;
                set_mark(marked_piece);
            }
        }
        if (n_pieces && lane == 0) atomicAdd(&s_served[(round >> calm_shift) & 1], n_pieces);
        if (n_pieces + step > kSoloEasy && lane == 0) {
            if (over) s_ctl[half].y = round;
            atomicMax(&s_ctl[half].z, (round << 8) | (n_pieces + step));
        }
        if (lane == 0) {
            if (todo != 0 || n_pieces) s_ctl[half].x = round;
            else if (any_open) s_ctl[half].w = round;
        }
        // the round's only barrier: all claims are in.  A wave that goes on to the next round writes the other
        // halves of the claims and of s_ctl, while slower ones still read these; the bitmap it marks then,
        // this round's, is not read behind the barrier
        __syncthreads();
        const int4 ctl = s_ctl[half];
        bool won = false;
        if (whole) won = solo_wins(tab, solo_word(round, int(job), low_gap));
        if (ctl.y == round) break;      // the launched rounds take this one over
        if (ctl.x != round) {           // nobody claims anything: the end
            // this round counts if a lane had lost the one before and found nothing more; in the first round one
            // had, else the block had ended above (list blocks used up by then never had their lanes opened)
            ended = 1; stable = 1;
            done = ctl.w == round || round == after + 1 ? round : round - 1;
            break;
        }
        auto grant = [&](bool mine, int l, uint32_t j) {       // lane l of this thread's list block gets job j
            const unsigned long long b = __ballot(mine);
            const int k = __popcll(b);
            if (n_log + k > kWave) flush();
            if (mine) {
                s_log[wave][n_log + __popcll(b & ((1ull << lane) - 1ull))] =
                    (static_cast<unsigned long long>(uint32_t(u * kWave + l)) << 32) | j;
                open &= ~(1ull << l);
                closed();
            }
            n_log += k;
        };
        if (__ballot(won)) grant(won, low_lane, job);
        if (n_pieces) {
            unsigned long long hits = __ballot(lane < n_pieces && solo_wins(tab, s_piece[wave][lane]));
            while (hits) {
                const int k = __ffsll((long long)hits) - 1;
                hits &= hits - 1;
                const int at = s_at[wave][k];
                grant(lane == at >> 6, at & 63, uint32_t(s_piece[wave][k] >> 20) & 0xfffffu);
            }
        }
        done = round;
        strain = max(strain + max((ctl.z >> 8) == round ? (ctl.z & 255) - kSoloEasy : 0, 0) - 1, 0);
        // (the other turn's count is complete, and cleared half a turn later)
        const int turn = round & ((1 << calm_shift) - 1);
        int *const served = &s_served[((round >> calm_shift) & 1) ^ 1];
        if (turn == 1 << (calm_shift - 1) && tid == 0) *served = 0;
        if (turn == 0 && round >= calm_from) calm = *served <= calm_pieces;
        if (round == cap || strain > kSoloPatience || calm) {
            // the block stops here.  A lane still open has lost this round; if there is none, the process has ended with it
            if (open) s_flag = 1;
            __syncthreads();
            const bool lost = s_flag != 0;
            ended = !lost || round == cap;
            stable = !lost;
            break;
        }
    }
    flush();
    if (tid == 0) {
        out[kSoloDone] = ended ? kSoloEnded : calm ? kSoloCalm : kSoloHandedBack; out[kSoloRounds] = done; out[kSoloStable] = stable;
        effort[0] = effort[1] = 0;
    }
    if (ended) return;
    // too much work: the state as a launched round leaves it, but for the outcome already known
    __syncthreads();
    // (the bitmap the next round would read: the jobs of the last one are marked in that one only)
    for (int i = tid; i < held_words; i += threads) held[i] = held[held_words + i] = s_held[(done + 1) & 1][i];
    for (int i = 0; i * waves + wave < n_lb; ++i) {
        const int slot = (i * waves + wave) * kWave + lane;
        const unsigned long long on = solo_readlane64(open, i);
        const int e_top = __builtin_amdgcn_readlane(e, i);
        const int flag = state[slot].w & 3;
        const bool highest = on != 0 && lane == 63 - __clzll((long long)on);
        if ((on >> lane) & 1ull) state[slot].x = max(state[slot].x, highest ? e_top : e_top - 63);
        else if (flag == 0) state[slot].w |= 2;
        else if (flag == 1) claim[state[slot].y] = claim_of(1, state[slot].w >> 2);     // any stamp of a past round says held
    }
}

}  // namespace sja
