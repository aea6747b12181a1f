// The claim tables of k_grant_solo: which gap gets a job that several list
// blocks name in one round.
//
// A round enters its claims, all waves meet at the round's only barrier, and
// then the wins are read.  A wave that has read its wins goes straight on and
// enters the next round's claims while a slower one may still be reading this
// round's, and a later claim replaces an earlier round's word in its slot.  So
// rounds take two tables in turn: a wave comes to the claims of round r + 2
// only through the barrier of round r + 1, which every wave reaches after its
// reads of round r.
//
// Nothing here but integer words in LDS, so that the order in which waves come
// by can be played through on the host as well.
#pragma once

#include <stdint.h>

namespace sja {

constexpr int kSoloTable = 2048;        // claim words: one per job named in a round (power of two)

struct SoloTables {
    unsigned long long word[2][kSoloTable];
};

__device__ __forceinline__ unsigned long long *solo_table(SoloTables &t, int round) { return t.word[round & 1]; }

// A claim: round (24 bits) : job (20) : inverted gap (20).  A word of an earlier round (two or more before,
// in the same table) is told from a current one by its stamp, so nothing is ever cleared.
__device__ __forceinline__ unsigned long long solo_word(int round, int job, int g)
{
    return (static_cast<unsigned long long>(uint32_t(round)) << 40) | (static_cast<unsigned long long>(uint32_t(job)) << 20) |
           (0xfffffu - uint32_t(g));
}

// Enters a claim in its round's table.  The larger of two words keeps a slot and the other one moves on, so
// all claims for a job end in one slot, the first from the job's own whose word is not larger, with the
// lowest gap.
__device__ __forceinline__ bool solo_enter(unsigned long long *tab, unsigned long long v)
{
    int h = int(v >> 20) & (kSoloTable - 1);
#pragma unroll 1
    for (int tries = 0; tries < kSoloTable; ++tries) {
        const unsigned long long old = atomicMax(&tab[h], v);
        if (__builtin_expect((old >> 40) != (v >> 40) || ((old ^ v) >> 20) == 0, 1)) return true;
        v = min(old, v);
        h = (h + 1) & (kSoloTable - 1);
    }
    return false;           // no slot left: the round is given up
}

// Whether the claim `v` is the one that stands for its job, once all claims of the round are in.
__device__ __forceinline__ bool solo_wins(const unsigned long long *tab, unsigned long long v)
{
    int h = int(v >> 20) & (kSoloTable - 1);
    unsigned long long x = tab[h];
#pragma unroll 1
    for (int tries = 1; __builtin_expect(((x ^ v) >> 20) != 0, 0) && tries < kSoloTable; ++tries) {
        h = (h + 1) & (kSoloTable - 1);
        x = tab[h];
    }
    return x == v;
}

}  // namespace sja
