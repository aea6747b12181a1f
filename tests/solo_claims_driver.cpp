// Plays the claim tables of k_claims.h through on the host, in the orders in which the waves of one
// thread block can come by: a round's claims of all waves, the barrier, and then for each wave its
// reads of the round's wins followed, some time before the others' reads, by its claims of the next
// round.  A claim wins exactly if it is the one with the lowest gap for its job.
#include <stdint.h>
#include <stdio.h>

#include <algorithm>
#include <map>
#include <random>
#include <vector>

#define __device__
#define __forceinline__ inline
static unsigned long long atomicMax(unsigned long long *p, unsigned long long v)
{
    const unsigned long long old = *p;
    *p = std::max(old, v);
    return old;
}
using std::min;

#include "k_claims.h"

using namespace sja;

struct Claim { int job, gap; };

int main()
{
    std::mt19937 rng(1);
    auto draw = [&](int n) { return int(rng() % unsigned(n)); };
    long wins = 0, checked = 0;
    for (int run = 0; run < 400; ++run) {
        static SoloTables t;
        t = SoloTables{};
        const int waves = 2 + draw(15), first_round = 5 + draw(1000), rounds = 6;
        // few slots, so that rounds meet in them: job ids that differ by multiples of the table's size
        const int slots = 1 + draw(run % 2 ? 8 : 2048), each = 1 + draw(run % 3 ? 6 : 64);
        std::vector<std::vector<std::vector<Claim>>> claims(rounds, std::vector<std::vector<Claim>>(waves));
        std::vector<std::map<int, int>> lowest(rounds);
        for (int r = 0; r < rounds; ++r)
            for (auto &of_wave : claims[r])
                for (int k = draw(each + 1); k > 0; --k) {
                    const Claim c{draw(slots) + kSoloTable * draw(64), draw(65536)};
                    of_wave.push_back(c);
                    auto at = lowest[r].emplace(c.job, c.gap).first;
                    at->second = std::min(at->second, c.gap);
                }
        auto enter = [&](int r, int w) {
            for (const Claim &c : claims[r][w])
                if (!solo_enter(solo_table(t, first_round + r), solo_word(first_round + r, c.job, c.gap))) return false;
            return true;
        };
        std::vector<int> order(waves);
        for (int w = 0; w < waves; ++w) order[w] = w;
        for (int w : order)
            if (!enter(0, w)) { printf("run %d: no slot\n", run); return 1; }
        for (int r = 0; r < rounds; ++r) {
            // behind the barrier of round r: each wave reads its wins and enters its next claims, one wave after the other
            std::shuffle(order.begin(), order.end(), rng);
            for (int w : order) {
                for (const Claim &c : claims[r][w]) {
                    const bool won = solo_wins(solo_table(t, first_round + r), solo_word(first_round + r, c.job, c.gap));
                    const bool should = lowest[r][c.job] == c.gap;
                    ++checked;
                    wins += won;
                    if (won != should) {
                        printf("run %d round %d: job %d gap %d %s\n", run, r, c.job, c.gap, should ? "lost its claim" : "won wrongly");
                        return 1;
                    }
                }
                if (r + 1 < rounds && !enter(r + 1, w)) { printf("run %d: no slot\n", run); return 1; }
            }
        }
    }
    // as many jobs as there are slots find one each, one more does not
    static SoloTables full;
    for (int j = 0; j < kSoloTable; ++j)
        if (!solo_enter(solo_table(full, 9), solo_word(9, 3 * j, j))) { printf("full table: job %d refused\n", j); return 1; }
    for (int j = 0; j < kSoloTable; ++j)
        if (!solo_wins(solo_table(full, 9), solo_word(9, 3 * j, j))) { printf("full table: job %d lost\n", j); return 1; }
    if (solo_enter(solo_table(full, 9), solo_word(9, 3 * kSoloTable, 1))) { printf("a full table took one more\n"); return 1; }
    printf("claims ok: %ld of %ld won\n", wins, checked);
    return 0;
}
