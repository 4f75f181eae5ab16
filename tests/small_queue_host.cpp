// Host model of the queue of a launch that holds whole sweeps (update_small_kernel):
// blocks of one XCD take (slice, group) items in order; each loads its link when it
// has the ticket, waits for all slices before, takes its next ticket once its
// staples are read and only then ends its update.  A random scheduler, with slow
// blocks among fast ones, lets every step that may happen happen in any order.
// Prints, per number of blocks, the links loaded before the same slice of the
// sweep before had written them, and the items left undone: with small_team's
// rule, and with all blocks let in.
#include <cstdint>
#include <cstdio>
#include <vector>

#include "layout.h"

static uint64_t g_state = 88172645463325252ull;
static uint32_t rnd(uint32_t n)
{
    g_state ^= g_state << 13; g_state ^= g_state >> 7; g_state ^= g_state << 17;  // xorshift64
    return uint32_t((g_state >> 11) % n);
}

struct Block {
    enum { kNew, kTicket, kLoaded, kRead, kGone } at = kNew;  // of the current item
    uint32_t item = 0, next = 0, weight = 1;
    bool has_next = false;
};

static void run(int D, uint32_t groups, uint32_t nblocks, uint32_t sweeps, bool rule, uint64_t &stale, uint64_t &undone)
{
    const uint32_t items = 2u * uint32_t(D) * sweeps * groups;
    const uint32_t stride = 8u * groups / nblocks;
    std::vector<uint32_t> done(groups, 0);
    std::vector<Block> b(nblocks);
    for (auto &x : b) x.weight = rnd(3) == 0 ? 1u : 60u;
    uint32_t ticket = 0, working = 0, left = nblocks;
    auto ready = [&](uint32_t n) {
        for (uint32_t d : done)
            if (d < n) return false;
        return true;
    };
    while (left) {
        const uint32_t i = rnd(nblocks);
        Block &x = b[i];
        if (x.at == Block::kGone || rnd(60) >= x.weight) continue;
        const uint32_t n = x.item / groups, g = x.item % groups;
        switch (x.at) {
        case Block::kNew: {
            // all on XCD 0; fewer blocks than 8 per group stand for as many XCDs
            const uint32_t team = su3hb::small_team(0, i * stride);
            if (working == 0) working = team;
            if (rule && working != team) {
                x.at = Block::kGone;
                --left;
                break;
            }
            x.item = ticket++;
            x.at = Block::kTicket;
            break;
        }
        case Block::kTicket:
            if (x.item >= items) {
                x.at = Block::kGone;
                --left;
                break;
            }
            // slice n - 2 D has written the link when done[g] > n - 2 D
            if (n >= 2u * uint32_t(D) && done[g] + 2u * uint32_t(D) <= n) ++stale;
            x.at = Block::kLoaded;
            break;
        case Block::kLoaded:
            if (ready(n)) x.at = Block::kRead;
            break;
        case Block::kRead:
            // the next ticket is wave 3's, the end of the update wave 0's: any order
            if (!x.has_next && rnd(2)) {
                x.next = ticket++;
                x.has_next = true;
            } else if (x.has_next) {
                done[g] = n + 1u;
                x.item = x.next;
                x.has_next = false;
                x.at = Block::kTicket;
            }
            break;
        default: break;
        }
    }
    for (uint32_t d : done)
        if (d != 2u * uint32_t(D) * sweeps) ++undone;
}

int main()
{
    for (int D : {2, 3, 4})
        for (uint32_t groups : {1u, 2u, 5u, 15u})
            for (uint32_t per : {1u, 4u, 8u}) {
                uint64_t stale[2] = {0, 0}, undone[2] = {0, 0};
                for (int k = 0; k < 60; ++k)
                    for (int rule = 0; rule < 2; ++rule) run(D, groups, per * groups, 3, rule != 0, stale[rule], undone[rule]);
                std::printf("D=%d groups=%u blocks=%u stale %llu undone %llu all let in: stale %llu undone %llu\n", D, groups,
                            per * groups, (unsigned long long)stale[1], (unsigned long long)undone[1],
                            (unsigned long long)stale[0], (unsigned long long)undone[0]);
            }
    return 0;
}
