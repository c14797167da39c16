// Hooks whose load returns any earlier state of the word (a cached copy): the
// transition from that state, an exchange, and the fold of what it replaced
// must find a race exactly when two of the accesses race.  One word, random
// blocks, waves, barriers and access kinds, 8-byte and 4-byte words.  Prints
// the number of histories with and without races; exits 1 at a difference.
#include <cstdio>
#include <random>
#include <vector>

#include "hr_fsm.h"

static std::mt19937_64 rng(11);
static uint32_t pick(uint32_t n) { return (uint32_t)(rng() % n); }

struct access {
    uint32_t block, thread, bc, wc, k;
};

static bool races(const access& a, const access& b, uint32_t s)
{
    if (a.block == b.block && a.thread == b.thread) return false;
    if (!hr::conflicts(a.k, b.k)) return false;
    if (a.block != b.block) return true;
    if (a.bc != b.bc) return false;
    return (a.thread >> s) != (b.thread >> s) || a.wc == b.wc;
}

// The accesses of one block in an order its barriers allow.
static std::vector<access> block_history(uint32_t block, uint32_t s)
{
    const uint32_t cls[3] = {hr::CL_R, hr::CL_A, hr::CL_X};
    const uint32_t mostly = cls[pick(3)], odd[3] = {2, 8, 64};
    const uint32_t purity = odd[pick(3)];
    std::vector<access> out;
    for (uint32_t bc = 0; bc < 3; ++bc) {
        std::vector<std::vector<access>> waves(2);
        for (uint32_t w = 0; w < 2; ++w)
            for (uint32_t wc = 0; wc < 2; ++wc)
                for (uint32_t n = pick(3); n-- > 0;)
                    waves[w].push_back({block, (w << s) + pick(2), bc, wc,
                                        pick(purity) ? mostly : cls[pick(3)]});
        size_t at[2] = {0, 0};
        while (at[0] < waves[0].size() || at[1] < waves[1].size()) {
            const uint32_t w = pick(2);
            if (at[w] < waves[w].size()) out.push_back(waves[w][at[w]++]);
        }
    }
    return out;
}

template <class W, class Step, class Merge, class Id>
static bool run(const std::vector<access>& log, Step step, Merge merge, Id id)
{
    std::vector<W> seen{(W)hr::T_INIT};         // every state the word has had
    W word = hr::T_INIT;
    for (const access& a : log) {
        const W old = seen[seen.size() - 1 - pick((uint32_t)seen.size())];
        const W nw = step(old, id(a), a.k);
        if (nw == old) continue;
        const W r = word;
        word = nw;
        seen.push_back(word);
        if (nw != hr::T_RACE && r != old) {
            const W m = merge(word, r);
            if (m != word) seen.push_back(word = m);
        }
    }
    return word == (W)hr::T_RACE;
}

int main()
{
    long with = 0, without = 0;
    for (long i = 0; i < 600000; ++i) {
        const uint32_t s = 1 + pick(6), blocks = 1 + pick(3);
        std::vector<std::vector<access>> hist;
        for (uint32_t b = 0; b < blocks; ++b) hist.push_back(block_history(b, s));
        std::vector<access> log;
        std::vector<size_t> at(blocks, 0);
        for (size_t left = 1; left;) {
            left = 0;
            const uint32_t b = pick(blocks);
            if (at[b] < hist[b].size()) log.push_back(hist[b][at[b]++]);
            for (uint32_t c = 0; c < blocks; ++c) left += hist[c].size() - at[c];
        }
        bool want = false;
        for (size_t x = 0; x < log.size(); ++x)
            for (size_t y = 0; y < x; ++y) want |= races(log[x], log[y], s);
        const uint64_t wm = hr::g::group_mask(s);
        const bool got8 = run<uint64_t>(
            log, [&](uint64_t o, uint64_t d, uint32_t k) { return hr::g::step(o, d, k, wm); },
            [&](uint64_t x, uint64_t y) { return hr::g::merge(x, y, wm); },
            [&](const access& a) { return hr::g::pack_id(1, a.block, a.thread, a.bc, a.wc); });
        const uint32_t lay = hr::c::layout(1, 2, 8), wm4 = hr::c::group_mask(s, lay);
        const bool got4 = run<uint32_t>(
            log, [&](uint32_t o, uint32_t d, uint32_t k) { return hr::c::step(o, d, k, wm4, lay); },
            [&](uint32_t x, uint32_t y) { return hr::c::merge(x, y, wm, lay); },
            [&](const access& a) { return hr::c::pack_id32(a.block, a.thread, a.bc, a.wc, lay); });
        if (got8 != want || got4 != want) {
            printf("history %ld: race %d, 8-byte %d, 4-byte %d\n", i, want, got8, got4);
            for (const access& a : log)
                printf("  block %u thread %u bc %u wc %u class %u\n", a.block, a.thread, a.bc, a.wc,
                       a.k);
            return 1;
        }
        ++(want ? with : without);
    }
    printf("%ld %ld\n", with, without);
    return 0;
}
