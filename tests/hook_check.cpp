// The hooks of one shadow word step by step: a load that returns any earlier
// state of the word (a cached copy; also one of an earlier launch, as between
// the phases of a batch), an exchange, and the fold of what the exchange
// replaced, each a step of its own that other threads' steps may come between.
// Some updates apply several accesses at once: the owner's and those of threads
// of other blocks, or of another thread of its wave.  Random threads, waves, blocks, barriers and launches; the
// outcome must be a race exactly when two accesses of a launch race.  8-byte
// words over several launches, 4-byte words over one.  Prints the numbers of
// programs with and without races and of steps that came between; exits 1 at a
// difference.
#include <cstdio>
#include <random>
#include <vector>

#include "hr_fsm.h"

static std::mt19937_64 rng(29);
static uint32_t pick(uint32_t n) { return (uint32_t)(rng() % n); }

struct access {
    uint32_t launch, block, thread, bc, wc, k;
};

static bool races(const access& a, const access& b, uint32_t s)
{
    if (a.launch != b.launch || (a.block == b.block && a.thread == b.thread)) return false;
    if (!hr::conflicts(a.k, b.k)) return false;
    if (a.block != b.block) return true;
    if (a.bc != b.bc) return false;
    return (a.thread >> s) != (b.thread >> s) || a.wc == b.wc;
}

enum { WAVE_BAR = 1, BLOCK_BAR = 2 };
struct item {
    int bar = 0;                 // or an update:
    std::vector<access> acc;
};
struct thread {
    uint32_t block, wave;
    std::vector<item> items;
    size_t pc = 0;
    int step = 0;                // of the update: 0 load, 1 exchange, 2 fold
    uint64_t old = 0, nw = 0, cur = 0, lost = 0;
    bool at_bar(int b) const { return pc < items.size() && items[pc].bar == b; }
};

// One launch of `blocks` blocks with two waves of two threads each; two
// further blocks' accesses, and some of these blocks', are made by owners.
static std::vector<thread> make(uint32_t launch, uint32_t blocks, uint32_t s,
                                std::vector<access>& all)
{
    const uint32_t cls[3] = {hr::CL_R, hr::CL_A, hr::CL_X};
    const uint32_t mostly = cls[pick(3)], odd[3] = {3, 12, 100};
    const uint32_t purity = odd[pick(3)], density = 2 + pick(5);
    std::vector<thread> out;
    const auto kind = [&] { return pick(purity) ? mostly : cls[pick(3)]; };
    for (uint32_t b = 0; b < blocks; ++b) {
        const uint32_t bcs = 1 + pick(3), wcs = 1 + pick(2);
        for (uint32_t w = 0; w < 2; ++w)
            for (uint32_t t = 0; t < 2; ++t) {
                thread th;
                th.block = b;
                th.wave = w;
                const uint32_t id = (w << s) + (t ? (1u << s) - 1 : 0u);
                for (uint32_t bc = 0; bc < bcs; ++bc) {
                    for (uint32_t wc = 0; wc < wcs; ++wc) {
                        for (uint32_t n = pick(density) ? 0 : 1 + pick(2); n-- > 0;) {
                            item u;
                            const uint32_t k = kind();
                            u.acc.push_back({launch, b, id, bc, wc, k});
                            if (pick(8) == 0)      // wave grouping: the wave's other thread
                                u.acc.push_back({launch, b, id ^ ((1u << s) - 1), bc, wc, k});
                            for (uint32_t o = pick(6) ? 0 : 1 + pick(2); o-- > 0;)
                                u.acc.push_back({launch, (b + 1 + pick(blocks + 1)) % (blocks + 2),
                                                 pick(2), bc, wc, k});
                            all.insert(all.end(), u.acc.begin(), u.acc.end());
                            th.items.push_back(u);
                        }
                        if (wc + 1 < wcs) th.items.push_back(item{WAVE_BAR, {}});
                    }
                    if (bc + 1 < bcs) th.items.push_back(item{BLOCK_BAR, {}});
                }
                out.push_back(th);
            }
    }
    return out;
}

static long between = 0;

template <class Step, class Merge, class Id>
struct word_model {
    Step step;
    Merge merge;
    Id id;
    uint64_t word = hr::T_INIT;
    std::vector<uint64_t> seen{(uint64_t)hr::T_INIT};   // every state the word has had
    long records = 0;

    void put(uint64_t w) { seen.push_back(word = w); }

    void run_step(thread& t)
    {
        const std::vector<access>& acc = t.items[t.pc].acc;
        if (t.step == 0) {
            const size_t back = pick(3) ? pick(2) : pick((uint32_t)seen.size());
            t.old = back < seen.size() ? seen[seen.size() - 1 - back] : seen[0];
            t.nw = t.old;
            for (const access& a : acc)
                if (t.nw != hr::T_RACE) t.nw = step(t.nw, id(a), a.k);
            if (t.nw == t.old) ++t.pc;
            else t.step = 1;
        } else if (t.step == 1) {
            t.lost = word;
            put(t.nw);
            if (t.nw == hr::T_RACE) {
                records += t.lost != hr::T_RACE;
                t.step = 0;
                ++t.pc;
            } else if (t.lost != t.old) {
                t.cur = t.nw;
                t.step = 2;
            } else {
                t.step = 0;
                ++t.pc;
            }
        } else {
            const uint64_t m = merge(t.cur, t.lost);
            if (m == t.cur) {
                t.step = 0;
                ++t.pc;
            } else if (word == t.cur) {
                put(m);
                records += m == hr::T_RACE && t.lost != hr::T_RACE;
                t.step = 0;
                ++t.pc;
            } else {
                ++between;
                t.cur = word;
            }
        }
    }

    void run_launch(std::vector<thread> ts)
    {
        for (;;) {
            std::vector<thread*> ready;
            for (thread& t : ts)
                if (t.pc < t.items.size() && !t.items[t.pc].bar) ready.push_back(&t);
            if (!ready.empty()) {
                run_step(*ready[pick((uint32_t)ready.size())]);
                // barriers are passed as soon as they can be, or later
                if (pick(2)) continue;
            }
            bool left = !ready.empty();
            for (thread& t : ts) {
                for (int bar : {WAVE_BAR, BLOCK_BAR}) {
                    if (!t.at_bar(bar)) continue;
                    bool all = true;
                    for (thread& o : ts)
                        if (o.block == t.block && (bar == BLOCK_BAR || o.wave == t.wave))
                            all &= o.at_bar(bar);
                    if (!all) continue;
                    for (thread& o : ts)
                        if (o.block == t.block && (bar == BLOCK_BAR || o.wave == t.wave)) ++o.pc;
                    left = true;
                }
            }
            if (!left) return;
        }
    }
};
template <class Step, class Merge, class Id>
static word_model<Step, Merge, Id> model(Step s, Merge m, Id i)
{
    return {s, m, i};
}

int main()
{
    long with = 0, without = 0;
    for (long i = 0; i < 150000; ++i) {
        const uint32_t s = 1 + pick(5), blocks = 1 + pick(2), launches = 1 + pick(3);
        std::vector<std::vector<thread>> prog;
        std::vector<access> all, one;
        for (uint32_t l = 0; l < launches; ++l) {
            prog.push_back(make(l, blocks, s, all));
            if (l == 0) one = all;
        }
        const auto racy = [&](const std::vector<access>& log) {
            for (size_t x = 0; x < log.size(); ++x)
                for (size_t y = 0; y < x; ++y)
                    if (races(log[x], log[y], s)) return true;
            return false;
        };
        const bool want8 = racy(all), want4 = racy(one);
        const uint64_t wm = hr::g::group_mask(s);
        auto m8 = model([&](uint64_t o, uint64_t d, uint32_t k) { return hr::g::step(o, d, k, wm); },
                        [&](uint64_t x, uint64_t y) { return hr::g::merge(x, y, wm); },
                        [&](const access& a) {
                            return hr::g::pack_id(a.launch, a.block, a.thread, a.bc, a.wc);
                        });
        for (const auto& p : prog) m8.run_launch(p);
        const uint32_t lay = hr::c::layout(1, 2, 8), wm4 = hr::c::group_mask(s, lay);
        auto m4 = model(
            [&](uint64_t o, uint64_t d, uint32_t k) {
                return (uint64_t)hr::c::step((uint32_t)o, (uint32_t)d, k, wm4, lay);
            },
            [&](uint64_t x, uint64_t y) {
                return (uint64_t)hr::c::merge((uint32_t)x, (uint32_t)y, wm, lay);
            },
            [&](const access& a) {
                return (uint64_t)hr::c::pack_id32(a.block, a.thread, a.bc, a.wc, lay);
            });
        m4.run_launch(prog[0]);
        const bool got8 = m8.word == hr::T_RACE, got4 = m4.word == hr::T_RACE;
        if (got8 != want8 || got4 != want4 || (m8.records > 0) != want8 ||
            (m4.records > 0) != want4) {
            printf("program %ld: race %d / %d, 8-byte %d (%ld records), 4-byte %d (%ld)\n", i, want8,
                   want4, got8, m8.records, got4, m4.records);
            for (const access& a : all)
                printf("  launch %u block %u thread %u bc %u wc %u class %u (wave bits %u)\n",
                       a.launch, a.block, a.thread, a.bc, a.wc, a.k, s);
            return 1;
        }
        ++(want8 ? with : without);
    }
    printf("%ld %ld %ld\n", with, without, between);
    return 0;
}
