// The closed forms of the owner updates (hr::g::fresh, hr::c::fresh,
// hr::l::fresh) against the transitions they stand for, one access after
// another, over random words reached by random accesses.  Prints the number
// of compared cases; exits 1 at the first difference.
#include <cstdio>
#include <random>

#include "hr_fsm.h"

static std::mt19937_64 rng(7);
static uint32_t pick(uint32_t n) { return (uint32_t)(rng() % n); }

int main()
{
    const uint32_t cls[3] = {hr::CL_R, hr::CL_A, hr::CL_X};
    long taken[3] = {0, 0, 0};
    for (long i = 0; i < 4000000; ++i) {
        const uint32_t s = 1 + pick(6);
        // identities close together, so that every relation comes up
        const auto id = [&](uint32_t launch, uint32_t block) {
            return hr::g::pack_id(launch, block, pick(4) * 16 + pick(70), pick(3), pick(2));
        };
        {
            const uint64_t wm = hr::g::group_mask(s);
            uint64_t w = pick(8) == 0 ? hr::T_RACE : 0;
            for (uint32_t n = pick(4); n-- > 0;) w = hr::g::step(w, id(pick(2), pick(3)), cls[pick(3)], wm);
            const uint32_t k = cls[pick(3)], others = pick(3), launch = pick(2);
            const uint64_t me = id(launch, 4);
            uint64_t want = hr::g::step(w, me, k, wm), got;
            for (uint32_t n = 0; n < others; ++n) want = hr::g::step(want, id(launch, 5 + n), k, wm);
            if (hr::g::fresh(w, me, k, others != 0, &got)) {
                ++taken[0];
                if (got != want) return printf("g %lx %lx %lx\n", w, got, want), 1;
            } else if ((w & hr::g::TAG_M) == hr::T_INIT && !(others && k == hr::CL_X)) {
                return printf("g refused %lx\n", w), 1;
            }
        }
        {
            const uint32_t lay = hr::c::layout(1 + pick(2), 2 + pick(2), 7 + pick(4));
            const uint32_t wm = hr::c::group_mask(s, lay);
            const auto cid = [&](uint32_t block) {
                return hr::c::pack_id32(block, pick(120), pick(3), pick(2), lay);
            };
            uint32_t w = pick(8) == 0 ? hr::T_RACE : 0;
            for (uint32_t n = pick(3); n-- > 0;) w = hr::c::step(w, cid(pick(3)), cls[pick(3)], wm, lay);
            const uint32_t k = cls[pick(3)], others = pick(3);
            const uint32_t me = cid(4);
            uint32_t want = hr::c::step(w, me, k, wm, lay), got;
            for (uint32_t n = 0; n < others; ++n) want = hr::c::step(want, cid(5 + n), k, wm, lay);
            if (hr::c::fresh(w, me, k, others != 0, &got)) {
                ++taken[1];
                if (got != want) return printf("c %x %x %x\n", w, got, want), 1;
            } else if (w == 0 && !(others && k == hr::CL_X)) {
                return printf("c refused %x\n", w), 1;
            }
        }
        {
            const uint32_t wm = hr::l::group_mask(s);
            uint32_t w = pick(8) == 0 ? hr::T_RACE : 0;
            for (uint32_t n = pick(4); n-- > 0;)
                w = hr::l::step(w, hr::l::pack_id(pick(256), pick(3), pick(2)), cls[pick(3)], wm);
            const uint32_t k = cls[pick(3)], t = pick(256), bc = pick(4), wc = pick(2);
            const uint32_t me = hr::l::pack_id(t, bc, wc);
            uint32_t want = hr::l::step(w, me, k, wm), got, others = 0;
            for (uint32_t n = pick(4); n-- > 0;) {
                const uint32_t u = (t & ~31u) + pick(64);
                const uint32_t o = hr::l::pack_id(u, bc, wc);
                if (u == t) continue;
                want = hr::l::step(want, o, k, wm);
                const uint32_t kind = ((o ^ me) & wm) ? 2u : 1u;
                if (kind > others) others = kind;
            }
            if (hr::l::fresh(w, me, k, others, wm, &got)) {
                ++taken[2];
                if (got != want) return printf("l %x %x %x\n", w, got, want), 1;
            } else if (w == 0 && !(others && k == hr::CL_X)) {
                return printf("l refused %x\n", w), 1;
            }
        }
    }
    printf("%ld %ld %ld\n", taken[0], taken[1], taken[2]);
    return 0;
}
