// Hook call sites of the workload bodies: each wrapper calls the device hook
// when CHECK is set and compiles to nothing in the plain kernels (CHECK 0).
// CHECK 1 is the checking kernel; CHECK 2 the same with the debug access
// log compiled in (hr_count<LOG>), for contexts made with an access log.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "hr_device.h"

// An element of a global region as a hook takes it: its index (checked
// against the region's length and reported) and the offset of its shadow
// word (the region's address-to-shadow map applied to the index).
struct hr_el {
    uint64_t index, off;
};

// A global region as the hooks see it: its shadow, length, report id and
// address-to-shadow map; hr_gref4 for a context with 4-byte words.  Bodies
// written over a region type G use G::word for a pre-loaded shadow word and
// G::pend for a split hook in flight, and name elements either by index
// (at) or, in a 2-D array, by row and column (at2, no division).
struct hr_gref {
    uint64_t* shadow;
    uint64_t n;
    uint32_t id;
    hr_lay lay;
    using word = uint64_t;
    using pend = hr_pend;
    static constexpr bool TABLE = false;   // transitions by the bit logic
    __device__ __forceinline__ const uint16_t* table() const { return nullptr; }
    __device__ __forceinline__ hr_el at(uint64_t index) const { return {index, hr_lay_off(lay, index)}; }
    __device__ __forceinline__ hr_el at2(uint32_t r, uint32_t c, uint64_t index) const
    {
        return {index, hr_lay_off2(lay, r, c)};
    }
};

// An 8-byte-word region whose hooks take their transitions from the flat
// table of the machine (hr::g::step_tab) at `tab`.
struct hr_gref_tab : hr_gref {
    const uint16_t* tab;
    static constexpr bool TABLE = true;
    __device__ __forceinline__ const uint16_t* table() const { return tab; }
};

// Overloads for the 8-byte-word region types (hr_gref and types built on it).
template <class G>
using hr_if8 = std::enable_if_t<std::is_base_of<hr_gref, G>::value, int>;

// LAY: the 4-byte word layout as a compile-time constant (0: the context's).
template <uint32_t LAY>
struct hr_gref4t {
    uint32_t* shadow;
    uint64_t n;
    uint32_t id;
    hr_lay lay;
    using word = uint32_t;
    using pend = hr_pend4;
    __device__ __forceinline__ hr_el at(uint64_t index) const { return {index, hr_lay_off(lay, index)}; }
    __device__ __forceinline__ hr_el at2(uint32_t r, uint32_t c, uint64_t index) const
    {
        return {index, hr_lay_off2(lay, r, c)};
    }
};
using hr_gref4 = hr_gref4t<0>;

// The row-major map of a region `cols` elements wide (or of a 1-D region).
__host__ __device__ __forceinline__ hr_lay hr_lay_rows(uint32_t cols)
{
    return hr_lay{cols, cols, 0u, 0u};
}

// Global hook at a lane-affine site (GROUP false) or a data-dependent one.
// Every global wrapper takes the element as an hr_el, or as an index (then
// the region's map gives the shadow offset).
template <int KIND, int CHECK, bool GROUP = false, class G, hr_if8<G> = 0>
__device__ __forceinline__ void hr_g(const hr_env& e, const hr_thread& t, const G& g, hr_el x,
                                     uint32_t site)
{
    if constexpr (CHECK)
        hr_check<KIND, GROUP, false, CHECK == 2, G::TABLE>(e, t, g.shadow, g.n, g.id, x.index,
                                                           x.off, site, 0, g.table());
}

// Global hook on a word loaded earlier by hr_gload.
template <int CHECK, class G, hr_if8<G> = 0>
__device__ __forceinline__ uint64_t hr_gload(const hr_thread& t, const G& g, hr_el x)
{
    if constexpr (CHECK) return hr_check_load(t, g.shadow, g.n, x.index, x.off);
    return 0;
}

template <int KIND, int CHECK, bool GROUP = true, class G, hr_if8<G> = 0>
__device__ __forceinline__ void hr_gpre(const hr_env& e, const hr_thread& t, const G& g, hr_el x,
                                        uint32_t site, uint64_t pre)
{
    if constexpr (CHECK)
        hr_check<KIND, GROUP, true, CHECK == 2, G::TABLE>(e, t, g.shadow, g.n, g.id, x.index,
                                                          x.off, site, pre, g.table());
}

// The two halves of a global hook at a lane-affine site (hr_check_issue /
// hr_check_settle; both take the call site); `pre` as for hr_gpre when PRE.
template <int KIND, int CHECK, bool PRE = false, class G, hr_if8<G> = 0>
__device__ __forceinline__ hr_pend hr_gi(const hr_env& e, const hr_thread& t, const G& g, hr_el x,
                                         uint32_t site, uint64_t pre = 0)
{
    if constexpr (CHECK)
        return hr_check_issue<KIND, PRE, CHECK == 2, G::TABLE>(e, t, g.shadow, g.n, g.id, x.index,
                                                               x.off, site, pre, g.table());
    return hr_pend{nullptr, 0, 0, 0};
}

template <int KIND, int CHECK, class G, hr_if8<G> = 0>
__device__ __forceinline__ void hr_gs(const hr_env& e, const hr_thread& t, const G& g,
                                      const hr_pend& p, uint64_t index, uint32_t site)
{
    if constexpr (CHECK) hr_check_settle<KIND>(e, t, p, g.id, index, site);
}

template <int KIND, int CHECK>
__device__ __forceinline__ void hr_l(const hr_env& e, const hr_thread& t, uint32_t* sh,
                                     uint32_t n, uint32_t id, uint32_t index, uint32_t site)
{
    if constexpr (CHECK) hr_access_lds<KIND, CHECK == 2>(e, t, sh, n, id, index, site);
}

template <int CHECK>
__device__ __forceinline__ void hr_bar(const hr_env& e, hr_thread& t)
{
    if constexpr (CHECK) hr_barrier_block(e, t);
    else __syncthreads();
}

// The global hooks on 4-byte words.
template <int KIND, int CHECK, bool GROUP = false, uint32_t LAY = 0>
__device__ __forceinline__ void hr_g(const hr_env& e, const hr_thread& t, const hr_gref4t<LAY>& g,
                                     hr_el x, uint32_t site)
{
    if constexpr (CHECK)
        hr_check4<KIND, GROUP, false, LAY, CHECK == 2>(e, t, g.shadow, g.n, g.id, x.index, x.off, site);
}

template <int CHECK, uint32_t LAY = 0>
__device__ __forceinline__ uint32_t hr_gload(const hr_thread& t, const hr_gref4t<LAY>& g, hr_el x)
{
    if constexpr (CHECK) return hr_check4_load(t, g.shadow, g.n, x.index, x.off);
    return 0;
}

template <int KIND, int CHECK, bool GROUP = true, uint32_t LAY = 0>
__device__ __forceinline__ void hr_gpre(const hr_env& e, const hr_thread& t,
                                        const hr_gref4t<LAY>& g, hr_el x, uint32_t site,
                                        uint32_t pre)
{
    if constexpr (CHECK)
        hr_check4<KIND, GROUP, true, LAY, CHECK == 2>(e, t, g.shadow, g.n, g.id, x.index, x.off, site, pre);
}

template <int KIND, int CHECK, bool PRE = false, uint32_t LAY = 0>
__device__ __forceinline__ hr_pend4 hr_gi(const hr_env& e, const hr_thread& t,
                                          const hr_gref4t<LAY>& g, hr_el x, uint32_t site,
                                          uint32_t pre = 0)
{
    if constexpr (CHECK)
        return hr_check4_issue<KIND, PRE, LAY, CHECK == 2>(e, t, g.shadow, g.n, g.id, x.index, x.off, site,
                                               pre);
    return hr_pend4{nullptr, 0, 0, 0};
}

template <int KIND, int CHECK, uint32_t LAY = 0>
__device__ __forceinline__ void hr_gs(const hr_env& e, const hr_thread& t, const hr_gref4t<LAY>& g,
                                      const hr_pend4& p, uint64_t index, uint32_t site)
{
    if constexpr (CHECK) hr_check4_settle<KIND>(e, t, p, g.id, index, site);
}

// The wrappers taking an element index: G is the region's own type, so a
// region type with a compile-time map (hr_map) turns the index into its
// shadow offset without the run-time map's division.
template <int KIND, int CHECK, bool GROUP = false, class G>
__device__ __forceinline__ void hr_g(const hr_env& e, const hr_thread& t, const G& g,
                                     uint64_t index, uint32_t site)
{
    if constexpr (CHECK) hr_g<KIND, CHECK, GROUP>(e, t, g, g.at(index), site);
}

template <int CHECK, class G>
__device__ __forceinline__ typename G::word hr_gload(const hr_thread& t, const G& g,
                                                     uint64_t index)
{
    if constexpr (CHECK) return hr_gload<CHECK>(t, g, g.at(index));
    return 0;
}

template <int KIND, int CHECK, bool GROUP = true, class G>
__device__ __forceinline__ void hr_gpre(const hr_env& e, const hr_thread& t, const G& g,
                                        uint64_t index, uint32_t site, typename G::word pre)
{
    if constexpr (CHECK) hr_gpre<KIND, CHECK, GROUP>(e, t, g, g.at(index), site, pre);
}

template <int KIND, int CHECK, bool PRE = false, class G>
__device__ __forceinline__ typename G::pend hr_gi(const hr_env& e, const hr_thread& t, const G& g,
                                                  uint64_t index, uint32_t site,
                                                  typename G::word pre = 0)
{
    if constexpr (CHECK) return hr_gi<KIND, CHECK, PRE>(e, t, g, g.at(index), site, pre);
    return typename G::pend{nullptr, 0, 0, 0};
}

// A region type whose map is fixed at compile time: TW = TH = 0 is the
// row-major map (the shadow offset is the element index itself; 1-D
// regions), TW, TH > 0 tiles of 2^TW x 2^TH elements with constant shifts,
// and TW < 0 the region's own map at run time.  Base: hr_gref or
// hr_gref4t<LAY>.
template <class Base, int TW, int TH>
struct hr_map : Base {
    __device__ __forceinline__ hr_el at(uint64_t index) const
    {
        if constexpr (TW == 0 && TH == 0) return {index, index};
        else return Base::at(index);
    }
    __device__ __forceinline__ hr_el at2(uint32_t r, uint32_t c, uint64_t index) const
    {
        if constexpr (TW < 0) {
            return Base::at2(r, c, index);
        } else if constexpr (TW == 0 && TH == 0) {
            return {index, index};
        } else {
            const uint64_t tile = (uint64_t)(r >> TH) * this->lay.tiles_x + (c >> TW);
            return {index, (tile << (TW + TH)) | ((uint64_t)(r & ((1u << TH) - 1u)) << TW) |
                               (uint64_t)(c & ((1u << TW) - 1u))};
        }
    }
};
template <int TW, int TH>
using hr_gref_map = hr_map<hr_gref, TW, TH>;
// 1-D regions under the identity map
using hr_gref_1d = hr_map<hr_gref, 0, 0>;
template <uint32_t LAY>
using hr_gref4_1d = hr_map<hr_gref4t<LAY>, 0, 0>;

// ---------------------------------------------------------------------------
// Owner updates.  Where a kernel's code fixes which threads access an element
// between two barriers (a stencil's halo), the accesses need not each be
// published on their own: one thread, the element's owner, applies all of
// them to its word, one transition each, and publishes once.  The accesses,
// their identities and the resulting summary are the ones the separate hooks
// would leave in that order; what goes is the traffic between the accessors.
// With every access to a word applied by one thread, the publishing needs no
// read-modify-write either, as long as no other kernel of the launch epoch
// runs beside this one (env.excl, decided by the host): a coherent store
// takes the exchange's place.  Without env.excl the update is the exchange
// and fold of hr_check.
// ---------------------------------------------------------------------------

// One access as an owner update takes it.
struct hr_by {
    uint32_t on;                  // 0: no such access
    uint32_t block, thread, site;
};

// The word operations of a region type: 8-byte words.
template <class G, hr_if8<G> = 0>
__device__ __forceinline__ uint64_t hr_own_id(const hr_env& e, const G&, uint32_t block,
                                              uint32_t thread, uint32_t bc, uint32_t wc)
{
    return hr::g::pack_id(e.launch, block, thread, bc, wc);
}
template <class G, hr_if8<G> = 0>
__device__ __forceinline__ uint64_t hr_own_step(const hr_env& e, const G& g, uint64_t old,
                                                uint64_t id, uint32_t k)
{
    return hr_step8<G::TABLE>(g.table(), old, id, k, hr::g::group_mask(e.wave_bits));
}
template <class G, hr_if8<G> = 0>
__device__ __forceinline__ uint64_t hr_own_widen(const hr_env&, const G&, uint64_t w)
{
    return w;
}
template <class G, hr_if8<G> = 0>
__device__ __forceinline__ uint64_t hr_own_fold(const hr_env& e, const G&, uint64_t* sp,
                                                uint64_t mine, uint64_t lost)
{
    return hr_fold(sp, mine, lost, hr::g::group_mask(e.wave_bits));
}

// ... and 4-byte words.
template <uint32_t LAY>
__device__ __forceinline__ uint32_t hr_own_id(const hr_env& e, const hr_gref4t<LAY>&,
                                              uint32_t block, uint32_t thread, uint32_t bc,
                                              uint32_t wc)
{
    return hr::c::pack_id32(block, thread, bc, wc, LAY ? LAY : e.word4);
}
template <uint32_t LAY>
__device__ __forceinline__ uint32_t hr_own_step(const hr_env& e, const hr_gref4t<LAY>&,
                                                uint32_t old, uint32_t id, uint32_t k)
{
    const uint32_t lay = LAY ? LAY : e.word4;
    return hr::c::step(old, id, k, hr::c::group_mask(e.wave_bits, lay), lay);
}
template <uint32_t LAY>
__device__ __forceinline__ uint64_t hr_own_widen(const hr_env& e, const hr_gref4t<LAY>&,
                                                 uint32_t w)
{
    return hr::c::widen(w, LAY ? LAY : e.word4);
}
template <uint32_t LAY>
__device__ __forceinline__ uint64_t hr_own_fold(const hr_env& e, const hr_gref4t<LAY>&,
                                                uint32_t* sp, uint32_t mine, uint32_t lost)
{
    const uint32_t b = hr_fold4(sp, mine, lost, hr::g::group_mask(e.wave_bits),
                                LAY ? LAY : e.word4);
    return b == HR_NO_REPORT4 ? HR_NO_REPORT : (uint64_t)b;
}

// The fresh case of an owner update, in closed form: the word `old` holds no
// access of this launch (and no race), so the owner's access makes it the
// owner's alone, or together with accesses of the same class by other blocks
// the several-blocks state.  False: another case (or a write with others);
// the update is hr_own's.  In a context with the flat table the transitions
// come from it, and every case without a race is taken.
template <int KIND, class G, hr_if8<G> = 0>
__device__ __forceinline__ bool hr_own_fresh(const hr_env& e, const hr_thread& t, const G& g,
                                             uint64_t old, const hr_by& b, const hr_by& c,
                                             uint64_t* nw)
{
    constexpr uint32_t k = KIND == 0 ? hr::CL_R : (KIND == 2 ? hr::CL_A : hr::CL_X);
    const uint64_t id = hr_own_id(e, g, t.block, t.thread, t.bc, t.wc);
    if constexpr (G::TABLE) {
        uint64_t w = hr_own_step(e, g, old, id, k);
        if (b.on) w = hr_own_step(e, g, w, hr_own_id(e, g, b.block, b.thread, t.bc, t.wc), k);
        if (c.on) w = hr_own_step(e, g, w, hr_own_id(e, g, c.block, c.thread, t.bc, t.wc), k);
        *nw = w;
        return w != hr::T_RACE;
    } else {
        return hr::g::fresh(old, id, k, b.on || c.on, nw);
    }
}
template <int KIND, uint32_t LAY>
__device__ __forceinline__ bool hr_own_fresh(const hr_env& e, const hr_thread& t,
                                             const hr_gref4t<LAY>& g, uint32_t old, const hr_by& b,
                                             const hr_by& c, uint32_t* nw)
{
    // other blocks must not look like the owner's (4-byte words fold ids)
    const uint32_t bm = hr::c::block_mask(LAY ? LAY : e.word4);
    if ((b.on && !((b.block ^ t.block) & bm)) || (c.on && !((c.block ^ t.block) & bm)))
        return false;
    return hr::c::fresh(old, hr_own_id(e, g, t.block, t.thread, t.bc, t.wc),
                        KIND == 0 ? hr::CL_R : (KIND == 2 ? hr::CL_A : hr::CL_X), b.on || c.on, nw);
}

// The fast half of an owner update, for a word loaded as `old` since the
// thread's last barrier: publishes it in the fresh case of an exclusive
// launch and returns true, else returns false with nothing done (hr_own is
// then due).  A store, no call: the rare rest of the update (races, words
// with accesses of this launch, shared launches) can follow at the kernel's
// end, where little is live, since no other thread updates the word.
template <int KIND, class G>
__device__ __forceinline__ bool hr_own_fast(const hr_env& e, const hr_thread& t, const G& g,
                                            hr_el x, typename G::word old, const hr_by& b,
                                            const hr_by& c)
{
    typename G::word nw;
    const bool ok = hr_own_fresh<KIND>(e, t, g, old, b, c, &nw);
    if (!g.shadow) return true;
    if (!e.excl) return false;
    const bool done = ok & (t.enabled == 1);
    if (done) __hip_atomic_store(g.shadow + x.off, nw, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return done;
}

// The owner update of element x: the owner's own access, then b and c, all
// of kind KIND and at the owner's clocks.  The accesses are counted by their
// own threads (hr_note).
template <int KIND, class G>
__device__ __forceinline__ void hr_own(const hr_env& e, const hr_thread& t, const G& g, hr_el x,
                                       uint32_t site, const hr_by& b, const hr_by& c)
{
    using W = typename G::word;
    constexpr uint32_t k = KIND == 0 ? hr::CL_R : (KIND == 2 ? hr::CL_A : hr::CL_X);
    if (t.enabled != 1 || !g.shadow) return;
    W* sp = g.shadow + x.off;
    const W old = __hip_atomic_load(sp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // the last transition made, and the access that made it: a race state is
    // never left, so that access completes the race if there is one
    hr_by by{1, t.block, t.thread, site};
    W before = old, id = hr_own_id(e, g, t.block, t.thread, t.bc, t.wc);
    W nw = hr_own_step(e, g, old, id, k);
    for (uint32_t i = 0; i < 2 && nw != hr::T_RACE; ++i) {
        const hr_by& next = i == 0 ? b : c;
        if (!next.on) continue;
        by = next;
        before = nw;
        id = hr_own_id(e, g, by.block, by.thread, t.bc, t.wc);
        nw = hr_own_step(e, g, nw, id, k);
    }
    if (nw == old) return;
    W r = old;
    if (e.excl) __hip_atomic_store(sp, nw, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else r = __hip_atomic_exchange(sp, nw, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    uint64_t was = HR_NO_REPORT, with = 0;
    uint32_t flags = 0;
    if (nw == hr::T_RACE) {
        if (r == hr::T_RACE) return;
        was = hr_own_widen(e, g, before);
        with = hr_own_widen(e, g, hr_own_step(e, g, (W)hr::T_INIT, id, k));
    } else if (r != old) {
        const uint64_t f = hr_own_fold(e, g, sp, nw, r);
        if (f == HR_NO_REPORT) return;
        was = hr_own_widen(e, g, (W)f);
        with = hr_own_widen(e, g, r);
        flags = HR_RACE_FOLD;
        by = hr_by{1, t.block, t.thread, site};
    } else {
        return;
    }
    hr_ring_push(e, 0, g.id, by.block, x.index, by.thread, KIND, by.site, was, with, flags);
}

// The same in LDS: the owner's access of word `index`, then that of thread
// `other` of its block (HR_NO_THREAD: none), both of kind KIND and at the
// owner's clocks.  Of several other threads that make the same access in
// that epoch, one stands for all: one of another synchronization group if
// there is one (after two accessors of different groups, or of one group,
// a further one of theirs does not change the word).
#define HR_NO_THREAD (~0u)
template <int KIND>
__device__ __forceinline__ void hr_own_lds(const hr_env& e, const hr_thread& t, uint32_t* sh,
                                           uint32_t array_id, uint32_t index, uint32_t site,
                                           uint32_t other = HR_NO_THREAD)
{
    constexpr uint32_t k = KIND == 0 ? hr::CL_R : (KIND == 2 ? hr::CL_A : hr::CL_X);
    if (t.enabled != 1) return;
    const uint32_t wm = hr::l::group_mask(e.wave_bits);
    const uint32_t old = sh[index];
    uint32_t before = old, by = t.thread, id = t.lid;
    uint32_t nw = hr::l::step(old, id, k, wm);
    if (other != HR_NO_THREAD && nw != hr::T_RACE) {
        before = nw;
        by = other;
        id = hr::l::pack_id(other, t.bc, t.wc);
        nw = hr::l::step(nw, id, k, wm);
    }
    if (nw == old) return;
    sh[index] = nw;
    if (nw == hr::T_RACE)
        hr_ring_push(e, 1, array_id, t.block, index, by, KIND, site, before,
                     hr::l::step(hr::T_INIT, id, k), 0);
}

// Its fast half: a word without an access of this block epoch, in closed
// form (hr::l::fresh).  others: 0 none, 1 other threads of the owner's
// group, 2 threads of other groups (too).
template <int KIND>
__device__ __forceinline__ bool hr_own_lds_fast(const hr_env& e, const hr_thread& t, uint32_t* sh,
                                                uint32_t index, uint32_t others)
{
    uint32_t nw;
    if (t.enabled != 1 ||
        !hr::l::fresh(sh[index], t.lid, KIND == 0 ? hr::CL_R : (KIND == 2 ? hr::CL_A : hr::CL_X),
                      others, hr::l::group_mask(e.wave_bits), &nw))
        return false;
    sh[index] = nw;
    return true;
}

// Count (and with CHECK 2 log) an access that an owner update applies.
template <int KIND, int CHECK, class G>
__device__ __forceinline__ void hr_note(const hr_env& e, const hr_thread& t, const G& g,
                                        uint64_t index, uint32_t site)
{
    if (t.enabled == 1 && g.shadow) hr_count<CHECK == 2>(e, t, 0, g.id, index, KIND, site);
}
template <int KIND, int CHECK>
__device__ __forceinline__ void hr_note_lds(const hr_env& e, const hr_thread& t, uint32_t id,
                                            uint32_t index, uint32_t site)
{
    if (t.enabled == 1) hr_count<CHECK == 2>(e, t, 1, id, index, KIND, site);
}
