// Bodies of the instrumented workloads, as device functions of one logical
// block.  The standalone kernels run one logical block per hardware block;
// the job executors run several logical blocks of one job side by side in a
// larger hardware block (each a group of `T` consecutive threads, a multiple
// of the wave size).  `t` is the thread's index in its logical block; a
// thread with t >= T has no logical block and only takes part in the block
// barriers, which every logical block of a hardware block reaches in the
// same order.  CHECK=false compiles the hooks out (plain kernels).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "hr_device.h"

#include "hr_hooks.h"
#include "hr_jacobi.h"

// Tree reduction of in[lb*n .. lb*n+n) (n a power of two, n <= 2T) by T
// threads in LDS: load, then log2(n) halving steps, step s adding
// a[t + (n >> (s+1))] into a[t] for t < n >> (s+1), with a block barrier
// after each step unless s == drop; every thread then writes a[0] to
// out[lb*T + t].  When n < 2T a thread's step-0 operand was loaded by
// another thread, so a barrier also follows the loads.
template <int CHECK, class G = hr_gref>
__device__ void reduce_body(const hr_env& e, const G& gin, const G& gout,
                            const int32_t* __restrict__ in, int32_t* __restrict__ out, uint32_t n,
                            uint32_t T, uint32_t lb, uint32_t t, int32_t drop, int32_t* s,
                            uint32_t* sh, uint32_t lds_id)
{
    const bool act = t < T;
    hr_thread th{};
    if constexpr (CHECK) {
        th = hr_thread_make(e, lb, t);
        if (act)
            for (uint32_t i = t; i < n; i += T) sh[i] = 0;
        __syncthreads();
    }
    const size_t base = (size_t)lb * n;
    const size_t o = (size_t)lb * T + t;
    if (act) {
        // A thread loads at most two input words (n <= 2T), t and t + T.
        // The shadow words of both are loaded together and both exchanges
        // are in flight together: a one-block launch is a chain of round
        // trips, and only this thread touches these words.
        const bool one = t < n, two = t + T < n;
        const typename G::word q0 = one ? hr_gload<CHECK>(th, gin, base + t) : 0;
        const typename G::word q1 = two ? hr_gload<CHECK>(th, gin, base + t + T) : 0;
        const int32_t v0 = one ? in[base + t] : 0;
        const int32_t v1 = two ? in[base + t + T] : 0;
        typename G::pend p0{}, p1{};
        if (one) p0 = hr_gi<0, CHECK, true>(e, th, gin, base + t, HR_SITE_REDUCE_LOAD, q0);
        if (two) p1 = hr_gi<0, CHECK, true>(e, th, gin, base + t + T, HR_SITE_REDUCE_LOAD, q1);
        if (one) {
            hr_l<1, CHECK>(e, th, sh, n, lds_id, t, HR_SITE_REDUCE_STAGE);
            s[t] = v0;
        }
        if (two) {
            hr_l<1, CHECK>(e, th, sh, n, lds_id, t + T, HR_SITE_REDUCE_STAGE);
            s[t + T] = v1;
        }
        hr_gs<0, CHECK>(e, th, gin, p0, base + t, HR_SITE_REDUCE_LOAD);
        hr_gs<0, CHECK>(e, th, gin, p1, base + t + T, HR_SITE_REDUCE_LOAD);
    }
    if (n != 2 * T) hr_bar<CHECK>(e, th);
    const int32_t steps = 31 - __builtin_clz(n);
    for (int32_t step = 0; step < steps; ++step) {
        const uint32_t h = n >> (step + 1);
        if (act && t < h) {
            const int32_t x = s[t];
            const int32_t y = s[t + h];
            s[t] = x + y;
            if constexpr (CHECK)
                hr_lds_rrw<CHECK == 2>(e, th, sh, n, lds_id, t, t + h, HR_SITE_REDUCE_LEFT,
                           HR_SITE_REDUCE_RIGHT, HR_SITE_REDUCE_SUM);
        }
        if (step != drop) hr_bar<CHECK>(e, th);
    }
    if (act) {
        // the output word's shadow load is in flight during the LDS read
        const typename G::word pre_out = hr_gload<CHECK>(th, gout, o);
        const int32_t r = s[0];
        hr_l<0, CHECK>(e, th, sh, n, lds_id, 0, HR_SITE_REDUCE_TOTAL);
        out[o] = r;
        hr_gpre<1, CHECK, false>(e, th, gout, o, HR_SITE_REDUCE_OUT, pre_out);
    }
}

// Label propagation, one logical thread per vertex v (thread v % T of logical
// block v / T): l = atomic load of label[v]; for every edge (v, u) an atomic
// min of l into label[u], or for a seeded edge a plain read and plain write
// of label[u].  grp / gcol: optional monitoring of the CSR reads (shadow null
// when off).  Two physical forms of the same accesses; this one:
//
// The hardware block takes the nv consecutive vertices v0 .. v0+nv, loads
// their labels and row pointers (one lane per vertex), and after a block
// barrier all its lanes walk the vertices' edges, which are consecutive in
// CSR, whichever vertex they belong to.  An edge is checked with the identity
// of its vertex's logical thread (block and thread index, found by a search
// of the row pointers in LDS), so the accesses and their happens-before are
// the program's; the hardware barrier is no barrier of the program.  A
// logical thread's edges then run side by side on several lanes: the job has
// no barrier, so all its accesses lie in one epoch, where the order of one
// thread's updates does not change a summary (step and merge take them as one
// thread's).  An atomic min that would not lower the label is only its atomic
// load (the same access class and the same value): the hubs' labels are hot,
// and memory-side atomics on one line run one after another.
//
// What bounds it: random requests past the L2, a label and a shadow word per
// edge (about 22 G requests/s here), and for small graphs the block that
// holds the largest hub.  R-MAT of 2^22 vertices and 2^25 edges: 3.0 ms per
// checked launch against 45.7 ms with one lane per vertex (a hub's lane walks
// tens of thousands of edges, a round trip each), and 7.0 ms with every
// atomic min performed.  One edge per lane at a time, in 64 registers (two
// 1024-thread blocks per compute unit), was as fast as 2 or 4 edges per lane
// (3.2 and 3.3 ms, with more registers) and as loading the next edge's words
// ahead (3.0 ms, the small graph slower).
template <int CHECK, class G>
__device__ __forceinline__ void labelprop_edges(const hr_env& e, const G& glab, const G& grp,
                                                const G& gcol, int32_t* __restrict__ label,
                                                const int32_t* __restrict__ rp,
                                                const int32_t* __restrict__ col,
                                                const uint8_t* __restrict__ mask, uint32_t n,
                                                uint32_t T, uint32_t v0, uint32_t nv, uint32_t* lds)
{
    int32_t* s_rp = (int32_t*)lds;               // nv + 1 row pointers
    int32_t* s_l = s_rp + nv + 1;                // labels
    uint32_t* s_id = (uint32_t*)(s_l + nv);      // logical block << 10 | thread
    for (uint32_t i = threadIdx.x; i < nv; i += blockDim.x) {
        const uint32_t v = v0 + i, lb = v / T, t = v - lb * T;
        hr_thread th{};
        if constexpr (CHECK) {
            th = hr_thread_make(e, lb, t);
            s_id[i] = lb << 10 | t;
        }
        const typename G::word q = hr_gload<CHECK>(th, glab, v);
        const int32_t l = __hip_atomic_load(label + v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const int32_t r = rp[v];
        if (i + 1 == nv) s_rp[nv] = rp[v + 1];
        const typename G::pend p = hr_gi<2, CHECK, true>(e, th, glab, v, HR_SITE_LP_OWN, q);
        s_l[i] = l;
        s_rp[i] = r;
        hr_gs<2, CHECK>(e, th, glab, p, v, HR_SITE_LP_OWN);
        if (CHECK && grp.shadow) {
            hr_g<0, CHECK>(e, th, grp, v, HR_SITE_LP_CSR);
            hr_g<0, CHECK>(e, th, grp, v + 1, HR_SITE_LP_CSR);
        }
    }
    __syncthreads();
    const int64_t e1 = s_rp[nv];
    for (int64_t k = (int64_t)s_rp[0] + threadIdx.x; k < e1; k += blockDim.x) {
        const uint32_t u = (uint32_t)col[k];
        const bool seeded = mask[k];
        typename G::word w = 0;
        if constexpr (CHECK) w = hr_gload<CHECK>(hr_thread_of(e, 0, 0), gcol, (uint64_t)k);
        // the edge's vertex: the last i with s_rp[i] <= k
        uint32_t lo = 0, hi = nv;
        while (hi - lo > 1) {
            const uint32_t mid = (lo + hi) >> 1;
            if (s_rp[mid] <= k) lo = mid;
            else hi = mid;
        }
        const int32_t l = s_l[lo];
        hr_thread th{};
        if constexpr (CHECK) th = hr_thread_of(e, s_id[lo] >> 10, s_id[lo] & 1023u);
        typename G::word q = 0;
        typename G::pend pu{}, pc{};
        int32_t cur = 0;
        if (u < n) {
            q = hr_gload<CHECK>(th, glab, u);
            cur = __hip_atomic_load(label + u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        if (CHECK && gcol.shadow)
            pc = hr_gi<0, CHECK, true>(e, th, gcol, (uint64_t)k, HR_SITE_LP_CSR, w);
        if (u < n && !seeded) {
            if (cur > l) atomicMin(label + u, l);
            pu = hr_gi<2, CHECK, true>(e, th, glab, u, HR_SITE_LP_MIN, q);
        }
        if (CHECK && gcol.shadow)
            hr_gs<0, CHECK>(e, th, gcol, pc, (uint64_t)k, HR_SITE_LP_CSR);
        hr_gs<2, CHECK>(e, th, glab, pu, u, HR_SITE_LP_MIN);
        if (u < n && seeded) {
            const int32_t r = label[u];
            hr_gpre<0, CHECK, false>(e, th, glab, u, HR_SITE_LP_SEED_READ, q);
            label[u] = r < l ? r : l;
            hr_g<1, CHECK>(e, th, glab, u, HR_SITE_LP_SEED_WRITE);
        }
    }
}

// LDS words labelprop_edges needs for nv vertices.
constexpr uint32_t labelprop_lds_words(uint32_t nv) { return 3 * nv + 1; }

// The other form: one lane per logical thread, vertices lb*T .. lb*T+T, one
// edge at a time.  For contexts with wave grouping, whose hook instructions
// must run one logical wave per hardware wave (hr_group).  While edge k is
// checked, the column index of edge k+2, and the seeded flag of edge k+1 and
// the shadow word of its target, are already in flight.
template <int CHECK, class G = hr_gref>
__device__ void labelprop_body(const hr_env& e, const G& glab, const G& grp, const G& gcol,
                               int32_t* __restrict__ label, const int32_t* __restrict__ rp,
                               const int32_t* __restrict__ col, const uint8_t* __restrict__ mask,
                               uint32_t n, uint32_t T, uint32_t lb, uint32_t t)
{
    const uint32_t v = lb * T + t;
    if (t >= T || v >= n) return;
    hr_thread th{};
    if constexpr (CHECK) th = hr_thread_make(e, lb, t);
    const int32_t l = __hip_atomic_load(label + v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    hr_g<2, CHECK>(e, th, glab, v, HR_SITE_LP_OWN);
    const int32_t e0 = rp[v], e1 = rp[v + 1];
    if (CHECK && grp.shadow) {
        hr_g<0, CHECK>(e, th, grp, v, HR_SITE_LP_CSR);
        hr_g<0, CHECK>(e, th, grp, v + 1, HR_SITE_LP_CSR);
    }
    uint32_t u0 = e0 < e1 ? (uint32_t)col[e0] : 0u;
    uint32_t u1 = e0 + 1 < e1 ? (uint32_t)col[e0 + 1] : 0u;
    typename G::word s0 = e0 < e1 ? hr_gload<CHECK>(th, glab, u0) : 0;
    uint8_t m0 = e0 < e1 ? mask[e0] : 0;
    for (int32_t k = e0; k < e1; ++k) {
        const uint32_t u2 = k + 2 < e1 ? (uint32_t)col[k + 2] : 0u;
        const typename G::word s1 = k + 1 < e1 ? hr_gload<CHECK>(th, glab, u1) : 0;
        const uint8_t m1 = k + 1 < e1 ? mask[k + 1] : 0;
        const uint32_t u = u0;
        const typename G::word su = s0;
        const uint8_t seeded = m0;
        u0 = u1;
        u1 = u2;
        s0 = s1;
        m0 = m1;
        if (CHECK && gcol.shadow) hr_g<0, CHECK>(e, th, gcol, (uint64_t)k, HR_SITE_LP_CSR);
        if (u >= n) continue;
        if (seeded) {
            const int32_t r = label[u];
            hr_gpre<0, CHECK>(e, th, glab, u, HR_SITE_LP_SEED_READ, su);
            label[u] = r < l ? r : l;
            hr_g<1, CHECK, true>(e, th, glab, u, HR_SITE_LP_SEED_WRITE);
        } else {
            atomicMin(label + u, l);
            hr_gpre<2, CHECK>(e, th, glab, u, HR_SITE_LP_MIN, su);
        }
    }
}
