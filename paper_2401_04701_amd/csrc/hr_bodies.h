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
__device__ __forceinline__ void reduce_body(const hr_env& e, const G& gin, const G& gout,
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
// A hardware block takes consecutive vertices and consecutive edges, loads
// the vertices' labels and row pointers (one lane per vertex), and after a
// block barrier all its lanes walk the edges, whichever vertex they belong
// to.  An edge is checked with the identity of its vertex's logical thread
// (block and thread index, found by a search of the row pointers in LDS), so
// the accesses and their happens-before are the program's; the hardware
// barrier is no barrier of the program.  A logical thread's edges then run
// side by side on several lanes: the job has no barrier, so all its accesses
// lie in one epoch, where the order of one thread's updates does not change a
// summary (step and merge take them as one thread's).  An atomic min that
// would not lower the label is only its atomic load (the same access class
// and the same value): the hubs' labels are hot, and memory-side atomics on
// one line run one after another.
//
// The blocks' shares are equal (lp_part): vertices and edges are put in one
// order, each vertex before its edges, and cut into pieces of one length, so
// a hub's edges spread over several blocks.  Its thread loads its label once,
// so those blocks take the value that was read where the pieces were cut.
// Cut by vertices instead, the block of the largest hubs bounded every
// launch: on R-MAT graphs of 50 K to 250 K vertices it holds 80 K to 180 K
// edges, 6 us a round of 1024.

// A seeded edge's plain read and write of a label.  COH: past the caches, for
// a batch's workers, which run several sweeps with only a counter between
// them.  (Elsewhere the caches take the write: 2^25 edges, 1 % seeded, 0.73 ms
// per launch against 1.28 past them.)
template <bool COH>
__device__ __forceinline__ int32_t lp_get(const int32_t* p)
{
    if constexpr (COH) return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else return *p;
}
template <bool COH>
__device__ __forceinline__ void lp_set(int32_t* p, int32_t v)
{
    if constexpr (COH) __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else *p = v;
}

// Where piece i of a job begins: its first vertex v, its first edge
// row_ptr[0] + i * length - v, and, when that edge belongs to vertex v - 1,
// that vertex's label.
struct lp_part {
    uint32_t v;
    int32_t label;
};

// Vertex v's edges are row_ptr[v] .. row_ptr[v + 1]; in a range of a larger
// graph's rows row_ptr[0] is not 0.  lp_edge: the edges before vertex v's.
__device__ __forceinline__ uint32_t lp_edge(const int32_t* __restrict__ rp, uint64_t v)
{
    return (uint32_t)max(rp[v], rp[0]) - (uint32_t)rp[0];
}

// The first position of piece i when n vertices and `edges` edges are cut
// into `pieces` of one length.
__device__ __forceinline__ uint64_t lp_begin(uint64_t edges, uint32_t n, uint32_t pieces,
                                             uint32_t i)
{
    const uint64_t total = edges + n, len = (total + pieces - 1) / pieces;
    return min(total, len * i);
}

// Find the begin of piece i (i <= pieces), one wave.  Vertex v lies at
// position v + lp_edge(v): the piece's first vertex is the first one at or
// past the piece's begin, found by 64 probes a round.
__device__ __forceinline__ void lp_cut(lp_part* __restrict__ part, const int32_t* label,
                                       const int32_t* __restrict__ rp, uint32_t n,
                                       uint32_t pieces, uint32_t i)
{
    const uint32_t lane = __lane_id();
    const uint64_t at = lp_begin(lp_edge(rp, n), n, pieces, i);
    uint32_t lo = 0, hi = n;               // the answer is in lo..hi
    while (lo < hi) {
        const uint32_t m = hi - lo, step = (m + 63u) / 64u;
        const uint64_t q = (uint64_t)lo + (uint64_t)lane * step + step - 1;
        const uint64_t hit = __ballot(q < hi && q + lp_edge(rp, q < hi ? q : lo) >= at);
        if (hit == 0) {
            lo += m / step * step;
        } else {
            const uint32_t f = (uint32_t)__builtin_ctzll(hit);
            lo += f * step;
            hi = lo + step - 1;
        }
    }
    if (lane == 0) {
        const bool cont = lo > 0 && at - lo < lp_edge(rp, lo);
        part[i].v = lo;
        part[i].label = cont ? __hip_atomic_load(label + (lo - 1), __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT)
                             : 0;
    }
}

// Vertices and edges of a hardware block.  Without pieces (cut false) the
// edges are those of its vertices.
struct lp_share {
    uint32_t v0, v1;
    bool cut;
    uint32_t e0, e1;         // cut: the edges
    int32_t l0;              // cut: label of v0 - 1, for edges below row_ptr[v0]
    int32_t l1;              // label of v1 - 1 when its edges go on in the
    bool cont;               // next piece (cont)
    bool pilot;              // one wave's edges first (labelprop_edges)
};

__device__ __forceinline__ lp_share lp_share_of(const lp_part* part, const int32_t* __restrict__ rp,
                                                uint32_t n, uint32_t pieces, uint32_t i)
{
    const uint64_t edges = lp_edge(rp, n);
    const uint32_t first = (uint32_t)rp[0];
    const auto load = [&](uint32_t k) {   // the batch's workers renew the labels
        const uint64_t w = __hip_atomic_load(reinterpret_cast<const uint64_t*>(part + k),
                                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return lp_part{(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)w),
                       __builtin_amdgcn_readfirstlane((int)(w >> 32))};
    };
    const lp_part p0 = load(i), p1 = load(i + 1);
    lp_share s;
    s.v0 = p0.v;
    s.v1 = max(p1.v, p0.v);
    s.cut = true;
    s.e0 = first + (uint32_t)min(edges, lp_begin(edges, n, pieces, i) - p0.v);
    s.e1 = first + (uint32_t)min(edges, lp_begin(edges, n, pieces, i + 1) - p1.v);
    s.l0 = p0.label;
    s.l1 = p1.label;
    s.cont = (int32_t)s.e1 < rp[s.v1];
    return s;
}

// What bounds it: whole lines read for one label or one shadow word of an
// edge's target (2^25 edges: 3.2 GB per launch, 4.4 times the words that the
// sweep needs, at 4.3 TB/s), and in smaller graphs the hubs' words: until the first update of a
// hub's word lands, every lane with an edge into the hub exchanges the word,
// and exchanges of one word run one after another.  So in the blocks that
// start the launch (sh.pilot) one wave's edges go first, and the others find
// the hubs' words settled.  Per checked launch, R-MAT: 100,003 vertices and
// 800,024 edges, CSR monitored, 0.070 ms (0.16 without the first wave's
// start, 0.26 cut by vertices); 2^22 vertices and 2^25 edges 0.64 to 0.76 ms
// (3.2 cut by vertices).  One edge per lane at a time, in 64
// registers (two 1024-thread blocks per compute unit), was as fast as 2 or 4
// edges per lane (with more registers) and as loading the next edge's words
// ahead.  vt: vertices loaded at a time.
template <int CHECK, class G, bool COH = false>
__device__ __forceinline__ void labelprop_edges(const hr_env& e, const G& glab, const G& grp,
                                                const G& gcol, int32_t* __restrict__ label,
                                                const int32_t* __restrict__ rp,
                                                const int32_t* __restrict__ col,
                                                const uint8_t* __restrict__ mask, uint32_t n,
                                                uint32_t T, const lp_share& sh, uint32_t vt,
                                                uint32_t* lds)
{
    uint32_t* s_rp = lds;                        // row pointers of v0 - 1 (where its
    int32_t* s_l = (int32_t*)(s_rp + vt + 2);    // edges begin here), the vertices, the end;
    uint32_t* s_id = (uint32_t*)(s_l + vt + 1);  // labels; logical block << 10 | thread
    for (uint32_t tv = sh.v0;;) {
        const uint32_t nv = min(vt, sh.v1 - tv);
        const bool head = tv == sh.v0, tail = tv + nv == sh.v1;
        if (threadIdx.x == 0) {
            s_rp[0] = sh.cut && head ? sh.e0 : (uint32_t)rp[tv];
            s_l[0] = sh.l0;
            s_id[0] = tv == 0 ? 0u : (tv - 1) / T << 10 | (tv - 1) % T;
        }
        for (uint32_t i = threadIdx.x; i < nv; i += blockDim.x) {
            const uint32_t v = tv + i, lb = v / T, t = v - lb * T;
            hr_thread th{};
            if constexpr (CHECK) {
                th = hr_thread_make(e, lb, t);
                s_id[i + 1] = lb << 10 | t;
            }
            const typename G::word q = hr_gload<CHECK>(th, glab, v);
            int32_t l = __hip_atomic_load(label + v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (sh.cut && sh.cont && v + 1 == sh.v1) l = sh.l1;
            const uint32_t r = (uint32_t)rp[v];
            if (i + 1 == nv) s_rp[nv + 1] = (uint32_t)rp[v + 1];
            const typename G::pend p = hr_gi<2, CHECK, true>(e, th, glab, v, HR_SITE_LP_OWN, q);
            s_l[i + 1] = l;
            s_rp[i + 1] = r;
            hr_gs<2, CHECK>(e, th, glab, p, v, HR_SITE_LP_OWN);
            if (CHECK && grp.shadow) {
                hr_g<0, CHECK>(e, th, grp, v, HR_SITE_LP_CSR);
                hr_g<0, CHECK>(e, th, grp, v + 1, HR_SITE_LP_CSR);
            }
        }
        __syncthreads();
        const uint32_t k0 = sh.cut && head ? sh.e0 : s_rp[1];
        const uint32_t k1 = sh.cut && tail ? sh.e1 : s_rp[nv + 1];
        const uint32_t rounds = k1 > k0 ? (k1 - k0 + blockDim.x - 1) / blockDim.x : 0;
        const bool pilot = sh.pilot && head;
        for (uint32_t j = pilot ? 0 : 1; j <= rounds; ++j) {       // uniform
            if (pilot && j == 1) __syncthreads();
            const uint32_t k = k0 + threadIdx.x + (j ? j - 1 : 0) * blockDim.x;
            if (k >= k1 || (pilot && j < 2 && (threadIdx.x < 64) != (j == 0))) continue;
            const uint32_t u = (uint32_t)col[k];
            const bool seeded = mask[k];
            typename G::word w = 0;
            if constexpr (CHECK) w = hr_gload<CHECK>(hr_thread_of(e, 0, 0), gcol, (uint64_t)k);
            // the edge's vertex: the last one whose edges begin at or before k
            uint32_t lo = 0, hi = nv + 1;
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
                const int32_t r = lp_get<COH>(label + u);
                hr_gpre<0, CHECK, false>(e, th, glab, u, HR_SITE_LP_SEED_READ, q);
                lp_set<COH>(label + u, r < l ? r : l);
                hr_g<1, CHECK>(e, th, glab, u, HR_SITE_LP_SEED_WRITE);
            }
        }
        tv += nv;
        if (tv >= sh.v1) return;
        __syncthreads();
    }
}

// LDS words labelprop_edges needs for vt vertices at a time.
constexpr uint32_t labelprop_lds_words(uint32_t vt) { return 3 * vt + 4; }

// The other form: one lane per logical thread, vertices lb*T .. lb*T+T, one
// edge at a time.  For contexts with wave grouping, whose hook instructions
// must run one logical wave per hardware wave (hr_group).  While edge k is
// checked, the column index of edge k+2, and the seeded flag of edge k+1 and
// the shadow word of its target, are already in flight.
template <int CHECK, class G = hr_gref, bool COH = false>
__device__ __forceinline__ void labelprop_body(const hr_env& e, const G& glab, const G& grp, const G& gcol,
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
            const int32_t r = lp_get<COH>(label + u);
            hr_gpre<0, CHECK>(e, th, glab, u, HR_SITE_LP_SEED_READ, su);
            lp_set<COH>(label + u, r < l ? r : l);
            hr_g<1, CHECK, true>(e, th, glab, u, HR_SITE_LP_SEED_WRITE);
        } else {
            atomicMin(label + u, l);
            hr_gpre<2, CHECK>(e, th, glab, u, HR_SITE_LP_MIN, su);
        }
    }
}
