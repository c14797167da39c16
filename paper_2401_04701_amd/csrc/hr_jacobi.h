// The 5-point Jacobi sweep: its body as a device function of one logical
// block, and its standalone kernel.  The sweep's device code lives here
// alone, so that its measured figures can be tied to these sources.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "hr_device.h"
#include "hr_hooks.h"

constexpr uint32_t JACOBI_TILE = 18;
constexpr uint32_t JACOBI_TILE_WORDS = JACOBI_TILE * JACOBI_TILE;

// The synchronization of a tile's threads in jacobi_body: the hardware
// block's barrier.
struct hr_block_sync {
    template <int CHECK>
    __device__ __forceinline__ void bar(const hr_env& e, hr_thread& t) { hr_bar<CHECK>(e, t); }
};

// The synchronization of the 256 threads (4 waves) of one tile when a
// hardware block runs several tiles side by side: a barrier of those waves
// alone, on an arrival counter in LDS, so that a tile's waves do not wait
// for the other tiles' slowest wave.  The kernel clears the counter, then
// passes one block barrier, before the body runs.  Every
// wave of the tile reaches each barrier (the body's barriers are not under
// divergent control), and all are resident with their block, so the wait
// ends; it is bounded all the same, and a wait that runs out is reported as
// a stall (HR_DEVF_STALL) and goes on.  For the checker it is the tile's
// block barrier: it advances the block clock as hr_barrier_block does.
struct hr_tile_sync {
    static constexpr uint32_t SPIN_LIMIT = 1u << 22;
    uint32_t* arrive;     // the tile's counter in LDS, zero before the body
    uint32_t target;      // arrivals that end the next barrier
    template <int CHECK>
    __device__ __forceinline__ void bar(const hr_env& e, hr_thread& t)
    {
        target += 4u;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        if (__lane_id() == 0)
            __hip_atomic_fetch_add(arrive, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        for (uint32_t spin = 0;
             __hip_atomic_load(arrive, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) < target;
             ++spin) {
            if (spin >= SPIN_LIMIT) {
                hr_set_flag(e, HR_DEVF_STALL);
                break;
            }
            __builtin_amdgcn_s_sleep(1);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
        if constexpr (CHECK) {
            t.bc += 1;
            t.wc = 0;
            if (t.bc > e.bc_max && (t.enabled & 1u)) {
                t.enabled &= ~1u;
                hr_set_flag(e, HR_DEVF_CLOCK);
            }
            hr_retag(e, t);
        }
    }
};

// One 16x16 tile (logical block lb of a grid nbx tiles wide) of the 5-point
// sweep u_new = 0.2 (c + n + s + w + e), staged through an 18x18 LDS tile.
// seeds: NULL or per-block (side << 8 | offset) entries (-1: none); a seeded
// block's edge thread also writes the neighbour-owned halo cell.
//
// Which threads access an element is fixed by the code, so each cell's thread
// applies all accesses to its shadow words (owner updates): to the old cell's
// word its own read and the halo reads of the blocks beside an edge cell, to
// the new cell's word its own write and a neighbour's seeded write of it, to
// the LDS tile's words the staging writes and then every read of them.  Each
// global word is loaded once, with the data, and stored once.
//
// COH: the cells are read and written past the caches (agent scope), for a
// kernel whose blocks run several sweeps with only a counter between them.
//
// What bounds it: memory.  4096 x 4096: 0.129 ms per launch, 5.2 TB/s of the
// 671 MB of grids and shadow words (copies of 0.5 to 8 GiB reach 4.5 to 5.6
// TB/s here, smaller ones up to 6.8 with the memory-side cache), against 0.278 ms with every access published by its own thread's exchange
// (100 memory-side requests per tile, which run at 25 G/s on the chip, and
// 530 vector instructions per wave).  The general transitions in place of
// the closed forms (hr_own_fast), with their rare paths inside the kernel
// and not at its end, took 0.184 ms, issue-bound; plain, nontemporal or
// coherent loads and stores of the words made no difference.  A launch that
// is not alone in its epoch (no env.excl) leaves every word to the general
// transitions and an exchange: 0.200 ms.
template <int CHECK, class G = hr_gref, class SYNC = hr_block_sync, bool COH = false>
__device__ __forceinline__ void jacobi_body(const hr_env& e, const G& gold, const G& gnew,
                            const float* __restrict__ uo, float* __restrict__ un, uint32_t ny,
                            uint32_t nx, uint32_t nbx, const int32_t* __restrict__ seeds,
                            uint32_t lb, uint32_t t, float* tile, uint32_t* tsh, uint32_t lds_id,
                            SYNC sync = SYNC{})
{
    constexpr uint32_t TL = JACOBI_TILE;
    const uint32_t tx = t & 15u, ty = (t >> 4) & 15u;
    const uint32_t bx = lb % nbx, by = lb / nbx;
    const uint32_t gx = bx * 16u + tx, gy = by * 16u + ty;
    const bool inside = t < 256 && gx < nx && gy < ny;
    uint32_t late = 0;        // owner updates left to the end (bits below)
    constexpr uint32_t OLD = 1, CENTRE = 2, ROW = 4, COL = 8, NEW = 16;
    hr_thread th{};
    if constexpr (CHECK) th = hr_thread_make(e, lb, t);
    const auto cell = [&](size_t i) {
        if constexpr (COH)
            return __hip_atomic_load(uo + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        else
            return uo[i];
    };
    const auto set = [&](size_t i, float v) {
        if constexpr (COH)
            __hip_atomic_store(un + i, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        else
            un[i] = v;
    };
    const size_t g = (size_t)gy * nx + gx;
    const uint32_t cl = (ty + 1) * TL + tx + 1;
    // An edge thread stages at most one row halo cell (north or south) and
    // one column halo cell (west or east).
    const bool hn = inside && ty == 0 && gy > 0, hs = inside && ty == 15 && gy + 1 < ny;
    const bool hw = inside && tx == 0 && gx > 0, he = inside && tx == 15 && gx + 1 < nx;
    const size_t gr = hn ? g - nx : g + nx, gc = hw ? g - 1 : g + 1;
    const uint32_t lr = hn ? tx + 1 : 17 * TL + tx + 1;
    const uint32_t lc = hw ? (ty + 1) * TL : (ty + 1) * TL + 17;
    const hr_el xo = gold.at2(gy, gx, g), xn = gnew.at2(gy, gx, g);
    // an edge cell is the halo cell of the tile beside it, read there by the
    // thread next to it
    const auto by_row = [&] {
        return hr_by{hn || hs, hn ? lb - nbx : lb + nbx, hn ? 240u + tx : tx, HR_SITE_JACOBI_HALO};
    };
    const auto by_col = [&] {
        return hr_by{hw || he, hw ? lb - 1 : lb + 1, ty * 16u + (hw ? 15u : 0u),
                     HR_SITE_JACOBI_HALO};
    };
    typename G::word qo = 0, qn = 0;
    // in place (one region as both grids) the new cell's word is the old
    // cell's, to be loaded after its first update
    bool in_place = false;
    if constexpr (CHECK) in_place = gold.shadow == gnew.shadow;
    if (inside) {
        const float vc = cell(g);
        const float vr = hn || hs ? cell(gr) : 0.0f;
        const float vk = hw || he ? cell(gc) : 0.0f;
        if constexpr (CHECK) {
            qo = hr_gload<CHECK>(th, gold, xo);
            if (!in_place) qn = hr_gload<CHECK>(th, gnew, xn);
            // the first access of a tile word this launch: no earlier word
            const uint32_t staged = hr::l::step(hr::T_INIT, th.lid, hr::CL_X);
            tsh[cl] = staged;
            if (hn || hs) tsh[lr] = staged;
            if (hw || he) tsh[lc] = staged;
            if (e.count) {
                hr_note<0, CHECK>(e, th, gold, g, HR_SITE_JACOBI_CENTRE);
                hr_note_lds<1, CHECK>(e, th, lds_id, cl, HR_SITE_JACOBI_STAGE);
                if (hn || hs) {
                    hr_note<0, CHECK>(e, th, gold, gr, HR_SITE_JACOBI_HALO);
                    hr_note_lds<1, CHECK>(e, th, lds_id, lr, HR_SITE_JACOBI_STAGE);
                }
                if (hw || he) {
                    hr_note<0, CHECK>(e, th, gold, gc, HR_SITE_JACOBI_HALO);
                    hr_note_lds<1, CHECK>(e, th, lds_id, lc, HR_SITE_JACOBI_STAGE);
                }
            }
        }
        tile[cl] = vc;
        if (hn || hs) tile[lr] = vr;
        if (hw || he) tile[lc] = vk;
        if constexpr (CHECK)
            if (!hr_own_fast<0>(e, th, gold, xo, qo, by_row(), by_col())) late |= OLD;
    }
    sync.template bar<CHECK>(e, th);
    // the centre word is read by its own thread and by the tile's threads
    // beside it; one of them stands for the others, of another
    // synchronization group if there is one (far)
    uint32_t other = HR_NO_THREAD;
    bool far = false;
    const auto reader = [&] {
        const uint32_t gm = 1023u >> e.wave_bits << e.wave_bits;
        const auto reads = [&](bool on, uint32_t u) {
            const bool f = ((t ^ u) & gm) != 0;
            if (on && !far) {
                other = u;
                far = f;
            }
        };
        reads(tx > 0, t - 1);
        reads(tx < 15 && gx + 1 < nx, t + 1);
        reads(ty > 0, t - 16);
        reads(ty < 15 && gy + 1 < ny, t + 16);
    };
    hr_by rows{0, 0, 0, 0}, cols{0, 0, 0, 0};
    if (inside) {
        // a neighbour outside the grid reads the centre (no branches)
        const float c = tile[cl];
        const float vn = tile[gy > 0 ? cl - TL : cl];
        const float vs = tile[gy + 1 < ny ? cl + TL : cl];
        const float vw = tile[gx > 0 ? cl - 1 : cl];
        const float ve = tile[gx + 1 < nx ? cl + 1 : cl];
        if constexpr (CHECK) {
            if (e.count) {
                hr_note_lds<0, CHECK>(e, th, lds_id, cl, HR_SITE_JACOBI_TILE);
                if (gy > 0) hr_note_lds<0, CHECK>(e, th, lds_id, cl - TL, HR_SITE_JACOBI_TILE);
                if (gy + 1 < ny) hr_note_lds<0, CHECK>(e, th, lds_id, cl + TL, HR_SITE_JACOBI_TILE);
                if (gx > 0) hr_note_lds<0, CHECK>(e, th, lds_id, cl - 1, HR_SITE_JACOBI_TILE);
                if (gx + 1 < nx) hr_note_lds<0, CHECK>(e, th, lds_id, cl + 1, HR_SITE_JACOBI_TILE);
            }
            // (whole waves of 4 rows: the rows above and below a wave's)
            uint32_t others;
            if (e.wave_bits == 6) {
                const bool up = ty > 0, down = (ty < 15) & (gy + 1 < ny);
                const bool beside = (tx > 0) | ((tx < 15) & (gx + 1 < nx));
                others = (((ty & 3u) == 0) & up) | (((ty & 3u) == 3) & down) ? 2u
                         : up | down | beside                               ? 1u
                                                                             : 0u;
            } else {
                reader();
                others = other == HR_NO_THREAD ? 0u : far ? 2u : 1u;
            }
            if (!hr_own_lds_fast<0>(e, th, tsh, cl, others)) late |= CENTRE;
            if ((hn || hs) && !hr_own_lds_fast<0>(e, th, tsh, lr, 0)) late |= ROW;
            if ((hw || he) && !hr_own_lds_fast<0>(e, th, tsh, lc, 0)) late |= COL;
        }
        const float r = 0.2f * (c + vn + vs + vw + ve);
        set(g, r);
        if constexpr (CHECK) {
            if (e.count) hr_note<1, CHECK>(e, th, gnew, g, HR_SITE_JACOBI_OUT);
        }
        if (seeds) {
            const int32_t sd = seeds[lb];
            if (sd >= 0) {
                const uint32_t side = (uint32_t)sd >> 8, off = (uint32_t)sd & 255u;
                size_t tgt = g;              // the neighbour-owned target cell
                if (side == 0 && ty == 0 && tx == off && gy > 0) tgt = g - nx;
                else if (side == 1 && ty == 15 && tx == off && gy + 1 < ny) tgt = g + nx;
                else if (side == 2 && tx == 0 && ty == off && gx > 0) tgt = g - 1;
                else if (side == 3 && tx == 15 && ty == off && gx + 1 < nx) tgt = g + 1;
                if (tgt != g) {
                    set(tgt, r);
                    if constexpr (CHECK) {
                        if (e.count) hr_note<1, CHECK>(e, th, gnew, tgt, HR_SITE_JACOBI_SEED);
                    }
                }
            }
            if constexpr (CHECK) {
                // the blocks beside this cell whose seeded write names it
                const auto names = [&](uint32_t block, uint32_t side, uint32_t off) {
                    return seeds[block] == (int32_t)(side << 8 | off);
                };
                if (hn) rows = hr_by{names(lb - nbx, 1, tx), lb - nbx, 240u + tx, HR_SITE_JACOBI_SEED};
                if (hs) rows = hr_by{names(lb + nbx, 0, tx), lb + nbx, tx, HR_SITE_JACOBI_SEED};
                if (hw) cols = hr_by{names(lb - 1, 3, ty), lb - 1, ty * 16u + 15u, HR_SITE_JACOBI_SEED};
                if (he) cols = hr_by{names(lb + 1, 2, ty), lb + 1, ty * 16u, HR_SITE_JACOBI_SEED};
            }
        }
        if constexpr (CHECK)
            if (in_place || !hr_own_fast<1>(e, th, gnew, xn, qn, rows, cols)) late |= NEW;
    }
    if constexpr (CHECK) {
        if (late == 0) return;
        if (late & OLD)
            hr_own<0>(e, hr_thread_of(e, lb, t), gold, xo, HR_SITE_JACOBI_CENTRE, by_row(),
                      by_col());
        if (late & CENTRE) {
            reader();
            hr_own_lds<0>(e, th, tsh, lds_id, cl, HR_SITE_JACOBI_TILE, other);
        }
        if (late & ROW) hr_own_lds<0>(e, th, tsh, lds_id, lr, HR_SITE_JACOBI_TILE);
        if (late & COL) hr_own_lds<0>(e, th, tsh, lds_id, lc, HR_SITE_JACOBI_TILE);
        if (late & NEW) hr_own<1>(e, th, gnew, xn, HR_SITE_JACOBI_OUT, rows, cols);
    }
}

namespace {

// The tile of a hardware block.  Blocks go to the chip's eight dies in turn,
// each with its own L2; of 256 consecutive tiles a die takes 32 consecutive
// ones, so that neighbours share the lines of their halos and of the data rows
// (a tile's row is half a 128-byte line) in one L2.  4096 x 4096: 0.145 to
// 0.136 ms per launch, each timed on its own (0.141 with 2, 0.139 with 8 at a
// time); with 4-byte words 0.066 to 0.063 ms at 2048 x 3072, the clear with it.
__device__ __forceinline__ uint32_t jacobi_tile()
{
    const uint32_t b = blockIdx.y * gridDim.x + blockIdx.x, n = gridDim.x * gridDim.y;
    return b < (n & ~255u) ? (b & ~255u) | (b & 7u) << 5 | ((b >> 3) & 31u) : b;
}

// One 16 x 16 tile per hardware block, on row-major shadow maps (CHECK 0:
// plain, 1: checked).  8 waves per SIMD: the hook's scalar registers would
// otherwise cap the occupancy at 7.
template <int CHECK>
__global__ __launch_bounds__(256, 8) void k_jacobi(hr_kargs a, hr_gref gold, hr_gref gnew,
                                                const float* __restrict__ uo,
                                                float* __restrict__ un, uint32_t ny, uint32_t nx,
                                                const int32_t* __restrict__ seeds)
{
    __shared__ float tile[JACOBI_TILE_WORDS];
    __shared__ uint32_t tsh[CHECK ? JACOBI_TILE_WORDS : 1];
    using G = hr_gref_map<0, 0>;
    jacobi_body<CHECK, G>(a.env, G{gold}, G{gnew}, uo, un, ny, nx, gridDim.x, seeds, jacobi_tile(),
                          threadIdx.x, tile, tsh, 0);
}

// Four consecutive tiles per 1024-thread block, each quarter of the block
// running the tuned body of k_jacobi on its own tile (row-major maps,
// checked), for launches that share the device with other streams' work:
// 1024-thread blocks of other kernels find room as this kernel's blocks
// retire, where 256-thread blocks would take every freed slot back.
// TILE_SYNC: each quarter syncs its own waves (hr_tile_sync) after one
// block barrier at the start; else the body's barriers are the whole
// block's.  Quarters past the last tile run the body without a cell.  A
// template, so that only the sources that launch it compile it.
template <int CHECK = 1, bool TILE_SYNC = true>
__global__ __launch_bounds__(1024, 8) void k_jacobi_x4(hr_kargs a, hr_gref gold, hr_gref gnew,
                                                    const float* __restrict__ uo,
                                                    float* __restrict__ un, uint32_t ny,
                                                    uint32_t nx, uint32_t nbx, uint32_t tiles,
                                                    const int32_t* __restrict__ seeds)
{
    __shared__ float tile[4][JACOBI_TILE_WORDS];
    __shared__ uint32_t tsh[4][JACOBI_TILE_WORDS];
    __shared__ uint32_t arrive[4];
    using G = hr_gref_map<0, 0>;
    const uint32_t q = threadIdx.x >> 8;
    uint32_t lb = blockIdx.x * 4u + q, t = threadIdx.x & 255u;
    if (lb >= tiles) {
        lb = blockIdx.x * 4u;
        t = UINT32_MAX;
    }
    if constexpr (TILE_SYNC) {
        if (threadIdx.x < 4) arrive[threadIdx.x] = 0;
        __syncthreads();
        jacobi_body<CHECK, G, hr_tile_sync>(a.env, G{gold}, G{gnew}, uo, un, ny, nx, nbx,
                                                  seeds, lb, t, tile[q], tsh[q], 0,
                                                  hr_tile_sync{&arrive[q], 0u});
    } else {
        jacobi_body<CHECK, G>(a.env, G{gold}, G{gnew}, uo, un, ny, nx, nbx, seeds, lb, t,
                                    tile[q], tsh[q], 0);
    }
}

// The checked sweep of k_jacobi with every global transition read from the
// flat table of the machine at `tab` (a context made with
// HR_CFG_FSM_TABLE; row-major maps).  LDS_TAB: each block first copies the
// table into its LDS (32 KiB, which leaves room for 4 blocks per compute
// unit) and reads it there (HR_CFG_FSM_TABLE_LDS).  A template, so that
// only the sources that launch it compile it.
template <int CHECK = 1, bool LDS_TAB = false>
__global__ __launch_bounds__(256, 8) void k_jacobi_tab(hr_kargs a, hr_gref gold, hr_gref gnew,
                                                    const float* __restrict__ uo,
                                                    float* __restrict__ un, uint32_t ny,
                                                    uint32_t nx, const int32_t* __restrict__ seeds,
                                                    const uint16_t* __restrict__ tab)
{
    __shared__ float tile[JACOBI_TILE_WORDS];
    __shared__ uint32_t tsh[CHECK ? JACOBI_TILE_WORDS : 1];
    using G = hr_map<hr_gref_tab, 0, 0>;
    const uint16_t* t = tab;
    if constexpr (LDS_TAB) {
        __shared__ uint4 stab[sizeof(hr::g::step_table) / sizeof(uint4)];
        const uint4* src = reinterpret_cast<const uint4*>(tab);
        for (uint32_t i = threadIdx.x; i < sizeof(stab) / sizeof(uint4); i += 256) stab[i] = src[i];
        __syncthreads();
        t = reinterpret_cast<const uint16_t*>(stab);
    }
    jacobi_body<CHECK, G>(a.env, G{hr_gref_tab{gold, t}}, G{hr_gref_tab{gnew, t}}, uo, un,
                                ny, nx, gridDim.x, seeds, jacobi_tile(), threadIdx.x, tile, tsh, 0);
}

// The checked sweep on tiled shadow maps: both grids tiled by 2^TW x 2^TH
// (constant shifts), or TW < 0: each grid's own map, read at run time.
// CHECK 2: with the debug access log (any map; row-major maps run here too).
template <int TW, int TH, int CHECK = 1>
__global__ __launch_bounds__(256, 8) void k_jacobi_tiled(hr_kargs a, hr_gref gold, hr_gref gnew,
                                                         const float* __restrict__ uo,
                                                         float* __restrict__ un, uint32_t ny,
                                                         uint32_t nx,
                                                         const int32_t* __restrict__ seeds)
{
    __shared__ float tile[JACOBI_TILE_WORDS];
    __shared__ uint32_t tsh[JACOBI_TILE_WORDS];
    using G = hr_gref_map<TW, TH>;
    jacobi_body<CHECK, G>(a.env, G{gold}, G{gnew}, uo, un, ny, nx, gridDim.x, seeds,
                               jacobi_tile(), threadIdx.x, tile, tsh, 0);
}

// The checked sweep on 4-byte shadow words, with the word layout as a
// constant (LAY) or the context's (LAY = 0); CHECK 2 adds the access log.  With a constant layout it fits
// 8 waves per SIMD; the context-layout kernel needs a few more registers
// and runs 7.
template <uint32_t LAY, int CHECK = 1>
__global__ __launch_bounds__(256, LAY ? 8 : 7) void k_jacobi4(hr_kargs a, hr_gref4t<LAY> gold,
                                                 hr_gref4t<LAY> gnew,
                                                 const float* __restrict__ uo,
                                                 float* __restrict__ un, uint32_t ny, uint32_t nx,
                                                 const int32_t* __restrict__ seeds)
{
    __shared__ float tile[JACOBI_TILE_WORDS];
    __shared__ uint32_t tsh[JACOBI_TILE_WORDS];
    jacobi_body<CHECK, hr_gref4t<LAY>>(a.env, gold, gnew, uo, un, ny, nx, gridDim.x, seeds,
                                            jacobi_tile(), threadIdx.x,
                                            tile, tsh, 0);
}

}  // namespace
