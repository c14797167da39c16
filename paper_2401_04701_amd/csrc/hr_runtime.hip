// Host runtime of the race checker: contexts, shadow regions, launch epochs
// and the race report.  See hr.h for the contract of each entry point.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <new>
#include <vector>

#include "hr.h"
#include "hr_device.h"
#include "hr_internal.h"

namespace {

// Clears and fills take several pieces of memory in one launch: a job's
// start is a chain of launches, about 2 us each on the device however
// little they clear.  16-byte stores over whole blocks of each piece.
constexpr uint32_t SEGS = 8;
struct segs {
    uint64_t* p[SEGS];
    size_t n[SEGS];      // 8-byte units; p is 16-byte aligned
    uint32_t count;
};

__global__ __launch_bounds__(256) void k_fill(segs g)
{
    const size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (uint32_t k = 0; k < g.count; ++k) {
        ulonglong2* p = reinterpret_cast<ulonglong2*>(g.p[k]);
        for (size_t i = t; i < g.n[k] / 2; i += stride) p[i] = make_ulonglong2(0, 0);
        if (t == 0 && (g.n[k] & 1)) g.p[k][g.n[k] - 1] = 0;
    }
}

// The launch-boundary clear of 4-byte words, two per 8-byte unit: back to
// the initial state, except that while some race record is missing from the
// ring (it overflowed, or a call site reached its record limit; read on the
// device) a word in the race state keeps it for the report's scan.
__global__ __launch_bounds__(256) void k_clear_word4(segs g, const uint32_t* __restrict__ ctr,
                                                     uint32_t ring_cap)
{
    const size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    const bool keep = ctr[HR_CTR_HEAD] > ring_cap || (ctr[HR_CTR_FLAGS] & HR_DEVF_LIMIT);
    const auto left = [keep](uint64_t v) {
        if (!keep) return (uint64_t)0;
        const uint64_t lo = (uint32_t)v == hr::T_RACE ? hr::T_RACE : 0u;
        const uint64_t hi = (uint32_t)(v >> 32) == hr::T_RACE ? hr::T_RACE : 0u;
        return lo | (hi << 32);
    };
    for (uint32_t k = 0; k < g.count; ++k) {
        ulonglong2* p = reinterpret_cast<ulonglong2*>(g.p[k]);
        for (size_t i = t; i < g.n[k] / 2; i += stride) {
            const ulonglong2 v = keep ? p[i] : make_ulonglong2(0, 0);
            p[i] = make_ulonglong2(left(v.x), left(v.y));
        }
        uint64_t* last = g.p[k] + g.n[k] - 1;
        if (t == 0 && (g.n[k] & 1)) *last = left(keep ? *last : 0);
    }
}

// Launch `kern` over pieces of memory, SEGS at a time: head[0 .. n_head), then
// the shadow allocations of c (may be null).  Nothing is allocated.
template <class K, class... A>
hipError_t launch_segs(K kern, hr_ctx c, const hr_piece* head, size_t n_head, hipStream_t s,
                       A... args)
{
    const size_t n = n_head + (c ? c->allocs.size() : 0);
    for (size_t at = 0; at < n;) {
        segs g{};
        size_t most = 0;
        for (; at < n && g.count < SEGS; ++at) {
            hr_piece p{nullptr, 0};
            if (at < n_head) p = head[at];
            else if (c->allocs[at - n_head].live)
                p = {c->allocs[at - n_head].mem, c->allocs[at - n_head].words};
            if (p.words == 0) continue;
            g.p[g.count] = (uint64_t*)p.mem;
            g.n[g.count++] = p.words;
            most = std::max(most, p.words);
        }
        if (g.count == 0) break;
        const size_t blocks = std::min<size_t>((most + 511) / 512, 4096);
        (void)hipGetLastError();   // drop stale errors of unrelated earlier calls
        hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(256), 0, s, g, args...);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// The global races among n shadow words: each word in the race state is
// appended to ring[] as a scanned record (only its key is valid) at the
// index taken from *count, or only counted when ring is null.  The caller
// sizes ring for every word it scans.
// The words are at offsets first .. first + n - 1 of the region's shadow;
// rows and lay give the region's map back to element indices.
__global__ void k_scan_races(const uint64_t* __restrict__ sh, size_t n, size_t first,
                             uint32_t word4, uint32_t region, hr_race_rec* __restrict__ ring,
                             uint32_t* __restrict__ count, uint32_t rows, hr_lay lay)
{
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (; i < n; i += stride) {
        const size_t o = first + i;
        const bool race = word4 ? ((const uint32_t*)sh)[o] == hr::T_RACE
                                : (sh[o] & hr::g::TAG_M) == hr::T_RACE;
        const uint64_t e = hr_lay_index(lay, rows, o);
        if (!race || e == UINT64_MAX) continue;
        const uint32_t slot =
            __hip_atomic_fetch_add(count, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (!ring) continue;
        uint4* p = reinterpret_cast<uint4*>(ring + slot);
        p[0] = make_uint4(0u, region, 0xFFFFFFFFu, 0xFFFFFFFFu);
        p[1] = make_uint4((uint32_t)e, (uint32_t)(e >> 32), 0u, 0u);
        p[2] = make_uint4(0u, 0u, 0xFFFFFFFFu, HR_RACE_SCANNED);
    }
}

}  // namespace

namespace {
uint32_t key_block(const hr_race& r) { return r.space == HR_LDS ? r.block : 0u; }

bool key_less(const hr_race& a, const hr_race& b)
{
    if (a.space != b.space) return a.space < b.space;
    if (a.region != b.region) return a.region < b.region;
    if (key_block(a) != key_block(b)) return key_block(a) < key_block(b);
    if (a.index != b.index) return a.index < b.index;
    return a.launch < b.launch;
}

bool key_same(const hr_race& a, const hr_race& b)
{
    return a.space == b.space && a.region == b.region && key_block(a) == key_block(b) &&
           a.index == b.index;
}
}  // namespace

namespace {

// Order of a record as one number (space, region, block if LDS, index), or
// false where a field does not fit.
bool key_pack(const hr_race& r, uint64_t* k)
{
    const uint64_t where = r.space == HR_LDS ? ((uint64_t)r.block << 17 | r.index) : r.index;
    *k = (uint64_t)(r.space == HR_LDS) << 63 | (uint64_t)r.region << 39 | where;
    return r.space <= HR_LDS && r.region < (1u << 24) &&
           (r.space == HR_LDS ? r.index < (1u << 17) && r.block < (1u << 22)
                              : r.index < (1ull << 39));
}

struct key_at {
    uint64_t key;
    size_t at;
};

}  // namespace

// Sorting moves 16-byte keys, not the 48-byte records, by counting passes
// over the key bits that differ between records (two for a grid or a graph
// of 4 M elements); then every kept record is moved once, to out.  (Reports of
// 5,000 records 0.07 ms against 0.45, of 260,000 14 against 37 with the
// comparison sort of the records, in turn on one host.)
bool hr_sort_records(const hr_race* recs, size_t n, hr_race* out, size_t cap, hr_host_buf& work,
                     size_t* n_out)
{
    *n_out = 0;
    if (n == 0) return true;
    key_at* k = (key_at*)work.get(2 * n * sizeof(key_at));
    if (!k) return false;
    key_at* other = k + n;
    uint64_t vary = 0;
    bool packed = n >= 256;   // below, the comparison sort is the faster one
    for (size_t i = 0; i < n; ++i) {
        packed &= key_pack(recs[i], &k[i].key);
        k[i].at = i;
        vary |= k[i].key ^ k[0].key;
    }
    if (!packed) {
        std::sort(k, k + n, [&](const key_at& a, const key_at& b) {
            return key_less(recs[a.at], recs[b.at]);
        });
    } else {
        constexpr uint32_t BITS = 11, N = 1u << BITS;
        for (uint32_t sh = 0; sh < 64 && vary >> sh;) {
            if (!((vary >> sh) & 1u)) {
                ++sh;
                continue;
            }
            size_t start[N + 1] = {};
            for (size_t i = 0; i < n; ++i) ++start[((k[i].key >> sh) & (N - 1)) + 1];
            for (uint32_t d = 0; d < N; ++d) start[d + 1] += start[d];
            for (size_t i = 0; i < n; ++i) other[start[(k[i].key >> sh) & (N - 1)]++] = k[i];
            std::swap(k, other);
            sh += BITS;
        }
    }
    // of records with one key the one of the earliest launch
    size_t m = 0;
    for (size_t i = 0; i < n; ++i) {
        if (m && (packed ? k[m - 1].key == k[i].key : key_same(recs[k[m - 1].at], recs[k[i].at]))) {
            if (recs[k[i].at].launch < recs[k[m - 1].at].launch) k[m - 1] = k[i];
        } else {
            k[m++] = k[i];
        }
    }
    *n_out = m;
    if (m > cap || !out) return true;
    constexpr size_t AHEAD = 24;   // the records lie anywhere in the ring
    for (size_t i = 0; i < m; ++i) {
        if (i + AHEAD < m) __builtin_prefetch(&recs[k[i + AHEAD].at]);
        out[i] = recs[k[i].at];
    }
    return true;
}

// In place and without any allocation.
size_t hr_sort_unique(hr_race* recs, size_t n)
{
    std::sort(recs, recs + n, key_less);
    size_t m = 0;
    for (size_t i = 0; i < n; ++i)
        if (m == 0 || !key_same(recs[m - 1], recs[i])) recs[m++] = recs[i];
    return m;
}

hipError_t hr_scan_races_dev(const uint64_t* sh, size_t n, size_t first, bool word4,
                             uint32_t region, hr_race_rec* ring, uint32_t* count, hipStream_t s,
                             uint32_t rows, const hr_lay& lay)
{
    if (n == 0) return hipSuccess;
    const size_t blocks = std::min<size_t>((n + 255) / 256, 8192);
    (void)hipGetLastError();
    hipLaunchKernelGGL(k_scan_races, dim3((unsigned)blocks), dim3(256), 0, s, sh, n, first,
                       word4 ? 1u : 0u, region, ring, count, rows, lay);
    return hipGetLastError();
}

// Clears run as kernels rather than hipMemsetAsync so the calls stay safe
// inside a captured HIP graph.
hipError_t hr_fill(const hr_piece* pieces, size_t count, hipStream_t s)
{
    return launch_segs(k_fill, nullptr, pieces, count, s);
}

hipStream_t hr_stream(hr_ctx c, void* stream)
{
    return stream ? (hipStream_t)stream : c->stream;
}

hr_env hr_env_of(const hr_config& cfg, hr_race_rec* ring, uint32_t* ctr,
                 unsigned long long* count, uint32_t launch_seq, hr_access_rec* log)
{
    hr_env e{};
    e.ring = ring;
    e.ctr = ctr;
    e.count = (cfg.flags & (HR_CFG_COUNT_CHECKS | HR_CFG_ACCESS_LOG)) ? count : nullptr;
    e.log = (cfg.flags & HR_CFG_ACCESS_LOG) ? log : nullptr;
    e.log_cap = e.log ? cfg.log_capacity : 0u;
    e.ring_cap = cfg.ring_capacity;
    e.launch = launch_seq & ((1u << hr::g::LAUNCH_BITS) - 1);
    e.launch_seq = launch_seq;
    e.bc_max = (1u << cfg.bc_bits) - 1;
    e.wc_max = (1u << cfg.wc_bits) - 1;
    e.group = (cfg.flags & HR_CFG_WAVE_GROUPING) ? cfg.coalesce_width : 0u;
    e.site_limit = cfg.site_limit;
    e.wave_bits = cfg.wave_bits;
    e.nested = (cfg.flags & HR_CFG_NESTED_TILES) ? 1u : 0u;
    e.word4 = (cfg.flags & HR_CFG_WORD4)
                  ? hr::c::layout(cfg.wc_bits, cfg.bc_bits, cfg.thread_bits)
                  : 0u;
    return e;
}

hr_env hr_make_env(hr_ctx c)
{
    return hr_env_of(c->cfg, c->ring, c->ctr, c->count, c->launch_seq, c->log);
}

void hr_fill_args(hr_ctx c, hr_kargs* a)
{
    *a = hr_kargs{};
    a->env = hr_make_env(c);
    const uint32_t n = (uint32_t)std::min<size_t>(c->reg.size(), HR_MAX_REGIONS);
    for (uint32_t r = 0; r < n; ++r) {
        if (!c->reg[r].live) continue;
        a->shadow[r] = c->reg[r].monitored ? c->reg[r].shadow : nullptr;
        a->n_elems[r] = c->reg[r].elems;
        a->data[r] = const_cast<void*>(c->reg[r].data);
        a->lay[r] = c->reg[r].lay;
    }
}

namespace {

// Calls that may wait or allocate while some stream records a graph.
struct relaxed_capture {
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    bool set = hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess;
    ~relaxed_capture()
    {
        if (set) (void)hipThreadExchangeStreamCaptureMode(&mode);
    }
};

// Its launches run now, not as a graph's (false too if the handle is invalid).
bool eager(hipStream_t s)
{
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &cap) == hipSuccess) return cap == hipStreamCaptureStatusNone;
    (void)hipGetLastError();
    return false;
}

// Record `ev` (made on first use) behind the work launched on s so far.
bool record(hipEvent_t& ev, hipStream_t s)
{
    const relaxed_capture r;
    if ((ev || hipEventCreateWithFlags(&ev, hipEventDisableTiming) == hipSuccess) &&
        hipEventRecord(ev, s) == hipSuccess)
        return true;
    (void)hipGetLastError();
    return false;
}

// Let s wait on the device for an event.  (Refused for an event whose stream
// has begun to record a graph since.)
bool follow(hipStream_t s, hipEvent_t ev)
{
    const relaxed_capture r;
    if (hipStreamWaitEvent(s, ev, 0) == hipSuccess) return true;
    (void)hipGetLastError();
    return false;
}

// Wait on the host for the work launched on the device so far, also while
// streams record graphs: hipDeviceSynchronize and hipEventSynchronize would
// end a recording, the wait that hipFree implies does not.
hipError_t wait_device()
{
    const relaxed_capture r;
    void* p = nullptr;
    const hipError_t err = hipMalloc(&p, 256);
    return err == hipSuccess ? hipFree(p) : err;
}

// From here on the epoch is shared.  What is launched next waits for its
// exclusive launches: on stream s, or where there is none (the caller's own
// kernels, a recorded launch) here on the host.
hr_status epoch_share(hr_ctx c, const hipStream_t* s)
{
    c->epoch_shared = true;
    if (!c->epoch_excl) return HR_OK;
    const bool here = !c->epoch_away && eager(c->stream);   // launched on c->stream
    if (!s && here) {
        const relaxed_capture r;
        if (hipStreamSynchronize(c->stream) != hipSuccess) return HR_E_HIP;
        c->epoch_excl = false;
        return HR_OK;
    }
    if (s && !c->epoch_recorded && here) c->epoch_recorded = record(c->epoch_event, c->stream);
    if (s && c->epoch_recorded && follow(*s, c->epoch_event)) return HR_OK;
    if (wait_device() != hipSuccess) return HR_E_HIP;
    c->epoch_excl = false;
    return HR_OK;
}

void epoch_begin(hr_ctx c)
{
    c->epoch_used = c->epoch_away = c->epoch_shared = c->epoch_excl = c->epoch_recorded = false;
}

}  // namespace

hr_status hr_epoch_enter(hr_ctx c, hipStream_t s, uint16_t* excl, bool away)
{
    const bool now = eager(s), one = now && s != hipStreamPerThread;
    const bool home = one && s == c->stream;
    if (!now) c->recorded = true;
    const bool alone = one && !c->epoch_shared && (home ? !c->epoch_away : !c->epoch_used);
    if (!alone) {
        const hr_status st = epoch_share(c, now ? &s : nullptr);
        if (st != HR_OK) return st;
    }
    c->epoch_used = true;
    c->epoch_away |= !home;
    if (excl) *excl = alone && !c->recorded && (home || away);
    return HR_OK;
}

hr_status hr_epoch_leave(hr_ctx c, hipStream_t s, uint16_t excl)
{
    if (!excl) return HR_OK;
    if (s != c->stream) {
        c->epoch_recorded = record(c->epoch_event, s);
        if (!c->epoch_recorded) return wait_device() == hipSuccess ? HR_OK : HR_E_HIP;
    }
    c->epoch_excl = true;
    return HR_OK;
}

lp_part* hr_lp_room(hr_ctx c, hipStream_t s)
{
    if (s == hipStreamPerThread || !eager(s)) return nullptr;
    const bool home = s == c->stream;
    if (c->lp_last == hr_ctx_s::LP_HOME && !home &&
        !(eager(c->stream) && record(c->lp_event, c->stream)))
        return nullptr;
    if ((c->lp_last == hr_ctx_s::LP_AWAY || (c->lp_last == hr_ctx_s::LP_HOME && !home)) &&
        !follow(s, c->lp_event))
        return nullptr;
    if (home) c->lp_last = hr_ctx_s::LP_HOME;
    return (lp_part*)(c->count + HR_COUNT_SLOTS);
}

hr_status hr_lp_leave(hr_ctx c, hipStream_t s)
{
    if (s == c->stream) return HR_OK;
    if (record(c->lp_event, s)) {
        c->lp_last = hr_ctx_s::LP_AWAY;
        return HR_OK;
    }
    if (wait_device() != hipSuccess) return HR_E_HIP;
    c->lp_last = hr_ctx_s::LP_NONE;
    return HR_OK;
}

bool hr_region_ok(hr_ctx c, uint32_t r, const void* data, size_t min_elems)
{
    return r < HR_MAX_REGIONS && r < c->reg.size() && c->reg[r].live && c->reg[r].data == data &&
           c->reg[r].elems >= min_elems;
}

hr_status hr_new_alloc(hr_ctx c, size_t words, uint32_t* alloc_out)
{
    const uint64_t bytes = (uint64_t)words * 8u;
    if (c->cfg.shadow_budget && c->shadow_bytes + bytes > c->cfg.shadow_budget) return HR_E_NOMEM;
    uint64_t* mem = nullptr;
    if (hipMalloc(&mem, bytes) != hipSuccess) return HR_E_NOMEM;
    const hr_piece piece{mem, words};
    if (hr_fill(&piece, 1, c->stream) != hipSuccess) {
        (void)hipFree(mem);
        return HR_E_HIP;
    }
    c->allocs.push_back(hr_alloc{mem, words, true});
    c->shadow_bytes += bytes;
    *alloc_out = (uint32_t)(c->allocs.size() - 1);
    return HR_OK;
}

uint32_t hr_new_region(hr_ctx c, const void* data, size_t elems, uint64_t* shadow, uint32_t alloc)
{
    c->reg.push_back(hr_region{data, elems, shadow, alloc, true, true});
    return (uint32_t)(c->reg.size() - 1);
}

size_t hr_region_words(const hr_region& r)
{
    return hr_lay_words(r.lay, r.rows, r.elems);
}

void hr_free_alloc(hr_ctx c, uint32_t alloc)
{
    hr_alloc& al = c->allocs[alloc];
    if (!al.live) return;
    (void)hipFree(al.mem);
    al.live = false;
    c->shadow_bytes -= (uint64_t)al.words * 8u;
    for (hr_region& r : c->reg)
        if (r.alloc == alloc) r.live = false;
}

// The flat transition table of the global-word machine, built at compile
// time from its bit logic (hr::g::make_step_table).
static constexpr hr::g::step_table FSM_TABLE = hr::g::make_step_table();
static_assert(hr::g::step_table_consistent(), "the flat table must rebuild hr::g::step");

bool hr_config_normalize(const hr_config* cfg, hr_config* out)
{
    hr_config k = {};
    if (cfg) k = *cfg;
    const bool word4 = (k.flags & HR_CFG_WORD4) != 0;
    const bool nested = (k.flags & HR_CFG_NESTED_TILES) != 0;
    if (nested) {
        // tiles of 2^wave_bits lanes inside whole waves; the nested words'
        // clock fields hold 5 and 4 bits, and the flat options do not apply
        if (k.wave_bits < 1 || k.wave_bits > 5 || word4 || (k.flags & HR_CFG_WAVE_GROUPING))
            return false;
        if (k.bc_bits == 0) k.bc_bits = 5;
        if (k.wc_bits == 0) k.wc_bits = 4;
        if (k.bc_bits > 5 || k.wc_bits > 4) return false;
    }
    if (k.ring_capacity == 0) k.ring_capacity = 65536;
    if (k.bc_bits == 0) k.bc_bits = word4 ? 2 : 8;
    if (k.wc_bits == 0) k.wc_bits = word4 ? 1 : 6;
    if (k.thread_bits == 0) k.thread_bits = word4 ? 8 : 10;
    if (k.bc_bits > 8 || k.wc_bits > 6 || k.ring_capacity > (1u << 26)) return false;
    if (k.thread_bits > 10 || (!word4 && k.thread_bits != 10)) return false;
    if (k.flags & HR_CFG_FSM_TABLE_LDS) k.flags |= HR_CFG_FSM_TABLE;
    if (k.flags & ~(HR_CFG_COUNT_CHECKS | HR_CFG_WAVE_GROUPING | HR_CFG_WORD4 |
                    HR_CFG_ACCESS_LOG | HR_CFG_NESTED_TILES | HR_CFG_FSM_TABLE |
                    HR_CFG_FSM_TABLE_LDS))
        return false;
    if ((k.flags & HR_CFG_FSM_TABLE) &&
        (k.flags & (HR_CFG_WORD4 | HR_CFG_NESTED_TILES | HR_CFG_ACCESS_LOG)))
        return false;
    if (k.flags & HR_CFG_ACCESS_LOG) {
        if (k.log_capacity == 0) k.log_capacity = 1u << 20;
        if (k.log_capacity > (1u << 28)) return false;
    } else if (k.log_capacity) {
        return false;   // a log size without the log
    }
    if (k.wave_bits == 0) k.wave_bits = 6;
    if (k.wave_bits > 6) return false;
    if (k.flags & HR_CFG_WAVE_GROUPING) {
        if (k.coalesce_width == 0) k.coalesce_width = 64;
        if (!hr_coalesce_width_ok(k.coalesce_width)) return false;
    } else if (k.coalesce_width) {
        return false;   // a width without grouping
    }
    *out = k;
    return true;
}

extern "C" hr_status hr_ctx_create(hr_ctx* out, const hr_config* cfg, void* stream)
{
    if (!out) return HR_E_INVAL;
    *out = nullptr;
    hr_config k;
    if (!hr_config_normalize(cfg, &k)) return HR_E_INVAL;
    hr_ctx c = new (std::nothrow) hr_ctx_s();
    if (!c) return HR_E_NOMEM;
    c->cfg = k;
    c->stream = (hipStream_t)stream;
    if (hipGetDevice(&c->device) != hipSuccess) {
        delete c;
        return HR_E_HIP;
    }
    if (hipMalloc(&c->ctr, HR_CTR_BYTES + sizeof(hr_race_rec) * (size_t)k.ring_capacity) !=
        hipSuccess) {
        hr_ctx_destroy(c);
        return HR_E_NOMEM;
    }
    c->ring = (hr_race_rec*)((uint8_t*)c->ctr + HR_CTR_BYTES);
    if (hipMalloc(&c->count, sizeof(unsigned long long) * HR_COUNT_SLOTS + HR_LP_ROOM_BYTES) !=
            hipSuccess ||
        ((k.flags & HR_CFG_ACCESS_LOG) &&
         hipMalloc(&c->log, sizeof(hr_access_rec) * (size_t)k.log_capacity) != hipSuccess) ||
        ((k.flags & HR_CFG_FSM_TABLE) && hipMalloc(&c->fsm_tab, sizeof(FSM_TABLE)) != hipSuccess)) {
        hr_ctx_destroy(c);
        return HR_E_NOMEM;
    }
    if (c->fsm_tab && hipMemcpy(c->fsm_tab, FSM_TABLE.e, sizeof(FSM_TABLE),
                                hipMemcpyHostToDevice) != hipSuccess) {
        hr_ctx_destroy(c);
        return HR_E_HIP;
    }
    const hr_piece pieces[] = {HR_CTR_PIECE(c->ctr), {c->count, HR_COUNT_SLOTS}};
    if (hr_fill(pieces, 2, c->stream) != hipSuccess) {
        hr_ctx_destroy(c);
        return HR_E_HIP;
    }
    *out = c;
    return HR_OK;
}

extern "C" hr_status hr_ctx_destroy(hr_ctx c)
{
    if (!c) return HR_E_INVAL;
    hipError_t e = hipStreamSynchronize(c->stream);
    for (hr_alloc& al : c->allocs)
        if (al.live) (void)hipFree(al.mem);
    if (c->ctr) (void)hipFree(c->ctr);   // the ring's memory too
    if (c->count) (void)hipFree(c->count);
    if (c->log) (void)hipFree(c->log);
    if (c->fsm_tab) (void)hipFree(c->fsm_tab);
    if (c->epoch_event) (void)hipEventDestroy(c->epoch_event);
    if (c->lp_event) (void)hipEventDestroy(c->lp_event);
    delete c;
    return e == hipSuccess ? HR_OK : HR_E_HIP;
}

extern "C" hr_status hr_shadow_alloc(hr_ctx c, const void* data_dev, size_t bytes,
                                     uint32_t elem_bytes, uint32_t* region_out)
{
    if (!c || !region_out || elem_bytes != 4 || bytes == 0 || bytes % 4 != 0) return HR_E_INVAL;
    if (c->reg.size() >= (1u << 24)) return HR_E_INVAL;
    const size_t elems = bytes / 4;
    uint32_t alloc = 0;
    const size_t words = (c->cfg.flags & HR_CFG_WORD4) ? (elems + 1) / 2 : elems;
    const hr_status st = hr_new_alloc(c, words, &alloc);
    if (st != HR_OK) return st;
    *region_out = hr_new_region(c, data_dev, elems, c->allocs[alloc].mem, alloc);
    return HR_OK;
}

extern "C" hr_status hr_shadow_alloc_2d(hr_ctx c, const void* data_dev, uint32_t rows,
                                        uint32_t cols, uint32_t elem_bytes, uint32_t tile_w_log2,
                                        uint32_t tile_h_log2, uint32_t* region_out)
{
    if (!c || !region_out || elem_bytes != 4 || rows == 0 || cols == 0) return HR_E_INVAL;
    if (tile_w_log2 > HR_TILE_LOG2_MAX || tile_h_log2 > HR_TILE_LOG2_MAX ||
        tile_w_log2 + tile_h_log2 > 2 * HR_TILE_LOG2_MAX)
        return HR_E_INVAL;
    if (c->reg.size() >= (1u << 24)) return HR_E_INVAL;
    hr_lay L{cols, (cols + (1u << tile_w_log2) - 1u) >> tile_w_log2, tile_w_log2, tile_h_log2};
    if ((tile_w_log2 | tile_h_log2) == 0) L = hr_lay{};   // row-major: the identity map
    const size_t elems = (size_t)rows * cols;
    const size_t lw = hr_lay_words(L, rows, elems);
    const size_t words = (c->cfg.flags & HR_CFG_WORD4) ? (lw + 1) / 2 : lw;
    uint32_t alloc = 0;
    const hr_status st = hr_new_alloc(c, words, &alloc);
    if (st != HR_OK) return st;
    *region_out = hr_new_region(c, data_dev, elems, c->allocs[alloc].mem, alloc);
    c->reg[*region_out].lay = L;
    c->reg[*region_out].rows = rows;
    return HR_OK;
}

extern "C" hr_status hr_shadow_free(hr_ctx c, uint32_t region)
{
    if (!c || region >= c->reg.size() || !c->reg[region].live) return HR_E_INVAL;
    const uint32_t alloc = c->reg[region].alloc;
    for (const hr_region& r : c->reg)
        if (r.live && r.alloc == alloc && &r != &c->reg[region]) return HR_E_STATE;   // shared arena
    if (hipStreamSynchronize(c->stream) != hipSuccess) return HR_E_HIP;
    hr_free_alloc(c, alloc);
    return HR_OK;
}

extern "C" hr_status hr_dev_args(hr_ctx c, void* out, size_t cap, size_t* size_out)
{
    if (!c) return HR_E_INVAL;
    if (size_out) *size_out = sizeof(hr_kargs);
    if (!out || cap < sizeof(hr_kargs)) return HR_E_INVAL;
    const hr_status st = epoch_share(c, nullptr);   // the caller's kernel may run on any stream
    if (st != HR_OK) return st;
    hr_fill_args(c, (hr_kargs*)out);
    return HR_OK;
}

static hr_race scanned_race(uint32_t region, size_t index)
{
    hr_race x = {};
    x.space = HR_GLOBAL;
    x.region = region;
    x.block = 0xFFFFFFFFu;
    x.launch = 0xFFFFFFFFu;
    x.index = index;
    x.tid = 0xFFFFFFFFu;
    x.flags = HR_RACE_SCANNED;
    return x;
}

// The global races held in the sticky race words of every live region.
static hr_status scan_races(hr_ctx c, std::vector<hr_race>& out)
{
    const bool word4 = (c->cfg.flags & HR_CFG_WORD4) != 0;
    for (uint32_t r = 0; r < c->reg.size(); ++r) {
        if (!c->reg[r].live) continue;
        const hr_region& g = c->reg[r];
        const size_t words = hr_region_words(g);
        if (word4) {
            std::vector<uint32_t> sh(words);
            if (hipMemcpy(sh.data(), g.shadow, sizeof(uint32_t) * sh.size(),
                          hipMemcpyDeviceToHost) != hipSuccess)
                return HR_E_HIP;
            for (size_t i = 0; i < sh.size(); ++i)
                if (sh[i] == hr::T_RACE && hr_lay_index(g.lay, g.rows, i) != UINT64_MAX)
                    out.push_back(scanned_race(r, hr_lay_index(g.lay, g.rows, i)));
            continue;
        }
        std::vector<uint64_t> sh(words);
        if (hipMemcpy(sh.data(), g.shadow, sizeof(uint64_t) * sh.size(),
                      hipMemcpyDeviceToHost) != hipSuccess)
            return HR_E_HIP;
        for (size_t i = 0; i < sh.size(); ++i) {
            if ((sh[i] & hr::g::TAG_M) == hr::T_RACE && hr_lay_index(g.lay, g.rows, i) != UINT64_MAX)
                out.push_back(scanned_race(r, hr_lay_index(g.lay, g.rows, i)));
        }
    }
    return HR_OK;
}

extern "C" hr_status hr_kernel_end(hr_ctx c, void* stream)
{
    if (!c) return HR_E_INVAL;
    c->launch_seq += 1;
    epoch_begin(c);
    if (c->cfg.flags & HR_CFG_WORD4) {
        // No launch field: every boundary returns the words to INIT.
        hipStream_t s = hr_stream(c, stream);
        if (launch_segs(k_clear_word4, c, nullptr, 0, s, (const uint32_t*)c->ctr,
                        c->cfg.ring_capacity) != hipSuccess)
            return HR_E_HIP;
        return HR_OK;
    }
    // The launch epoch in a shadow word has 9 bits: before it wraps, return
    // every word to the initial state.  Exact: all earlier accesses happen
    // before all later ones, and the races found so far are in the ring.
    // If the ring has overflowed or a call site reached its record limit,
    // the races whose records are missing live only in the race words, so
    // they are recovered before the clear and carried to the report.
    if ((c->launch_seq & ((1u << hr::g::LAUNCH_BITS) - 1)) == 0) {
        hipStream_t s = hr_stream(c, stream);
        uint32_t hf[2] = {0, 0};   // HR_CTR_HEAD, HR_CTR_FLAGS
        if (hipMemcpyAsync(hf, c->ctr, sizeof(hf), hipMemcpyDeviceToHost, s) != hipSuccess ||
            hipStreamSynchronize(s) != hipSuccess)
            return HR_E_HIP;
        if (hf[HR_CTR_HEAD] > c->cfg.ring_capacity || (hf[HR_CTR_FLAGS] & HR_DEVF_LIMIT)) {
            const hr_status st = scan_races(c, c->carried);
            if (st != HR_OK) return st;
        }
        return launch_segs(k_fill, c, nullptr, 0, s) == hipSuccess ? HR_OK : HR_E_HIP;
    }
    return HR_OK;
}

extern "C" hr_status hr_reset(hr_ctx c, void* stream)
{
    if (!c) return HR_E_INVAL;
    hipStream_t s = hr_stream(c, stream);
    const hr_piece head[] = {HR_CTR_PIECE(c->ctr), {c->count, HR_COUNT_SLOTS}};
    if (launch_segs(k_fill, c, head, 2, s) != hipSuccess) return HR_E_HIP;
    c->launch_seq = 0;
    c->carried.clear();
    epoch_begin(c);
    return HR_OK;
}

extern "C" hr_status hr_region_enable(hr_ctx c, uint32_t region, uint32_t on)
{
    if (!c || region >= c->reg.size() || !c->reg[region].live) return HR_E_INVAL;
    c->reg[region].monitored = on != 0;
    return HR_OK;
}

extern "C" hr_status hr_report(hr_ctx c, hr_race* out, size_t cap, size_t* n_out, void* stream)
{
    if (!c || !n_out) return HR_E_INVAL;
    hipStream_t s = hr_stream(c, stream);
    // One copy, after the stream's work, reads the counters and as many ring
    // records as the last report found (at least 64); a second copy reads
    // the rest when there are more.
    const uint32_t pre = std::min(c->cfg.ring_capacity, std::max(64u, c->last_head));
    const size_t first = HR_CTR_BYTES + sizeof(hr_race_rec) * (size_t)pre;
    uint8_t* buf = (uint8_t*)c->h_ring.get(first);
    if (!buf) return HR_E_NOMEM;
    if (hipMemcpyAsync(buf, c->ctr, first, hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess)
        return HR_E_HIP;
    uint32_t ctr[HR_CTR_SITES];
    std::memcpy(ctr, buf, sizeof(ctr));
    const uint32_t head = ctr[HR_CTR_HEAD];
    const uint32_t n_ring = std::min(head, c->cfg.ring_capacity);
    c->last_head = n_ring;
    if (n_ring > pre) {
        buf = (uint8_t*)c->h_ring.get(HR_CTR_BYTES + sizeof(hr_race_rec) * (size_t)n_ring, first);
        if (!buf) return HR_E_NOMEM;
        if (hipMemcpy(buf + first, c->ring + pre, sizeof(hr_race_rec) * (size_t)(n_ring - pre),
                      hipMemcpyDeviceToHost) != hipSuccess)
            return HR_E_HIP;
    }
    const hr_race* recs = (const hr_race*)(buf + HR_CTR_BYTES);
    size_t n_recs = n_ring;
    std::vector<hr_race> all;
    int warn = 0;
    if (ctr[HR_CTR_FLAGS] & HR_DEVF_CLOCK) warn |= HR_W_CLOCK_OVERFLOW;
    if (ctr[HR_CTR_FLAGS] & HR_DEVF_RANGE) warn |= HR_W_OUT_OF_RANGE;
    if (ctr[HR_CTR_FLAGS] & HR_DEVF_STALL) warn |= HR_W_STALLED;
    if (ctr[HR_CTR_FLAGS] & HR_DEVF_LIMIT) warn |= HR_W_REPORT_LIMITED;
    if (ctr[HR_CTR_FLAGS] & HR_DEVF_FOLD) warn |= HR_W_FOLDED;
    if (ctr[HR_CTR_FLAGS] & HR_DEVF_MASK) warn |= HR_W_PARTIAL_BARRIER;
    if (head > c->cfg.ring_capacity) warn |= HR_W_RING_OVERFLOW;
    if (head > c->cfg.ring_capacity || (ctr[HR_CTR_FLAGS] & HR_DEVF_LIMIT)) {
        // Race records are missing (ring overflow, or a site past its record
        // limit): race states are sticky in global shadow memory, so the
        // global part of the flagged set is recovered from it exactly (and
        // from the races carried over a shadow clear).
        all.assign(recs, recs + n_ring);
        const hr_status st = scan_races(c, all);
        if (st != HR_OK) return st;
        all.insert(all.end(), c->carried.begin(), c->carried.end());
        recs = all.data();
        n_recs = all.size();
    }
    if (!hr_sort_records(recs, n_recs, out, cap, c->h_keys, n_out)) return HR_E_NOMEM;
    if (*n_out > cap || (*n_out && !out)) return HR_E_INVAL;
    return (hr_status)warn;
}

extern "C" hr_status hr_check_count(hr_ctx c, uint64_t* out, void* stream)
{
    if (!c || !out) return HR_E_INVAL;
    if (hipStreamSynchronize(hr_stream(c, stream)) != hipSuccess) return HR_E_HIP;
    unsigned long long slots[HR_COUNT_SLOTS];
    if (hipMemcpy(slots, c->count, sizeof(slots), hipMemcpyDeviceToHost) != hipSuccess)
        return HR_E_HIP;
    uint64_t sum = 0;
    for (int i = 0; i < HR_COUNT_SLOTS; ++i) sum += slots[i];
    *out = sum;
    return HR_OK;
}

extern "C" hr_status hr_access_log(hr_ctx c, hr_access_rec* out, size_t cap, size_t* n_out,
                                   void* stream)
{
    if (!c || !n_out || !c->log) return HR_E_INVAL;
    if (hipStreamSynchronize(hr_stream(c, stream)) != hipSuccess) return HR_E_HIP;
    uint32_t head = 0;
    if (hipMemcpy(&head, c->ctr + HR_CTR_LOG, sizeof(head), hipMemcpyDeviceToHost) != hipSuccess)
        return HR_E_HIP;
    const size_t n = std::min<size_t>(head, c->cfg.log_capacity);
    *n_out = n;
    if (n > cap || (n && !out)) return HR_E_INVAL;
    if (n && hipMemcpy(out, c->log, sizeof(hr_access_rec) * n, hipMemcpyDeviceToHost) != hipSuccess)
        return HR_E_HIP;
    return head > c->cfg.log_capacity ? HR_W_LOG_TRUNCATED : HR_OK;
}

extern "C" hr_status hr_fsm_step(uint32_t space, uint64_t old, uint32_t kind, uint32_t launch,
                                 uint32_t block, uint32_t thread, uint32_t bc, uint32_t wc,
                                 uint32_t wave_bits, uint64_t* new_out)
{
    if (!new_out || kind > 2 || space > 1 || thread > 1023) return HR_E_INVAL;
    if (wave_bits < 1 || wave_bits > 6) return HR_E_INVAL;
    const uint32_t k = hr::kind_class(kind);
    if (space == HR_GLOBAL) {
        if (block >= hr::g::BLOCK_LIMIT) return HR_E_INVAL;
        *new_out = hr::g::step(old, hr::g::pack_id(launch, block, thread, bc, wc), k,
                               hr::g::group_mask(wave_bits));
    } else {
        *new_out = hr::l::step((uint32_t)old, hr::l::pack_id(thread, bc, wc), k,
                               hr::l::group_mask(wave_bits));
    }
    return HR_OK;
}

extern "C" hr_status hr_fsm_step_table(uint32_t space, uint64_t old, uint32_t kind,
                                       uint32_t launch, uint32_t block, uint32_t thread,
                                       uint32_t bc, uint32_t wc, uint32_t wave_bits,
                                       uint64_t* new_out)
{
    if (!new_out || kind > 2 || space != HR_GLOBAL || thread > 1023) return HR_E_INVAL;
    if (wave_bits < 1 || wave_bits > 6 || block >= hr::g::BLOCK_LIMIT) return HR_E_INVAL;
    *new_out = hr::g::step_tab(FSM_TABLE.e, old, hr::g::pack_id(launch, block, thread, bc, wc),
                               hr::kind_class(kind), hr::g::group_mask(wave_bits));
    return HR_OK;
}

extern "C" hr_status hr_describe(uint32_t space, uint64_t word, uint32_t wave_bits,
                                 hr_summary* out)
{
    if (!out || space > HR_LDS || wave_bits < 1 || wave_bits > 6) return HR_E_INVAL;
    const uint32_t none = UINT32_MAX;
    hr_summary d = {};
    d.launch = d.block = d.bc = d.wave = d.wc = d.thread = none;
    uint32_t tag, cl = 0, cb, cw, bc, wc, th;
    if (space == HR_GLOBAL) {
        namespace g = hr::g;
        tag = (uint32_t)(word & g::TAG_M);
        cl = (uint32_t)(word >> g::CL_SH) & 3u;
        cb = (uint32_t)(word >> g::CB_SH) & 3u;
        cw = (uint32_t)(word >> g::CW_SH) & 3u;
        bc = (uint32_t)(word >> g::BC_SH) & 255u;
        wc = (uint32_t)(word >> g::WC_SH) & 63u;
        th = (uint32_t)(word >> g::TH_SH) & 1023u;
        if (tag > hr::T_ST) return HR_E_INVAL;
        if (tag >= hr::T_MB) d.launch = (uint32_t)(word >> g::LA_SH) & 511u;
        if (tag >= hr::T_MW) d.block = (uint32_t)(word >> g::BL_SH) & (g::BLOCK_LIMIT - 1);
    } else {
        namespace l = hr::l;
        const uint32_t w = (uint32_t)word;
        tag = w & l::TAG_M;
        cb = (w >> l::CB_SH) & 3u;
        cw = (w >> l::CW_SH) & 3u;
        bc = (w >> l::BC_SH) & 255u;
        wc = (w >> l::WC_SH) & 63u;
        th = (w >> l::TH_SH) & 1023u;
        if (tag > hr::T_ST || tag == hr::T_MB) return HR_E_INVAL;
    }
    d.state = tag;
    if (tag >= hr::T_MW) {
        d.class_launch = cl;
        d.bc = bc;
    }
    if (tag == hr::T_MB || tag == hr::T_MW) d.class_block = cb;
    if (tag >= hr::T_MT) {
        d.class_block = cb;
        d.wave = th >> wave_bits;
        d.wc = wc;
    }
    if (tag == hr::T_MW || tag == hr::T_MT) d.class_wave = tag == hr::T_MT ? cw : 0;
    if (tag == hr::T_ST) {
        d.class_wave = cw;
        d.thread = th;
    }
    *out = d;
    return HR_OK;
}

extern "C" hr_status hr_describe_nested(uint32_t space, uint64_t word, uint32_t tile_bits,
                                        hr_summary_nested* out)
{
    if (!out || space > HR_LDS || tile_bits < 1 || tile_bits > 5) return HR_E_INVAL;
    const uint32_t none = UINT32_MAX;
    hr_summary_nested d = {};
    d.launch = d.block = d.bc = d.wave = d.wc = d.tile = d.tc = d.thread = none;
    uint32_t tag, cl = 0, cb, cw, ct, bc, wc, tc, th;
    if (space == HR_GLOBAL) {
        namespace n = hr::n;
        tag = (uint32_t)(word & n::TAG_M);
        cl = (uint32_t)(word >> n::CL_SH) & 3u;
        cb = (uint32_t)(word >> n::CB_SH) & 3u;
        cw = (uint32_t)(word >> n::CW_SH) & 3u;
        ct = (uint32_t)(word >> n::CT_SH) & 3u;
        bc = (uint32_t)(word >> n::BC_SH) & 63u;
        wc = (uint32_t)(word >> n::WC_SH) & 15u;
        tc = (uint32_t)(word >> n::TC_SH) & 15u;
        th = (uint32_t)(word >> n::TH_SH) & 1023u;
        if (tag > hr::T_MTI) return HR_E_INVAL;
        if (tag >= hr::T_MB) d.launch = (uint32_t)(word >> n::LA_SH) & 511u;
        if (tag >= hr::T_MW) d.block = (uint32_t)(word >> n::BL_SH) & (n::BLOCK_LIMIT - 1);
    } else {
        namespace nl = hr::nl;
        const uint32_t w = (uint32_t)word;
        tag = w & nl::TAG_M;
        cb = (w >> nl::CB_SH) & 3u;
        cw = (w >> nl::CW_SH) & 3u;
        ct = (w >> nl::CT_SH) & 3u;
        bc = (w >> nl::BC_SH) & 31u;
        wc = (w >> nl::WC_SH) & 15u;
        tc = (w >> nl::TC_SH) & 15u;
        th = (w >> nl::TH_SH) & 1023u;
        if (tag > hr::T_MTI || tag == hr::T_MB) return HR_E_INVAL;
    }
    // Tag order of the nested machine, from the widest group down: MB
    // (blocks), MW (waves), MTI (tiles of one wave), MT (threads of one
    // tile), ST (one thread).
    const bool mw = tag == hr::T_MW, mti = tag == hr::T_MTI, mt = tag == hr::T_MT,
               st = tag == hr::T_ST;
    d.state = mti ? (uint32_t)HR_S_TILES : tag;
    if (tag == hr::T_MB) d.class_block = cb;
    if (mw || mti || mt || st) {
        d.class_launch = cl;
        d.class_block = cb;
        d.bc = bc;
    }
    if (mti || mt || st) {
        d.class_wave = cw;
        d.wave = th >> 6;
        d.wc = wc;
    }
    if (mt || st) {
        d.class_tile = ct;
        d.tile = th >> tile_bits;
        d.tc = tc;
    }
    if (st) d.thread = th;
    *out = d;
    return HR_OK;
}

static bool word4_widths(uint32_t* wc_bits, uint32_t* bc_bits, uint32_t* thread_bits)
{
    if (*wc_bits == 0) *wc_bits = 1;
    if (*bc_bits == 0) *bc_bits = 2;
    if (*thread_bits == 0) *thread_bits = 8;
    return *wc_bits <= 6 && *bc_bits <= 8 && *thread_bits <= 10;   // the block keeps >= 3 bits
}

extern "C" hr_status hr_fsm_step_word4(uint32_t old, uint32_t kind, uint32_t block,
                                       uint32_t thread, uint32_t bc, uint32_t wc,
                                       uint32_t wave_bits, uint32_t wc_bits, uint32_t bc_bits,
                                       uint32_t thread_bits, uint32_t* new_out)
{
    if (!new_out || kind > 2 || wave_bits < 1 || wave_bits > 6 ||
        !word4_widths(&wc_bits, &bc_bits, &thread_bits) || bc >= (1u << bc_bits) ||
        wc >= (1u << wc_bits) || (old & 31u) >= hr::c::N_STATES)
        return HR_E_INVAL;
    const uint32_t lay = hr::c::layout(wc_bits, bc_bits, thread_bits);
    *new_out = hr::c::step(old, hr::c::pack_id32(block, thread, bc, wc, lay),
                           hr::kind_class(kind), hr::c::group_mask(wave_bits, lay), lay);
    return HR_OK;
}

extern "C" hr_status hr_word4_widen(uint32_t word, uint32_t wc_bits, uint32_t bc_bits,
                                    uint32_t thread_bits, uint64_t* out)
{
    if (!out || !word4_widths(&wc_bits, &bc_bits, &thread_bits) ||
        (word & 31u) >= hr::c::N_STATES)
        return HR_E_INVAL;
    *out = hr::c::widen(word, hr::c::layout(wc_bits, bc_bits, thread_bits));
    return HR_OK;
}

extern "C" hr_status hr_fsm_step_nested(uint32_t space, uint64_t old, uint32_t kind,
                                        uint32_t launch, uint32_t block, uint32_t thread,
                                        uint32_t bc, uint32_t wc, uint32_t tc, uint32_t tile_bits,
                                        uint64_t* new_out)
{
    if (!new_out || kind > 2 || space > 1 || thread > 1023 || tile_bits < 1 || tile_bits > 5)
        return HR_E_INVAL;
    if (block >= hr::n::BLOCK_LIMIT || bc >= hr::n::BC_LIMIT || wc >= hr::n::WC_LIMIT ||
        tc >= hr::n::TC_LIMIT)
        return HR_E_INVAL;
    const uint32_t k = hr::kind_class(kind);
    if (space == HR_GLOBAL)
        *new_out = hr::n::step(old, hr::n::pack_id(launch, block, thread, bc, wc, tc), k,
                               hr::n::tile_mask(tile_bits));
    else
        *new_out = hr::nl::step((uint32_t)old, hr::nl::pack_id(thread, bc, wc, tc), k,
                                hr::nl::tile_mask(tile_bits));
    return HR_OK;
}

extern "C" hr_status hr_fsm_merge_nested(uint64_t x, uint64_t y, uint32_t tile_bits,
                                         uint64_t* out)
{
    if (!out || tile_bits < 1 || tile_bits > 5) return HR_E_INVAL;
    *out = hr::n::merge(x, y, hr::n::tile_mask(tile_bits));
    return HR_OK;
}

extern "C" hr_status hr_fsm_merge(uint64_t x, uint64_t y, uint32_t wave_bits, uint64_t* out)
{
    if (!out || wave_bits < 1 || wave_bits > 6) return HR_E_INVAL;
    *out = hr::g::merge(x, y, hr::g::group_mask(wave_bits));
    return HR_OK;
}
