// Host side of the C ABI declared in include/monta.h: argument validation,
// workspace layout, launch shapes, the slice pipeline and event profiling.
// Everything that touches data runs in the kernels of monta_kernels.hpp.
#include "monta.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cstdlib>
#include <cmath>
#include <cstring>
#include <mutex>
#include <vector>

#include "monta_kernels.hpp"
#include "monta_planner.hpp"

namespace {

using namespace monta;


thread_local int g_last_hip = 0;
std::atomic<int> g_pipeline_mode{-1};  // -1: one pass; 0, 1, 2: separate passes, one slice per launch
std::atomic<int> g_plan_mode{-1};      // -1: per-workgroup rebuild when the histogram table is small; 0: always the scan kernel
std::atomic<int> g_cache_policy{-1};   // -1: chosen from the working-set size

// The process-wide switches as one entry point saw them when it was called: every decision of that call, and of
// the internal steps it is made of, uses this snapshot, so a switch flipped by another thread takes effect at
// the next call and never in the middle of one.
struct Modes {
    int pipeline, plan, cache;
};
Modes snapshot_modes() { return {g_pipeline_mode.load(), g_plan_mode.load(), g_cache_policy.load()}; }

#define HIP_TRY(expr)                          \
    do {                                       \
        hipError_t e__ = (expr);               \
        if (e__ != hipSuccess) {               \
            g_last_hip = (int)e__;             \
            (void)hipGetLastError();           \
            return MONTA_ERR_HIP;              \
        }                                      \
    } while (0)

inline int64_t align_up(int64_t v, int64_t a) { return (v + a - 1) / a * a; }

int pow2ceil(int v)
{
    int p = 1;
    while (p < v) p <<= 1;
    return p;
}

constexpr size_t kRouteTileBudget = 120 * 1024;     // route_tile_bytes
constexpr size_t kRouteLdsBudget = 120 * 1024;      // dynamic LDS of the kernels that route
constexpr int64_t kFewRouteBlocks = 128;
// Routing and plan with 8192 counters: 73 us if every workgroup reduces them and only 32 workgroups run it (2048 tokens, 256
// experts), 35 if a kernel scans them; with 256 workgroups 35 and 37.  At 2048 counters the launch costs more than it saves.
constexpr int64_t kRebuildMax = 4096;

struct Geometry {
    Shape s;
    Modes modes;
    int64_t max_rows;
    int64_t row_bytes;
    size_t route_lds;
    int route_threads;   // workgroup size of the route kernel: TB * lanes per token
    int64_t blocks_by_tile;  // route workgroups if only route_tile_bytes limited their tokens
};

// Per-expert capacity: C = min(T, ceil(cf*T*k/E)), cf = 0 meaning "no drop".
int64_t capacity_of(const monta_cfg *c)
{
    if (c->capacity_factor <= 0.f) return c->tokens;
    double v = std::ceil((double)c->capacity_factor * (double)c->tokens * (double)c->top_k / (double)c->experts);
    if (v > (double)c->tokens) return c->tokens;
    return (int64_t)v;
}

// lanes that share one token in the route kernel: each lane should still scan at least 8 experts
int route_lanes_per_token(int TB, int E)
{
    int rl = 1;
    while (rl < 8 && E / (2 * rl) >= 8 && TB * 2 * rl <= 1024) rl *= 2;
    return rl;
}

// What decides how many tokens a route workgroup takes, and with it the layout of the workspace and the limit of the static entry point: the
// bytes of its logits, its bit masks, and three words per choice.  The workgroup's LDS (route_lds) is smaller by the logits, which are in
// registers: 11 KiB for 64 tokens on 256 experts, top-8, which is all that fit this budget.
size_t route_tile_bytes(int TB, int E, int k)
{
    const int NW = TB > kWave ? TB / kWave : 1, L = route_lanes_per_token(TB, E);
    const int stride = L * (((E + L - 1) / L) | 1);
    size_t b = ((size_t)TB * stride * 4 + (size_t)TB * k * 4 + 7) & ~(size_t)7;
    return b + (size_t)E * NW * 8 + (size_t)TB * k * 8 + (size_t)TB * 8;
}

int validate(const monta_cfg *c, Geometry *g)
{
    if (!c) return MONTA_ERR_NULL;
    g->modes = snapshot_modes();
    if (c->tokens < 1 || c->hidden < 1 || c->experts < 1 || c->top_k < 1 || c->ep < 1 || c->tp < 1 || c->slices < 1)
        return MONTA_ERR_INVALID;
    if (c->dtype != MONTA_FP32 && c->dtype != MONTA_BF16) return MONTA_ERR_INVALID;
    if (c->renorm != 0 && c->renorm != 1) return MONTA_ERR_INVALID;
    if (c->padded != 0 && c->padded != 1) return MONTA_ERR_INVALID;
    if (c->top_k > c->experts) return MONTA_ERR_INVALID;
    if (c->experts % c->ep != 0) return MONTA_ERR_INVALID;
    if (!(c->capacity_factor >= 0.f) || !std::isfinite(c->capacity_factor)) return MONTA_ERR_INVALID;
    const int64_t U = (int64_t)c->slices * c->tp;
    if (c->tokens % U != 0) return MONTA_ERR_INVALID;
    const int64_t row = (int64_t)c->hidden * (c->dtype == MONTA_FP32 ? 4 : 2);
    if (row % 16 != 0) return MONTA_ERR_INVALID;
    if (c->experts > 256 || c->top_k > 32) return MONTA_ERR_UNSUPPORTED;
    if (c->tokens * (int64_t)c->top_k > 0x7fffffffLL) return MONTA_ERR_UNSUPPORTED;
    if (row / 16 > 0x7fffffffLL || U * c->experts > 0x7fffffffLL) return MONTA_ERR_UNSUPPORTED;

    Shape &s = g->s;
    s.T = (int32_t)c->tokens;
    s.E = c->experts;
    s.k = c->top_k;
    s.ep = c->ep;
    s.tp = c->tp;
    s.S = c->slices;
    s.U = (int32_t)U;
    s.Tu = (int32_t)(c->tokens / U);
    s.C = (int32_t)capacity_of(c);
    s.renorm = c->renorm;
    s.by_E = fast_div(s.E);
    s.by_k = fast_div(s.k);
    s.by_k1 = fast_div(s.k > 1 ? s.k - 1 : 1);
    s.by_Tu = fast_div(s.Tu < 1 << 14 ? s.Tu : 1);      // used for small problems
    s.by_ep = fast_div(s.ep);
    s.vpr = (int32_t)(row / 16);
    const int lpr_max = kMoverThreads;
    s.lpr = pow2ceil(s.vpr) < lpr_max ? pow2ceil(s.vpr) : lpr_max;
    // route workgroup: as many tokens as fit route_tile_bytes' budget, at most 256, no more than a unit needs
    int TB = 256;
    while (TB > 32 && (route_tile_bytes(TB, s.E, s.k) > kRouteTileBudget || TB / 2 >= s.Tu)) TB >>= 1;
    if (route_tile_bytes(TB, s.E, s.k) > kRouteTileBudget) return MONTA_ERR_UNSUPPORTED;
    // ... and no more than leaves every second CU a workgroup (down to one wave of tokens): 8192 tokens, 64 experts, top-8:
    // 28.5 us for routing and plan in workgroups of 256 tokens, 24.2 in 64; 16384 tokens, 32 experts: 19.1 and 18.2
    auto blocks = [&](int tb) { return (int64_t)((s.Tu + tb - 1) / tb) * U; };
    g->blocks_by_tile = blocks(TB);
    while (TB > kWave && blocks(TB) < kFewRouteBlocks) TB >>= 1;
    s.TB = TB;
    s.bpu = (s.Tu + TB - 1) / TB;
    const int64_t nb = (int64_t)s.bpu * U;
    if (nb * s.E > 0x7fffffffLL) return MONTA_ERR_UNSUPPORTED;
    s.num_blocks = (int32_t)nb;
    // the per-workgroup rebuild of the scans reads num_blocks*E counters in every workgroup; a larger table is scanned by a
    // kernel of its own
    s.fast_plan = (g->modes.plan != 0 && nb * s.E <= kRebuildMax) ? 1 : 0;
    g->route_lds = (size_t)route_lds(TB, s.E, s.k).bytes;
    const int rl = route_lanes_per_token(TB, s.E);
    s.rl = rl;
    g->route_threads = TB * rl < kWave ? kWave : TB * rl;
    const int64_t tk = c->tokens * (int64_t)c->top_k, ec = (int64_t)c->experts * s.C;
    if (c->padded && ec > 0x7fffffffLL) return MONTA_ERR_UNSUPPORTED;
    s.padded = c->padded;
    g->max_rows = c->padded ? ec : (tk < ec ? tk : ec);
    s.max_rows = (int32_t)g->max_rows;
    {
        // Measured on MI355X (256 MB memory-side cache): a producer's cacheable stores pay when the
        // consumer kernel reads them back soon; beyond the cache everything but the pack stores streams.
        const int pol = g->modes.cache;
        const int64_t touched = (2 * c->tokens + 2 * g->max_rows) * row;   // x + out + STAGE + FINAL
        if (pol >= 0) s.cache = pol;
        else if (touched <= (512ll << 20)) s.cache = NT_REG_LD | NT_COMB_LD | NT_COMB_ST;
        else if (touched <= (1024ll << 20)) s.cache = NT_REG_LD | NT_REG_ST | NT_COMB_LD | NT_COMB_ST;
        else s.cache = NT_PACK_LD | NT_REG_LD | NT_REG_ST | NT_COMB_LD | NT_COMB_ST;
    }
    g->row_bytes = row;
    return MONTA_OK;
}

void fill_layout(const Geometry &g, monta_ws_layout *L)
{
    const Shape &s = g.s;
    int64_t off = 0;
    auto take = [&](int64_t ints) {
        int64_t o = off;
        off = align_up(off + ints * 4, 256);
        return o;
    };
    L->max_rows = g.max_rows;
    L->capacity = s.C;
    L->units = s.U;
    L->tokens_per_unit = s.Tu;
    L->block_tokens = s.TB;
    L->num_blocks = s.num_blocks;
    L->off_meta = take(META_SLOTS);
    L->off_counts = take(s.E);
    L->off_kept = take(s.E);
    L->off_offsets = take(s.E + 1);
    L->off_n = take((int64_t)s.U * s.E);
    L->off_stage_off = take((int64_t)s.U * s.E);
    L->off_unit_base = take((int64_t)s.U * s.E);
    L->off_send_rows = take((int64_t)s.U * s.ep);
    L->off_unit_rows = take((int64_t)s.U + 1);
    L->off_pos_final = take((int64_t)s.T * s.k);
    L->off_pos_stage = take((int64_t)s.T * s.k);
    L->off_row_map = take(g.max_rows);
    L->off_block_counts = take((int64_t)s.num_blocks * s.E);
    L->off_block_base = take((int64_t)s.num_blocks * s.E);
    L->off_local_rank = take((int64_t)s.T * s.k);
    L->off_kept_prefix = take(s.E + 1);
    L->ws_bytes = off;
}

int64_t ws_bytes(const Geometry &g)
{
    monta_ws_layout L;
    fill_layout(g, &L);
    return L.ws_bytes;
}

PlanPtrs plan_ptrs(const Geometry &g, const void *ws)
{
    monta_ws_layout L;
    fill_layout(g, &L);
    char *b = const_cast<char *>(static_cast<const char *>(ws));
    auto at = [&](int64_t o) { return reinterpret_cast<int32_t *>(b + o); };
    PlanPtrs p;
    p.meta = at(L.off_meta);
    p.counts = at(L.off_counts);
    p.kept = at(L.off_kept);
    p.offsets = at(L.off_offsets);
    p.n = at(L.off_n);
    p.stage_off = at(L.off_stage_off);
    p.unit_base = at(L.off_unit_base);
    p.send_rows = at(L.off_send_rows);
    p.unit_rows = at(L.off_unit_rows);
    p.pos_final = at(L.off_pos_final);
    p.pos_stage = at(L.off_pos_stage);
    p.row_map = at(L.off_row_map);
    p.block_counts = at(L.off_block_counts);
    p.block_base = at(L.off_block_base);
    p.local_rank = at(L.off_local_rank);
    p.kept_prefix = at(L.off_kept_prefix);
    return p;
}

inline bool misaligned(const void *p, uintptr_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) != 0; }

// ------------------------------------------------------------- profiling
//
// One event is recorded after every kernel launch, on the launching stream.  A
// kernel's duration is the time from the previous such event on the same stream
// (the end of the previous kernel) to its own event, so consecutive kernels are
// timed back to back without a second marker between them; the first kernel of a
// chain, or one that follows a cross-stream wait, gets a start event of its own.

struct ProfRec {
    int kid;
    hipEvent_t a, b;
};
std::mutex g_prof_mu;
std::atomic<int> g_prof_on{0};
std::vector<ProfRec> g_prof_recs;
std::vector<hipEvent_t> g_prof_events;                        // everything created, destroyed when drained
std::vector<std::pair<hipStream_t, hipEvent_t>> g_prof_last;  // last end event per stream
double g_prof_ms[MONTA_K_COUNT] = {0};
int64_t g_prof_n[MONTA_K_COUNT] = {0};

void prof_break_chain(hipStream_t st)
{
    if (!g_prof_on.load()) return;
    std::lock_guard<std::mutex> lk(g_prof_mu);
    for (auto &pr : g_prof_last)
        if (pr.first == st) pr.second = nullptr;
}

struct ProfScope {
    hipStream_t st;
    int kid;
    hipEvent_t a = nullptr;
    bool on;
    ProfScope(int kid_, hipStream_t st_) : st(st_), kid(kid_), on(g_prof_on.load() != 0)
    {
        if (!on) return;
        std::lock_guard<std::mutex> lk(g_prof_mu);
        for (auto &pr : g_prof_last)
            if (pr.first == st) a = pr.second;
        if (!a) {
            if (hipEventCreate(&a) != hipSuccess) {
                on = false;
                a = nullptr;
                return;
            }
            g_prof_events.push_back(a);
            (void)hipEventRecord(a, st);
        }
    }
    ~ProfScope()
    {
        if (!on) return;
        hipEvent_t b = nullptr;
        if (hipEventCreate(&b) != hipSuccess) return;
        (void)hipEventRecord(b, st);
        std::lock_guard<std::mutex> lk(g_prof_mu);
        g_prof_events.push_back(b);
        g_prof_recs.push_back({kid, a, b});
        bool found = false;
        for (auto &pr : g_prof_last)
            if (pr.first == st) {
                pr.second = b;
                found = true;
            }
        if (!found) g_prof_last.push_back({st, b});
    }
};

int prof_drain()
{
    std::lock_guard<std::mutex> lk(g_prof_mu);
    int rc = MONTA_OK;
    for (auto &r : g_prof_recs) {
        float ms = 0.f;
        hipError_t e = hipEventSynchronize(r.b);
        if (e == hipSuccess) e = hipEventElapsedTime(&ms, r.a, r.b);
        if (e == hipSuccess) {
            g_prof_ms[r.kid] += ms;
            g_prof_n[r.kid] += 1;
        } else {
            g_last_hip = (int)e;
            rc = MONTA_ERR_HIP;
        }
    }
    for (hipEvent_t ev : g_prof_events) (void)hipEventDestroy(ev);
    g_prof_events.clear();
    g_prof_recs.clear();
    g_prof_last.clear();
    return rc;
}

// ------------------------------------------------- side stream for mode 0

struct DevState {
    std::mutex mu;              // held while a call enqueues work that uses the side stream or the events
    hipStream_t side = nullptr;
    std::vector<hipEvent_t> ev;
    hipEvent_t done = nullptr;
};
std::mutex g_dev_mu;
DevState g_dev[64];

int dev_state(int nslices, DevState **out)
{
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= 64) return MONTA_ERR_UNSUPPORTED;
    std::lock_guard<std::mutex> lk(g_dev_mu);
    DevState &d = g_dev[dev];
    if (!d.side) HIP_TRY(hipStreamCreateWithFlags(&d.side, hipStreamNonBlocking));
    if (!d.done) HIP_TRY(hipEventCreateWithFlags(&d.done, hipEventDisableTiming));
    while ((int)d.ev.size() < nslices) {
        hipEvent_t e;
        HIP_TRY(hipEventCreateWithFlags(&e, hipEventDisableTiming));
        d.ev.push_back(e);
    }
    *out = &d;
    return MONTA_OK;
}

// ------------------------------------------------------------ launch shapes

constexpr int kMaxMoverGrid = 1 << 16;
constexpr int kResidentMoverWgs = 2048;         // mover workgroups the chip holds at once: 256 CUs x 8
constexpr int64_t kGroupBytes = 256ll << 20;   // a launch group's share of STAGE: the size of the memory-side cache

int mover_grid(const Shape &s, int64_t rows)
{
    const int rows_per_wg = kMoverThreads / s.lpr;
    int64_t g = (rows + rows_per_wg - 1) / rows_per_wg;
    if (g < 1) g = 1;
    if (g > kMaxMoverGrid) g = kMaxMoverGrid;
    return (int)g;
}

// The row count of a slice is only known on the device; the grid is sized from the host-side bound.
// With capacity drops most of those workgroups would find nothing to do, and an idle workgroup still
// costs dispatch time (measured on the largest workload, 55 % of the pairs dropped: a cap of 65536 workgroups
// makes the step 4 % longer than 32768, 16384 is another 0.5 % shorter, 8192 is slower again), so the grid stops
// at 16384 workgroups and the kernel strides over the rest.
constexpr int kMaxRegatherGrid = 16384;
int regather_grid(const Shape &s, int64_t rows_bound)
{
    const int g = mover_grid(s, rows_bound);
    return g < kMaxRegatherGrid ? g : kMaxRegatherGrid;
}

int64_t slice_rows_bound(const Geometry &g, int nslices_covered)
{
    int64_t r = (int64_t)g.s.tp * g.s.Tu * nslices_covered * g.s.k;
    return r < g.max_rows ? r : g.max_rows;
}

// The launch helpers below take a range of slices [j0, j1).
int launch_pack(const Geometry &g, const PlanPtrs &p, const void *x, void *stage, int j0, int j1, hipStream_t st)
{
    const Shape &s = g.s;
    const int per_slice = s.tp * s.Tu;
    const int t0 = j0 * per_slice, nt = (j1 - j0) * per_slice;
    ProfScope ps(MONTA_K_PACK, st);
    hipLaunchKernelGGL(pack_kernel, dim3(mover_grid(s, nt)), dim3(kMoverThreads), 0, st,
                       static_cast<const u32x4 *>(x), static_cast<u32x4 *>(stage), p, s, t0, nt);
    HIP_TRY(hipGetLastError());
    return MONTA_OK;
}

int launch_regather(const Geometry &g, const PlanPtrs &p, const void *stage, void *fin, int j0, int j1, hipStream_t st)
{
    const Shape &s = g.s;
    const int64_t bound = slice_rows_bound(g, j1 - j0);
    ProfScope ps(MONTA_K_REGATHER, st);
    hipLaunchKernelGGL(regather_kernel, dim3(regather_grid(s, bound)), dim3(kMoverThreads), 0, st,
                       static_cast<const u32x4 *>(stage), static_cast<u32x4 *>(fin), p, s, j0 * s.tp, j1 * s.tp);
    HIP_TRY(hipGetLastError());
    return MONTA_OK;
}

// packs slices [pj0, pj1) and regathers slices [rj0, rj1) in disjoint workgroups of one grid
int launch_pack_regather(const Geometry &g, const PlanPtrs &p, const void *x, void *stage, void *fin, int pj0, int pj1,
                         int rj0, int rj1, hipStream_t st)
{
    const Shape &s = g.s;
    const int per_slice = s.tp * s.Tu;
    const int n_pack = mover_grid(s, (pj1 - pj0) * per_slice);
    const int n_reg = regather_grid(s, slice_rows_bound(g, rj1 - rj0));
    ProfScope ps(MONTA_K_PACK_REGATHER, st);
    hipLaunchKernelGGL(pack_regather_kernel, dim3(n_pack + n_reg), dim3(kMoverThreads), 0, st,
                       static_cast<const u32x4 *>(x), static_cast<u32x4 *>(stage), static_cast<u32x4 *>(fin), p, s,
                       pj0 * per_slice, (pj1 - pj0) * per_slice, rj0 * s.tp, rj1 * s.tp, n_pack);
    HIP_TRY(hipGetLastError());
    return MONTA_OK;
}

int check_act_ptrs(const void *a, const void *b)
{
    if (!a || !b) return MONTA_ERR_NULL;
    if (misaligned(a, 16) || misaligned(b, 16)) return MONTA_ERR_ALIGN;
    return MONTA_OK;
}

// Dynamic LDS above the default limit has to be asked for once per kernel and device.
struct LdsOptIn {
    std::atomic<int> done[64];
};

int opt_in_lds(const void *kernel, int bytes, LdsOptIn &state)
{
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= 64) return MONTA_ERR_UNSUPPORTED;
    if (!state.done[dev].load()) {
        HIP_TRY(hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes));
        state.done[dev].store(1);
    }
    return MONTA_OK;
}

template <int MT, int NT, int KS, bool DEEP, bool SPLIT = false, bool STREAM = false>
int launch_gate(const u32x4 *x, const u32x4 *w, float *logits, int64_t T, int H, int E, hipStream_t st)
{
    using G = GateTile<MT, NT, KS>;
    static LdsOptIn lds_opt_in;
    if (int rc = opt_in_lds(reinterpret_cast<const void *>(gate_bf16_kernel<MT, NT, KS, DEEP, SPLIT, STREAM>),
                            (int)G::lds_bytes(32 * NT, !SPLIT), lds_opt_in))
        return rc;
    const unsigned grid = (unsigned)((T + G::kTokens - 1) / G::kTokens);
    hipLaunchKernelGGL((gate_bf16_kernel<MT, NT, KS, DEEP, SPLIT, STREAM>), dim3(grid), dim3(kGateThreads), G::lds_bytes(E, !SPLIT), st, x, w, logits,
                       T, H, E);
    return MONTA_OK;
}

template <int NCH, int THREADS, int MAXCHUNK>
int launch_gate_small(const u32x4 *x, const u32x4 *w, float *logits, int64_t T, int H, int E, int wgs_per_cu,
                      hipStream_t st)
{
    static LdsOptIn lds_opt_in;
    if (int rc = opt_in_lds(reinterpret_cast<const void *>(gate_small_kernel<NCH, THREADS, MAXCHUNK>),
                            (int)gate_small_lds_bytes(MAXCHUNK, THREADS), lds_opt_in))
        return rc;
    static std::atomic<int> cus{0};
    if (!cus.load()) {
        int dev = 0, n = 0;
        HIP_TRY(hipGetDevice(&dev));
        HIP_TRY(hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev));
        cus.store(n > 0 ? n : 256);
    }
    const int64_t ngroups = (T + kGateSmallTokens - 1) / kGateSmallTokens;
    const int64_t resident = (int64_t)wgs_per_cu * cus.load();
    const unsigned grid = (unsigned)(ngroups < resident ? ngroups : resident);
    hipLaunchKernelGGL((gate_small_kernel<NCH, THREADS, MAXCHUNK>), dim3(grid), dim3(THREADS),
                       gate_small_lds_bytes(H / NCH, THREADS), st, x, w, logits, T, H, E, ngroups);
    return MONTA_OK;
}

template <int XR, int WR, int NST, bool F32, bool SPREAD>
int launch_gate_short_t(const u32x4 *x, const u32x4 *w, float *logits, int64_t T, int H, int E, hipStream_t st)
{
    using G = ShortTile<XR, WR, NST>;
    static LdsOptIn lds_opt_in;
    if (int rc = opt_in_lds(reinterpret_cast<const void *>(gate_short_kernel<XR, WR, NST, F32, SPREAD>), G::kLdsBytes, lds_opt_in)) return rc;
    const int64_t grid = (T + XR - 1) / XR * ((E + WR - 1) / WR);
    if (grid > 0x7fffffff) return MONTA_ERR_UNSUPPORTED;
    hipLaunchKernelGGL((gate_short_kernel<XR, WR, NST, F32, SPREAD>), dim3((unsigned)grid), dim3(256), G::kLdsBytes, st, x, w, logits, T, H, E);
    return MONTA_OK;
}

// Spread starts (walk_start) up to 2 MiB of weights, half an L2: the tiles then read them at different places.  Three sets of activations in
// turn, in step and spread, us: 9000 x 4096, 20 experts 22.7 and 16.5; 16384 x 2048, 64 experts 15.0 and 13.8; 16384 x 8192 70.3 and 61.1;
// 10000 x 4096, 256 experts 64.8 and 58.8; 30000 x 2048, 128 experts 41.9 and 41.4.  The line is a cautious one: 12000 x 8192, 160 experts,
// 2.5 MiB, 116.8 and 93.7, 10000 x 8192, 256 experts, 4 MiB, 114 and 107.  In fp32 the matrix rate decides (16384 x 4096, 64 experts:
// 95.9 and 96.3).
template <int XR, int WR, int NST, bool F32 = false>
int launch_gate_short(const u32x4 *x, const u32x4 *w, float *logits, int64_t T, int H, int E, hipStream_t st)
{
    const int64_t row = (int64_t)H * 2;
    if constexpr (!F32)
        if (row % 4096 == 0 && E * row <= (2 << 20)) return launch_gate_short_t<XR, WR, NST, false, true>(x, w, logits, T, H, E, st);
    return launch_gate_short_t<XR, WR, NST, F32, false>(x, w, logits, T, H, E, st);
}

// The whole-row kernel for at most 8 experts; returns 1 if the shape does not fit it.  Measured on MI355X: tiles
// of 8 rows x 4 KiB serve rows of up to 8 KiB best (a workgroup then sees more, smaller tiles and starts
// sooner), tiles of 8 rows x 8 KiB longer rows; there more than one workgroup per CU only repeats the weight set-up.
int launch_gate_small_any(const u32x4 *x, const u32x4 *w, float *logits, int64_t T, int H, int E, hipStream_t st)
{
    if (E > kGateSmallExperts) return 1;
    // short rows: two workgroups per CU, a tile's latency under the other's (65536 x 2048, 8 experts 60 and 50 us, 8192 x 1536 9.9 and
    // 8.8); up to 2 KiB, where even 8 rows are little to wait for, the 32 x 64 tiles of the larger expert counts (65536 x 512: 32 and
    // 13 us, 8192 x 1024: 8.2 and 6.0; 30000 x 2048: 24 and 29)
    if (H <= 1024 && T > 2048) return launch_gate_short<32, 64, 4>(x, w, logits, T, H, E, st);
    if (H <= 2048 && H % 64 == 0) return launch_gate_small<1, 512, 2048>(x, w, logits, T, H, E, 2, st);
    if (H <= 4096 && H % 128 == 0) return launch_gate_small<2, 512, 2048>(x, w, logits, T, H, E, 1, st);
    if (H <= 4096 && H % 64 == 0) return launch_gate_small<1, 512, 4096>(x, w, logits, T, H, E, 1, st);
    if (H <= 8192 && H % 128 == 0) return launch_gate_small<2, 512, 4096>(x, w, logits, T, H, E, 1, st);
    return 1;
}

// nb: groups of 16 experts per workgroup, 1 or 2 (bf16), 1 or 4 (fp32)
template <bool BF16>
int launch_gate_split(const u32x4 *x, const u32x4 *w, float *logits, int64_t T, int64_t cpr, int E, int nb, hipStream_t st)
{
    const int64_t grid = (T + 15) / 16 * ((E + 16 * nb - 1) / (16 * nb));
    if (grid > 0x7fffffff) return MONTA_ERR_UNSUPPORTED;
    constexpr int kMany = BF16 ? 2 : 4;
    if (nb == kMany) hipLaunchKernelGGL((gate_split_kernel<BF16, kMany>), dim3((unsigned)grid), dim3(512), 0, st, x, w, logits, T, cpr, E);
    else if (nb == 1) hipLaunchKernelGGL((gate_split_kernel<BF16, 1>), dim3((unsigned)grid), dim3(512), 0, st, x, w, logits, T, cpr, E);
    else return MONTA_ERR_UNSUPPORTED;
    return MONTA_OK;
}

template <int XB, int CB, int W, int NST>
int launch_gate_ring(const u32x4 *x, const u32x4 *w, float *logits, int64_t T, int H, int E, hipStream_t st)
{
    using G = SplitTile<XB, CB, W, NST>;
    static LdsOptIn lds_opt_in;
    if (int rc = opt_in_lds(reinterpret_cast<const void *>(gate_ring_kernel<XB, CB, W, NST>), G::kLdsBytes, lds_opt_in)) return rc;
    const int64_t grid = (T + 16 * XB - 1) / (16 * XB) * ((E + 16 * CB - 1) / (16 * CB));
    if (grid > 0x7fffffff) return MONTA_ERR_UNSUPPORTED;
    hipLaunchKernelGGL((gate_ring_kernel<XB, CB, W, NST>), dim3((unsigned)grid), dim3(G::kThreads), G::kLdsBytes, st, x, w, logits, T, H / 8, E);
    return MONTA_OK;
}

// bf16, few tiles: with the hidden axis split (gate_ring_kernel), 1 if they are not few.  About one tile per CU: 16 x 16, 16 x 32, 32 x 32 and,
// on rows of 2048 elements and more, 32 x 64, whichever is the first to be few enough; eight waves for the longest rows and half a tile per
// CU.  Measured on MI355X, three sets in turn, us, the forms before (split tiles straight into registers, 32 x 64 tiles, whole rows for up to 8
// experts) and these: 1 x 5264, 128 experts 6.8 and 5.2; 64 x 7168, 256 experts 15.8 and 6.9; 376 x 4096, 256 experts 14.2 and 6.9;
// 4559 x 5120, 16 experts 23.0 and 10.3; 1513 x 2048, 256 experts 10.8 and 9.5; 8192 x 4096, 8 experts 13.1 and 12.1; 2000 x 8192, 8 experts 10.4 and
// 7.3; 1003 x 792, 256 experts, 256 tiles of 32 x 32 on 13 steps 5.6 and 5.7; 8000 x 8192, 8 experts, 125 MiB of activations 27.4 and 29.6.
// Over 60 shapes of up to 300 tiles of 32 x 64 1.44 times as fast.  Error against 64 bits nowhere larger (at split_tile).
int launch_gate_few(const u32x4 *x, const u32x4 *w, float *logits, int64_t T, int H, int E, hipStream_t st)
{
    auto tiles = [&](int64_t R, int64_t C) { return (T + R - 1) / R * ((E + C - 1) / C); };
    const int64_t steps = ((int64_t)H * 2 + 127) / 128, small = tiles(16, 16);
    if (H > kBigMaxHidden || steps < 8 || T * H * 2 > (96ll << 20)) return 1;
    if (steps >= 128 && small <= 128) return launch_gate_ring<1, 1, 8, 4>(x, w, logits, T, H, E, st);
    if (small <= 200) return launch_gate_ring<1, 1, 4, 3>(x, w, logits, T, H, E, st);
    if (tiles(16, 32) <= 256) return launch_gate_ring<1, 2, 4, 3>(x, w, logits, T, H, E, st);
    if (tiles(32, 32) <= (steps >= 16 ? 256 : 160)) return launch_gate_ring<2, 2, 4, 3>(x, w, logits, T, H, E, st);
    if (tiles(32, 64) <= 256 && steps >= 32) return launch_gate_ring<2, 4, 4, 3>(x, w, logits, T, H, E, st);
    return 1;
}

int launch_gate_f32_few(const float4 *x, const float4 *w, float *logits, int64_t T, int H, int E, hipStream_t st)
{
    const dim3 grid((unsigned)((T + 3) / 4)), block(256);
    const int vpr = H / 4;
    if (E == 1) hipLaunchKernelGGL(gate_f32_few_kernel<1>, grid, block, 0, st, x, w, logits, T, vpr);
    else if (E == 2) hipLaunchKernelGGL(gate_f32_few_kernel<2>, grid, block, 0, st, x, w, logits, T, vpr);
    else if (E == 3) hipLaunchKernelGGL(gate_f32_few_kernel<3>, grid, block, 0, st, x, w, logits, T, vpr);
    else hipLaunchKernelGGL(gate_f32_few_kernel<4>, grid, block, 0, st, x, w, logits, T, vpr);
    return MONTA_OK;
}

template <bool RAGGED_LAST, bool DEEP_W, bool TAIL>
int launch_expert_big_k(const void *x_final, const void *w_exp, void *y, const ExpertArgs &a, int64_t grid, hipStream_t st)
{
    static LdsOptIn lds_opt_in;
    constexpr int lds = big_lds_bytes(DEEP_W);
    if (int rc = opt_in_lds(reinterpret_cast<const void *>(expert_big_kernel<RAGGED_LAST, DEEP_W, TAIL>), lds, lds_opt_in)) return rc;
    hipLaunchKernelGGL((expert_big_kernel<RAGGED_LAST, DEEP_W, TAIL>), dim3((unsigned)grid), dim3(kBigThreads), lds, st,
                       static_cast<const u32x4 *>(x_final), static_cast<const u32x4 *>(w_exp),
                       static_cast<unsigned short *>(y), a);
    return MONTA_OK;
}

template <bool RAGGED_LAST, bool DEEP_W>
int launch_expert_big_t(const void *x_final, const void *w_exp, void *y, const ExpertArgs &a, int64_t grid, hipStream_t st)
{
    return a.H % 64 ? launch_expert_big_k<RAGGED_LAST, DEEP_W, true>(x_final, w_exp, y, a, grid, st)
                    : launch_expert_big_k<RAGGED_LAST, DEEP_W, false>(x_final, w_exp, y, a, grid, st);
}

int launch_expert_big(const void *x_final, const void *w_exp, void *y, ExpertArgs a, int64_t rows_bound,
                      int64_t rows_per_expert, hipStream_t st)
{
    // Weights are streamed only on rows of more than 4096 elements.  Plain and streamed, three sets of weights in turn, us: 256
    // experts of 512 x 7936, 74 rows 532 and 574, 128 of 2048 x 2048, 100 rows 271 and 282, 64 of 4096 x 2048, 150 rows 269 and 271,
    // 4096 x 4096, 200 rows 546 and 545; but 5120 x 2560, 150 rows 382 and 380, 7168 x 2048, 120 rows 355 and 345, 32 of 8192 x 4096
    // 449 and 434.
    if (a.H <= 4096) a.stream_from = (int64_t)a.E * a.N;
    const int64_t row_tiles = (rows_bound + kBigBM - 1) / kBigBM + a.E;      // each expert may end in a ragged tile
    const int64_t nct = (a.N + kBigBN - 1) / kBigBN;
    // whole blocks of 256 workgroups: the kernel hands out tile numbers in such blocks, 32 per XCD
    auto rounded = [](int64_t n) { return (n + 32 * kXcds - 1) / (32 * kXcds) * (32 * kXcds); };
    const int64_t grid = rounded(row_tiles * nct), grid_last = rounded((row_tiles + a.E) * nct);     // ragged tiles may come in halves
    if (grid_last > 0x7fffffff) return MONTA_ERR_UNSUPPORTED;
    // The segments' ragged last tiles go to the end of the numbering only when there are few of them, at most one round
    // of 256 workgroups: measured on MI355X, eight segments of about 2048 rows 464 us against 480 with the ragged tiles in
    // place; 64 segments of 191 rows, where every tile is ragged, 448 against 440.
    const bool ragged_last = (int64_t)a.E * nct <= 256;
    // The third stage of weights in LDS: where a weight tile has one user, or two, the second of them a ragged tile that runs at
    // the end, after the first (8 experts, 8192 x 8192, 320 rows: 550 us, with the third stage 502; 64 experts, 4096 x 512: 182 and
    // 164; but 32 experts, 4096 x 4096, where the ragged tile runs beside it, 391 and 433, and 1024 x 1024, whose walk is short,
    // 84 and 85).
    const bool deep_w = rows_per_expert <= kBigBM || (ragged_last && a.H >= 4096 && rows_per_expert <= kBigBM * 3 / 2);
    // Spread starts (walk_start), by expert, with the third stage of weights: us, in step and spread, 64 experts of 4096 x 2048, 120 rows 263 and
    // 212, 190 rows 285 and 238; 128 of 2048 x 2048, 190 rows 308 and 259; 256 of 2048 x 1024, 70 rows 264 and 221.
    a.spread = (int64_t)a.H * 2 % 4096 == 0;
    if (ragged_last) return deep_w ? launch_expert_big_t<true, true>(x_final, w_exp, y, a, grid_last, st)
                                   : launch_expert_big_t<true, false>(x_final, w_exp, y, a, grid_last, st);
    return deep_w ? launch_expert_big_t<false, true>(x_final, w_exp, y, a, grid, st)
                  : launch_expert_big_t<false, false>(x_final, w_exp, y, a, grid, st);
}

template <int XR, int WR, int NST, bool F32 = false, bool FINE = false>
int launch_expert_short_t(const void *x_final, const void *w_exp, void *y, ExpertArgs a, int64_t rows_bound, int64_t rows_per_expert,
                          hipStream_t st)
{
    using G = ShortTile<XR, WR, NST>;
    // No streamed weights in 64 x 128 tiles on rows below 1536 elements.  Plain and streamed, three sets of weights in turn, us: 256
    // experts of 512 x 2048, 40 rows 124 and 126, 128 of 1024 x 2048 103 and 106, 128 of 1152 x 1536 88.5 and 91.0; but 128 of 1536 x
    // 1024 80.0 and 79.5, 64 of 2048 x 2048, 48 rows 118 and 115, and in 32 x 64 tiles 128 of 1024 x 2048, 8 rows 90 and 82.
    if (WR == 128 && a.H < 1536) a.stream_from = (int64_t)a.E * a.N;
    // Spread starts (walk_start) where most experts fit one tile's rows; with more row tiles the rows, too, are read at many places at
    // a time and leave the L2 (16 experts of 8192 x 1024, 37 rows in 32 x 64 tiles: in step 64, spread 76 us).  Three sets of weights in turn, in
    // step and spread, us: 16 experts of 4096 x 2048, 8 rows 48.8 and 40.7; 6144 x 2048 68.9 and 60.7; 8192 x 1024 49.3 and 41.1; 32 of
    // 2048 x 2048, 25 rows 56 and 43; 16 of 4096 x 2048, 37 rows in 64 x 128 tiles 58.5 and 43.4; fp32, 16 of 5120 x 1024, 8 rows 63.0
    // and 53.0; 1024 x 2048 31.5 and 25.1.  With one set, part of it in the memory-side cache, 0.94 to 1.08 times as fast over these.  On rows
    // of other lengths it loses: 7168 x 1024 41.2 and 43.6, 1024 x 4096 70 and 72.
    a.spread = (int64_t)a.H * (F32 ? 4 : 2) % 4096 == 0 && rows_per_expert * 8 <= XR * 7;
    // Tile numbers go to the XCDs in blocks of 32, so that an XCD's tiles share rows and weights.  Up to two tiles per CU of one row tile per
    // expert in blocks of 8: an XCD reads about 1 TB/s, and half a block of 256 is four of them (one set of weights and three in turn, us: 8
    // experts of 4096 x 2560, 4 rows 33.0, 38.8, in eights 26.4, 34.4; 4 of 7168 x 3072, 32 rows 42.3, 55.7 and 37.1, 55.4; 2 of 4096 x
    // 4504, 20 rows 20.4 and 14.8; 32 of 1064 x 1616, one row 9.4, 10.8 and 10.0, 10.4; but 512 tiles, 8 of 4096 x 4096, 16 rows 40.0, 41.5 and, in fours, 41.8, 43.8; and with several row
    // tiles, 4 of 4096 x 2048, 100 rows, 20.0 and 20.7, one by one 38).
    a.deal = rows_per_expert <= XR && std::min<int64_t>(a.E, rows_bound) * ((a.N + WR - 1) / WR) < 512 ? 3 : 5;
    static LdsOptIn lds_opt_in;
    if (int rc = opt_in_lds(reinterpret_cast<const void *>(expert_short_kernel<XR, WR, NST, F32, FINE>), G::kLdsBytes, lds_opt_in)) return rc;
    const int64_t row_tiles = rows_bound / XR + std::min<int64_t>(a.E, rows_bound);
    const int64_t nct = (a.N + WR - 1) / WR;
    const int64_t grid = (row_tiles * nct + 32 * kXcds - 1) / (32 * kXcds) * (32 * kXcds);
    if (grid > 0x7fffffff) return MONTA_ERR_UNSUPPORTED;
    hipLaunchKernelGGL((expert_short_kernel<XR, WR, NST, F32, FINE>), dim3((unsigned)grid), dim3(256), G::kLdsBytes, st,
                       static_cast<const u32x4 *>(x_final), static_cast<const u32x4 *>(w_exp), y, a);
    return MONTA_OK;
}

template <int XB, int CB, int W, int NST, bool F32>
int launch_expert_split(const void *x_final, const void *w_exp, void *y, const ExpertArgs &a, int64_t rows_bound, hipStream_t st)
{
    using G = SplitTile<XB, CB, W, NST>;
    static LdsOptIn lds_opt_in;
    if (int rc = opt_in_lds(reinterpret_cast<const void *>(expert_split_kernel<XB, CB, W, NST, F32>), G::kLdsBytes, lds_opt_in)) return rc;
    const int64_t row_tiles = rows_bound / (16 * XB) + std::min<int64_t>(a.E, rows_bound), nct = (a.N + 16 * CB - 1) / (16 * CB);
    const int64_t grid = (row_tiles * nct + 8 * kXcds - 1) / (8 * kXcds) * (8 * kXcds);
    if (grid > 0x7fffffff) return MONTA_ERR_UNSUPPORTED;
    hipLaunchKernelGGL((expert_split_kernel<XB, CB, W, NST, F32>), dim3((unsigned)grid), dim3(G::kThreads), G::kLdsBytes, st,
                       static_cast<const u32x4 *>(x_final), static_cast<const u32x4 *>(w_exp), y, a);
    return MONTA_OK;
}

// Few tiles: with the hidden axis split, 1 if they are not few.  The tiles counted as in launch_expert_tiled.  Measured on MI355X over
// 64 shapes (2 to 64 experts, 1 to 616 rows per expert, 88 to 8192 elements, 64 to 5600 features, a third of them fp32; three sets of weights in
// turn), these lines and the 32 x 64 tiles beyond take 1.03 of the best of fourteen forms' time and 0.68 of those tiles' alone.
//  - 16 x 16 where experts have up to 32 rows, about one and a half tiles per CU (us in 32 x 64, 16 x 16, 16 x 32, 32 x 32: 4 experts of 4096 x
//    1024, 4 rows 15.7, 8.0, 8.1, 8.6; 16 of 2048 x 120, 14 rows 9.8, 4.6, 5.3, 6.0; 8 of 2048 x 704, 19 rows, 594 tiles 10.0, 8.8,
//    8.9, 7.4; 2 of 4096 x 4504, 20 rows, 987 tiles 15.8 in blocks of 8, 17.2, 17.9, 19.4); eight waves for long rows and half a tile
//    per CU (fp32, 8 of 8192 x 136: four waves 18.7, eight 14.1);
//  - 16 x 32, then 32 x 32, up to one tile per CU, where rows are more: 3 of 6176 x 336, 83 rows 21.9, 14.6, 12.5, 15.2; 4 of 8192 x 688,
//    47 rows 28.5, 19.7, 19.7, 14.5; but 2 of 5120 x 1984, 130 rows, 564 tiles of 32 x 32 25.1, 35.6, 31.5, 29.9.  An expert with rows has one
//    row tile at the least, which the estimate of its tiles falls short of where rows are less than half a tile's: a second round of few
//    tiles costs a whole walk (in 32 x 64 and 32 x 32: 8 of 2504 x 1352, 6 rows, 344 tiles 11.7, 15.6, 64 of 4096 x 152, 8 rows, 320
//    tiles 15.0, 18.8; fp32, 16 of 5788 x 784, 4 rows, 400 tiles 59.6, 73.5; in 32 x 64 and 16 x 32: 6 of 2504 x 1600, 5 rows 11.1, 12.9;
//    fp32, whose 32 x 64 tiles take longer, 19.2, 14.9 for 64 of 2000 x 192, one row, 384 tiles);
//  - fp32, whose MFMAs take four times as long, in 16 x 32 up to less than four tiles per CU if rows are more than one of 32 x 32, and up to
//    1300 where 32 x 64 tiles are past one per CU and take two walks' time (us in 32 x 64, 16 x 32: 3 of 4096 x 664, 121 rows, 507 tiles
//    50.9, 23.3; 2 of 2048 x 1836, 116 rows, 899 tiles 34.0, 24.8; 16 of 2048 x 340, 73 rows, 891 tiles 40.1, 27.5; beyond 4 of 2500 x
//    1020, 114 rows, 976 tiles 33.1, 37.9, 8 of 5788 x 1048, 75 rows, 1369 tiles 119, 152; with 317 tiles of 32 x 64 3 of 4096 x 2416, 73
//    rows, 1154 tiles 77.4, 56.2, with 400 32 of 8192 x 208, 84 rows, 1288 tiles 157, 142, with 345 2 of 2500 x 1320, 247 rows, 1338 tiles
//    51.5, 52.8; and 8 of 2172 x 1380, 20 rows 29, 39).  At the worst 1.16 of the better form's time (32 of 5788 x 160, 58 rows 72, 84);
//  - fp32 beyond these lines, up to about three tiles of 32 x 32 per CU: 32 x 64 with sums as exact as the split tiles' (FINE, error against 64
//    bits 2.1e-7 at 1024 to 8192 elements in split tiles);
//  - not on short walks (4 of 208 x 232, 467 rows 4.2, 9.0, 6.9, 6.7), up to 23 steps only where the tiles are fewest (32 of 1024 x 112,
//    4 rows, 168 tiles 5.9, 3.9; 2 of 512 x 4752, 3 rows, 408 tiles 5.2, 5.0, 4.8, 6.9, in blocks of 8 4.5).
template <bool F32>
int launch_expert_few(const void *x_final, const void *w_exp, void *y, const ExpertArgs &a, int64_t rows_bound, int64_t active, int64_t r,
                      hipStream_t st)
{
    auto tiles = [&](int64_t R, int64_t C) { return active * ((a.N + C - 1) / C) * (2 * r + R) / (2 * R); };
    auto whole_tiles = [&](int64_t R, int64_t C) { return std::max(tiles(R, C), active * ((a.N + C - 1) / C)); };
    const int64_t steps = ((int64_t)a.H * (F32 ? 4 : 2) + 127) / 128, small = tiles(16, 16);
    if (steps < 8 || (steps < 24 && small > 256)) return 1;
    if (steps >= 128 && small <= 128) return launch_expert_split<1, 1, 8, 4, F32>(x_final, w_exp, y, a, rows_bound, st);
    if (r <= 32 && small <= 400) return launch_expert_split<1, 1, 4, 3, F32>(x_final, w_exp, y, a, rows_bound, st);
    if ((F32 ? tiles(16, 32) : whole_tiles(16, 32)) <= 256) return launch_expert_split<1, 2, 4, 3, F32>(x_final, w_exp, y, a, rows_bound, st);
    if (whole_tiles(32, 32) <= 256) return launch_expert_split<2, 2, 4, 3, F32>(x_final, w_exp, y, a, rows_bound, st);
    if (F32 && r > 40 && (tiles(16, 32) <= 950 || (tiles(32, 64) > 272 && tiles(16, 32) <= 1300)))
        return launch_expert_split<1, 2, 4, 3, F32>(x_final, w_exp, y, a, rows_bound, st);
    if constexpr (F32)
        if (tiles(32, 32) <= (r > 40 ? 800 : 256))
            return r <= 24 ? launch_expert_short_t<32, 64, 4, true, true>(x_final, w_exp, y, a, rows_bound, r, st)
                           : launch_expert_short_t<32, 64, 3, true, true>(x_final, w_exp, y, a, rows_bound, r, st);
    return 1;
}

template <int BM, int BN, int WM, int WN>
int launch_expert(const void *x_final, const void *w_exp, void *y, ExpertArgs a, int64_t rows_bound, hipStream_t st)
{
    using G = ExpertTile<BM, BN, WM, WN>;
    static LdsOptIn lds_opt_in;
    if (int rc = opt_in_lds(reinterpret_cast<const void *>(expert_bf16_kernel<BM, BN, WM, WN>), G::kLdsBytes, lds_opt_in))
        return rc;
    const int64_t row_tiles = (rows_bound + BM - 1) / BM + a.E;      // each expert may end in a ragged tile
    const int64_t nct = (a.N + BN - 1) / BN;
    constexpr int64_t block = 32 * G::kWgsPerCu * kXcds;            // the kernel numbers its tiles in such blocks
    const int64_t grid8 = (row_tiles * nct + block - 1) / block * block;
    if (grid8 > 0x7fffffff) return MONTA_ERR_UNSUPPORTED;
    hipLaunchKernelGGL((expert_bf16_kernel<BM, BN, WM, WN>), dim3((unsigned)grid8), dim3(G::kThreads), G::kLdsBytes, st,
                       static_cast<const u32x4 *>(x_final), static_cast<const u32x4 *>(w_exp),
                       static_cast<unsigned short *>(y), a);
    return MONTA_OK;
}

// Which tile: with r rows per expert, a kernel of R x C tiles has about experts * (r / R + 1/2) * N / C of them, and a
// launch that leaves CUs idle is slower with large tiles than with small ones.  Measured on MI355X (us for tiles of 32 x 64,
// 64 x 128, 256 x 256, and the register-staged 128 x 256):
//   8 experts, 4096 x 4096:   r = 16: 41, 41, 45, 147   48: 57, 44, 45, 150   96: 90, 60, 82, 156   128: 109, 93, 87, 155
//   2 experts, 8192 x 8192:   r = 16: 40, 70, 71, 260   48: 58, 79, 77, 262   128: 108, 103, 148, 273   384: 257, 188, 193, 266
//   64 experts, 2048 x 2048:  r = 16: 98, 112, 123, 130   48: 128, 117, 131, 139   96: 181, 137, 142, 143   128: 225, 161, 144, 187
//   64 experts, 7168 x 2048:  r = 16: 310, 311, 309, 312   64: 511, 389, 333, 333   96: 630, 431, 341, 343   192: -, 671, 408, 590
// So a tile is taken where most experts fit one of its rows' tiles, or where its tiles number at most 2.5 per CU; on short rows,
// where a large tile's first loads and its stores weigh most, at most 5 per CU (64 experts, 1024 x 1024, r = 96: 45, 35, 38, 48;
// 128 experts, 512 x 512, r = 96: 33, 24, 37, 33).  The register-staged tile, which has no such rule of its own, is not taken on long
// rows (64 experts of 4096 x 2048, large tiles with their short ragged ones and it, three sets of weights in turn: r = 57 189 and 191, 76
// 195 and 197, with a skewed load 182 and 281, 217 and 287; 4992 x 2040, r = 66: 228 and 239), but
//  - on rows of at most 512 (128 experts, 512 x 512, r = 192: 56, 39, 43, 29; 256 experts: 120, 74, 57, 55, skewed 60, 35, 40, 32);
//  - on rows that are not whole steps, whose lines the large tile fetches twice, where an expert's second large tile would be
//    half empty (16 experts, 8184 x 2048, r = 300: 614, 378, 363, 326; 64 experts, 3000 x 1024: 472, 279, 285, 265; r = 1000: 1537,
//    773, 536, 614; r = 150: 270, 176, 121, 152);
//  - on such rows of up to 448 elements wherever the tiles are many, as a larger tile's walk is over before its loads are in flight
//    (64 experts, 32 x 4096, r = 844: 407, 254, 218, 154; 256 experts, 120 x 256, r = 175: 37, 24, 58, 20).  Up to 56 rows per expert
//    64 x 128 (256 experts, 88 x 3880, r = 19: 110, 79, 86, 85; 64 experts, 392 x 4096, r = 36: 54, 41, 52, 60), on rows of one step
//    only up to 8 (256 experts, 48 x 1024, r = 22: 27, 19, 25, 18); 32 x 64 up to 5 tiles per CU where r is at most 16 (256
//    experts, 48 x 4096, r = 4: 79, 60, 64, 59; 64 experts, 264 x 1184, r = 5: 10.9, 12.4, 15.3, 18.1).  Over 2600 shapes of such
//    rows the choice takes 1.01 of the best form's time;
//  - on such rows of up to 1104 elements and at most 256 features, one column tile (256 experts, 560 x 256, r = 196: 66, 44, 75, 37;
//    64 experts, 1032 x 256, r = 766: 97, 60, 60, 50).
int launch_expert_tiled(const void *x_final, const void *w_exp, void *y, const ExpertArgs &a, int64_t rows_bound,
                        int64_t kept_bound, hipStream_t st)
{
    const int64_t active = std::min<int64_t>(a.E, kept_bound), r = kept_bound / active;
    auto tiles = [&](int64_t R, int64_t C) { return active * ((a.N + C - 1) / C) * (2 * r + R) / (2 * R); };
    constexpr int64_t kFewTiles = 640, kFewTilesShortRows = 1300, kOddShortRow = 448, kOddNarrowRow = 1104;
    if (const int rc = launch_expert_few<false>(x_final, w_exp, y, a, rows_bound, active, r, st); rc <= 0) return rc;
    if (a.H % 64 && a.H <= kOddShortRow) {
        if (tiles(32, 64) <= (r <= 16 ? kFewTilesShortRows : kFewTiles)) return launch_expert_short_t<32, 64, 4>(x_final, w_exp, y, a, rows_bound, r, st);
        if (r <= (a.H <= 64 ? 8 : 56) || tiles(64, 128) <= kFewTilesShortRows)
            return launch_expert_short_t<64, 128, 3>(x_final, w_exp, y, a, rows_bound, r, st);
        return launch_expert<128, 256, 2, 2>(x_final, w_exp, y, a, rows_bound, st);
    }
    if (r <= 24 || tiles(32, 64) <= kFewTiles) return launch_expert_short_t<32, 64, 4>(x_final, w_exp, y, a, rows_bound, r, st);
    if (r <= 56 || tiles(64, 128) <= (a.H <= 1024 ? kFewTilesShortRows : kFewTiles))
        return launch_expert_short_t<64, 128, 3>(x_final, w_exp, y, a, rows_bound, r, st);
    if (a.H <= 512 && a.E <= 128 && r <= 384) return launch_expert<128, 256, 2, 2>(x_final, w_exp, y, a, rows_bound, st);
    if (a.H % 64 && a.H <= kOddNarrowRow && a.N <= kBigBN) return launch_expert<128, 256, 2, 2>(x_final, w_exp, y, a, rows_bound, st);
    if (a.H % 64 && r > kBigBM && r <= kBigBM * 3 / 2) return launch_expert<128, 256, 2, 2>(x_final, w_exp, y, a, rows_bound, st);
    return launch_expert_big(x_final, w_exp, y, a, rows_bound, r, st);
}

// fp32: tiles of 32 x 64, three stages, up to four workgroups per CU (up to 24 rows per expert, where the weights' trip from memory
// is what takes the time, four: 16 experts of 2048 x 1024, 2 rows 27.9 and 24.9 us; 8 of 1024 x 1024, 200 rows 42 and 52); 64 x 64 where most experts fit one tile's rows and not the
// half, which reads the weights once instead of twice, unless that leaves CUs without two tiles.  Measured on MI355X, 32 x 64 and
// 64 x 64, 48 rows per expert: 16 experts of 5120 x 2048 214 and 190 us, 256 of 512 x 512 99 and 91; 2 of 4096 x 4096 62 and 87, 8 of
// 516 x 516 10.9 and 15.5.  200 rows: 256 of 512 x 512 289 and 295, 64 of 1000 x 512 145 and 147.  Wider tiles, 32 x 128 and 64 x
// 128, were nowhere faster by more than 3 % and up to twice slower.
int launch_expert_f32(const void *x_final, const void *w_exp, void *y, const ExpertArgs &a, int64_t rows_bound,
                      int64_t kept_bound, hipStream_t st)
{
    if (a.H > kBigMaxHidden) {
        const int64_t row_tiles = rows_bound / kF32Tile + a.E, nct = (a.N + kF32Tile - 1) / kF32Tile;
        const int64_t grid = (row_tiles * nct + 32 * kXcds - 1) / (32 * kXcds) * (32 * kXcds);
        if (grid > 0x7fffffff) return MONTA_ERR_UNSUPPORTED;
        hipLaunchKernelGGL(expert_f32_kernel, dim3((unsigned)grid), dim3(256), 0, st, static_cast<const u32x4 *>(x_final),
                           static_cast<const u32x4 *>(w_exp), static_cast<float *>(y), a);
        return MONTA_OK;
    }
    const int64_t active = std::min<int64_t>(a.E, kept_bound), r = kept_bound / active;
    if (const int rc = launch_expert_few<true>(x_final, w_exp, y, a, rows_bound, active, r, st); rc <= 0) return rc;
    if (r > 32 && r <= 64 && active * ((a.N + 63) / 64) >= 512) return launch_expert_short_t<64, 64, 3, true>(x_final, w_exp, y, a, rows_bound, r, st);
    if (r <= 24) return launch_expert_short_t<32, 64, 4, true>(x_final, w_exp, y, a, rows_bound, r, st);
    return launch_expert_short_t<32, 64, 3, true>(x_final, w_exp, y, a, rows_bound, r, st);
}

int launch_route(const Geometry &g, const PlanPtrs &p, const float *logits, int32_t *topk_idx, float *gates,
                 hipStream_t st)
{
    const int per_lane = (g.s.E + g.s.rl - 1) / g.s.rl;
    auto launch = [&](auto lc, auto ne) -> int {
        constexpr int L = decltype(lc)::value, NE = decltype(ne)::value;
        static LdsOptIn lds_opt_in;
        if (g.route_lds > 48 * 1024)
            if (int rc = opt_in_lds(reinterpret_cast<const void *>(route_plan_kernel<L, NE>), (int)kRouteLdsBudget, lds_opt_in))
                return rc;
        ProfScope ps(MONTA_K_ROUTE, st);
        hipLaunchKernelGGL((route_plan_kernel<L, NE>), dim3(g.s.num_blocks), dim3(g.route_threads), g.route_lds, st, logits,
                           topk_idx, gates, p, g.s);
        HIP_TRY(hipGetLastError());
        return MONTA_OK;
    };
    auto with_groups = [&](auto lc) -> int {        // a lane's elements
        if (per_lane <= 8) return launch(lc, std::integral_constant<int, 8>{});
        if (per_lane <= 16) return launch(lc, std::integral_constant<int, 16>{});
        // one or two lanes share a token only below 16 and 32 experts, four or eight have at most 28 and 32 each (LDS budget)
        if constexpr (decltype(lc)::value >= 4)
            if (per_lane <= 32) return launch(lc, std::integral_constant<int, 32>{});
        return MONTA_ERR_UNSUPPORTED;
    };
    int rc;
    if (g.s.rl == 1) rc = with_groups(std::integral_constant<int, 1>{});
    else if (g.s.rl == 2) rc = with_groups(std::integral_constant<int, 2>{});
    else if (g.s.rl == 4) rc = with_groups(std::integral_constant<int, 4>{});
    else rc = with_groups(std::integral_constant<int, 8>{});
    if (rc || g.s.fast_plan) return rc;
    ProfScope ps(MONTA_K_SCAN, st);
    hipLaunchKernelGGL(block_scan_kernel, dim3((g.s.E + kScanExperts - 1) / kScanExperts), dim3(kScanExperts * kWave), 0, st, p, g.s);
    HIP_TRY(hipGetLastError());
    return MONTA_OK;
}

// Do the bytes [a, a + na) and [b, b + nb) share any?
bool overlap(const void *a, int64_t na, const void *b, int64_t nb)
{
    const uintptr_t pa = reinterpret_cast<uintptr_t>(a), pb = reinterpret_cast<uintptr_t>(b);
    return pa < pb + (uintptr_t)nb && pb < pa + (uintptr_t)na;
}

// Lanes per token of small_step_kernel, 0 if the problem is not a small one: all tokens have to be covered by one pass of a
// workgroup's threads, their choices and the plan by its LDS.  And routing them all in every workgroup must not take longer than
// routing a share of them and waiting for the others, which grows with tokens x experts and, where each row's workgroup does it, with
// the choices.  Measured on MI355X, GPU time in us, several launches and one: routing 64 x 8, top-2 8.2 and 4.3; 128 x 64, top-8 9.2 and 7.8,
// 256 x 64 9.5 and 11.0; 512 x 16, top-2 8.4 and 6.2, top-8 10.6 and 11.7, 512 x 32, top-4 8.7 and 9.5; 64 x 256, top-8 12.0 and 9.0;
// 1024 x 8 8.3 and 7.1.  With the rows (4096 elements): 64 x 8, top-2 8.8 and 5.2, 512 x 8 10.7 and 7.7, 1024 x 8 12.5 and 13.2; 256 x 32, top-4
// 11.2 and 10.1, 512 x 32 12.9 and 13.1; 128 x 64, top-8 11.9 and 12.7, 256 x 64 13.5 and 15.7; 512 x 16, top-8 19.4 and 17.2.  The
// whole step, which takes the same line, could take one launch further: 64 x 8 12.0 and 6.4, 512 x 8 15.8 and 9.0, 128 x 64, top-8 17.2 and
// 14.6, 512 x 32, top-4 18.7 and 14.8, 1024 x 8 19.3 and 15.5.
constexpr int kSmallTokens = 512, kSmallUnits = 4096, kSmallPerLogits = 8192, kSmallPerChoices = 32768, kSmallAnyway = 64;
int small_lanes(const Geometry &g, bool rows)
{
    const Shape &s = g.s;
    if (g.modes.plan >= 0 || s.T > kSmallTokens || (int64_t)s.U * s.E > kSmallUnits) return 0;
    if (s.T > kSmallAnyway && (s.T * s.E > kSmallPerLogits || (rows && s.T * s.E * s.k > kSmallPerChoices))) return 0;
    int L = 1;
    while (L < 16 && s.E / (2 * L) >= 8 && s.T * 2 * L <= 1024) L *= 2;
    const int per_lane = (s.E + L - 1) / L;
    if (s.T * L > 1024 || per_lane > 16 || small_lds(s.T, s.E, s.k, s.U).bytes > (int)kRouteLdsBudget) return 0;
    return L;
}

int launch_small(const Geometry &g, const PlanPtrs &p, int L, SmallWhat what, const float *logits, const void *x, int32_t *topk_idx,
                 float *gates, void *stage, void *final_, void *out, bool bf16, hipStream_t st)
{
    const Shape &s = g.s;
    int threads = kMoverThreads;
    while (threads < s.T * L || (threads < 1024 && threads < s.U * kWave)) threads *= 2;     // a wave per unit, up to 16
    const int rows = threads / s.lpr;
    const unsigned grid = 3 + (what == SMALL_ROUTE ? 0u : (unsigned)((s.T + rows - 1) / rows));
    const SmallLds lay = small_lds(s.T, s.E, s.k, s.U);
    const size_t lds = (size_t)lay.bytes;
    const int per_lane = (s.E + L - 1) / L;
    auto launch = [&](auto lc, auto ne) -> int {
        constexpr int LN = decltype(lc)::value, NE = decltype(ne)::value;
        static LdsOptIn lds_opt_in;
        if (lds > 48 * 1024)
            if (int rc = opt_in_lds(reinterpret_cast<const void *>(small_step_kernel<LN, NE>), (int)kRouteLdsBudget, lds_opt_in)) return rc;
        ProfScope ps(MONTA_K_SMALL_STEP, st);
        hipLaunchKernelGGL((small_step_kernel<LN, NE>), dim3(grid), dim3(threads), lds, st, logits, static_cast<const u32x4 *>(x), topk_idx,
                           gates, static_cast<u32x4 *>(stage), static_cast<u32x4 *>(final_), static_cast<u32x4 *>(out), p, s, lay, (int)what,
                           bf16 ? 1 : 0);
        HIP_TRY(hipGetLastError());
        return MONTA_OK;
    };
    auto with_groups = [&](auto lc) -> int {        // a lane's elements: the limits above leave it 16 at most
        return per_lane <= 8 ? launch(lc, std::integral_constant<int, 8>{}) : launch(lc, std::integral_constant<int, 16>{});
    };
    if (L == 1) return with_groups(std::integral_constant<int, 1>{});
    if (L == 2) return with_groups(std::integral_constant<int, 2>{});
    if (L == 4) return with_groups(std::integral_constant<int, 4>{});
    if (L == 8) return with_groups(std::integral_constant<int, 8>{});
    return with_groups(std::integral_constant<int, 16>{});
}

// May workgroups store while others still read the logits and the rows (small_step_kernel)?  Only if nothing that is stored shares
// memory with what is read; the launches one after the other read a workgroup's logits before it stores, and all of them before a
// row is stored.  A buffer that the call does not have is null; the plan tables are null, too, where they are the library's own.
bool small_apart(const Geometry &g, const float *logits, const int32_t *topk_idx, const float *gates, const void *ws, const void *x = nullptr,
                 const void *stage = nullptr, const void *final_ = nullptr, const void *out = nullptr)
{
    struct Range {
        const void *p;
        int64_t n;
    };
    const Shape &s = g.s;
    const int64_t xb = (int64_t)s.T * g.row_bytes, fb = g.max_rows * g.row_bytes, tk = (int64_t)s.T * s.k * 4;
    const Range read[] = {{logits, (int64_t)s.T * s.E * 4}, {x, xb}};
    const Range stored[] = {{topk_idx, tk}, {gates, tk}, {stage, fb}, {final_, fb}, {out, xb}, {ws, ws_bytes(g)}};
    auto share = [](const Range &a, const Range &b) { return a.p && b.p && overlap(a.p, a.n, b.p, b.n); };
    constexpr int kStored = sizeof(stored) / sizeof(stored[0]);
    for (int i = 0; i < kStored; ++i) {
        for (const Range &r : read)
            if (share(r, stored[i])) return false;
        for (int j = 0; j < i; ++j)                 // what two launches would store one after the other
            if (share(stored[i], stored[j])) return false;
    }
    return true;
}

int check_ws(const void *ws)
{
    if (!ws) return MONTA_ERR_NULL;
    if (misaligned(ws, 16)) return MONTA_ERR_ALIGN;
    return MONTA_OK;
}

int check_route_ptrs(const float *logits, const int32_t *topk_idx, const float *gates, const void *ws)
{
    if (!logits || !topk_idx || !gates) return MONTA_ERR_NULL;
    if (misaligned(logits, 4) || misaligned(topk_idx, 4) || misaligned(gates, 4)) return MONTA_ERR_ALIGN;
    return check_ws(ws);
}

int check_expert_args(const monta_cfg *cfg, const Geometry &g, const void *x_final, const void *w_exp, int32_t out_features,
                      const void *y, const void *ws, int slice)
{
    if (!x_final || !w_exp || !y || !ws) return MONTA_ERR_NULL;
    if (misaligned(x_final, 16) || misaligned(w_exp, 16) || misaligned(y, 16) || misaligned(ws, 16)) return MONTA_ERR_ALIGN;
    const int bpe = cfg->dtype == MONTA_BF16 ? 2 : 4;
    if (out_features < 1 || ((int64_t)out_features * bpe) % 16 != 0) return MONTA_ERR_INVALID;
    if (slice < -1 || slice >= g.s.S) return MONTA_ERR_INVALID;
    if (x_final == y) return MONTA_ERR_INVALID;
    return MONTA_OK;
}

constexpr double kStreamWeightsFrom = 240 << 20, kCacheableWeights = 96 << 20;

int launch_expert_layer(const monta_cfg *cfg, const Geometry &g, const void *x_final, const void *w_exp, int32_t out_features,
                        void *y, const void *ws, int slice, hipStream_t st)
{
    const Shape &s = g.s;
    int rc = MONTA_OK;
    PlanPtrs p = plan_ptrs(g, const_cast<void *>(ws));
    ExpertArgs a;
    a.spread = 0;
    a.E = (int16_t)s.E;
    a.H = cfg->hidden;
    a.N = out_features;
    a.max_rows = s.max_rows;
    // Weights about as large as the memory-side cache (256 MiB) do not stay in it from one call to the next as a whole.  A part of 96 MiB
    // does, if the rest is streamed past it, and it costs nothing where other weights come between two calls.  8 experts of
    // 4096 x 4096, 256 MiB, 16 rows, one set of weights used again, three in turn, five: plain 40.7, 54.1, 54.2 us, all streamed
    // 46.6, 47.5, 47.4, all but 96 MiB 39.9, 47.3, 48.9; 16 of 2048 x 6144, 384 MiB 78, 77, 76, then 68, 68, 67 and 64, 68, 69; over 30
    // shapes of 240 to 512 MiB the part is 0.82 to 1.05 of the better of the other two with one set, 0.97 to 1.03 with five.
    // The line lies at 240 MiB (8 of 4096 x 3840, 16 rows: 38.1, 49.7, 49.8, all but 96 MiB 39.2, 44.1, 45.2); below it plain weights stay whole:
    // 16 of 2048 x 2048, 128 MiB, 40 rows 21.5, 33.8 in turn, all streamed 28.7, 30.1.
    // What counts are the weights of the experts that have rows, in the mean of an even load (16 tokens, top-4 of 64, 5120 x 464: 290
    // MiB, 40 experts with rows, one set 21.8 us and, by all 64, 24.1); as nobody knows which, each row of the weights has the same
    // share.
    // Rows and base have to be whole 128-byte lines.
    const int64_t w_row = (int64_t)cfg->hidden * (cfg->dtype == MONTA_BF16 ? 2 : 4);
    const int64_t w_rows = (int64_t)s.E * out_features, kept_bound = std::min<int64_t>((int64_t)s.T * s.k, (int64_t)s.E * s.C);
    const double with_rows = s.E * (1.0 - std::pow(1.0 - 1.0 / s.E, (double)kept_bound)), touched = with_rows * out_features * w_row;
    a.stream_from = touched >= kStreamWeightsFrom && w_row % 128 == 0 && !misaligned(w_exp, 128)
                        ? (int64_t)(w_rows * (kCacheableWeights / touched)) : w_rows;
    // rows of expert e: its whole kept segment [offsets[e], offsets[e] + kept[e]), or the part of it filled by the
    // slice's units, which starts at unit_base[first unit of the slice][e] and ends where the next slice's starts
    a.lo = slice < 0 ? p.offsets : p.unit_base + (int64_t)slice * s.tp * s.E;
    if (slice >= 0 && slice + 1 < s.S) {
        a.hi_base = p.unit_base + (int64_t)(slice + 1) * s.tp * s.E;
        a.hi_len = nullptr;
    } else {
        a.hi_base = p.offsets;
        a.hi_len = p.kept;
    }
    // worst case of the rows in play: every pair of the slice's tokens kept, as far as the capacity lets them (the rows of a
    // padded layout beyond them are never multiplied)
    const int64_t rows_bound = slice < 0 ? kept_bound : std::min<int64_t>(kept_bound, (int64_t)(s.T / s.S) * s.k);
    ProfScope ps(MONTA_K_EXPERT, st);
    if (cfg->dtype == MONTA_BF16) {
        // The offsets inside a direct-to-LDS tile have 31 bits.  The choice of tile looks at the whole problem, not at the slice,
        // so that a slice runs as the whole would.
        if (cfg->hidden <= kBigMaxHidden)
            rc = launch_expert_tiled(x_final, w_exp, y, a, rows_bound, kept_bound, st);
        else
            rc = launch_expert<128, 256, 2, 2>(x_final, w_exp, y, a, rows_bound, st);
        if (rc) return rc;
    } else {
        rc = launch_expert_f32(x_final, w_exp, y, a, rows_bound, kept_bound, st);
        if (rc) return rc;
    }
    HIP_TRY(hipGetLastError());
    return MONTA_OK;
}

// How the two passes of the slice pipeline are launched where they are kept apart (single_pass() says when they are not):
// the realisation (0, 1 or 2) and how many consecutive slices one launch covers.
struct PipePlan {
    int mode;
    int first;      // slices in the first launch group
    int spg;        // slices in every later group
};

// What the calls do.  An explicit mode keeps one slice per launch.  With the default they come here only because FINAL shares
// memory with x: every row of x has to be packed before the first row of FINAL is written, so one launch packs all slices and
// the next regathers them.
PipePlan pipeline_plan(const Geometry &g)
{
    if (g.modes.pipeline >= 0) return {g.modes.pipeline, 1, 1};
    return {1, g.s.S, g.s.S};
}

// Can the kernel that finishes the plan also pack (plan_pack_kernel)?  It needs a histogram table small enough to
// rebuild in every pack workgroup and token groups that never straddle two route workgroups.
bool plan_pack_shape_ok(const Geometry &g)
{
    const Shape &s = g.s;
    const int rows_per_wg = kMoverThreads / s.lpr;
    return s.fast_plan && (int64_t)s.num_blocks * s.E <= 2048 && s.Tu % s.TB == 0 && rows_per_wg <= s.TB &&
           kMoverThreads >= s.TB;
}

// By default the dispatch runs in one pass (place_kernel): each row is read once and stored to its rows in STAGE and in
// FINAL.  An explicit pipeline mode asks for the two passes, and they are kept where FINAL shares memory with x: rows of x
// still to be read would be overwritten (pipeline_plan() then packs everything first).
bool single_pass(const Geometry &g, const void *x, const void *final_)
{
    return g.modes.pipeline < 0 && !overlap(x, (int64_t)g.s.T * g.row_bytes, final_, g.max_rows * g.row_bytes);
}

// Cache policy of the single pass: nothing reads STAGE again, so its stores stream; x and FINAL stay cacheable (the combine
// or the experts read FINAL next).  Measured against the other seven choices, step of 8192 x 8 KiB rows, top-2: 90 us
// against 94-120, of 8192 x 16 KiB, top-1: 106 against 107-139; beyond the memory-side cache the choice moves 1-3 %.
// lazy: a capacity below the number of tokens may leave tokens without a kept choice, and their rows need not be read.  Not where
// the capacity is twice an even load, which rarely drops anything, nor where all of x is small.  Measured on MI355X, dispatch alone:
// 31880 x 16 KiB on 64 experts, top-1, a Zipf load at 1.25, 83 % dropped 146 -> 58 us; 43712 x 14 KiB, top-2, 78 % dropped 238 -> 162;
// 5952 x 16 KiB 43 -> 33; with nothing dropped 0.97 to 1.01 of the time over 40 shapes.
Shape place_shape(const Geometry &g)
{
    Shape s = g.s;
    if (g.modes.cache < 0) s.cache = NT_PACK_ST;
    s.lazy = s.C < s.T && (int64_t)s.C * s.E < 2 * (int64_t)s.T * s.k && (int64_t)s.T * g.row_bytes >= (16 << 20);
    return s;
}

int launch_place(const Geometry &g, const PlanPtrs &p, const void *x, void *stage, void *final_, hipStream_t st)
{
    const Shape s = place_shape(g);
    ProfScope ps(MONTA_K_PLACE, st);
    const dim3 grid(mover_grid(s, s.T)), block(kMoverThreads);
    const u32x4 *xv = static_cast<const u32x4 *>(x);
    u32x4 *sv = static_cast<u32x4 *>(stage), *fv = static_cast<u32x4 *>(final_);
    if (s.lpr >= kWave) hipLaunchKernelGGL(place_kernel<true>, grid, block, 0, st, xv, sv, fv, p, s);
    else hipLaunchKernelGGL(place_kernel<false>, grid, block, 0, st, xv, sv, fv, p, s);
    HIP_TRY(hipGetLastError());
    return MONTA_OK;
}

// Tokens per workgroup of plan_place_kernel, 0 if the shape is better served (or only served) by the plan and the rows in
// kernels of their own.  The tokens of a workgroup must belong to one route workgroup; one round of resident workgroups
// rebuilds the plan once each, more rows per workgroup keep it at one round.
int plan_place_span(const Geometry &g)
{
    const Shape &s = g.s;
    // A table that every workgroup reduces must be small.  Otherwise the rows' own time decides: a launch less is worth it for
    // short jobs, long ones run better in the plain kernel, whose workgroups take their rows in order.  Scans there already: 2048
    // tokens x 2 KiB, top-8 of 256 45.6 -> 39.9 us, 32768 x 512 B, 285 MB 92.6 -> 85.9, but 8192 x 4 KiB, 570 MB 113.6 -> 116.3.  A
    // small table, whole step in one kernel and in two over 80 shapes: from 1 GiB on two are never behind (1205 MiB 396 and 349 us,
    // 1688 MiB 542 and 487, 2619 MiB 797 and 775, 1.00 to 1.14 times).  Below it bytes part them poorly, 0.92 to 1.31 times: mostly one
    // leads (168 MiB 46.7 and 49.5, 492 MiB 139 and 144), but not on some rows of 2 to 8 KiB, several to a workgroup (29184 x 4 KiB,
    // top-2, 570 MiB 213 and 167; 25088 x 8 KiB, 980 MiB 311 and 269).
    if (s.fast_plan && (int64_t)s.num_blocks * s.E > 2048) return 0;
    if (((int64_t)s.T + 2 * slice_rows_bound(g, s.S)) * g.row_bytes > (s.fast_plan ? 1024ll : 320ll) << 20) return 0;
    auto fits = [&](int span) { return span <= s.TB && s.TB % span == 0 && (s.Tu % span == 0 || s.U == 1); };
    int span = kMoverThreads / s.lpr;
    if (!fits(span)) return 0;
    while ((s.T + span - 1) / span > kResidentMoverWgs && fits(2 * span)) span *= 2;
    return span;
}

int launch_plan_place(const Geometry &g, const PlanPtrs &p, int span, const int32_t *topk_idx, const void *x, void *stage,
                      void *final_, hipStream_t st)
{
    const Shape s = place_shape(g);
    ProfScope ps(MONTA_K_PLAN_PLACE, st);
    const dim3 grid(s.num_blocks + (s.T + span - 1) / span), block(kMoverThreads);
    const u32x4 *xv = static_cast<const u32x4 *>(x);
    u32x4 *sv = static_cast<u32x4 *>(stage), *fv = static_cast<u32x4 *>(final_);
    if (s.lpr >= kWave)
        hipLaunchKernelGGL(plan_place_kernel<true>, grid, block, 0, st, topk_idx, xv, sv, fv, p, s, span, s.num_blocks);
    else
        hipLaunchKernelGGL(plan_place_kernel<false>, grid, block, 0, st, topk_idx, xv, sv, fv, p, s, span, s.num_blocks);
    HIP_TRY(hipGetLastError());
    return MONTA_OK;
}

// What monta_pipeline_query answers.  With the default mode, whose calls launch no groups, it is the grouping that suits the
// sizes for a program that issues the passes itself, as the paper's planner chooses its chunk count from the traffic (section
// "Network-traffic-aware"): measured on MI355X,
//  - a launch boundary costs a few microseconds of idle memory system, so slices that move only tens of
//    megabytes are grouped until a launch's share of STAGE reaches 256 MiB (the size of the memory-side cache:
//    what the pack writes is still there when the regather reads it); a problem that fits one group runs as
//    plan + pack of everything, then one regather;
//  - co-scheduling pack(j) with regather(j-1) in one grid saves a boundary per slice, which decides it while
//    a group's copies take a few tens of microseconds; once they take hundreds, two plain kernels run faster
//    than the mixed grid (the regather alone reaches 6.6-7.0 TB/s, the mixed grid 6.2-6.7).
PipePlan grouping_by_size(const Geometry &g)
{
    if (g.modes.pipeline >= 0) return pipeline_plan(g);
    const int S = g.s.S;
    const int64_t slice_bytes = slice_rows_bound(g, 1) * g.row_bytes;      // what one slice may put into STAGE
    if (slice_bytes >= kGroupBytes) return {2, 1, 1};
    int spg = (int)(kGroupBytes / slice_bytes);
    if (spg > S) spg = S;
    int groups = (S + spg - 1) / spg;
    spg = (S + groups - 1) / groups;                                       // even groups
    if (groups > 1) return {spg * slice_bytes >= kGroupBytes * 3 / 4 ? 2 : 1, spg, spg};
    // Everything fits one group.  The pack workgroups of the fused plan-and-pack kernel each rebuild the plan's
    // scans before their first store; with one round of them resident on the chip that hides behind the row
    // reads, with several rounds it is paid every round (measured: 8192 of them pack 192 MiB at 5.0 TB/s, the
    // plain pack at 6.3).  So the first launch takes about one round of workgroups (whole slices), the rest
    // of the slices form the second group: plan + pack(first), pack(rest) with regather(first), regather(rest).
    if (!plan_pack_shape_ok(g) || S == 1) return {1, S, S};
    const int64_t round_tokens = (int64_t)kResidentMoverWgs * (kMoverThreads / g.s.lpr);
    int first = (int)(round_tokens / ((int64_t)g.s.tp * g.s.Tu));
    if (first < 1) first = 1;
    if (first >= S) first = S - 1;
    return {1, first, S - first};
}

int route_impl(const Geometry &g, const float *logits, int32_t *topk_idx, float *gates, void *ws, hipStream_t st)
{
    const Shape &s = g.s;
    PlanPtrs p = plan_ptrs(g, ws);
    const int L = small_lanes(g, false);
    if (L && small_apart(g, logits, topk_idx, gates, ws))
        return launch_small(g, p, L, SMALL_ROUTE, logits, nullptr, topk_idx, gates, nullptr, nullptr, nullptr, false, st);
    if (int rc = launch_route(g, p, logits, topk_idx, gates, st)) return rc;
    ProfScope ps(MONTA_K_POSITIONS, st);
    hipLaunchKernelGGL(plan_positions_kernel, dim3(s.num_blocks), dim3(kPlanThreads), 0, st, topk_idx, p, s);
    HIP_TRY(hipGetLastError());
    return MONTA_OK;
}

// the pipeline from group `first` on (group 0 may have been packed already by the kernel that finishes the plan)
int pipeline_impl(const Geometry &g, const PipePlan &pp, const void *x, void *stage, void *final_, const void *ws,
                  bool group0_packed, hipStream_t st)
{
    int rc = MONTA_OK;
    const PlanPtrs p = plan_ptrs(g, ws);
    const int S = g.s.S;
    const int first = pp.first < S ? pp.first : S, spg = pp.spg;
    auto lo = [&](int gi) { return gi == 0 ? 0 : first + (gi - 1) * spg; };
    auto hi = [&](int gi) { const int h = first + gi * spg; return h < S ? h : S; };
    const int G = 1 + (S - first + spg - 1) / spg;
    if (pp.mode == 2) {
        for (int gi = 0; gi < G; ++gi) {
            if (!(gi == 0 && group0_packed))
                if ((rc = launch_pack(g, p, x, stage, lo(gi), hi(gi), st))) return rc;
            if ((rc = launch_regather(g, p, stage, final_, lo(gi), hi(gi), st))) return rc;
        }
        return MONTA_OK;
    }
    if (pp.mode == 1) {
        if (!group0_packed)
            if ((rc = launch_pack(g, p, x, stage, lo(0), hi(0), st))) return rc;
        for (int gi = 1; gi < G; ++gi)
            if ((rc = launch_pack_regather(g, p, x, stage, final_, lo(gi), hi(gi), lo(gi - 1), hi(gi - 1), st))) return rc;
        return launch_regather(g, p, stage, final_, lo(G - 1), hi(G - 1), st);
    }
    // mode 0: packs on the caller's stream, regathers on the side stream, one event per slice.  The side stream
    // and its events are shared by every caller on this device: the whole enqueue holds the device's lock, so
    // that each wait pairs with the record made just before it (a wait refers to the event's latest record at
    // the time the wait is enqueued; what another call records later does not change it).
    DevState *d = nullptr;
    if ((rc = dev_state(G, &d))) return rc;
    std::lock_guard<std::mutex> lk(d->mu);
    for (int gi = 0; gi < G; ++gi) {
        if (!(gi == 0 && group0_packed))
            if ((rc = launch_pack(g, p, x, stage, lo(gi), hi(gi), st))) return rc;
        HIP_TRY(hipEventRecord(d->ev[gi], st));
        HIP_TRY(hipStreamWaitEvent(d->side, d->ev[gi], 0));
        prof_break_chain(d->side);
        if ((rc = launch_regather(g, p, stage, final_, lo(gi), hi(gi), d->side))) return rc;
    }
    HIP_TRY(hipEventRecord(d->done, d->side));
    HIP_TRY(hipStreamWaitEvent(st, d->done, 0));
    prof_break_chain(st);
    return MONTA_OK;
}

int dispatch_regather_impl(const Geometry &g, const void *x, void *stage, void *final_, const void *ws, hipStream_t st)
{
    if (single_pass(g, x, final_)) return launch_place(g, plan_ptrs(g, ws), x, stage, final_, st);
    return pipeline_impl(g, pipeline_plan(g), x, stage, final_, ws, false, st);
}

// Does monta_route_dispatch_regather finish the plan and pack the first launch group in one grid?  An explicit
// mode 0 or 2 keeps the plain sequence of kernels.
bool plan_pack_fused(const Geometry &g, const PipePlan &pp)
{
    return pp.mode != 0 && (pp.mode == 1 || g.modes.pipeline < 0) && plan_pack_shape_ok(g);
}

int route_dispatch_regather_impl(const Geometry &g, const float *logits, const void *x, int32_t *topk_idx, float *gates,
                                 void *stage, void *final_, void *ws, hipStream_t st)
{
    int rc = MONTA_OK;
    const Shape &s = g.s;
    if (single_pass(g, x, final_)) {
        const PlanPtrs p = plan_ptrs(g, ws);
        const int L = g.modes.cache < 0 ? small_lanes(g, true) : 0;
        if (L && small_apart(g, logits, topk_idx, gates, ws, x, stage, final_))
            return launch_small(g, p, L, SMALL_PLACE, logits, x, topk_idx, gates, stage, final_, nullptr, false, st);
        if (const int span = plan_place_span(g)) {
            if ((rc = launch_route(g, p, logits, topk_idx, gates, st))) return rc;
            return launch_plan_place(g, p, span, topk_idx, x, stage, final_, st);
        }
        if ((rc = route_impl(g, logits, topk_idx, gates, ws, st))) return rc;
        return launch_place(g, p, x, stage, final_, st);
    }
    const PipePlan pp = pipeline_plan(g);
    const int rows_per_wg = kMoverThreads / s.lpr;
    if (!plan_pack_fused(g, pp)) {
        if ((rc = route_impl(g, logits, topk_idx, gates, ws, st))) return rc;
        return pipeline_impl(g, pp, x, stage, final_, ws, false, st);
    }
    PlanPtrs p = plan_ptrs(g, ws);
    if ((rc = launch_route(g, p, logits, topk_idx, gates, st))) return rc;
    {
        const int nt = (pp.first < s.S ? pp.first : s.S) * s.tp * s.Tu;      // tokens of the first group
        const int n_pack = (nt + rows_per_wg - 1) / rows_per_wg;           // one token group per workgroup, no striding
        ProfScope ps(MONTA_K_PLAN_PACK, st);
        hipLaunchKernelGGL(plan_pack_kernel, dim3(s.num_blocks + n_pack), dim3(kMoverThreads), 0, st, topk_idx,
                           static_cast<const u32x4 *>(x), static_cast<u32x4 *>(stage), p, s, 0, nt, s.num_blocks);
        HIP_TRY(hipGetLastError());
    }
    return pipeline_impl(g, pp, x, stage, final_, ws, true, st);
}

int64_t combine_unit_count(const Shape &s)
{
    const int tokens = s.vpr >= kWave ? 1 : kWave / s.lpr;          // of a wave
    return s.vpr >= kWave ? (int64_t)s.T * ((s.vpr + kWave - 1) / kWave) : (s.T + tokens - 1) / tokens;
}
// How many choices combine_units_t has on their way, 0 where the forms of 256 lanes per row are the better ones.  Measured on MI355X, the
// combine alone (three sets in turn, us, 256 lanes and a wave per 64 vectors; bf16 unless said):
//  - rows of up to 4 KiB: 7500 x 1632, top-2 20.4 and 16.5; 30000 x 1024, top-2 39.2 and 32.5; 8000 x 512, top-8 17.4 and 13.8;
//    60000 x 2048, top-1 100 and 96;
//  - longer ones that leave more than three tenths of the lanes' vectors unused: 30595 x 5120, top-3 226 and 204; 8407 x 5008, top-3 64 and
//    57; but 4876 x 5120, fp32, top-2, half of it dropped 29.4 and 32.1, and with full lanes 30000 x 4096, top-2 120 and 123, 65536 x 7168,
//    top-8, half dropped 712 and 735;
//  - few tokens, whose chain of row after row is what takes the time: 492 x 4096, top-8 9.0 and 5.6; 285 x 3200, top-6 7.2 and 4.5; 675 x
//    8192, top-8 19.0 and 18.2; but top-1, 1123 x 7168 7.0 and 7.7.
// Eight rows on their way pay where waves are few (500 x 512, top-8, two 4.9, eight 4.0; 8000 x 512 13.8 and 14.3).  Over 150 shapes 1.08
// times as fast.  The return path, which also stores the rows, gains less (13347 x 1024, top-3 13.7 and 12.0; 3658 x 132, fp32, top-6 6.1 and 5.2)
// and loses with one or two choices on rows of 4 KiB (39259 x 1024, fp32, top-2 141 and 146; 335 x 4096, fp32 5.4 and 5.8).
int combine_units(const Shape &s, bool bf16, bool returned)
{
    if (s.k > s.lpr) return 0;
    const bool few = combine_unit_count(s) <= 4096;
    if (s.vpr <= kMoverThreads) {
        if (returned && s.k <= 2 && s.vpr > 192 && !few) return 0;
    } else if (s.k < 2) {
        return 0;
    } else if (s.T <= 1024) {
        if (returned && s.k == 2 && !few) return 0;
    } else {
        const int pass = kMoverThreads * (s.vpr > 2 * kMoverThreads ? 4 : 2);
        if (s.vpr * 10ll > (s.vpr + pass - 1) / pass * pass * 7ll) return 0;
        if (!bf16 && (returned || (s.C < s.T && (int64_t)s.C * s.E < 2ll * s.T * s.k))) return 0;
    }
    return s.k > 2 && (few || s.T <= 1024) ? 8 : 2;
}
dim3 combine_units_grid(const Shape &s)
{
    constexpr int kPerWg = kMoverThreads / kWave;
    return dim3((unsigned)std::min<int64_t>((combine_unit_count(s) + kPerWg - 1) / kPerWg, 1 << 20));
}
// launch(is bf16, choices on their way at a time, rows of whole waves)
template <typename F>
void with_units(int dtype, const Shape &s, int K, F launch)
{
    auto by_k = [&](auto bf, auto wave) {
        if (K == 8) launch(bf, std::integral_constant<int, 8>{}, wave);
        else launch(bf, std::integral_constant<int, 2>{}, wave);
    };
    auto by_rows = [&](auto bf) {
        if (s.vpr >= kWave) by_k(bf, std::true_type{});
        else by_k(bf, std::false_type{});
    };
    if (dtype == MONTA_BF16) by_rows(std::true_type{});
    else by_rows(std::false_type{});
}

int combine_impl(const Geometry &g, int dtype, const void *y, const float *gates, void *out, const void *ws, hipStream_t st)
{
    const Shape &s = g.s;
    const PlanPtrs p = plan_ptrs(g, ws);
    ProfScope ps(MONTA_K_COMBINE, st);
    const dim3 grid(mover_grid(s, s.T)), block(kMoverThreads);
    const bool wide = s.vpr > 2 * s.lpr;   // more than two vectors per lane: 4 per pass
    const u32x4 *yv = static_cast<const u32x4 *>(y);
    u32x4 *ov = static_cast<u32x4 *>(out);
    if (const int K = combine_units(s, dtype == MONTA_BF16, false)) {
        const dim3 ugrid = combine_units_grid(s);
        with_units(dtype, s, K, [&](auto bf, auto kc, auto wave) {
            hipLaunchKernelGGL((combine_units_kernel<decltype(bf)::value, decltype(kc)::value, decltype(wave)::value>), ugrid, block, 0, st, yv, gates,
                               ov, p, s);
        });
        HIP_TRY(hipGetLastError());
        return MONTA_OK;
    }
    // Otherwise, with three or more choices per token, the software-pipelined form wins (measured on MI355X, 65536 tokens of
    // 14 KiB, top-8 with drops: 802 -> 707 us); with one or two there is nothing to pipeline and its extra
    // registers cost 2-4 %.  It needs the token's k positions to fit the lanes that share its row.
    if (s.k >= 3 && s.k <= s.lpr) {
        if (dtype == MONTA_BF16) {
            if (wide) hipLaunchKernelGGL((combine_pf_kernel<true, 4>), grid, block, 0, st, yv, gates, ov, p, s);
            else hipLaunchKernelGGL((combine_pf_kernel<true, 2>), grid, block, 0, st, yv, gates, ov, p, s);
        } else {
            if (wide) hipLaunchKernelGGL((combine_pf_kernel<false, 4>), grid, block, 0, st, yv, gates, ov, p, s);
            else hipLaunchKernelGGL((combine_pf_kernel<false, 2>), grid, block, 0, st, yv, gates, ov, p, s);
        }
        HIP_TRY(hipGetLastError());
        return MONTA_OK;
    }
    if (dtype == MONTA_BF16) {
        if (wide) hipLaunchKernelGGL((combine_kernel<true, 4>), grid, block, 0, st, yv, gates, ov, p, s);
        else hipLaunchKernelGGL((combine_kernel<true, 2>), grid, block, 0, st, yv, gates, ov, p, s);
    } else {
        if (wide) hipLaunchKernelGGL((combine_kernel<false, 4>), grid, block, 0, st, yv, gates, ov, p, s);
        else hipLaunchKernelGGL((combine_kernel<false, 2>), grid, block, 0, st, yv, gates, ov, p, s);
    }
    HIP_TRY(hipGetLastError());
    return MONTA_OK;
}

}  // namespace

extern "C" {

int monta_workspace_bytes(const monta_cfg *cfg, size_t *ws_bytes, int64_t *max_rows)
{
    if (!ws_bytes || !max_rows) return MONTA_ERR_NULL;
    Geometry g;
    int rc = validate(cfg, &g);
    if (rc) return rc;
    monta_ws_layout L;
    fill_layout(g, &L);
    *ws_bytes = (size_t)L.ws_bytes;
    *max_rows = L.max_rows;
    return MONTA_OK;
}

int monta_ws_layout_query(const monta_cfg *cfg, monta_ws_layout *layout)
{
    if (!layout) return MONTA_ERR_NULL;
    Geometry g;
    int rc = validate(cfg, &g);
    if (rc) return rc;
    fill_layout(g, layout);
    return MONTA_OK;
}

int monta_ws_init(const monta_cfg *cfg, void *ws, void *stream)
{
    Geometry g;
    int rc = validate(cfg, &g);
    if (rc) return rc;
    if ((rc = check_ws(ws))) return rc;
    PlanPtrs p = plan_ptrs(g, ws);
    hipLaunchKernelGGL(ws_init_kernel, dim3(1), dim3(kWave), 0, static_cast<hipStream_t>(stream), p.meta);
    HIP_TRY(hipGetLastError());
    return MONTA_OK;
}

int monta_gate(const monta_cfg *cfg, const void *x, const void *w_gate, float *logits, void *stream)
{
    Geometry g;
    int rc = validate(cfg, &g);
    if (rc) return rc;
    if (!x || !w_gate || !logits) return MONTA_ERR_NULL;
    if (misaligned(x, 16) || misaligned(w_gate, 16) || misaligned(logits, 4)) return MONTA_ERR_ALIGN;
    const Shape &s = g.s;
    const int64_t T = s.T;
    const int H = cfg->hidden, E = s.E;
    hipStream_t st = static_cast<hipStream_t>(stream);
    ProfScope ps(MONTA_K_GATE, st);
    if (cfg->dtype == MONTA_BF16) {
        // validate() guarantees H % 8 == 0 (rows are whole 16-byte vectors) and E <= 256 (at most 8 tiles).
        //  - Few tiles: launch_gate_few.  What it leaves, up to 8 experts on whole rows: launch_gate_small_any.  The rest, as follows.
        //  - Up to a round of tiles of 16 tokens x 16 experts, two rounds for up to 16 experts on rows over 2 KiB, or a round of 16 x 32 on such
        //    rows: the hidden axis is split, too.  launch_gate_few leaves these only rows below 456 elements, activations of more than
        //    96 MiB and rows beyond 2^20 (three sets in turn, us, split and in 32 x 64: 6500 x 8192, 9 experts 29 and 31; 4096 x 16384, 16 / 24
        //    experts 39 / 48 and 58; 2048 x 28672, 32 experts 59 and 101; but 8192 x 8192, 16 experts 37 and 32).
        //  - Up to 32736 tokens, and short rows on up to 32 experts beyond: direct-to-LDS tiles.  32 x 64 come three per CU, the
        //    others two; the larger, the fewer bytes, and the longer a workgroup's walk.
        //    Up to 64 experts one tile of 32 x 64 holds them all: those up to three rounds' worth of tiles and, on short rows, always
        //    (64 x 128 beyond: 25592 x 5120, 64 experts 60 and 56 us, three sets of activations in turn 86 and 70).
        //    More experts: 32 x 64 up to a round of 256.  32 x 128 up to a round of those, unless the rows are short (4096 x 512, 256
        //    experts: 7.7 us in 32 x 64, 8.4) or the last tile's columns are mostly idle (4644 x 5120, 160 experts: 31, 43 and in 64 x
        //    128 40; but 4096 x 4096, 256 experts 31, 22 and 33).  Then 32 x 64 up to two rounds, and 64 x 128, except that rows of up to
        //    4 KiB stay in 32 x 128 up to two rounds (12571 x 512, 65 experts: 11.9, 8.5 and 9.8; 12000 x 7168, 128 experts: 83, 77
        //    and 60), as do rows of 8 KiB on more than 128 experts, a stride at which the 128 rows of weights of a larger tile
        //    fall on few channels (8192 x 4096, 256 experts: 58, 37 and 43, in turn 61, 45 and 44; 192 experts 42, 36 and 43, in
        //    turn 44, 39 and 43).
        //    Rows that are not whole steps, whose lines every tile fetches twice: no two rounds of the smaller tiles (6188 x 1784, 192
        //    experts: 24, 25 and 21), 64 x 128 from 33 experts on (12000 x 4104, 64 experts: 47 and 39), the k-split form up to 32
        //    experts and from 16353 tokens on (24000 x 8184, 24 experts: 104 and 82).
        //  - Otherwise a workgroup per 32 tokens whose waves share the hidden axis, or per 128 tokens.
        // Over 1415 shapes of whole steps (64 to 8192 elements, 512 to 32736 tokens, 65 to 256 experts), one set of activations and
        // several in turn, this takes 1.02 of the best tile's time.
        const int64_t tiles32 = (T + 31) / 32;
        const u32x4 *xv = static_cast<const u32x4 *>(x), *wv = static_cast<const u32x4 *>(w_gate);
        rc = launch_gate_few(xv, wv, logits, T, H, E, st);
        if (rc > 0) rc = launch_gate_small_any(xv, wv, logits, T, H, E, st);
        auto tiles = [&](int64_t R, int64_t C) { return (T + R - 1) / R * ((E + C - 1) / C); };
        const int64_t tiles16 = tiles(16, 16), round = 256, n64 = tiles(32, 64), n128 = tiles(32, 128);
        const bool stream_x = T * H * 2 >= (300ll << 20);
        const bool whole = H % 64 == 0, short_rows = H <= 1024, many = tiles32 >= 1024, odd = !whole && H >= 2048;
        const bool k_split = (many && !(short_rows && E <= 32)) || (odd && E <= 32 && tiles32 >= 512);
        auto use_32x64 = [&] {
            if (odd && E > 32 && E <= 64 && T > 8192) return false;
            if (E <= 64) return n64 <= 3 * round || short_rows;
            if (n64 <= round) return true;
            const bool wider = whole && !short_rows && n128 <= round && (H <= 2048 ? n64 == 2 * n128 : 2 * n64 >= 3 * n128);
            return whole && !wider && n64 <= 2 * round;
        };
        auto use_32x128 = [&] {
            if (E <= 64) return false;
            return n128 <= (whole && (H <= 2048 || (H == 4096 && E > 128)) ? 2 * round : round);
        };
        if (rc <= 0) {
            if (rc) return rc;
        }
        else if (tiles16 <= (E <= 16 && !short_rows ? 2 * round : round) || (!k_split && H > kBigMaxHidden))
            rc = launch_gate_split<true>(xv, wv, logits, T, H / 8, E, 1, st);
        else if (E > 16 && tiles(16, 32) <= round && !short_rows)
            rc = launch_gate_split<true>(xv, wv, logits, T, H / 8, E, 2, st);
        else if (!k_split && use_32x64()) rc = launch_gate_short<32, 64, 4>(xv, wv, logits, T, H, E, st);
        else if (!k_split && use_32x128()) rc = launch_gate_short<32, 128, 4>(xv, wv, logits, T, H, E, st);
        else if (!k_split) rc = launch_gate_short<64, 128, 3>(xv, wv, logits, T, H, E, st);
        else if (E <= 32) rc = launch_gate<1, 1, 512, true>(xv, wv, logits, T, H, E, st);
        // More experts: at least one 128-token workgroup per CU, in which every wave owns whole output tiles (W_g is re-read once
        // per 128 tokens, and the small tiles let 3 workgroups share a CU).
        // Activations well beyond the memory-side cache (256 MB) leave nothing in it for the dispatch behind the gate: then they are
        // streamed.  At 256 MiB most of them are still there from whoever wrote them (32768 x 4096, 40 experts: one set used again
        // 49 us and, streamed, 60, three in turn 66 and 59), at 300 no longer (38400 x 4096: 80 and 71, in turn 80 and 73); 65536 x
        // 7168, 64 experts 175 -> 155, 128 experts 201 -> 192, 256 experts 336 and 333.
        else if (E <= 64)
            rc = stream_x ? launch_gate<4, 2, 128, false, true, true>(xv, wv, logits, T, H, E, st)
                                            : launch_gate<4, 2, 128, false, true>(xv, wv, logits, T, H, E, st);
        else if (E <= 128)
            rc = stream_x ? launch_gate<4, 4, 64, false, true, true>(xv, wv, logits, T, H, E, st)
                                            : launch_gate<4, 4, 64, false, true>(xv, wv, logits, T, H, E, st);
        else rc = launch_gate<4, 8, 64, false, true>(xv, wv, logits, T, H, E, st);
        if (rc) return rc;
    } else {
        // At most four experts: a wave per token, as long as its loads of the weights stay fewer than a tile's idle work: 4096 x
        // 4096, 3 / 4 experts 13.2 / 15.1 us against 12.9 / 13.1; 65536 x 4096, 1 / 2 experts 167 / 204 against 173 / 174.
        // Otherwise 64 experts per workgroup read x a quarter as often, 16 give four times the workgroups.
        // More than 16 experts and a tile of 32 x 64 for every CU: those, or 64 x 64 where they are two rounds (8192 x 4096, 32 / 128 /
        // 256 experts: 79 / 171 / 328 us, in 32 x 64 62 / 99 / 166, in 64 x 64 100 / 106 / 164; 32000 x 4096, 64 experts: 348, 177 and 170;
        // 2048 x 4096, 128 experts, half a round: 42 and 52).  Their sums are the more exact ones from about 800 elements on (1000:
        // 9.6e-8 against 9.9e-8; 8192: 1.4e-7 and 2.1e-7; but 512: 9.1e-8 and 8.6e-8).
        const int64_t tiles16 = (T + 15) / 16 * ((E + 15) / 16), experts64 = (E + 63) / 64;
        const bool short_tiles = E > 16 && H >= 896 && H <= kBigMaxHidden && (T + 31) / 32 * experts64 >= 256;
        const u32x4 *xv = static_cast<const u32x4 *>(x), *wv = static_cast<const u32x4 *>(w_gate);
        if (E <= 4 && (E == 1 || H <= 512 || T * E <= 12288))
            rc = launch_gate_f32_few(static_cast<const float4 *>(x), static_cast<const float4 *>(w_gate), logits, T, H, E, st);
        else if (short_tiles && (T + 63) / 64 * experts64 >= 500) rc = launch_gate_short<64, 64, 3, true>(xv, wv, logits, T, H, E, st);
        else if (short_tiles) rc = launch_gate_short<32, 64, 3, true>(xv, wv, logits, T, H, E, st);
        else rc = launch_gate_split<false>(xv, wv, logits, T, H / 4, E, E <= 16 || tiles16 <= 256 ? 1 : 4, st);
        if (rc) return rc;
    }
    HIP_TRY(hipGetLastError());
    return MONTA_OK;
}

int monta_expert_linear(const monta_cfg *cfg, const void *x_final, const void *w_exp, int32_t out_features, void *y,
                        const void *ws, int slice, void *stream)
{
    Geometry g;
    int rc = validate(cfg, &g);
    if (rc) return rc;
    if ((rc = check_expert_args(cfg, g, x_final, w_exp, out_features, y, ws, slice))) return rc;
    return launch_expert_layer(cfg, g, x_final, w_exp, out_features, y, ws, slice, static_cast<hipStream_t>(stream));
}

int monta_route_dispatch_expert(const monta_cfg *cfg, const float *logits, const void *x, int32_t *topk_idx, float *gates,
                                void *stage, void *final_, const void *w_exp, int32_t out_features, void *y, void *ws,
                                int overlap, void *stream)
{
    Geometry g;
    int rc = validate(cfg, &g);
    if (rc) return rc;
    if ((rc = check_route_ptrs(logits, topk_idx, gates, ws))) return rc;
    if ((rc = check_act_ptrs(x, stage))) return rc;
    if ((rc = check_act_ptrs(stage, final_))) return rc;
    if (stage == final_ || y == stage || y == x) return MONTA_ERR_INVALID;
    if ((rc = check_expert_args(cfg, g, final_, w_exp, out_features, y, ws, -1))) return rc;
    if (overlap != 0 && overlap != 1) return MONTA_ERR_INVALID;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (!overlap) {
        if ((rc = route_dispatch_regather_impl(g, logits, x, topk_idx, gates, stage, final_, ws, st))) return rc;
        return launch_expert_layer(cfg, g, final_, w_exp, out_features, y, ws, -1, st);
    }
    // Overlapped: the slice pipeline of pipeline mode 1 on the caller's stream, an event behind the kernel that
    // completes a slice's rows of FINAL, and that slice's expert layer on the side stream: the matrix cores work
    // on slice j while the movers stream slice j+1.
    const int S = g.s.S;
    DevState *d = nullptr;
    if ((rc = dev_state(S, &d))) return rc;
    std::lock_guard<std::mutex> lk(d->mu);      // the side stream and its events are shared per device
    if ((rc = route_impl(g, logits, topk_idx, gates, ws, st))) return rc;
    const PlanPtrs p = plan_ptrs(g, ws);
    if ((rc = launch_pack(g, p, x, stage, 0, 1, st))) return rc;
    for (int j = 0; j < S; ++j) {
        rc = j + 1 < S ? launch_pack_regather(g, p, x, stage, final_, j + 1, j + 2, j, j + 1, st)      // pack(j+1) and regather(j)
                       : launch_regather(g, p, stage, final_, j, j + 1, st);
        if (rc) return rc;
        HIP_TRY(hipEventRecord(d->ev[j], st));
        HIP_TRY(hipStreamWaitEvent(d->side, d->ev[j], 0));
        prof_break_chain(d->side);
        if ((rc = launch_expert_layer(cfg, g, final_, w_exp, out_features, y, ws, j, d->side))) return rc;
    }
    HIP_TRY(hipEventRecord(d->done, d->side));
    HIP_TRY(hipStreamWaitEvent(st, d->done, 0));
    prof_break_chain(st);
    return MONTA_OK;
}

int monta_route(const monta_cfg *cfg, const float *logits, int32_t *topk_idx, float *gates, void *ws, void *stream)
{
    Geometry g;
    int rc = validate(cfg, &g);
    if (rc) return rc;
    if ((rc = check_route_ptrs(logits, topk_idx, gates, ws))) return rc;
    return route_impl(g, logits, topk_idx, gates, ws, static_cast<hipStream_t>(stream));
}

int monta_route_dispatch_regather(const monta_cfg *cfg, const float *logits, const void *x, int32_t *topk_idx,
                                  float *gates, void *stage, void *final_, void *ws, void *stream)
{
    Geometry g;
    int rc = validate(cfg, &g);
    if (rc) return rc;
    if ((rc = check_route_ptrs(logits, topk_idx, gates, ws))) return rc;
    if ((rc = check_act_ptrs(x, stage))) return rc;
    if ((rc = check_act_ptrs(stage, final_))) return rc;
    if (stage == final_) return MONTA_ERR_INVALID;
    return route_dispatch_regather_impl(g, logits, x, topk_idx, gates, stage, final_, ws, static_cast<hipStream_t>(stream));
}

int monta_dispatch(const monta_cfg *cfg, const void *x, void *stage, const void *ws, int slice, void *stream)
{
    Geometry g;
    int rc = validate(cfg, &g);
    if (rc) return rc;
    if (slice < -1 || slice >= cfg->slices) return MONTA_ERR_INVALID;
    if ((rc = check_act_ptrs(x, stage))) return rc;
    if ((rc = check_ws(ws))) return rc;
    return launch_pack(g, plan_ptrs(g, ws), x, stage, slice < 0 ? 0 : slice, slice < 0 ? g.s.S : slice + 1,
                       static_cast<hipStream_t>(stream));
}

int monta_regather(const monta_cfg *cfg, const void *stage, void *final_, const void *ws, int slice, void *stream)
{
    Geometry g;
    int rc = validate(cfg, &g);
    if (rc) return rc;
    if (slice < -1 || slice >= cfg->slices) return MONTA_ERR_INVALID;
    if ((rc = check_act_ptrs(stage, final_))) return rc;
    if (stage == final_) return MONTA_ERR_INVALID;
    if ((rc = check_ws(ws))) return rc;
    return launch_regather(g, plan_ptrs(g, ws), stage, final_, slice < 0 ? 0 : slice, slice < 0 ? g.s.S : slice + 1,
                           static_cast<hipStream_t>(stream));
}

int monta_dispatch_regather(const monta_cfg *cfg, const void *x, void *stage, void *final_, const void *ws,
                            void *stream)
{
    Geometry g;
    int rc = validate(cfg, &g);
    if (rc) return rc;
    if ((rc = check_act_ptrs(x, stage))) return rc;
    if ((rc = check_act_ptrs(stage, final_))) return rc;
    if (stage == final_) return MONTA_ERR_INVALID;
    if ((rc = check_ws(ws))) return rc;
    return dispatch_regather_impl(g, x, stage, final_, ws, static_cast<hipStream_t>(stream));
}

int monta_combine(const monta_cfg *cfg, const void *y, const float *gates, void *out, const void *ws, void *stream)
{
    Geometry g;
    int rc = validate(cfg, &g);
    if (rc) return rc;
    if (!gates) return MONTA_ERR_NULL;
    if (misaligned(gates, 4)) return MONTA_ERR_ALIGN;
    if ((rc = check_act_ptrs(y, out))) return rc;
    if (y == out) return MONTA_ERR_INVALID;
    if ((rc = check_ws(ws))) return rc;
    return combine_impl(g, cfg->dtype, y, gates, out, ws, static_cast<hipStream_t>(stream));
}

namespace {

int allgather_grid(const Geometry &g, int nslices)
{
    const int64_t vecs = slice_rows_bound(g, nslices) * g.s.vpr;
    int64_t wg = (vecs + (int64_t)kMoverThreads * kVecInFlight - 1) / ((int64_t)kMoverThreads * kVecInFlight);
    if (wg < 1) wg = 1;
    if (wg > 32768) wg = 32768;
    return (int)wg;
}

int launch_allgather(const Geometry &g, const PlanPtrs &p, const void *stage, void *gathered, int j0, int j1, hipStream_t st)
{
    const Shape &s = g.s;
    ProfScope ps(MONTA_K_ALLGATHER, st);
    hipLaunchKernelGGL(allgather_kernel, dim3((unsigned)allgather_grid(g, j1 - j0)), dim3(kMoverThreads), 0, st,
                       static_cast<const u32x4 *>(stage), static_cast<u32x4 *>(gathered), p, s, j0 * s.tp, j1 * s.tp);
    HIP_TRY(hipGetLastError());
    return MONTA_OK;
}

}  // namespace

int monta_allgather(const monta_cfg *cfg, const void *stage, void *gathered, const void *ws, int slice, void *stream)
{
    Geometry g;
    int rc = validate(cfg, &g);
    if (rc) return rc;
    if (slice < -1 || slice >= cfg->slices) return MONTA_ERR_INVALID;
    if ((rc = check_act_ptrs(stage, gathered))) return rc;
    if (stage == gathered) return MONTA_ERR_INVALID;
    if ((rc = check_ws(ws))) return rc;
    return launch_allgather(g, plan_ptrs(g, ws), stage, gathered, slice < 0 ? 0 : slice, slice < 0 ? g.s.S : slice + 1,
                            static_cast<hipStream_t>(stream));
}

int monta_allgather_regather(const monta_cfg *cfg, const void *stage, void *gathered, void *final_, const void *ws,
                             int schedule, void *stream)
{
    Geometry g;
    int rc = validate(cfg, &g);
    if (rc) return rc;
    if (schedule < 0 || schedule > 2) return MONTA_ERR_INVALID;
    if ((rc = check_act_ptrs(stage, gathered))) return rc;
    if ((rc = check_act_ptrs(gathered, final_))) return rc;
    if (stage == gathered || gathered == final_ || stage == final_) return MONTA_ERR_INVALID;
    if ((rc = check_ws(ws))) return rc;
    const Shape &s = g.s;
    const PlanPtrs p = plan_ptrs(g, ws);
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int S = s.S;
    if (schedule == 0) {            // chunk by chunk, gather then copy: no overlap
        for (int j = 0; j < S; ++j) {
            if ((rc = launch_allgather(g, p, stage, gathered, j, j + 1, st))) return rc;
            if ((rc = launch_regather(g, p, gathered, final_, j, j + 1, st))) return rc;
        }
        return MONTA_OK;
    }
    if (schedule == 1) {            // launch j gathers chunk j and, in disjoint workgroups, copies chunk j-1
        if ((rc = launch_allgather(g, p, stage, gathered, 0, 1, st))) return rc;
        for (int j = 1; j < S; ++j) {
            const int n_gather = allgather_grid(g, 1), n_copy = regather_grid(s, slice_rows_bound(g, 1));
            ProfScope ps(MONTA_K_ALLGATHER_REGATHER, st);
            hipLaunchKernelGGL(allgather_regather_kernel, dim3(n_gather + n_copy), dim3(kMoverThreads), 0, st,
                               static_cast<const u32x4 *>(stage), static_cast<u32x4 *>(gathered), static_cast<u32x4 *>(final_),
                               p, s, j * s.tp, (j + 1) * s.tp, (j - 1) * s.tp, j * s.tp, n_gather);
            HIP_TRY(hipGetLastError());
        }
        return launch_regather(g, p, gathered, final_, S - 1, S, st);
    }
    // schedule 2: the paper's stream picture: gathers on the caller's stream, copies on the library's side stream
    // (default priority), one event per chunk, joined back into the caller's stream
    DevState *d = nullptr;
    if ((rc = dev_state(S, &d))) return rc;
    std::lock_guard<std::mutex> lk(d->mu);
    for (int j = 0; j < S; ++j) {
        if ((rc = launch_allgather(g, p, stage, gathered, j, j + 1, st))) return rc;
        HIP_TRY(hipEventRecord(d->ev[j], st));
        HIP_TRY(hipStreamWaitEvent(d->side, d->ev[j], 0));
        prof_break_chain(d->side);
        if ((rc = launch_regather(g, p, gathered, final_, j, j + 1, d->side))) return rc;
    }
    HIP_TRY(hipEventRecord(d->done, d->side));
    HIP_TRY(hipStreamWaitEvent(st, d->done, 0));
    prof_break_chain(st);
    return MONTA_OK;
}

// mirrored return path -------------------------------------------------------------------------

int monta_unregather(const monta_cfg *cfg, const void *y, void *y_stage, const void *ws, int slice, void *stream)
{
    Geometry g;
    int rc = validate(cfg, &g);
    if (rc) return rc;
    if (slice < -1 || slice >= cfg->slices) return MONTA_ERR_INVALID;
    if ((rc = check_act_ptrs(y, y_stage))) return rc;
    if (y == y_stage) return MONTA_ERR_INVALID;
    if ((rc = check_ws(ws))) return rc;
    const Shape &s = g.s;
    const PlanPtrs p = plan_ptrs(g, ws);
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int u0 = slice < 0 ? 0 : slice * s.tp;
    const int u1 = slice < 0 ? s.U : (slice + 1) * s.tp;
    ProfScope ps(MONTA_K_UNREGATHER, st);
    hipLaunchKernelGGL(unregather_kernel, dim3(regather_grid(s, slice_rows_bound(g, slice < 0 ? s.S : 1))),
                       dim3(kMoverThreads), 0, st, static_cast<const u32x4 *>(y), static_cast<u32x4 *>(y_stage), p, s,
                       u0, u1);
    HIP_TRY(hipGetLastError());
    return MONTA_OK;
}

namespace {

// launches unregather(units [u0,u1)) and / or combine of tokens [t0, t0+nt) from the unit-major layout
int launch_unregather_combine(const Geometry &g, const PlanPtrs &p, int dtype, const void *y, void *y_stage,
                              const float *gates, void *out, int u0, int u1, int t0, int nt, hipStream_t st)
{
    Shape s = g.s;
    // the rows fetched back are read exactly once by the staged combine: stream them unless the caller set a policy
    if (g.modes.cache < 0) s.cache |= NT_COMB_LD;
    const int n_unreg = u0 < u1 ? regather_grid(s, slice_rows_bound(g, (u1 - u0) / s.tp)) : 0;
    const int n_comb = nt > 0 ? mover_grid(s, nt) : 0;
    if (n_unreg + n_comb == 0) return MONTA_OK;
    const bool wide = s.vpr > 2 * s.lpr;
    const u32x4 *yv = static_cast<const u32x4 *>(y);
    u32x4 *sv = static_cast<u32x4 *>(y_stage), *ov = static_cast<u32x4 *>(out);
    const dim3 grid(n_unreg + n_comb), block(kMoverThreads);
    ProfScope ps(n_unreg && n_comb ? MONTA_K_UNREGATHER_COMBINE : (n_unreg ? MONTA_K_UNREGATHER : MONTA_K_COMBINE), st);
    const bool pf = s.k >= 3 && s.k <= s.lpr;       // as in monta_combine
#define MONTA_LAUNCH_UC(BF, NV_, PF_)                                                                                    \
    hipLaunchKernelGGL((unregather_combine_kernel<BF, NV_, PF_>), grid, block, 0, st, yv, sv, gates, ov, p, s, u0, u1, t0, \
                       nt, n_unreg)
    if (dtype == MONTA_BF16) {
        if (pf) { if (wide) MONTA_LAUNCH_UC(true, 4, true); else MONTA_LAUNCH_UC(true, 2, true); }
        else { if (wide) MONTA_LAUNCH_UC(true, 4, false); else MONTA_LAUNCH_UC(true, 2, false); }
    } else {
        if (pf) { if (wide) MONTA_LAUNCH_UC(false, 4, true); else MONTA_LAUNCH_UC(false, 2, true); }
        else { if (wide) MONTA_LAUNCH_UC(false, 4, false); else MONTA_LAUNCH_UC(false, 2, false); }
    }
#undef MONTA_LAUNCH_UC
    HIP_TRY(hipGetLastError());
    return MONTA_OK;
}

int launch_return(const Geometry &g, const PlanPtrs &p, int dtype, const void *y, void *y_stage, const float *gates,
                  void *out, hipStream_t st)
{
    Shape s = g.s;
    // y_stage and out are not read again here; y streams only where it does not fit the memory-side cache anyway (8192
    // tokens, top-2, 8 KiB rows: 49.9 us with y cacheable, 64.7 streamed; 65536 tokens of 14 KiB, top-8: 1417 and 1394)
    if (g.modes.cache < 0) {
        const int64_t touched = ((int64_t)s.T + 2 * g.max_rows) * g.row_bytes;
        s.cache = NT_REG_ST | NT_COMB_ST | (touched > (1024ll << 20) ? NT_REG_LD : 0);
    }
    const bool wide = s.vpr > 2 * s.lpr, pf = s.k >= 3 && s.k <= s.lpr;       // as in monta_combine
    const u32x4 *yv = static_cast<const u32x4 *>(y);
    u32x4 *sv = static_cast<u32x4 *>(y_stage), *ov = static_cast<u32x4 *>(out);
    const dim3 grid(mover_grid(s, s.T)), block(kMoverThreads);
    ProfScope ps(MONTA_K_RETURN, st);
    if (const int K = combine_units(s, dtype == MONTA_BF16, true)) {
        const dim3 ugrid = combine_units_grid(s);
        with_units(dtype, s, K, [&](auto bf, auto kc, auto wave) {
            hipLaunchKernelGGL((return_units_kernel<decltype(bf)::value, decltype(kc)::value, decltype(wave)::value>), ugrid, block, 0, st, yv, sv, gates,
                               ov, p, s);
        });
        HIP_TRY(hipGetLastError());
        return MONTA_OK;
    }
    auto launch = [&](auto bf, auto nv, auto pfc) {
        hipLaunchKernelGGL((return_kernel<decltype(bf)::value, decltype(nv)::value, decltype(pfc)::value>), grid, block, 0, st,
                           yv, sv, gates, ov, p, s);
    };
    auto by_form = [&](auto bf) {
        using two = std::integral_constant<int, 2>;
        using four = std::integral_constant<int, 4>;
        if (pf) { if (wide) launch(bf, four{}, std::true_type{}); else launch(bf, two{}, std::true_type{}); }
        else { if (wide) launch(bf, four{}, std::false_type{}); else launch(bf, two{}, std::false_type{}); }
    };
    if (dtype == MONTA_BF16) by_form(std::true_type{});
    else by_form(std::false_type{});
    HIP_TRY(hipGetLastError());
    return MONTA_OK;
}

int check_staged_combine(const monta_cfg *cfg, Geometry *g, const void *y_stage, const float *gates, void *out,
                         const void *ws)
{
    int rc = validate(cfg, g);
    if (rc) return rc;
    if (!gates) return MONTA_ERR_NULL;
    if (misaligned(gates, 4)) return MONTA_ERR_ALIGN;
    if ((rc = check_act_ptrs(y_stage, out))) return rc;
    if (y_stage == out) return MONTA_ERR_INVALID;
    return check_ws(ws);
}

}  // namespace

int monta_combine_staged(const monta_cfg *cfg, const void *y_stage, const float *gates, void *out, const void *ws,
                         int slice, void *stream)
{
    Geometry g;
    int rc = check_staged_combine(cfg, &g, y_stage, gates, out, ws);
    if (rc) return rc;
    if (slice < -1 || slice >= cfg->slices) return MONTA_ERR_INVALID;
    const Shape &s = g.s;
    const int per_slice = s.tp * s.Tu;
    const int t0 = slice < 0 ? 0 : slice * per_slice, nt = slice < 0 ? s.T : per_slice;
    return launch_unregather_combine(g, plan_ptrs(g, ws), cfg->dtype, y_stage, const_cast<void *>(y_stage), gates, out,
                                     0, 0, t0, nt, static_cast<hipStream_t>(stream));
}

int monta_unregather_combine(const monta_cfg *cfg, const void *y, void *y_stage, const float *gates, void *out,
                             const void *ws, void *stream)
{
    Geometry g;
    int rc = check_staged_combine(cfg, &g, y_stage, gates, out, ws);
    if (rc) return rc;
    if ((rc = check_act_ptrs(y, y_stage))) return rc;
    if (y == y_stage || y == out) return MONTA_ERR_INVALID;
    const Shape &s = g.s;
    const PlanPtrs p = plan_ptrs(g, ws);
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int64_t y_bytes = g.max_rows * g.row_bytes, out_bytes = (int64_t)s.T * g.row_bytes;
    if (g.modes.pipeline < 0 && !overlap(y, y_bytes, y_stage, y_bytes) && !overlap(y, y_bytes, out, out_bytes) &&
        !overlap(y_stage, y_bytes, out, out_bytes))
        return launch_return(g, p, cfg->dtype, y, y_stage, gates, out, st);
    const int per_slice = s.tp * s.Tu;
    // One slice per launch with an explicit pipeline mode: launch j fetches slice j back and, in disjoint workgroups of the
    // same grid, combines the tokens of slice j-1; with mode 2 both are kernels of their own.  By default the two passes are
    // apart only because out shares memory with y (or a buffer with another beyond the rows in use): every row of y has to be
    // fetched before the first row of out is written, so one launch fetches all slices and the next combines them.
    const int spg = g.modes.pipeline < 0 ? s.S : 1;
    const int G = s.S / spg;
    if (g.modes.pipeline < 0 || g.modes.pipeline == 2) {
        for (int gi = 0; gi < G; ++gi) {
            if ((rc = launch_unregather_combine(g, p, cfg->dtype, y, y_stage, gates, out, gi * spg * s.tp, (gi + 1) * spg * s.tp, 0, 0, st)))
                return rc;
            if ((rc = launch_unregather_combine(g, p, cfg->dtype, y, y_stage, gates, out, 0, 0, gi * spg * per_slice, spg * per_slice, st)))
                return rc;
        }
        return MONTA_OK;
    }
    for (int gi = 0; gi <= G; ++gi) {
        const int u0 = gi < G ? gi * s.tp : 0, u1 = gi < G ? (gi + 1) * s.tp : 0;
        const int t0 = gi > 0 ? (gi - 1) * per_slice : 0, nt = gi > 0 ? per_slice : 0;
        if ((rc = launch_unregather_combine(g, p, cfg->dtype, y, y_stage, gates, out, u0, u1, t0, nt, st))) return rc;
    }
    return MONTA_OK;
}

// ---- one entry point that allocates nothing -------------------------------------------------------
//
// The plan tables of the whole step live in a file-scope device array instead of a caller workspace.
// In host code the array's name is only a stand-in for the symbol: the device address is looked up once
// per device (every GPU holds its own copy at its own address) and only that address is ever handed to
// kernels.

constexpr size_t kStaticScratchBytes = 16u << 20;
// fewer than 256 route workgroups where there could be fewer than 128 (validate), two tables, at most 256 experts
constexpr size_t kStaticFinerBytes = 512u << 10;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes + kStaticFinerBytes];

namespace {

std::mutex g_scratch_mu;
void *g_scratch_ptr[64] = {nullptr};

int static_scratch(void **out)
{
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= 64) return MONTA_ERR_UNSUPPORTED;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *ptr = nullptr;
        HIP_TRY(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));      // the current device's copy of the array
        if (!ptr) return MONTA_ERR_HIP;
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return MONTA_OK;
}

}  // namespace

int monta_route_dispatch_combine_static(const monta_cfg *cfg, const float *logits, const void *x, int32_t *topk_idx,
                                        float *gates, void *stage, void *final_, void *out, void *stream)
{
    Geometry g;
    int rc = validate(cfg, &g);
    if (rc) return rc;
    if (!logits || !topk_idx || !gates) return MONTA_ERR_NULL;
    if (misaligned(logits, 4) || misaligned(topk_idx, 4) || misaligned(gates, 4)) return MONTA_ERR_ALIGN;
    if ((rc = check_act_ptrs(x, stage))) return rc;
    if ((rc = check_act_ptrs(final_, out))) return rc;
    if (stage == final_ || final_ == out || stage == out || x == out) return MONTA_ERR_INVALID;
    monta_ws_layout L;
    fill_layout(g, &L);
    // the limit is on the tables as they are with as few route workgroups as fit: what the finer histograms of small
    // problems add does not count against it
    const int64_t finer = 2 * (align_up((int64_t)g.s.num_blocks * g.s.E * 4, 256) - align_up(g.blocks_by_tile * g.s.E * 4, 256));
    if ((size_t)(L.ws_bytes - finer) > kStaticScratchBytes || finer > (int64_t)kStaticFinerBytes) return MONTA_ERR_TOO_LARGE;
    // event profiling creates events per launch and the two-stream pipeline creates a stream: neither belongs
    // in a call that must not allocate
    if (g_prof_on.load()) return MONTA_ERR_INVALID;
    if (g.modes.pipeline == 0) g.modes.pipeline = -1;      // pipeline_plan() then never answers 0
    void *ws = nullptr;
    if ((rc = static_scratch(&ws))) return rc;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int lanes = g.modes.cache < 0 && single_pass(g, x, final_) ? small_lanes(g, true) : 0;
    if (lanes && small_apart(g, logits, topk_idx, gates, nullptr, x, stage, final_, out))
        return launch_small(g, plan_ptrs(g, ws), lanes, SMALL_COMBINE, logits, x, topk_idx, gates, stage, final_, out, cfg->dtype == MONTA_BF16, st);
    // the array keeps the previous call's contents, possibly of another shape: no kernel reads what this call has not written
    if ((rc = route_dispatch_regather_impl(g, logits, x, topk_idx, gates, stage, final_, ws, st))) return rc;
    return combine_impl(g, cfg->dtype, final_, gates, out, ws, st);
}

int monta_pipeline_query(const monta_cfg *cfg, int32_t *mode, int32_t *first_slices, int32_t *slices_per_launch,
                         int32_t *plan_fused)
{
    if (!mode || !first_slices || !slices_per_launch || !plan_fused) return MONTA_ERR_NULL;
    Geometry g;
    int rc = validate(cfg, &g);
    if (rc) return rc;
    const PipePlan pp = grouping_by_size(g);
    *mode = pp.mode;
    *first_slices = pp.first < g.s.S ? pp.first : g.s.S;
    *slices_per_launch = pp.spg;
    *plan_fused = plan_pack_fused(g, pp) ? 1 : 0;
    return MONTA_OK;
}

int monta_set_pipeline_mode(int mode)
{
    if (mode < -1 || mode > 2) return MONTA_ERR_INVALID;
    g_pipeline_mode.store(mode);
    return MONTA_OK;
}

int monta_get_pipeline_mode(void) { return g_pipeline_mode.load(); }

int monta_set_plan_mode(int mode)
{
    if (mode != -1 && mode != 0) return MONTA_ERR_INVALID;
    g_plan_mode.store(mode);
    return MONTA_OK;
}

int monta_get_plan_mode(void) { return g_plan_mode.load(); }

int monta_set_cache_policy(int policy)
{
    if (policy < -1 || policy > 63) return MONTA_ERR_INVALID;
    g_cache_policy.store(policy);
    return MONTA_OK;
}

int monta_get_cache_policy(void) { return g_cache_policy.load(); }

int monta_copy(void *dst, const void *src, size_t bytes, void *stream)
{
    if (!dst || !src) return MONTA_ERR_NULL;
    if (bytes == 0 || bytes % 16 != 0) return MONTA_ERR_INVALID;
    if (misaligned(dst, 16) || misaligned(src, 16)) return MONTA_ERR_ALIGN;
    const size_t nvec = bytes / 16;
    size_t wg = (nvec + (size_t)kMoverThreads * kVecInFlight - 1) / ((size_t)kMoverThreads * kVecInFlight);
    if (wg > (size_t)kMaxMoverGrid) wg = kMaxMoverGrid;
    hipStream_t st = static_cast<hipStream_t>(stream);
    ProfScope ps(MONTA_K_COPY, st);
    hipLaunchKernelGGL(copy_kernel, dim3((unsigned)wg), dim3(kMoverThreads), 0, st, static_cast<const u32x4 *>(src),
                       static_cast<u32x4 *>(dst), nvec);
    HIP_TRY(hipGetLastError());
    return MONTA_OK;
}

int monta_profile_enable(int on)
{
    g_prof_on.store(on ? 1 : 0);
    std::lock_guard<std::mutex> lk(g_prof_mu);
    for (auto &pr : g_prof_last) pr.second = nullptr;     // work enqueued while disabled must not be timed
    return MONTA_OK;
}

int monta_profile_reset(void)
{
    int rc = prof_drain();
    std::lock_guard<std::mutex> lk(g_prof_mu);
    for (int i = 0; i < MONTA_K_COUNT; ++i) {
        g_prof_ms[i] = 0.0;
        g_prof_n[i] = 0;
    }
    return rc;
}

int monta_profile_read(int kernel_id, double *total_ms, int64_t *launches)
{
    if (!total_ms || !launches) return MONTA_ERR_NULL;
    if (kernel_id < 0 || kernel_id >= MONTA_K_COUNT) return MONTA_ERR_INVALID;
    int rc = prof_drain();
    std::lock_guard<std::mutex> lk(g_prof_mu);
    *total_ms = g_prof_ms[kernel_id];
    *launches = g_prof_n[kernel_id];
    return rc;
}

const char *monta_strerror(int code)
{
    switch (code) {
        case MONTA_OK: return "ok";
        case MONTA_ERR_INVALID: return "invalid argument (size, flag or slice violates the preconditions)";
        case MONTA_ERR_UNSUPPORTED: return "shape outside the library's limits";
        case MONTA_ERR_NULL: return "required pointer is NULL";
        case MONTA_ERR_HIP: return "HIP runtime call failed (see monta_last_hip_error)";
        case MONTA_ERR_ALIGN: return "pointer is not aligned as required";
        case MONTA_ERR_TOO_LARGE: return "problem needs more plan-table space than the library's static scratch array holds (16 MiB)";
        default: return "unknown monta status";
    }
}

int monta_last_hip_error(void) { return g_last_hip; }

int monta_shutdown(void)
{
    int rc = prof_drain();
    std::lock_guard<std::mutex> lk(g_dev_mu);
    int cur = 0;
    HIP_TRY(hipGetDevice(&cur));
    for (int dev = 0; dev < 64; ++dev) {
        DevState &d = g_dev[dev];
        if (!d.side && !d.done && d.ev.empty()) continue;
        std::lock_guard<std::mutex> dl(d.mu);
        HIP_TRY(hipSetDevice(dev));
        if (d.side) {
            HIP_TRY(hipStreamSynchronize(d.side));
            HIP_TRY(hipStreamDestroy(d.side));
            d.side = nullptr;
        }
        for (hipEvent_t e : d.ev) HIP_TRY(hipEventDestroy(e));
        d.ev.clear();
        if (d.done) {
            HIP_TRY(hipEventDestroy(d.done));
            d.done = nullptr;
        }
    }
    HIP_TRY(hipSetDevice(cur));
    return rc;
}

}  // extern "C"
