// lbm.hip -- host side of the C ABI declared in include/lbm.h.
//
// A domain holds one population array, updated in place by two alternating
// kernels (streaming step and local step), the list of 64-cell tiles that
// contain updated cells, and for tiles that touch a wall, inlet, box face or
// non-updated cell a 32-bit link mask per cell.  Interior tiles (every cell
// updated, every link a plain pull after periodic wrap) carry no mask and
// take the kernels' branch-free path.  Long runs of steps are replayed from
// a HIP graph built node by node, short ones launched step by step.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdarg>
#include <atomic>
#include <chrono>
#include <cmath>
#include <condition_variable>
#include <cstdio>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <thread>
#include <vector>

#define LBM_HOST_TU
#include "lbm_device.hpp"
#include "lbm_instances.hpp"
#include "../../include/lbm.h"

// the step and state-access kernels are compiled per storage format in
// lbm_kern.hip
namespace lbm {
LBM_INSTANCES(extern template, ST_FP32)
LBM_INSTANCES(extern template, ST_FP16S)
LBM_INSTANCES(extern template, ST_BF16S)
LBM_INSTANCES_WIDE(extern template, ST_FP32)
LBM_INSTANCES_WIDE(extern template, ST_FP16S)
LBM_INSTANCES_WIDE(extern template, ST_BF16S)
} // namespace lbm

using namespace lbm;

// Read-back buffer of lbm_get_moments_noalloc (see scratch_address).
constexpr uint64_t kScratchFloats = (uint64_t)16 << 20;
static __device__ __align__(256) float scratch[kScratchFloats];

namespace {

thread_local std::string g_err;

int fail(int code, const char *fmt, ...) __attribute__((format(printf, 2, 3)));
int fail(int code, const char *fmt, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_err = buf;
    return code;
}

#define HIP_TRY(expr)                                                                                            \
    do {                                                                                                         \
        hipError_t e_ = (expr);                                                                                  \
        if (e_ != hipSuccess)                                                                                    \
            return fail(LBM_ERR_DEVICE, "%s failed: %s", #expr, hipGetErrorString(e_));                          \
    } while (0)

size_t storage_bytes(int st) { return st == LBM_FP32 ? 4 : 2; }

FastDiv make_fastdiv(uint32_t d)
{
    FastDiv f{};
    uint32_t l = 0;
    while ((1ull << l) < d)
        ++l;
    f.m = (uint32_t)((((1ull << 32) * ((1ull << l) - d)) / d) + 1);
    f.s1 = l < 1 ? l : 1;
    f.s2 = l > 0 ? l - 1 : 0;
    f.d = d;
    return f;
}

// Step graph: 64 steps (an even length ends in the phase it starts in).
// Below 64 steps a replay is never faster than launching the steps one by
// one (32^3 FP32: 8 steps 83 us against 68, 32 steps 182 against 167, 64
// steps 310 against 299; a 128^3 box runs the same either way, its kernels
// being longer than a launch).  Long runs gain from replays where the
// kernels are short (640 steps: 8^3 2246 us against 2352, 32^3 2549 against
// 2691) and cost the host a third of the time (0.8 us a step against 2.4).
// Building the graph costs about 100 us of host time, so it is built once
// kGraphBuild steps have been asked for since the last change, in however
// many runs, and by a run that can use it; any run uses it once it is there
// (20 runs of 100 steps of a 16^3 box 7.5 ms, of which the host takes 3.2 to
// enqueue them; launched one by one 8.3 and 6.3).
constexpr int kGraphSteps = 64;
constexpr int kGraphBuild = 256;

// Largest population array the buffer-instruction kernels address (their
// byte offsets are 32-bit); larger arrays take the 64-bit kernels.
constexpr uint64_t kNarrowBytes = (1ull << 32) - (1ull << 16);

// Bytes of a domain's population array: the tile blocks, then 2 x 9 side
// rows of ny * nz elements, rounded up to 256 bytes.
uint64_t array_bytes(uint64_t P, int ny, int nz, int storage)
{
    const uint64_t es = storage_bytes(storage);
    return (Q * P * es + 18ull * ny * nz * es + 255) / 256 * 256;
}

// Status words of domains: 4 bytes each of pinned host memory that the first
// unstable waves write (check_state), so that waiting for steps is one stream
// synchronisation and a host read, with no copy behind it (one step of a 16^3
// box, waited for: 34.8 -> 14.5 us).  The words come from blocks of 1024.
// Pinned memory is given back (give_back_pinned) only where the library waits
// for the device anyway: hipHostFree waits for all work on it, other
// libraries' included, and a domain is destroyed beside that.
struct StatusWord {
    uint32_t *host = nullptr, *dev = nullptr;
};

struct StatusBlock {
    uint32_t *host = nullptr, *dev = nullptr;
    std::vector<uint32_t> unused;
};
constexpr uint32_t kStatusBlockWords = 1024;
std::mutex g_status_mutex;
std::vector<StatusBlock> g_status_blocks;

hipError_t status_alloc(StatusWord &w)
{
    std::lock_guard<std::mutex> lock(g_status_mutex);
    StatusBlock *b = nullptr;
    for (auto &c : g_status_blocks)
        if (!c.unused.empty())
            b = &c;
    if (!b) {
        StatusBlock n;
        void *p = nullptr, *q = nullptr;
        hipError_t e = hipHostMalloc(&p, kStatusBlockWords * sizeof(uint32_t), hipHostMallocPortable | hipHostMallocMapped);
        if (e == hipSuccess && (e = hipHostGetDevicePointer(&q, p, 0)) != hipSuccess)
            (void)hipHostFree(p);
        if (e != hipSuccess) {
            (void)hipGetLastError();
            return e;
        }
        n.host = (uint32_t *)p;
        n.dev = (uint32_t *)q;
        for (uint32_t i = 0; i < kStatusBlockWords; ++i)
            n.unused.push_back(i);
        g_status_blocks.push_back(std::move(n));
        b = &g_status_blocks.back();
    }
    const uint32_t i = b->unused.back();
    b->unused.pop_back();
    w.host = b->host + i;
    w.dev = b->dev + i;
    *w.host = 0;
    return hipSuccess;
}

void status_free(StatusWord &w)
{
    if (!w.host)
        return;
    std::lock_guard<std::mutex> lock(g_status_mutex);
    for (size_t k = 0; k < g_status_blocks.size(); ++k) {
        StatusBlock &b = g_status_blocks[k];
        if (w.host < b.host || w.host >= b.host + kStatusBlockWords)
            continue;
        b.unused.push_back((uint32_t)(w.host - b.host));
        break;
    }
    w = StatusWord{};
}

// Frees the blocks without a word in use, but one.
void status_give_back()
{
    std::lock_guard<std::mutex> lock(g_status_mutex);
    for (size_t k = g_status_blocks.size(); k-- > 0 && g_status_blocks.size() > 1;)
        if (g_status_blocks[k].unused.size() == kStatusBlockWords) {
            (void)hipHostFree(g_status_blocks[k].host);
            g_status_blocks.erase(g_status_blocks.begin() + (ptrdiff_t)k);
        }
}

// What the host knows of a status word once the steps are complete.
bool status_set(const StatusWord &w) { return __atomic_load_n(w.host, __ATOMIC_ACQUIRE) != 0; }

} // namespace

struct lbm_domain {
    int nx = 0, ny = 0, nz = 0, storage = 0;
    unsigned periodic = 0;
    uint64_t ncells = 0, P = 0;
    hipStream_t stream = nullptr;
    bool own_stream = false;
    bool own_buffers = true;
    int device = 0;
    char *buf = nullptr;  // the population array
    uint64_t bytes = 0;   // its size
    int phase = 0;        // phase of the stored state (k_stream_collide)
    bool outlets = false; // the domain has outlet cells
    int outlet_kind = LBM_OUTLET_ZERO_GRADIENT;
    double rho_out = 1.0; // outlet density of the constant-pressure outlet
    double *d_stats = nullptr;  // statistics sums, [15][64 ntiles]
    bool stats_on = false;
    uint64_t stats_samples = 0; // local steps accumulated
    uint8_t *d_flags = nullptr;
    char *d_tables = nullptr; // one allocation: the tile list, wall masks, inlet tables, terms and velocity, outlet targets
    TileRec *d_tiles = nullptr;
    uint32_t *d_wall = nullptr, *d_inlet = nullptr, *d_inlrec = nullptr;
    float *d_uin = nullptr;                // [3][n_inlet], null until set
    float *uin_room = nullptr;             // where it goes
    uint16_t *d_targets = nullptr;         // outlet cells fed by each last-plane cell, [nz][ny]
    float *d_iterm = nullptr;              // inlet terms, [27][64] per inlet tile
    float *d_bzc = nullptr;                // curved-wall coefficients, [27][64] per wall tile
    float *d_bzaux = nullptr;              // f*_k of the curved links, [27][64] per wall tile
    uint64_t n_inlrec = 0;                 // inlet records
    uint32_t n_inl = 0;                    // inlet tiles
    std::vector<uint64_t> inlet_cells;     // inlet cells, ascending (index = inlet ordinal)
    StatusWord status;                     // set by a step that goes unstable, and ...
    StatusTwin *d_status = nullptr;        // ... its twin in device memory, in front of the flags
    uint64_t ntiles = 0, nwall = 0, n_updated = 0;
    double omega = 1.0, omega_b = 1.0;
    double omega_o[4] = {1.0, 1.0, 1.0, 1.0}; // orders 3..6
    int feq_order = 6;                        // 6: the full equilibrium; 2..5: explicit truncated one
    bool high1() const { return omega_o[0] == 1.0 && omega_o[1] == 1.0 && omega_o[2] == 1.0 && omega_o[3] == 1.0; }
    bool curved() const { return d_bzc != nullptr; }
    bool explicit_feq() const { return feq_order < 6; }
    int variant() const
    {
        return (explicit_feq() ? kVarFeq : (high1() ? kVarH1 : 0)) | (curved() ? kVarCurved : 0) |
               (outlet_kind == LBM_OUTLET_PRESSURE ? kVarPressure : 0);
    }
    bool force_wide = false; // lbm_debug_wide_addressing
    uint32_t grid_blocks = 0; // lbm_debug_step_grid: blocks of a step launch (0: one wave per tile)
    // the step kernels address the array with 64-bit global instructions
    // (past the 4 GiB that buffer instructions reach)
    bool wide() const { return force_wide || bytes > kNarrowBytes; }
    bool unstable = false;
    hipGraphExec_t graph = nullptr; // kGraphSteps steps from phase 0
    hipGraph_t graph_def = nullptr;
    bool graph_dirty = true;
    uint64_t asked = 0; // steps asked for since the step kernels or their arguments last changed
    void changed()
    {
        graph_dirty = true;
        asked = 0;
    }
    lbm_batch *batch = nullptr;    // resident in this batch
    uint64_t device_bytes = 0;
    uint64_t flags_hash = 0;       // FNV-1a 64 of the creation flags (state images name it)
};

namespace {

// Device memory of domains comes from the stream-ordered allocator: a free
// does not synchronise the device (a service frees domains while other
// domains keep running), and freed memory stays in the device's pool for
// the next domain.
std::mutex g_pool_mutex;
bool g_pool_ready[64];

void pool_setup(int device)
{
    std::lock_guard<std::mutex> lock(g_pool_mutex);
    if (device < 0 || device >= 64 || g_pool_ready[device])
        return;
    hipMemPool_t pool;
    if (hipDeviceGetDefaultMemPool(&pool, device) == hipSuccess) {
        uint64_t keep = UINT64_MAX;
        (void)hipMemPoolSetAttribute(pool, hipMemPoolAttrReleaseThreshold, &keep);
    }
    (void)hipGetLastError();
    g_pool_ready[device] = true;
}

hipError_t dalloc(hipStream_t s, void **p, size_t n)
{
    *p = nullptr;
    if (n == 0)
        return hipSuccess;
    hipError_t e = hipMallocAsync(p, n, s);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        *p = nullptr;
    }
    return e;
}

void dfree(hipStream_t s, void *p)
{
    if (p)
        (void)hipFreeAsync(p, s);
}

// Copies between host memory and the domain's memory, in the domain's
// stream order; they return once the copy is complete.
hipError_t copy_sync(hipStream_t s, void *dst, const void *src, size_t n, hipMemcpyKind kind)
{
    if (n == 0)
        return hipSuccess;
    hipError_t e = hipMemcpyAsync(dst, src, n, kind, s);
    if (e != hipSuccess)
        return e;
    return hipStreamSynchronize(s);
}

KDomain kdomain(const lbm_domain *d)
{
    KDomain k{};
    k.buf = d->buf;
    k.flags = d->d_flags;
    k.stats = d->stats_on ? d->d_stats : nullptr;
    k.sstride = (uint32_t)(d->ntiles * 64);
    k.wall = d->d_wall;
    k.targets = d->d_targets;
    k.iterm = d->d_iterm;
    k.bzc = d->d_bzc;
    k.bzaux = d->d_bzaux;
    k.rowtiles = d->nx % 64 == 0 ? (uint32_t)(d->nx / 64) : 0u;
    k.drow = make_fastdiv(k.rowtiles ? k.rowtiles : 1u);
    k.status = &d->d_status->word;
    k.P = (uint32_t)d->P;
    k.tbytes = (uint32_t)(Q * 64 * storage_bytes(d->storage));
    k.side = d->P / 64 * k.tbytes;
    k.bufbytes = d->bytes <= kNarrowBytes ? (uint32_t)d->bytes : 0u; // read by the narrow kernels only
    k.nx = d->nx;
    k.ny = d->ny;
    k.nz = d->nz;
    k.ncells = (uint32_t)d->ncells;
    k.dnx = make_fastdiv(d->nx);
    k.dny = make_fastdiv(d->ny);
    k.periodic = d->periodic;
    k.omega = (float)d->omega;
    k.omega_b = (float)d->omega_b;
    for (int n = 0; n < 4; ++n)
        k.omega_o[n] = (float)d->omega_o[n];
    k.outlet = d->outlet_kind == LBM_OUTLET_PRESSURE ? 1u : 0u;
    k.high1 = d->high1() ? 1u : 0u;
    k.rho_out = (float)d->rho_out;
    k.feq_order = (uint32_t)d->feq_order;
    return k;
}

uint32_t grid8(uint64_t blocks) { return (uint32_t)((blocks + 7) / 8 * 8); }

// Grid of the single-domain kernels: one wave per tile (a wave's loads and
// collision do not overlap within the wave, and tiles per wave beyond one
// measured slower).
uint32_t step_grid(const lbm_domain *d)
{
    if (d->grid_blocks)
        return d->grid_blocks;
    return grid8((d->ntiles + kWavesPerBlock - 1) / kWavesPerBlock);
}

template <typename F> decltype(auto) dispatch_storage(int st, F &&f)
{
    if (st == LBM_FP32)
        return f(std::integral_constant<int, ST_FP32>{});
    else if (st == LBM_FP16S)
        return f(std::integral_constant<int, ST_FP16S>{});
    else
        return f(std::integral_constant<int, ST_BF16S>{});
}

int sync_status(lbm_domain *d)
{
    HIP_TRY(hipStreamSynchronize(d->stream));
    if (status_set(d->status))
        d->unstable = true;
    return LBM_OK;
}

int check_domain(const lbm_domain *d)
{
    if (!d)
        return fail(LBM_ERR_ARG, "null domain");
    return LBM_OK;
}

void release_graph(lbm_domain *d)
{
    if (d->graph)
        (void)hipGraphExecDestroy(d->graph);
    if (d->graph_def)
        (void)hipGraphDestroy(d->graph_def);
    d->graph = nullptr;
    d->graph_def = nullptr;
    d->graph_dirty = true;
}

void free_domain(lbm_domain *d)
{
    release_graph(d);
    if (d->stream) {
        hipStream_t s = d->stream;
        // (the status word and the flags lie behind an own array)
        dfree(s, d->own_buffers ? (void *)d->buf : (void *)d->d_status);
        dfree(s, d->d_tables);
        dfree(s, d->d_bzc);
        dfree(s, d->d_bzaux);
        dfree(s, d->d_stats);
        if (d->own_stream)
            (void)hipStreamDestroy(s);
    }
    status_free(d->status);
    delete d;
}

// Calls fn(std::integral_constant<int, ST>, std::integral_constant<int, V>)
// for a storage and a kernel variant known at run time.
// The explicit equilibrium always takes the general collision, so a variant
// with both bits set runs as the one without the reduced-collision bit.
template <class Fn> decltype(auto) with_kernel(int storage, int v, Fn &&fn)
{
    return dispatch_storage(storage, [&](auto st) {
        switch ((v & kVarFeq) ? (v & ~kVarH1) : v) {
        case 0:
            return fn(st, std::integral_constant<int, 0>{});
        case 1:
            return fn(st, std::integral_constant<int, 1>{});
        case 2:
            return fn(st, std::integral_constant<int, 2>{});
        case 3:
            return fn(st, std::integral_constant<int, 3>{});
        case 4:
            return fn(st, std::integral_constant<int, 4>{});
        case 5:
            return fn(st, std::integral_constant<int, 5>{});
        case 6:
            return fn(st, std::integral_constant<int, 6>{});
        case 7:
            return fn(st, std::integral_constant<int, 7>{});
        case 8:
            return fn(st, std::integral_constant<int, 8>{});
        case 10:
            return fn(st, std::integral_constant<int, 10>{});
        case 12:
            return fn(st, std::integral_constant<int, 12>{});
        default:
            return fn(st, std::integral_constant<int, 14>{});
        }
    });
}

// The step kernel of a phase: the streaming step (phase 0) with row-aligned
// or general addressing, or the local step; narrow or wide (Pops).
const void *step_kernel(int storage, int v, uint32_t phase, bool rows, bool wide)
{
    return with_kernel(storage, v, [&](auto st, auto vc) -> const void * {
        constexpr int ST = decltype(st)::value, V = decltype(vc)::value;
        if (wide) {
            if (phase == 1)
                return (const void *)k_local_collide<ST, V, true>;
            return rows ? (const void *)k_stream_collide<ST, V, true, true>
                        : (const void *)k_stream_collide<ST, V, false, true>;
        }
        if (phase == 1)
            return (const void *)k_local_collide<ST, V, false>;
        return rows ? (const void *)k_stream_collide<ST, V, true, false>
                    : (const void *)k_stream_collide<ST, V, false, false>;
    });
}

hipError_t launch_step(const lbm_domain *d, uint32_t phase)
{
    if (d->ntiles == 0)
        return hipSuccess;
    KDomain k = kdomain(d);
    const TileRec *tiles = d->d_tiles;
    uint32_t nt = (uint32_t)d->ntiles;
    void *args[] = {&k, &tiles, &nt};
    const hipError_t e = hipLaunchKernel(step_kernel(d->storage, d->variant(), phase, k.rowtiles != 0, d->wide()),
                                         dim3(step_grid(d)), dim3(kBlock), args, 0, d->stream);
    return e != hipSuccess ? e : hipGetLastError();
}

// Rebuild the inlet terms of the inlet tiles from the inlet velocity (all
// zero while none is set).
hipError_t build_inlet_terms(const lbm_domain *d)
{
    if (d->n_inl == 0)
        return hipSuccess;
    const uint32_t blocks = (uint32_t)((d->ntiles + 3) / 4);
    hipLaunchKernelGGL(k_inlet_terms, dim3(blocks), dim3(256), 0, d->stream, (const TileRec *)d->d_tiles,
                       (uint32_t)d->ntiles, (const uint32_t *)d->d_inlet, (const uint32_t *)d->d_inlrec,
                       (const float *)d->d_uin, (uint32_t)d->inlet_cells.size(), d->d_iterm);
    return hipGetLastError();
}

// First side rows of a phase-0 state (the outlet cells' clamped values).
hipError_t side_refresh(const lbm_domain *d)
{
    if (!d->outlets)
        return hipSuccess;
    const KDomain k = kdomain(d);
    const uint32_t blocks = (uint32_t)(((uint64_t)d->ny * d->nz + 255) / 256);
    dispatch_storage(d->storage, [&](auto st) {
        hipLaunchKernelGGL((k_side_refresh<decltype(st)::value>), dim3(blocks), dim3(256), 0, d->stream, k);
    });
    return hipGetLastError();
}

// Curved-wall values of a phase-0 state (k_curved_refresh).
hipError_t curved_refresh(const lbm_domain *d)
{
    if (!d->d_bzaux || !d->ntiles)
        return hipSuccess;
    const KDomain k = kdomain(d);
    const uint32_t blocks = (uint32_t)((d->ntiles + 3) / 4);
    dispatch_storage(d->storage, [&](auto st) {
        hipLaunchKernelGGL((k_curved_refresh<decltype(st)::value>), dim3(blocks), dim3(256), 0, d->stream, k,
                           (const TileRec *)d->d_tiles, (uint32_t)d->ntiles);
    });
    return hipGetLastError();
}

// Bring the stored state to phase 0, the form every state access uses.
hipError_t normalise(lbm_domain *d)
{
    if (d->phase == 0)
        return hipSuccess;
    if (d->ntiles) {
        const KDomain k = kdomain(d);
        const uint32_t blocks = (uint32_t)((d->ntiles + 3) / 4);
        dispatch_storage(d->storage, [&](auto st) {
            hipLaunchKernelGGL((k_normalise<decltype(st)::value>), dim3(blocks), dim3(256), 0, d->stream, k,
                               (const TileRec *)d->d_tiles, (uint32_t)d->ntiles);
        });
        if (hipError_t e = hipGetLastError())
            return e;
    }
    d->phase = 0;
    return hipSuccess;
}

// f^eq in the cells [c0, c0 + count), phase 0, from the fields of the first n
// of them (null: rho = 1, u = 0).
void launch_init_eq(const lbm_domain *d, const float *rho, const float *u, uint32_t c0, uint32_t n, uint32_t count)
{
    const KDomain k = kdomain(d);
    dispatch_storage(d->storage, [&](auto st) {
        hipLaunchKernelGGL((k_init_eq<decltype(st)::value>), dim3((count + 255) / 256), dim3(256), 0, d->stream, k, rho,
                           u, c0, n, count);
    });
}

// What follows an f^eq in every cell.  The caller waits for the stream and
// clears the status word then.
int init_done(lbm_domain *d)
{
    HIP_TRY(hipGetLastError());
    d->phase = 0;
    HIP_TRY(side_refresh(d));
    HIP_TRY(curved_refresh(d));
    return LBM_OK;
}

// A new state (no step in flight): stable until a step says otherwise.  The
// device word is set exactly when the host word is.
int clear_status(lbm_domain *d)
{
    if (status_set(d->status)) {
        HIP_TRY(hipMemsetAsync(&d->d_status->word, 0, sizeof(uint32_t), d->stream));
        HIP_TRY(hipStreamSynchronize(d->stream));
        *d->status.host = 0;
    }
    d->unstable = false;
    return LBM_OK;
}

// Cells rounded up to whole 64-cell tiles.
uint64_t plane_stride(uint64_t ncells) { return (ncells + 63) / 64 * 64; }

// Read-back buffer of lbm_get_moments_noalloc, for callers that cannot
// allocate: a fixed device array (64 MiB, 4 floats per cell) that each
// device holds from the library's load to the end of the process.  Host
// code uses it only through the device address hipGetSymbolAddress gives
// for the current device, resolved once per device.  Calls on one device
// share it, so they are serialised by a lock.
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex[kMaxDevices];
std::mutex g_scratch_resolve;
float *g_scratch_ptr[kMaxDevices];

int scratch_address(int device, float **out)
{
    if (device < 0 || device >= kMaxDevices)
        return fail(LBM_ERR_DEVICE, "device %d out of range", device);
    std::lock_guard<std::mutex> lock(g_scratch_resolve);
    if (!g_scratch_ptr[device]) {
        int cur = 0;
        HIP_TRY(hipGetDevice(&cur));
        HIP_TRY(hipSetDevice(device));
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        (void)hipSetDevice(cur);
        if (e != hipSuccess || !p)
            return fail(LBM_ERR_DEVICE, "read-back buffer address: %s", hipGetErrorString(e));
        g_scratch_ptr[device] = (float *)p;
    }
    *out = g_scratch_ptr[device];
    return LBM_OK;
}

} // namespace

namespace {

// Test hook (lbm_debug_fail_after): the n-th fallible allocation or upload
// of the batch calls, pinned pair or chunk of a field transfer from now on
// fails as if memory were exhausted.
std::atomic<int> g_fail_countdown{0};

bool injected_failure()
{
    int c = g_fail_countdown.load();
    while (c > 0)
        if (g_fail_countdown.compare_exchange_weak(c, c - 1))
            return c == 1;
    return false;
}

} // namespace

#include "lbm_build.inc"
#include "lbm_transfer.inc"

namespace {

// The tables of a new domain from its flags (d->d_flags, host copy in
// flags), with the population array as scratch memory; d's counts and the
// hash of the flags.  One host wait, for the counts the tables are
// allocated by.
int build_tables(lbm_domain *d, const uint8_t *flags)
{
    const KDomain k = kdomain(d);
    const uint32_t nt = (uint32_t)(d->P / 64), ngroups = (nt + kGroupTiles - 1) / kGroupTiles;
    const uint64_t hash_groups = d->ncells / kGroupCells, n_inlet = d->inlet_cells.size();
    const BuildScratch w = build_scratch(d->buf, nt, ngroups, hash_groups, n_inlet);
    if (w.bytes > d->bytes)
        return fail(LBM_ERR_STATE, "scratch of %llu bytes exceeds the array", (unsigned long long)w.bytes);
    const std::vector<uint32_t> cells(d->inlet_cells.begin(), d->inlet_cells.end());
    HIP_TRY(copy_sync(d->stream, w.inlet_cells, cells.data(), cells.size() * 4, hipMemcpyHostToDevice));
    const dim3 tiles((nt + 3) / 4);
    hipLaunchKernelGGL(k_tile_count, tiles, dim3(256), 0, d->stream, k, nt, w.tile, w.nupd);
    hipLaunchKernelGGL(k_group_count, dim3(ngroups), dim3(kGroupTiles), 0, d->stream, nt, (const uint64_t *)w.tile,
                       (const uint8_t *)w.nupd, w.group);
    hipLaunchKernelGGL(k_group_scan, dim3(1), dim3(kScanThreads), 0, d->stream, ngroups, w.group, w.total,
                       d->d_status, d->status.dev);
    if (hash_groups)
        hipLaunchKernelGGL(k_flags_hash, dim3((uint32_t)hash_groups), dim3(kGroupTiles), 0, d->stream,
                           (const uint8_t *)d->d_flags, w.maps);
    HIP_TRY(hipGetLastError());
    std::vector<uint64_t> back(8 + hash_groups * sizeof(FnvMap) / 8);
    HIP_TRY(copy_sync(d->stream, back.data(), w.total, back.size() * 8, hipMemcpyDeviceToHost));
    d->ntiles = back[0];
    d->nwall = back[1];
    d->n_inl = (uint32_t)back[2];
    d->n_inlrec = back[3];
    d->n_updated = back[4];
    d->flags_hash = fnv_finish((const FnvMap *)(back.data() + 8), hash_groups, flags + hash_groups * kGroupCells,
                               d->ncells - hash_groups * kGroupCells);
    const uint64_t size[7] = {d->ntiles * sizeof(TileRec),
                              d->nwall * 256,
                              d->nwall * 256,
                              d->n_inlrec * kRecWords * 4,
                              (uint64_t)d->n_inl * Q * 64 * sizeof(float),
                              3 * n_inlet * sizeof(float),
                              d->outlets ? (uint64_t)d->ny * d->nz * sizeof(uint16_t) : 0};
    uint64_t at[8] = {0};
    for (int j = 0; j < 7; ++j) {
        at[j + 1] = at[j] + (size[j] + 255) / 256 * 256;
        d->device_bytes += j != 5 ? size[j] : 0; // the inlet velocity counts once it is set
    }
    if (dalloc(d->stream, (void **)&d->d_tables, at[7]) != hipSuccess)
        return fail(LBM_ERR_OOM, "domain tables");
    d->d_tiles = (TileRec *)d->d_tables;
    d->d_wall = (uint32_t *)(d->d_tables + at[1]);
    d->d_inlet = (uint32_t *)(d->d_tables + at[2]);
    d->d_inlrec = (uint32_t *)(d->d_tables + at[3]);
    d->d_iterm = (float *)(d->d_tables + at[4]);
    d->uin_room = (float *)(d->d_tables + at[5]);
    d->d_targets = (uint16_t *)(d->d_tables + at[6]);
    if (d->outlets)
        hipLaunchKernelGGL(k_outlet_targets, dim3((uint32_t)(((uint64_t)d->ny * d->nz + 255) / 256)), dim3(256), 0,
                           d->stream, k, d->d_targets);
    hipLaunchKernelGGL(k_tile_write, tiles, dim3(256), 0, d->stream, k, nt, (const uint64_t *)w.tile,
                       (const uint32_t *)w.group, d->outlets ? 1u : 0u, (const uint32_t *)w.inlet_cells,
                       (uint32_t)n_inlet, d->d_tiles, d->d_wall, d->d_inlet, d->d_inlrec);
    HIP_TRY(hipGetLastError());
    return LBM_OK;
}

// Host copies of the tile list ...
int host_tiles(const lbm_domain *d, std::vector<TileRec> &tiles)
{
    tiles.resize(d->ntiles);
    HIP_TRY(copy_sync(d->stream, tiles.data(), d->d_tiles, tiles.size() * sizeof(TileRec), hipMemcpyDeviceToHost));
    return LBM_OK;
}

// ... and, per lane of the wall tiles, of the link masks and the inlet links.
int host_links(const lbm_domain *d, std::vector<uint32_t> &wall, std::vector<uint32_t> &inlm)
{
    wall.resize(d->nwall * 64);
    inlm.resize(d->nwall * 64);
    std::vector<uint32_t> rec(d->n_inlrec * kRecWords);
    HIP_TRY(copy_sync(d->stream, wall.data(), d->d_wall, wall.size() * 4, hipMemcpyDeviceToHost));
    HIP_TRY(copy_sync(d->stream, inlm.data(), d->d_inlet, inlm.size() * 4, hipMemcpyDeviceToHost));
    HIP_TRY(copy_sync(d->stream, rec.data(), d->d_inlrec, rec.size() * 4, hipMemcpyDeviceToHost));
    for (uint32_t &v : inlm)
        v = v == kNoRec ? 0u : rec[(size_t)v * kRecWords];
    return LBM_OK;
}

int create(const uint8_t *flags, int nx, int ny, int nz, unsigned periodic, int storage, void *hip_stream, void *fa,
           lbm_domain **out)
{
    if (!out)
        return fail(LBM_ERR_ARG, "out is null");
    *out = nullptr;
    if (!flags)
        return fail(LBM_ERR_ARG, "flags is null");
    if (nx < 1 || ny < 1 || nz < 1 || nx > 65535 || ny > 65535 || nz > 65535)
        return fail(LBM_ERR_ARG, "bad grid %d x %d x %d", nx, ny, nz);
    if (storage < LBM_FP32 || storage > LBM_BF16S)
        return fail(LBM_ERR_ARG, "bad storage %d", storage);
    if (periodic > 7u)
        return fail(LBM_ERR_ARG, "bad periodic mask %u", periodic);
    const uint64_t ncells = (uint64_t)nx * ny * nz;
    const uint64_t P = plane_stride(ncells);
    const uint64_t bufbytes = array_bytes(P, ny, nz, storage);
    // cell indices are 32-bit
    if (P > (1ull << 32) - 64)
        return fail(LBM_ERR_ARG, "domain of %llu cells; the limit is 2^32 - 64 cells", (unsigned long long)ncells);
    std::vector<uint64_t> inlet_cells;
    bool outlets = false;
    if (int rc = check_flags(flags, nx, ncells, periodic, inlet_cells, outlets))
        return rc;

    lbm_domain *d = new lbm_domain();
    d->nx = nx;
    d->ny = ny;
    d->nz = nz;
    d->storage = storage;
    d->periodic = periodic;
    d->ncells = ncells;
    d->P = P;
    d->bytes = bufbytes;
    d->outlets = outlets;
    d->inlet_cells = std::move(inlet_cells);
    auto bail = [&](int code) {
        free_domain(d);
        return code;
    };
    if (hipGetDevice(&d->device) != hipSuccess)
        return bail(fail(LBM_ERR_DEVICE, "no HIP device"));
    if (hip_stream) {
        d->stream = (hipStream_t)hip_stream;
    } else {
        if (hipStreamCreateWithFlags(&d->stream, hipStreamNonBlocking) != hipSuccess)
            return bail(fail(LBM_ERR_DEVICE, "hipStreamCreate failed"));
        d->own_stream = true;
    }
    pool_setup(d->device);
    auto up = [&](void *dst, const void *src, size_t n) {
        return copy_sync(d->stream, dst, src, n, hipMemcpyHostToDevice) == hipSuccess;
    };
    if (fa) {
        d->own_buffers = false;
        d->buf = (char *)fa;
        if ((uintptr_t)fa & 255u)
            return bail(fail(LBM_ERR_ARG, "an adopted population array must be 256-byte aligned"));
        d->device_bytes += bufbytes;
    }
    // an own array with the status word and the flags behind it is one
    // allocation, the tables another: a freed pair is found again whole by
    // the next domain of its size, where of many pieces the pool gave some
    // back to the device and had to ask for them again (freeing a domain of
    // 64 x 64 x 256 cells 577 -> 120 us)
    constexpr size_t kStatusRoom = 256; // keeps the flags aligned
    const size_t before = fa ? 0 : bufbytes;
    char *own = nullptr;
    if (dalloc(d->stream, (void **)&own, before + kStatusRoom + ncells) != hipSuccess)
        return bail(fail(LBM_ERR_OOM, "population array (%llu bytes)", (unsigned long long)bufbytes));
    if (!fa)
        d->buf = own;
    d->d_status = (StatusTwin *)(own + before);
    d->d_flags = (uint8_t *)own + before + kStatusRoom;
    d->device_bytes += before + kStatusRoom + ncells;
    if (status_alloc(d->status) != hipSuccess)
        return bail(fail(LBM_ERR_OOM, "status word"));
    if (!up(d->d_flags, flags, ncells))
        return bail(fail(LBM_ERR_DEVICE, "upload of the flags failed"));
    if (int rc = build_tables(d, flags))
        return bail(rc);
    if (build_inlet_terms(d) != hipSuccess)
        return bail(fail(LBM_ERR_DEVICE, "inlet terms"));
    d->omega = d->omega_b = 1.0 / 0.6;
    // the side rows' elements that no outlet cell uses, and the padding
    // after them, are never written: zero, so that state images are
    // deterministic (the tile blocks are written by init_eq)
    const uint64_t tile_bytes = (uint64_t)Q * P * storage_bytes(storage);
    if (hipMemsetAsync(d->buf + tile_bytes, 0, bufbytes - tile_bytes, d->stream) != hipSuccess)
        return bail(fail(LBM_ERR_DEVICE, "side rows"));
    launch_init_eq(d, nullptr, nullptr, 0, (uint32_t)ncells, (uint32_t)P);
    int rc = init_done(d);
    if (rc == LBM_OK && hipStreamSynchronize(d->stream) != hipSuccess)
        rc = fail(LBM_ERR_DEVICE, "initialisation failed");
    if (rc != LBM_OK)
        return bail(rc);
    *out = d;
    return LBM_OK;
}

// Append a kernel node after `prev` (or as a root when prev is null).  The
// argument values are copied into the node.
hipError_t add_kernel_node(hipGraph_t g, hipGraphNode_t prev, const void *func, uint32_t grid, uint32_t block,
                           void **args, hipGraphNode_t *out)
{
    hipKernelNodeParams p{};
    p.func = const_cast<void *>(func);
    p.gridDim = dim3(grid);
    p.blockDim = dim3(block);
    p.sharedMemBytes = 0;
    p.kernelParams = args;
    p.extra = nullptr;
    return hipGraphAddKernelNode(out, g, prev ? &prev : nullptr, prev ? 1 : 0, &p);
}


// Build (not capture) the step graph: kGraphSteps step nodes in a chain,
// starting in phase 0.  Built node by node so that work other threads issue
// meanwhile cannot interfere.
int build_graph(lbm_domain *d)
{
    release_graph(d);
    KDomain k = kdomain(d);
    const TileRec *tiles = d->d_tiles;
    uint32_t nt = (uint32_t)d->ntiles;
    HIP_TRY(hipGraphCreate(&d->graph_def, 0));
    hipGraphNode_t prev = nullptr;
    for (int s = 0; s < kGraphSteps; ++s) {
        const void *fn = step_kernel(d->storage, d->variant(), (uint32_t)(s & 1), k.rowtiles != 0, d->wide());
        void *args[] = {&k, &tiles, &nt};
        hipGraphNode_t node = nullptr;
        HIP_TRY(add_kernel_node(d->graph_def, prev, fn, step_grid(d), kBlock, args, &node));
        prev = node;
    }
    HIP_TRY(hipGraphInstantiate(&d->graph, d->graph_def, nullptr, nullptr, 0));
    d->graph_dirty = false;
    return LBM_OK;
}

} // namespace

// ===========================================================================
// C ABI
// ===========================================================================
extern "C" {

const char *lbm_last_error(void) { return g_err.c_str(); }

const char *lbm_version(void) { return "lbm-d3q27-chm gfx950 0.1"; }

uint64_t lbm_array_bytes(int nx, int ny, int nz, int storage)
{
    if (nx < 1 || ny < 1 || nz < 1 || nx > 65535 || ny > 65535 || nz > 65535 || storage < LBM_FP32 ||
        storage > LBM_BF16S)
        return 0;
    return array_bytes(plane_stride((uint64_t)nx * ny * nz), ny, nz, storage);
}

int lbm_create_domain(const uint8_t *flags, int nx, int ny, int nz, unsigned periodic, int storage,
                      void *hip_stream, lbm_domain **out)
{
    return create(flags, nx, ny, nz, periodic, storage, hip_stream, nullptr, out);
}

int lbm_create_domain_ext(const uint8_t *flags, int nx, int ny, int nz, unsigned periodic, int storage,
                          void *hip_stream, void *f, lbm_domain **out)
{
    if (!f)
        return fail(LBM_ERR_ARG, "adopted population array is null");
    return create(flags, nx, ny, nz, periodic, storage, hip_stream, f, out);
}

int lbm_set_rates(lbm_domain *d, double omega, double omega_bulk, double omega_high)
{
    if (int rc = check_domain(d))
        return rc;
    if (!(omega >= 0 && omega <= 2) || !(omega_bulk >= 0 && omega_bulk <= 2) ||
        !(omega_high >= 0 && omega_high <= 2))
        return fail(LBM_ERR_ARG, "rates must lie in [0, 2]");
    if (d->batch)
        return fail(LBM_ERR_STATE, "domain is resident in a batch");
    d->omega = omega;
    d->omega_b = omega_bulk;
    for (int n = 0; n < 4; ++n)
        d->omega_o[n] = omega_high;
    d->changed();
    return LBM_OK;
}

int lbm_set_order_rates(lbm_domain *d, double omega3, double omega4, double omega5, double omega6)
{
    if (int rc = check_domain(d))
        return rc;
    const double w[4] = {omega3, omega4, omega5, omega6};
    for (double v : w)
        if (!(v >= 0 && v <= 2))
            return fail(LBM_ERR_ARG, "rates must lie in [0, 2]");
    if (d->batch)
        return fail(LBM_ERR_STATE, "domain is resident in a batch");
    for (int n = 0; n < 4; ++n)
        d->omega_o[n] = w[n];
    d->changed();
    return LBM_OK;
}

int lbm_set_equilibrium_order(lbm_domain *d, int order)
{
    if (int rc = check_domain(d))
        return rc;
    if (order < 2 || order > 6)
        return fail(LBM_ERR_ARG, "equilibrium order %d outside 2..6", order);
    if (d->batch)
        return fail(LBM_ERR_STATE, "domain is resident in a batch");
    d->feq_order = order;
    d->changed();
    return LBM_OK;
}

int lbm_debug_wide_addressing(lbm_domain *d, int on)
{
    if (int rc = check_domain(d))
        return rc;
    if (on != 0 && on != 1)
        return fail(LBM_ERR_ARG, "on must be 0 or 1");
    if (d->batch)
        return fail(LBM_ERR_STATE, "domain is resident in a batch");
    d->force_wide = on == 1;
    d->changed();
    return LBM_OK;
}

int lbm_debug_step_grid(lbm_domain *d, int blocks)
{
    if (int rc = check_domain(d))
        return rc;
    if (blocks < 0 || blocks % 8 != 0 || blocks > (1 << 20))
        return fail(LBM_ERR_ARG, "blocks must be 0 or a positive multiple of 8 up to 2^20, got %d", blocks);
    if (d->batch)
        return fail(LBM_ERR_STATE, "domain is resident in a batch");
    d->grid_blocks = (uint32_t)blocks;
    d->changed();
    return LBM_OK;
}

int lbm_is_wide(const lbm_domain *d, int *wide)
{
    if (int rc = check_domain(d))
        return rc;
    if (!wide)
        return fail(LBM_ERR_ARG, "wide is null");
    *wide = d->wide() ? 1 : 0;
    return LBM_OK;
}

int lbm_set_outlet(lbm_domain *d, int kind, double rho_out)
{
    if (int rc = check_domain(d))
        return rc;
    if (kind != LBM_OUTLET_ZERO_GRADIENT && kind != LBM_OUTLET_PRESSURE)
        return fail(LBM_ERR_ARG, "unknown outlet kind %d", kind);
    if (!(rho_out > 0) || !std::isfinite(rho_out))
        return fail(LBM_ERR_ARG, "rho_out must be positive and finite");
    if (d->batch)
        return fail(LBM_ERR_STATE, "domain is resident in a batch");
    HIP_TRY(normalise(d));
    d->outlet_kind = kind;
    d->rho_out = rho_out;
    HIP_TRY(side_refresh(d));
    d->changed();
    return LBM_OK;
}

int lbm_set_wall_distances(lbm_domain *d, const float *q)
{
    if (int rc = check_domain(d))
        return rc;
    if (d->batch)
        return fail(LBM_ERR_STATE, "domain is resident in a batch");
    if (!q && !d->curved()) { // the halfway rule, as it is
        HIP_TRY(normalise(d));
        return LBM_OK;
    }
    const size_t nco = (size_t)d->nwall * Q * 64;
    std::vector<TileRec> tiles;
    if (int rc = host_tiles(d, tiles))
        return rc;
    std::vector<float> coef;
    std::vector<uint32_t> bz(tiles.size(), 0u), far(tiles.size(), 0u);
    if (q) {
        std::vector<uint32_t> wall, inlm;
        if (int rc = host_links(d, wall, inlm))
            return rc;
        coef.assign(nco, 1.f);
        for (size_t t = 0; t < tiles.size(); ++t) {
            const TileRec &r = tiles[t];
            if (r.wall < 0)
                continue;
            for (uint32_t l = 0; l < 64; ++l) {
                if (!((r.act[l >> 5] >> (l & 31)) & 1u))
                    continue;
                const uint64_t c = (uint64_t)r.tile * 64 + l;
                const size_t wl = (size_t)r.wall * 64 + l;
                const uint32_t m = wall[wl], il = inlm[wl];
                for (int k = 0; k < Q; ++k) {
                    if (!((m >> k) & 1u) || ((il >> k) & 1u))
                        continue; // not a wall link
                    const double qq = q[(size_t)k * d->ncells + c];
                    if (!(qq > 0.0 && qq <= 1.0))
                        return fail(LBM_ERR_ARG, "wall fraction %g of link %d of cell %llu outside (0, 1]", qq, k,
                                    (unsigned long long)c);
                    if (qq == 0.5 || (qq < 0.5 && ((m >> (Q - 1 - k)) & 1u)))
                        continue; // halfway rule
                    const bool near = qq < 0.5;
                    const float a = (float)(near ? 2.0 * qq : 1.0 / (2.0 * qq));
                    coef[((size_t)r.wall * Q + k) * 64 + l] = near ? a : -a;
                    far[t] |= near ? 0u : 1u << k;
                    bz[t] |= 1u << k;
                }
            }
        }
    }
    bool any = false;
    for (uint32_t b : bz)
        any |= b != 0;
    HIP_TRY(normalise(d));
    if (any && !d->d_bzc) {
        if (dalloc(d->stream, (void **)&d->d_bzc, nco * sizeof(float)) != hipSuccess ||
            dalloc(d->stream, (void **)&d->d_bzaux, nco * sizeof(float)) != hipSuccess) {
            dfree(d->stream, d->d_bzc);
            d->d_bzc = nullptr;
            d->d_bzaux = nullptr;
            return fail(LBM_ERR_OOM, "curved-wall tables");
        }
        d->device_bytes += nco * 2 * sizeof(float);
    }
    if (!any && d->d_bzc) {
        dfree(d->stream, d->d_bzc);
        dfree(d->stream, d->d_bzaux);
        d->d_bzc = nullptr;
        d->d_bzaux = nullptr;
        d->device_bytes -= nco * 2 * sizeof(float);
    }
    for (size_t t = 0; t < bz.size(); ++t) {
        tiles[t].bz = bz[t];
        tiles[t].edge = (tiles[t].edge & kEdge) | far[t];
    }
    HIP_TRY(copy_sync(d->stream, d->d_tiles, tiles.data(), tiles.size() * sizeof(TileRec), hipMemcpyHostToDevice));
    if (any) {
        HIP_TRY(copy_sync(d->stream, d->d_bzc, coef.data(), nco * sizeof(float), hipMemcpyHostToDevice));
        // kept values of lanes and links without a curved coefficient are
        // never written: zero, so that state images are deterministic
        HIP_TRY(hipMemsetAsync(d->d_bzaux, 0, nco * sizeof(float), d->stream));
        HIP_TRY(curved_refresh(d));
        HIP_TRY(hipStreamSynchronize(d->stream));
    }
    d->changed();
    return LBM_OK;
}

int lbm_set_params(lbm_domain *d, double tau, double omega_bulk, double omega_high)
{
    if (int rc = check_domain(d))
        return rc;
    if (!(tau > 0.5) || !std::isfinite(tau))
        return fail(LBM_ERR_ARG, "tau must be > 0.5");
    if (!(omega_bulk > 0 && omega_bulk < 2))
        return fail(LBM_ERR_ARG, "omega_bulk must lie in (0, 2)");
    if (!(omega_high > 0 && omega_high <= 2))
        return fail(LBM_ERR_ARG, "omega_high must lie in (0, 2]");
    return lbm_set_rates(d, 1.0 / tau, omega_bulk, omega_high);
}

int lbm_set_inlet_cells(lbm_domain *d, const float *u_inlet)
{
    if (int rc = check_domain(d))
        return rc;
    if (!u_inlet)
        return fail(LBM_ERR_ARG, "u_inlet is null");
    if (d->batch)
        return fail(LBM_ERR_STATE, "domain is resident in a batch");
    const size_t n = d->inlet_cells.size();
    if (n == 0)
        return LBM_OK;
    if (!d->d_uin) {
        d->d_uin = d->uin_room;
        d->device_bytes += 3 * n * sizeof(float);
        d->changed();
    }
    // a phase-1 state carries the old terms in its bounce-back slots
    HIP_TRY(normalise(d));
    HIP_TRY(copy_sync(d->stream, d->d_uin, u_inlet, 3 * n * sizeof(float), hipMemcpyHostToDevice));
    HIP_TRY(build_inlet_terms(d));
    HIP_TRY(hipStreamSynchronize(d->stream));
    return LBM_OK;
}

int lbm_set_inlet(lbm_domain *d, const float *u_in)
{
    if (int rc = check_domain(d))
        return rc;
    if (!u_in)
        return fail(LBM_ERR_ARG, "u_in is null");
    const size_t n = d->inlet_cells.size();
    std::vector<float> compact(3 * n);
    for (int a = 0; a < 3; ++a)
        for (size_t k = 0; k < n; ++k)
            compact[a * n + k] = u_in[a * d->ncells + d->inlet_cells[k]];
    return lbm_set_inlet_cells(d, compact.data());
}

int lbm_init_fields(lbm_domain *d, const float *rho, const float *u)
{
    if (int rc = check_domain(d))
        return rc;
    if (d->batch)
        return fail(LBM_ERR_STATE, "domain is resident in a batch");
    if (!rho && !u) {
        launch_init_eq(d, nullptr, nullptr, 0, (uint32_t)d->ncells, (uint32_t)d->P);
    } else {
        // chunks of rho, then u; the last one also covers the padding cells
        const int first = rho ? 0 : 1, comps = (rho ? 1 : 0) + (u ? 3 : 0);
        const Moved m = move_fields<false, const float>(
            d, comps,
            [&](uint32_t c0, uint32_t n, const float *dev) {
                const uint32_t count = c0 + n == d->ncells ? (uint32_t)d->P - c0 : n;
                launch_init_eq(d, rho ? dev : nullptr, u ? dev + (rho ? n : 0) : nullptr, c0, n, count);
            },
            [&](int k) { return k + first == 0 ? rho : u + (size_t)(k + first - 1) * d->ncells; });
        if (int rc = moved_in(d, m, "upload of the fields"))
            return rc;
    }
    d->unstable = true; // until the new state is complete
    if (int rc = init_done(d))
        return rc;
    HIP_TRY(hipStreamSynchronize(d->stream));
    return clear_status(d);
}

int lbm_step_async(lbm_domain *d, int n)
{
    if (int rc = check_domain(d))
        return rc;
    if (n < 0)
        return fail(LBM_ERR_ARG, "negative step count");
    if (d->batch)
        return fail(LBM_ERR_STATE, "domain is resident in a batch");
    if (d->unstable)
        return fail(LBM_ERR_UNSTABLE, "domain went unstable earlier; re-initialise it");
    if (d->ntiles == 0) // nothing is updated, the state stays as it is
        return LBM_OK;
    d->asked += (uint64_t)n;
    if (d->graph_dirty && d->asked >= (uint64_t)kGraphBuild && n - (d->phase == 1) >= kGraphSteps)
        if (int rc = build_graph(d))
            return rc;
    int left = n;
    uint64_t local_steps = 0;
    if (left > 0 && d->phase == 1) {
        HIP_TRY(launch_step(d, 1));
        d->phase = 0;
        --left;
        ++local_steps;
    }
    while (!d->graph_dirty && left >= kGraphSteps) {
        HIP_TRY(hipGraphLaunch(d->graph, d->stream));
        left -= kGraphSteps;
        local_steps += (uint64_t)kGraphSteps / 2;
    }
    while (left > 0) {
        HIP_TRY(launch_step(d, (uint32_t)d->phase));
        local_steps += (uint64_t)d->phase;
        d->phase ^= 1;
        --left;
    }
    if (d->stats_on)
        d->stats_samples += local_steps;
    return LBM_OK;
}

int lbm_step_wait(lbm_domain *d)
{
    if (int rc = check_domain(d))
        return rc;
    if (d->batch)
        return fail(LBM_ERR_STATE, "domain is resident in a batch");
    if (int rc = sync_status(d))
        return rc;
    if (d->unstable)
        return fail(LBM_ERR_UNSTABLE, "a step produced rho <= 0 or a non-finite value");
    return LBM_OK;
}

int lbm_step(lbm_domain *d, int n)
{
    if (int rc = lbm_step_async(d, n))
        return rc;
    if (d->ntiles == 0) // nothing is updated, the state stays as it is
        return LBM_OK;
    return lbm_step_wait(d);
}

int lbm_prepare_steps(lbm_domain *d)
{
    if (int rc = check_domain(d))
        return rc;
    if (d->batch)
        return fail(LBM_ERR_STATE, "domain is resident in a batch");
    if (d->ntiles && d->graph_dirty)
        return build_graph(d);
    return LBM_OK;
}

int lbm_get_moments_device(lbm_domain *d, float *rho_dev, float *u_dev)
{
    if (int rc = check_domain(d))
        return rc;
    if (!rho_dev || !u_dev)
        return fail(LBM_ERR_ARG, "null output");
    if (d->batch)
        return fail(LBM_ERR_STATE, "domain is resident in a batch");
    HIP_TRY(normalise(d));
    const KDomain k = kdomain(d);
    const uint32_t blocks = (uint32_t)((d->ncells + 255) / 256);
    dispatch_storage(d->storage, [&](auto st) {
        hipLaunchKernelGGL((k_moments<decltype(st)::value>), dim3(blocks), dim3(256), 0, d->stream, k, rho_dev, u_dev,
                           0u, (uint32_t)d->ncells);
    });
    HIP_TRY(hipGetLastError());
    HIP_TRY(hipStreamSynchronize(d->stream));
    return LBM_OK;
}

int lbm_get_moments_noalloc(lbm_domain *d, float *rho, float *u)
{
    if (int rc = check_domain(d))
        return rc;
    if (!rho || !u)
        return fail(LBM_ERR_ARG, "null output");
    if (d->batch)
        return fail(LBM_ERR_STATE, "domain is resident in a batch");
    if (d->ncells > kScratchFloats / 4)
        return fail(LBM_ERR_ARG, "domain of %llu cells exceeds the %llu cells of the static read-back buffer",
                    (unsigned long long)d->ncells, (unsigned long long)(kScratchFloats / 4));
    float *buf = nullptr;
    if (int rc = scratch_address(d->device, &buf))
        return rc;
    std::lock_guard<std::mutex> lock(g_scratch_mutex[d->device]);
    HIP_TRY(normalise(d));
    const KDomain k = kdomain(d);
    const uint32_t blocks = (uint32_t)((d->ncells + 255) / 256);
    dispatch_storage(d->storage, [&](auto st) {
        hipLaunchKernelGGL((k_moments<decltype(st)::value>), dim3(blocks), dim3(256), 0, d->stream, k, buf,
                           buf + d->ncells, 0u, (uint32_t)d->ncells);
    });
    HIP_TRY(hipGetLastError());
    HIP_TRY(hipMemcpyAsync(rho, buf, d->ncells * sizeof(float), hipMemcpyDeviceToHost, d->stream));
    HIP_TRY(hipMemcpyAsync(u, buf + d->ncells, 3 * d->ncells * sizeof(float), hipMemcpyDeviceToHost, d->stream));
    HIP_TRY(hipStreamSynchronize(d->stream));
    return LBM_OK;
}

int lbm_get_moments(lbm_domain *d, float *rho, float *u)
{
    if (int rc = check_domain(d))
        return rc;
    if (!rho || !u)
        return fail(LBM_ERR_ARG, "null output");
    if (d->batch)
        return fail(LBM_ERR_STATE, "domain is resident in a batch");
    HIP_TRY(normalise(d));
    const KDomain k = kdomain(d);
    const Moved m = move_fields<true, float>(
        d, 4,
        [&](uint32_t c0, uint32_t n, float *dev) {
            dispatch_storage(d->storage, [&](auto st) {
                hipLaunchKernelGGL((k_moments<decltype(st)::value>), dim3((n + 255) / 256), dim3(256), 0, d->stream, k,
                                   dev, dev + n, c0, n);
            });
        },
        [&](int c) { return c == 0 ? rho : u + (size_t)(c - 1) * d->ncells; });
    return moved_out(m, "moments");
}

int lbm_get_populations(lbm_domain *d, float *f)
{
    if (int rc = check_domain(d))
        return rc;
    if (!f)
        return fail(LBM_ERR_ARG, "null output");
    if (d->batch)
        return fail(LBM_ERR_STATE, "domain is resident in a batch");
    HIP_TRY(normalise(d));
    const KDomain k = kdomain(d);
    const Moved m = move_fields<true, float>(
        d, Q,
        [&](uint32_t c0, uint32_t n, float *dev) {
            dispatch_storage(d->storage, [&](auto st) {
                hipLaunchKernelGGL((k_export<decltype(st)::value>), dim3((n + 255) / 256), dim3(256), 0, d->stream, k,
                                   dev, c0, n);
            });
        },
        [&](int i) { return f + (size_t)i * d->ncells; });
    return moved_out(m, "population export");
}

int lbm_set_populations(lbm_domain *d, const float *f)
{
    if (int rc = check_domain(d))
        return rc;
    if (!f)
        return fail(LBM_ERR_ARG, "null input");
    if (d->batch)
        return fail(LBM_ERR_STATE, "domain is resident in a batch");
    const KDomain k = kdomain(d);
    const Moved m = move_fields<false, const float>(
        d, Q,
        [&](uint32_t c0, uint32_t n, const float *dev) {
            dispatch_storage(d->storage, [&](auto st) {
                hipLaunchKernelGGL((k_import<decltype(st)::value>), dim3((n + 255) / 256), dim3(256), 0, d->stream, k,
                                   dev, c0, n);
            });
        },
        [&](int i) { return f + (size_t)i * d->ncells; });
    if (int rc = moved_in(d, m, "population import"))
        return rc;
    d->phase = 0;
    if (side_refresh(d) != hipSuccess || curved_refresh(d) != hipSuccess ||
        hipStreamSynchronize(d->stream) != hipSuccess) {
        d->unstable = true;
        return fail(LBM_ERR_DEVICE, "population import failed");
    }
    return LBM_OK;
}

namespace {

// State images (lbm_save_state): a header of eight uint64 words, then the
// population array, then the kept curved-wall values.
constexpr uint64_t kStateTag = 0x31544154534d424cull; // "LBMSTAT1", little-endian
constexpr size_t kStateHeader = 64;

uint64_t aux_bytes(const lbm_domain *d)
{
    return d->d_bzaux ? d->nwall * Q * 64 * sizeof(float) : 0;
}

void state_header(const lbm_domain *d, uint64_t (&h)[8])
{
    h[0] = kStateTag;
    h[1] = (uint64_t)d->nx | (uint64_t)d->ny << 16 | (uint64_t)d->nz << 32 | (uint64_t)d->periodic << 48 |
           (uint64_t)d->storage << 56;
    h[2] = d->bytes;
    h[3] = aux_bytes(d);
    h[4] = d->flags_hash;
    h[5] = (uint64_t)d->phase | (uint64_t)d->unstable << 1;
    h[6] = h[7] = 0;
}

} // namespace

int lbm_state_bytes(const lbm_domain *d, size_t *bytes)
{
    if (int rc = check_domain(d))
        return rc;
    if (!bytes)
        return fail(LBM_ERR_ARG, "null output");
    *bytes = kStateHeader + d->bytes + aux_bytes(d);
    return LBM_OK;
}

int lbm_save_state(lbm_domain *d, void *buf, size_t bytes)
{
    if (int rc = check_domain(d))
        return rc;
    if (!buf)
        return fail(LBM_ERR_ARG, "null buffer");
    if (d->batch)
        return fail(LBM_ERR_STATE, "domain is resident in a batch");
    const uint64_t aux = aux_bytes(d);
    if (bytes < kStateHeader + d->bytes + aux)
        return fail(LBM_ERR_ARG, "buffer of %zu bytes; the state takes %llu", bytes,
                    (unsigned long long)(kStateHeader + d->bytes + aux));
    uint64_t h[8];
    state_header(d, h);
    std::memcpy(buf, h, sizeof h);
    char *p = (char *)buf + kStateHeader;
    if (int rc = moved_out(copy_out(d, p, d->buf, d->bytes), "state download"))
        return rc;
    return moved_out(copy_out(d, p + d->bytes, d->d_bzaux, aux), "state download");
}

int lbm_load_state(lbm_domain *d, const void *buf, size_t bytes)
{
    if (int rc = check_domain(d))
        return rc;
    if (!buf)
        return fail(LBM_ERR_ARG, "null buffer");
    if (d->batch)
        return fail(LBM_ERR_STATE, "domain is resident in a batch");
    if (bytes < kStateHeader)
        return fail(LBM_ERR_ARG, "state image of %zu bytes is shorter than its header", bytes);
    uint64_t h[8], mine[8];
    std::memcpy(h, buf, sizeof h);
    state_header(d, mine);
    if (h[0] != kStateTag || h[6] != 0 || h[7] != 0 || h[5] > 3)
        return fail(LBM_ERR_ARG, "not a state image");
    if (h[1] != mine[1] || h[2] != mine[2])
        return fail(LBM_ERR_ARG, "state image of another grid, periodicity or storage");
    if (h[4] != mine[4])
        return fail(LBM_ERR_STATE, "state image of a domain with other flags");
    if (h[3] != mine[3])
        return fail(LBM_ERR_STATE, "state image %s curved walls and the domain %s", h[3] ? "has" : "has no",
                    mine[3] ? "has" : "has none");
    if (bytes != kStateHeader + h[2] + h[3])
        return fail(LBM_ERR_ARG, "state image of %zu bytes; its header gives %llu", bytes,
                    (unsigned long long)(kStateHeader + h[2] + h[3]));
    const char *p = (const char *)buf + kStateHeader;
    if (int rc = moved_in(d, copy_in(d, d->buf, p, d->bytes), "state upload"))
        return rc;
    d->unstable = true; // until the new state is complete
    if (int rc = moved_in(d, copy_in(d, d->d_bzaux, p + d->bytes, h[3]), "state upload"))
        return rc;
    HIP_TRY(hipStreamSynchronize(d->stream));
    d->phase = (int)(h[5] & 1u);
    if (int rc = clear_status(d))
        return rc;
    d->unstable = (h[5] >> 1) != 0;
    return LBM_OK;
}

int lbm_stats_enable(lbm_domain *d, int on)
{
    if (int rc = check_domain(d))
        return rc;
    if (d->batch)
        return fail(LBM_ERR_STATE, "domain is resident in a batch");
    if (on) {
        const size_t bytes = (size_t)15 * d->ntiles * 64 * sizeof(double);
        if (!d->d_stats && bytes) {
            if (dalloc(d->stream, (void **)&d->d_stats, bytes) != hipSuccess)
                return fail(LBM_ERR_OOM, "statistics sums (%zu bytes)", bytes);
            d->device_bytes += bytes;
        }
        if (bytes)
            HIP_TRY(hipMemsetAsync(d->d_stats, 0, bytes, d->stream));
        HIP_TRY(hipStreamSynchronize(d->stream));
        d->stats_samples = 0;
    }
    d->stats_on = on != 0;
    d->changed();
    return LBM_OK;
}

int lbm_stats_get(lbm_domain *d, double *mean_u, double *mean_uu, double *mean_sigma, uint64_t *samples)
{
    if (int rc = check_domain(d))
        return rc;
    if (!mean_u || !mean_uu || !mean_sigma || !samples)
        return fail(LBM_ERR_ARG, "null output");
    if (d->batch)
        return fail(LBM_ERR_STATE, "domain is resident in a batch");
    *samples = d->stats_samples;
    const size_t n = d->ncells;
    double *dout = nullptr;
    if (dalloc(d->stream, (void **)&dout, 15 * n * sizeof(double)) != hipSuccess)
        return fail(LBM_ERR_OOM, "staging buffer");
    int rc = LBM_OK;
    if (hipMemsetAsync(dout, 0, 15 * n * sizeof(double), d->stream) != hipSuccess)
        rc = fail(LBM_ERR_DEVICE, "staging clear failed");
    if (rc == LBM_OK && d->d_stats && d->stats_samples && d->ntiles) {
        KDomain k = kdomain(d);
        k.stats = d->d_stats;
        const uint32_t blocks = (uint32_t)((d->ntiles + 3) / 4);
        hipLaunchKernelGGL(k_stats_export, dim3(blocks), dim3(256), 0, d->stream, k, (const TileRec *)d->d_tiles,
                           (uint32_t)d->ntiles, 1.0 / (double)d->stats_samples, dout);
        if (hipGetLastError() != hipSuccess)
            rc = fail(LBM_ERR_DEVICE, "statistics export failed");
    }
    if (rc == LBM_OK)
        rc = moved_out(copy_out(d, mean_u, dout, 3 * n * sizeof(double)), "statistics download");
    if (rc == LBM_OK)
        rc = moved_out(copy_out(d, mean_uu, dout + 3 * n, 6 * n * sizeof(double)), "statistics download");
    if (rc == LBM_OK)
        rc = moved_out(copy_out(d, mean_sigma, dout + 9 * n, 6 * n * sizeof(double)), "statistics download");
    dfree(d->stream, dout);
    return rc;
}

int lbm_domain_get_info(const lbm_domain *d, lbm_domain_info *info)
{
    if (!d || !info)
        return fail(LBM_ERR_ARG, "null argument");
    info->nx = d->nx;
    info->ny = d->ny;
    info->nz = d->nz;
    info->storage = d->storage;
    info->periodic = d->periodic;
    info->ncells = d->ncells;
    info->plane_stride = d->P;
    info->n_updated = d->n_updated;
    info->n_tiles = d->ntiles;
    info->n_wall_tiles = d->nwall;
    info->n_inlet = d->inlet_cells.size();
    info->device_bytes = d->device_bytes;
    info->bytes_per_cell_update = 2ull * Q * storage_bytes(d->storage);

    return LBM_OK;
}

int lbm_destroy(lbm_domain *d)
{
    if (int rc = check_domain(d))
        return rc;
    if (d->batch)
        return fail(LBM_ERR_STATE, "domain is resident in a batch; release it first");
    (void)hipStreamSynchronize(d->stream);
    free_domain(d);
    return LBM_OK;
}

} // extern "C"

#include "lbm_batch.inc"
#include "lbm_selftest.inc"
