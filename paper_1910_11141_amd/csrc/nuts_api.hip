// Host side of the C ABI declared in include/nuts.h: argument validation,
// target construction (device copies in kernel-friendly layouts), workspace
// management, kernel selection and launch.  There is no CPU fallback: if the
// device is missing or a launch fails the call returns NUTS_E_DEVICE.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdlib>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <new>
#include <thread>
#include <vector>

#include "../../include/nuts.h"
#include "nuts_dev.h"
#include "nuts_band.h"
#include "nuts_block.h"
#include "nuts_chip.h"
#include "nuts_dense.h"
#include "nuts_elem.h"
#include "nuts_grid.h"
#include "nuts_quad.h"
#include "nuts_tile.h"
#include "nuts_wave.h"
#include "nuts_wide.h"

namespace {

thread_local char g_err[512] = "";
thread_local hipStream_t g_stream = nullptr;

int fail(int code, const char* fmt, ...)
{
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof(g_err), fmt, ap);
    va_end(ap);
    return code;
}

#define HIP_TRY(expr, code)                                                                      \
    do {                                                                                         \
        hipError_t e_ = (expr);                                                                  \
        if (e_ != hipSuccess) return fail((code), "%s failed: %s", #expr, hipGetErrorString(e_)); \
    } while (0)

constexpr int kLdsBytes = 160 * 1024;  // of a compute unit,
constexpr int kLdsGranule = 1280;      // handed out in pieces of this size

size_t elem_size(int dtype) { return dtype == NUTS_F64 ? sizeof(double) : sizeof(float); }

// Scratch memory of nuts_sample_static: one array per GPU, part of the loaded code object, never
// allocated or freed.  The first kStaticHeader bytes hold the call's counters, the rest its workspace.
// In host code the array's name is only a handle for hipGetSymbolAddress; kernels get the address that
// call returned for the current device.
constexpr size_t kStaticHeader = 256;
constexpr int kMaxDevices = 64;
static __device__ __align__(256) unsigned char scratch[NUTS_STATIC_SCRATCH_BYTES];
unsigned char* g_scratch_ptr[kMaxDevices] = {};  // device address of `scratch` on each device, looked up once
std::mutex g_scratch_mutex;

// Looks up the current device's copy of `scratch` (set-up time: target creation or a first regular call).
int resolve_scratch(int dev)
{
    if (dev < 0 || dev >= kMaxDevices) return fail(NUTS_E_UNSUPPORTED, "device index %d out of range", dev);
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)), NUTS_E_DEVICE);
        g_scratch_ptr[dev] = static_cast<unsigned char*>(p);
    }
    return NUTS_OK;
}

}  // namespace

struct nuts_target {
    int32_t kind = 0, dtype = 0;
    int64_t dim = 0, n = 0;
    double prior_scale = 1.0;
    int device = -1;  // -1: no device data (standard normal before its first use)
    // device copies
    void* dPT = nullptr;
    void* dFtab = nullptr;  // table of the logistic function for the weight merges of the grid kernels
    void* dBand = nullptr;  // banded precision matrices: the band, see DevTarget::band
    void* dDiag = nullptr;  // banded precision matrices of 128 < dim <= kBandMaxDim: the diagonals, see nuts_band_kernel
    int diag_present = 0;
    void* dInvVar = nullptr;
    void* dX = nullptr;
    void* dXT = nullptr;
    void* dY = nullptr;
    nuts::TileData tile;  // operand-order copies of X for the tile and wide kernels (logistic regression)
    nuts::GridData grid;  // operand-order copy of X for the grid kernels (binary32 logistic regression)
    nuts::ChipData chip;  // padded copy of X~ for the chip kernel (binary32 logistic regression, in the grid kernels' place)
    nuts::QuadData quad;  // operand-order copy of P for the quad kernel (binary64 dense Gaussian, dim <= 128)
    nuts::BlockData block;  // operand-order copy of P for the block kernel (dense Gaussian, 128 < dim <= 512, not banded)
    // per-call scratch, grown on demand and kept
    char* workspace = nullptr;
    size_t workspace_bytes = 0;
    bool workspace_captured = false;      // a captured call uses it
    std::vector<char*> workspaces_kept;   // those that captured calls use and later calls do not
    size_t workspace_refused = SIZE_MAX;  // least size that a call did without because it could not be allocated
    size_t workspace_most = SIZE_MAX;     // nuts_debug_workspace
    int workspace_refusals = 0;           // (how often an allocation was asked for in vain)
    long turn_steps = -1;                 // nuts_debug_turns
    unsigned* turns_cur = nullptr;        // the queue of chains in turns of the launch in progress
    unsigned long long* counters = nullptr;
    // where the call in progress keeps its workspace and counters: the target's own allocations, or the
    // device's static scratch array (nuts_sample_static)
    bool static_call = false;
    char* ws_cur = nullptr;
    unsigned long long* counters_cur = nullptr;
    hipEvent_t ev_start = nullptr, ev_stop = nullptr;
    // grid kernels: the sets of chains beyond the first run their rounds on these streams
    hipStream_t side_stream[nuts::kGridMaxStreams - 1] = {};
    hipEvent_t ev_fork = nullptr, ev_join[nuts::kGridMaxStreams - 1] = {};
    unsigned* chip_state = nullptr;     // chip kernel: pinned, how the last run ended
    int chip_most = 0;                  // chip kernel: the most workgroups of the call's further launches, 0: no bound
    int chip_refuse = 0, chip_bound = 0;  // nuts_debug_chip_starts
    int wide_apart = 0;                   // nuts_debug_wide_apart
    int* halted_host = nullptr;         // grid kernels: pinned, two snapshots of the "halted" flags
    hipEvent_t ev_batch[2 * nuts::kGridMaxStreams] = {};  // [snapshot][stream]
    bool has_run = false;
    int32_t last_variant = 0, last_grid = 0;
    long last_slots = 0;       // chain slots of the last launch if the host charges them (wave, element-wise), else 0
    void* carry = nullptr;     // states handed from launch to launch under the trajectory schedule
    size_t carry_bytes = 0;
};

namespace {

// The tables of the logistic function and of the logarithm: constants, fitted on first use (1.4 ms, as much as the rest of
// a small target's creation).
const std::vector<double>& softplus_table()
{
    static const std::vector<double> table = [] {
        std::vector<double> t;
        nuts::build_softplus_table(&t);
        return t;
    }();
    return table;
}
const std::vector<double>& tile_tables()  // logistic function, then logarithm
{
    static const std::vector<double> tables = [] {
        std::vector<double> t = softplus_table(), log;
        nuts::build_log_table(&log);
        t.insert(t.end(), log.begin(), log.end());
        return t;
    }();
    return tables;
}

template <typename T>
int upload(const std::vector<T>& host, void** dev)
{
    HIP_TRY(hipMalloc(dev, host.size() * sizeof(T)), NUTS_E_ALLOC);
    HIP_TRY(hipMemcpy(*dev, host.data(), host.size() * sizeof(T), hipMemcpyHostToDevice), NUTS_E_DEVICE);
    return NUTS_OK;
}

// Binary32 logistic regression whose rows are worth spreading over the chip (chip or grid kernels) instead of giving a
// group of chains to each compute unit (wide kernel).  The line was drawn for the grid kernels against the wave kernel (N d = 800:
// 2-5 times slower; 25 000: 3-7 times faster, at 8 to 1024 chains) and stands because the kernels add up in different orders.
bool grid_pays(int64_t n, int64_t d) { return n * d >= (1 << 14); }

// Pairs of components per lane that the one-chain-per-wave kernels are instantiated for.
int row_chunks(int64_t d) { return d <= 128 ? 1 : d <= 256 ? 2 : d <= 512 ? 4 : d <= 1024 ? 8 : 16; }

// X~ for the chip kernel, from the target's own copies on the device ([n][d] and [n]); cd has the sizes.
__global__ void chip_pack_kernel(const float* __restrict__ X, const float* __restrict__ y, nuts::ChipData cd)
{
    const int pitch = nuts::chip_pitch(cd.mt);
    const size_t total = (size_t)cd.n_tiles * nuts::kChipRows * pitch;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (size_t)gridDim.x * blockDim.x) {
        const size_t r = i / pitch;
        const int k = (int)(i % pitch);
        const bool there = (long)r < cd.n_rows && k < cd.d;
        const float v = there ? X[r * cd.d + k] : 0.0f;
        cd.x[i] = there && y[r] == 0.0f ? -v : v;
    }
}

template <typename T>
int build_device_data(nuts_target* t, const nuts_target_desc* desc)
{
    const int64_t d = desc->dim;
    switch (desc->kind) {
    case NUTS_TARGET_STD_NORMAL:
        return NUTS_OK;
    case NUTS_TARGET_GAUSS_DENSE_PRECISION: {
        const T* P = static_cast<const T*>(desc->precision);
        std::vector<T> PT((size_t)d * d);
        for (int64_t i = 0; i < d; ++i)
            for (int64_t k = 0; k < d; ++k) PT[(size_t)k * d + i] = P[(size_t)i * d + k];
        // structure: a matrix that is exactly zero beyond kBandHalf off-diagonals is also kept as a band
        int64_t half = 0;
        for (int64_t i = 0; i < d; ++i)
            for (int64_t k = 0; k < d; ++k)
                if (P[(size_t)i * d + k] != (T)0 && std::llabs(i - k) > half) half = std::llabs(i - k);
        if (half <= nuts::kBandHalf) {
            const int w = 2 * nuts::kBandHalf + 1;
            std::vector<T> band((size_t)std::max<int64_t>(d, nuts::kBandRows) * w, (T)0);
            for (int64_t i = 0; i < d; ++i)
                for (int64_t k = std::max<int64_t>(0, i - nuts::kBandHalf); k <= std::min<int64_t>(d - 1, i + nuts::kBandHalf); ++k)
                    band[(size_t)i * w + (size_t)(k - i + nuts::kBandHalf)] = P[(size_t)i * d + k];
            int rc = upload(band, &t->dBand);
            if (rc) return rc;
            if (d > nuts::kDenseMaxDim && d <= nuts::kBandMaxDim) {
                const int64_t pitch = 128 * row_chunks(d);
                std::vector<T> diag((size_t)w * pitch, (T)0);
                for (int64_t i = 0; i < d; ++i)
                    for (int k = 0; k < w; ++k) {
                        diag[(size_t)(k * pitch + i)] = band[(size_t)i * w + k];
                        if (band[(size_t)i * w + k] != (T)0) t->diag_present |= 1 << k;
                    }
                rc = upload(diag, &t->dDiag);
                if (rc) return rc;
            }
        }
        if (sizeof(T) == sizeof(double) && d <= nuts::kQuadMaxDim) {
            std::vector<double> op;
            nuts::quad_pack_operands(reinterpret_cast<const double*>(P), d, &t->quad, &op);
            void* dev = nullptr;
            int rc = upload(op, &dev);
            if (rc) return rc;
            t->quad.ops = static_cast<double*>(dev);
        }
        if (d > nuts::kDenseMaxDim && d <= nuts::kBlockMaxDim && !t->dBand) {
            std::vector<double> op;
            nuts::block_pack_operands(P, d, &t->block, &op);
            void* dev = nullptr;
            int rc = upload(op, &dev);
            if (rc) return rc;
            t->block.ops = static_cast<double*>(dev);
        }
        return upload(PT, &t->dPT);
    }
    case NUTS_TARGET_GAUSS_DIAG: {
        const T* s = static_cast<const T*>(desc->scales);
        std::vector<T> w((size_t)d);
        for (int64_t i = 0; i < d; ++i) w[(size_t)i] = (T)(1.0 / ((double)s[i] * (double)s[i]));
        return upload(w, &t->dInvVar);
    }
    case NUTS_TARGET_LOGISTIC_REGRESSION: {
        const T* X = static_cast<const T*>(desc->X);
        const T* y = static_cast<const T*>(desc->y);
        const int64_t n = desc->n_data;
        std::vector<T> Xh(X, X + (size_t)n * d), yh(y, y + n), XT((size_t)n * d);
        for (int64_t r = 0; r < n; ++r)
            for (int64_t k = 0; k < d; ++k) XT[(size_t)k * n + r] = X[(size_t)r * d + k];
        int rc = upload(Xh, &t->dX);
        if (rc) return rc;
        rc = upload(XT, &t->dXT);
        if (rc) return rc;
        rc = upload(yh, &t->dY);
        if (rc) return rc;
        if (sizeof(T) == sizeof(double) ? nuts::tile_supports_shape(d, n) || nuts::wide_supports_shape(d, n)
                                        : nuts::wide_supports_shape(d, n) && !grid_pays(n, d)) {
            std::vector<double> op, colsum;
            if (sizeof(T) == sizeof(double)) {
                nuts::tile_pack_operands(reinterpret_cast<const double*>(X), reinterpret_cast<const double*>(y), n, d,
                                         nuts::wide_uses_residuals(d, sizeof(T)), &t->tile, &op, &colsum);
            } else {
                const std::vector<double> Xd(X, X + (size_t)n * d), yd(y, y + n);
                nuts::tile_pack_operands(Xd.data(), yd.data(), n, d, nuts::wide_uses_residuals(d, sizeof(T)), &t->tile, &op, &colsum);
            }
            void* dev = nullptr;
            rc = upload(op, &dev);
            if (rc) return rc;
            t->tile.base = static_cast<double*>(dev);
            rc = upload(colsum, &dev);
            if (rc) return rc;
            t->tile.colsum = static_cast<double*>(dev);
            rc = upload(tile_tables(), &dev);
            if (rc) return rc;
            t->tile.ftab = static_cast<double*>(dev);
        }
        if constexpr (sizeof(T) == sizeof(float)) {
            if (nuts::chip_pays(n, d)) {
                nuts::ChipData* const cd = &t->chip;
                cd->d = (int)d;
                cd->mt = (int)((d + 15) / 16);
                cd->n_rows = (long)n;
                cd->n_tiles = (int)((n + nuts::kChipRows - 1) / nuts::kChipRows);
                HIP_TRY(hipMalloc((void**)&cd->x, (size_t)cd->n_tiles * nuts::kChipRows * nuts::chip_pitch(cd->mt) * sizeof(float)), NUTS_E_ALLOC);
                hipLaunchKernelGGL(chip_pack_kernel, dim3(1024), dim3(256), 0, nullptr, static_cast<const float*>(t->dX),
                                   static_cast<const float*>(t->dY), *cd);
                HIP_TRY(hipGetLastError(), NUTS_E_DEVICE);
                HIP_TRY(hipStreamSynchronize(nullptr), NUTS_E_DEVICE);
            } else if (nuts::grid_supports_shape(d)) {
                std::vector<float> op;
                nuts::grid_pack_operands(X, y, n, d, &t->grid, &op);
                void* dev = nullptr;
                rc = upload(op, &dev);
                if (rc) return rc;
                t->grid.ops = static_cast<float*>(dev);
            }
        }
        return NUTS_OK;
    }
    default:
        return fail(NUTS_E_INVALID_ARG, "unknown target kind %d", desc->kind);
    }
}

template <typename T>
int check_values(const nuts_target_desc* desc)
{
    const int64_t d = desc->dim;
    if (desc->kind == NUTS_TARGET_GAUSS_DENSE_PRECISION) {
        const T* P = static_cast<const T*>(desc->precision);
        for (int64_t i = 0; i < d * d; ++i)
            if (!std::isfinite((double)P[i])) return fail(NUTS_E_INVALID_ARG, "precision[%lld] is not finite", (long long)i);
    } else if (desc->kind == NUTS_TARGET_GAUSS_DIAG) {
        const T* s = static_cast<const T*>(desc->scales);
        for (int64_t i = 0; i < d; ++i)
            if (!(s[i] > 0) || !std::isfinite((double)s[i]))
                return fail(NUTS_E_INVALID_ARG, "scales[%lld] must be finite and > 0", (long long)i);
    } else if (desc->kind == NUTS_TARGET_LOGISTIC_REGRESSION) {
        const T* X = static_cast<const T*>(desc->X);
        const T* y = static_cast<const T*>(desc->y);
        for (int64_t i = 0; i < desc->n_data * d; ++i)
            if (!std::isfinite((double)X[i])) return fail(NUTS_E_INVALID_ARG, "X[%lld] is not finite", (long long)i);
        for (int64_t i = 0; i < desc->n_data; ++i)
            if (!(y[i] == (T)0 || y[i] == (T)1)) return fail(NUTS_E_INVALID_ARG, "y[%lld] is not 0 or 1", (long long)i);
    }
    return NUTS_OK;
}

void release(nuts_target* t)
{
    if (!t) return;
    if (t->device >= 0) {
        (void)hipFree(t->dPT);
        (void)hipFree(t->dBand);
        (void)hipFree(t->dDiag);
        (void)hipFree(t->dFtab);
        (void)hipFree(t->dInvVar);
        (void)hipFree(t->dX);
        (void)hipFree(t->dXT);
        (void)hipFree(t->dY);
        (void)hipFree(t->tile.base);
        (void)hipFree(t->grid.ops);
        (void)hipFree(t->quad.ops);
        (void)hipFree(t->block.ops);
        (void)hipFree(t->chip.x);
        (void)hipFree(t->tile.ftab);
        (void)hipFree(t->tile.colsum);
        (void)hipFree(t->workspace);
        for (char* w : t->workspaces_kept) (void)hipFree(w);
        (void)hipFree(t->carry);
        (void)hipFree(t->counters);
        if (t->ev_start) (void)hipEventDestroy(t->ev_start);
        if (t->ev_stop) (void)hipEventDestroy(t->ev_stop);
        if (t->ev_fork) (void)hipEventDestroy(t->ev_fork);
        for (hipEvent_t e : t->ev_join)
            if (e) (void)hipEventDestroy(e);
        for (hipStream_t q : t->side_stream)
            if (q) (void)hipStreamDestroy(q);
        for (hipEvent_t e : t->ev_batch)
            if (e) (void)hipEventDestroy(e);
        if (t->halted_host) (void)hipHostFree(t->halted_host);
        if (t->chip_state) (void)hipHostFree(t->chip_state);
    }
    delete t;
}

int ensure_device(nuts_target* t)
{
    int count = 0;
    if (hipGetDeviceCount(&count) != hipSuccess || count < 1)
        return fail(NUTS_E_DEVICE, "no HIP device available (this library has no CPU path)");
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev), NUTS_E_DEVICE);
    if (t->device >= 0 && t->device != dev)
        return fail(NUTS_E_INVALID_ARG, "target was created on device %d, current device is %d", t->device, dev);
    t->device = dev;
    int rc = resolve_scratch(dev);
    if (rc) return rc;
    if (!t->counters)
        HIP_TRY(hipMalloc((void**)&t->counters, nuts::kCtrCount * sizeof(unsigned long long) + nuts::kWideMaxPairs * sizeof(unsigned)), NUTS_E_ALLOC);
    if (!t->ev_start) HIP_TRY(hipEventCreate(&t->ev_start), NUTS_E_DEVICE);
    if (!t->ev_stop) HIP_TRY(hipEventCreate(&t->ev_stop), NUTS_E_DEVICE);
    return NUTS_OK;
}

hipError_t workspace_alloc(nuts_target* t, char** p, size_t bytes)
{
    const hipError_t e = bytes > t->workspace_most ? hipErrorOutOfMemory : hipMalloc((void**)p, bytes);
    if (e != hipSuccess) t->workspace_refusals += 1;
    return e;
}

// Nothing can be allocated while a graph is captured (nor where that cannot be found out: another stream of the process is capturing).
bool stream_captures()
{
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(g_stream, &status) == hipSuccess) return status != hipStreamCaptureStatusNone;
    (void)hipGetLastError();
    return true;
}

// The workspace makes way for another one.  A graph of a captured call may be replayed at any time, so what such a call uses stays as long as the target.
int leave_workspace(nuts_target* t)
{
    if (!t->workspace) return NUTS_OK;
    if (t->workspace_captured) {
        try {
            t->workspaces_kept.push_back(t->workspace);
        } catch (const std::bad_alloc&) {
            return fail(NUTS_E_ALLOC, "out of host memory");
        }
    } else {
        HIP_TRY(hipDeviceSynchronize(), NUTS_E_DEVICE);
        (void)hipFree(t->workspace);
    }
    t->workspace = nullptr;
    t->workspace_bytes = 0;
    t->workspace_captured = false;
    return NUTS_OK;
}

int ensure_workspace(nuts_target* t, size_t bytes)
{
    if (t->static_call) {  // no allocation: the workspace is the device's static array, or the call is refused
        if (bytes > (size_t)NUTS_STATIC_SCRATCH_BYTES - kStaticHeader)
            return fail(NUTS_E_UNSUPPORTED, "this run needs %zu bytes of scratch memory; nuts_sample_static has %zu",
                        bytes, (size_t)NUTS_STATIC_SCRATCH_BYTES - kStaticHeader);
        t->ws_cur = reinterpret_cast<char*>(g_scratch_ptr[t->device]) + kStaticHeader;
        return NUTS_OK;
    }
    if (bytes > t->workspace_bytes) {
        const int rc = leave_workspace(t);
        if (rc) return rc;
        HIP_TRY(workspace_alloc(t, &t->workspace, bytes), NUTS_E_ALLOC);
        t->workspace_bytes = bytes;
        if (bytes >= t->workspace_refused) t->workspace_refused = SIZE_MAX;
    }
    t->workspace_captured = t->workspace_captured || stream_captures();
    t->ws_cur = t->workspace;
    return NUTS_OK;
}

// For runs that are faster with a workspace of `most` bytes and do with `least`: *has says which of them there is.  An allocation that was
// refused is not tried again before one of that size was to be had, and costs the workspace that is there only if that would not do either.
int ensure_workspace_or(nuts_target* t, size_t least, size_t most, bool* has)
{
    *has = !t->static_call && most <= t->workspace_bytes;
    if (!*has && !t->static_call && most < t->workspace_refused && !stream_captures()) {
        if (least <= t->workspace_bytes) {
            char* larger = nullptr;
            if (workspace_alloc(t, &larger, most) == hipSuccess) {
                const int rc = leave_workspace(t);
                if (rc) {
                    (void)hipFree(larger);
                    return rc;
                }
                t->workspace = larger;
                t->workspace_bytes = most;
                *has = true;
            }
        } else {
            const int rc = ensure_workspace(t, most);
            if (rc != NUTS_OK && rc != NUTS_E_ALLOC) return rc;
            *has = rc == NUTS_OK;
        }
        if (!*has) {
            (void)hipGetLastError();
            t->workspace_refused = most;
        }
    }
    return ensure_workspace(t, *has ? most : least);
}

// The logistic table of the grid kernels' weight merges.  Built when the target is created; never by nuts_sample_static.
int ensure_ftab(nuts_target* t)
{
    if (t->dFtab) return NUTS_OK;
    if (t->static_call)
        return fail(NUTS_E_UNSUPPORTED, "the target was created without a GPU: nuts_sample_static cannot build its tables");
    return upload(softplus_table(), &t->dFtab);
}

__global__ void fill_words_kernel(unsigned* p, int n, unsigned value)
{
    for (int i = threadIdx.x; i < n; i += blockDim.x) p[i] = value;
}

__global__ void begin_turns_kernel(unsigned* words, nuts::RowTurns plan)
{
    for (int i = threadIdx.x; i < nuts::kTurnPlan; i += blockDim.x) words[i] = 0u;
    for (unsigned i = threadIdx.x; i <= plan.mask; i += blockDim.x) words[nuts::kTurnRing + i] = 0u;
    if (threadIdx.x == 0) *reinterpret_cast<nuts::RowTurns*>(words + nuts::kTurnPlan) = plan;
}

// (behind the counters: the words at which the wide kernel's pairs of workgroups meet, of which a call without them has none)
__global__ void zero_counters_kernel(unsigned long long* c, int words)
{
    if (threadIdx.x < nuts::kCtrCount) c[threadIdx.x] = 0ull;
    for (int i = threadIdx.x; i < words; i += blockDim.x) reinterpret_cast<unsigned*>(c + nuts::kCtrCount)[i] = 0u;
}

// After every launch: the wave and element-wise kernels hold `slots` chain slots for as long as the
// busiest of them works, so that many slots x its gradient count were issued; the chain queue restarts.
__global__ void close_launch_kernel(unsigned long long* c, unsigned long long slots, int words, const unsigned* turns)
{
    for (int i = threadIdx.x; i < words; i += blockDim.x) {
        unsigned* const word = reinterpret_cast<unsigned*>(c + nuts::kCtrCount) + i;
        if ((*word & nuts::kMeetBoth) == nuts::kMeetBoth && !(*word & nuts::kMeetAlone)) atomicAdd(&c[nuts::kCtrPairsMet], 1ull);
        if (*word & nuts::kMeetLost) atomicAdd(&c[nuts::kCtrPairsLost], 1ull);
        *word = 0u;
    }
    if (threadIdx.x == 0) {
        c[nuts::kCtrIssued] += slots * c[nuts::kCtrSlotMax];
        c[nuts::kCtrSlotMax] = 0ull;
        c[nuts::kCtrQueue] = 0ull;
        if (turns) c[nuts::kCtrTurns] += turns[nuts::kTurnTail];
    }
}

int next_pow2(int x)
{
    int p = 1;
    while (p < x) p <<= 1;
    return p;
}

template <typename T>
nuts::DevTarget<T> dev_target(const nuts_target* t)
{
    nuts::DevTarget<T> g{};
    g.kind = t->kind;
    g.d = (int)t->dim;
    g.dstride = (int)((t->dim + 15) / 16 * 16);
    g.kl = next_pow2((int)(t->dim < 64 ? t->dim : 64));
    g.n = (long)t->n;
    g.PT = static_cast<const T*>(t->dPT);
    g.band = static_cast<const T*>(t->dBand);
    g.inv_var = static_cast<const T*>(t->dInvVar);
    g.X = static_cast<const T*>(t->dX);
    g.XT = static_cast<const T*>(t->dXT);
    g.y = static_cast<const T*>(t->dY);
    g.prior_prec = 1.0 / (t->prior_scale * t->prior_scale);
    return g;
}

// Launch shape of the general wave kernel.
struct WavePlan {
    size_t lds_bytes, slot;
    bool lds_matrix;
    long blocks;
};
constexpr int kWaveBlock = 4;  // waves per workgroup

template <typename T>
int wave_plan(const nuts_target* t, const nuts::DevSample& sa, WavePlan* wp)
{
    const nuts::DevTarget<T> tg = dev_target<T>(t);
    wp->lds_bytes = (size_t)kWaveBlock * tg.dstride * sizeof(T);
    if (wp->lds_bytes > 64 * 1024) return fail(NUTS_E_UNSUPPORTED, "dim %lld too large for the wave kernel", (long long)t->dim);
    const size_t mat_bytes = (size_t)t->dim * t->dim * sizeof(T);
    wp->lds_matrix = t->kind == NUTS_TARGET_GAUSS_DENSE_PRECISION && wp->lds_bytes + mat_bytes <= 128 * 1024;
    if (wp->lds_matrix) {
        wp->lds_bytes += mat_bytes;
        HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(nuts::nuts_wave_kernel<T>),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)wp->lds_bytes), NUTS_E_DEVICE);
    }
    size_t slot = ((size_t)nuts::wave_num_vectors(sa.max_depth) * tg.dstride * sizeof(T) + 15) & ~(size_t)15;
    if (t->kind == NUTS_TARGET_LOGISTIC_REGRESSION) slot += (size_t)t->n * sizeof(double);
    wp->slot = (slot + 255) & ~(size_t)255;
    int per_cu = 0, cus = 0;
    HIP_TRY(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, nuts::nuts_wave_kernel<T>, kWaveBlock * nuts::kWave, wp->lds_bytes),
            NUTS_E_DEVICE);
    HIP_TRY(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, t->device), NUTS_E_DEVICE);
    if (per_cu < 1) per_cu = 1;
    wp->blocks = (sa.n_chains + kWaveBlock - 1) / kWaveBlock;
    const long resident = (long)per_cu * cus;
    if (wp->blocks > resident) wp->blocks = resident;
    return NUTS_OK;
}

template <typename T>
int launch_wave(nuts_target* t, nuts::DevSample sa)
{
    nuts::DevTarget<T> tg = dev_target<T>(t);
    WavePlan wp;
    int rc = wave_plan<T>(t, sa, &wp);
    if (rc) return rc;
    tg.lds_matrix = wp.lds_matrix ? 1 : 0;
    rc = ensure_workspace(t, wp.slot * (size_t)wp.blocks * kWaveBlock);
    if (rc) return rc;
    sa.workspace = t->ws_cur;
    sa.slot_bytes = wp.slot;
    hipLaunchKernelGGL(nuts::nuts_wave_kernel<T>, dim3((unsigned)wp.blocks), dim3(kWaveBlock * nuts::kWave), wp.lds_bytes, g_stream, tg, sa);
    HIP_TRY(hipGetLastError(), NUTS_E_DEVICE);
    t->last_variant = NUTS_VARIANT_WAVE;
    t->last_grid = (int)wp.blocks;
    t->last_slots = wp.blocks * kWaveBlock < sa.n_chains ? wp.blocks * kWaveBlock : sa.n_chains;  // waves that get a chain
    return NUTS_OK;
}

// nuts_sample_static: a kernel that stands in for the wave kernel takes and refuses the runs that that one would, by its
// workspace.  (What it takes it can run in less: on fewer workgroups, with more chains in the queue.)
int static_check(nuts_target* t, const nuts::DevSample& sa)
{
    if (!t->static_call) return NUTS_OK;
    WavePlan wp;
    int rc = t->dtype == NUTS_F64 ? wave_plan<double>(t, sa, &wp) : wave_plan<float>(t, sa, &wp);
    if (rc) return rc;
    return ensure_workspace(t, wp.slot * (size_t)wp.blocks * kWaveBlock);
}

// Largest dimension of the element-wise variant, per dtype.  The kernel itself goes on to kElemMaxDim: AUTO takes it there
// in place of the wave kernel, as which it is reported (one wavefront per chain, too).
constexpr int kElemMaxDim = 2048;
int elem_max_dim(int dtype) { return dtype == NUTS_F64 ? 512 : 1024; }

bool elem_eligible(const nuts_target* t)
{
    return (t->kind == NUTS_TARGET_STD_NORMAL || t->kind == NUTS_TARGET_GAUSS_DIAG) && t->dim <= elem_max_dim(t->dtype);
}

// LDS for the shallow levels of the trees of one-chain-per-wave workgroups of four: what the `blocks` workgroups leave
// of each compute unit's LDS beyond `base` bytes each.
nuts::RowLds row_lds(long blocks, int cus, size_t base, int kc, size_t elem, int max_depth, bool grad)
{
    const long share = (blocks + cus - 1) / cus;
    const size_t budget = (size_t)(kLdsBytes / share) / kLdsGranule * kLdsGranule;
    return nuts::row_lds_split(budget > base ? (budget - base) / 4 : 0, kc, elem, max_depth, grad);
}

// How many steps a slot takes with one of a call's last chains before it turns to another (nuts_row.h; 0: it keeps its chain): where chains wait for
// slots, where there are iterations enough to turn between, and where a chain can take that many steps before its last one.  Time without turns over time with:
//   diagonal, 2000 to 16384 chains, 8 to 40 iterations of 200 to 760 steps: d = 2 1.10, d = 60 1.13, d = 130 1.11 and 1.24 (binary32, 64), d = 300 1.18,
//   d = 400 1.22, d = 700 1.11, d = 1000 1.07, d = 1500 1.11; four iterations of 75 steps 0.99; equal scales, d = 100 to 1000, 0.98 to 1.10
//   banded up to d = 128, 2100 to 4096 chains, 10 to 40 iterations of 30 to 90 steps: d = 10 1.03, d = 50 1.12, d = 100 1.11 and 1.30, d = 120 1.17; in a
//   call of 0.4 ms 0.97, of 0.8 ms 0.98
//   full matrix up to d = 128, 1300 to 4096 chains, 30 to 40 iterations of 31 steps: binary64 1.18 and 1.35, binary32 1.00 to 1.07; 10 iterations 0.99
// Not two or three iterations (0.98), nor banded matrices beyond d = 128 (nuts_band.h, 0.97 to 1.02: the code for turns takes registers that the
// state needs), nor nuts_sample_static, whose memory is fixed.
// Chains of the standard normal take about as many steps each, some 4.5 / eps an iteration.  So slots would turn all at once, and idle only in the last of the
// rounds in which they take the chains, if those do not fill it.  After 256 and 1024 steps, 1.1, 1.35, 1.48 and 3.3 times as many chains as slots:
//   one wave a SIMD (d = 649 and 1000 in binary64, 1100 and 2000 in binary32): 360 steps 1.04 to 1.12 and 0.97 to 1.04, 600 1.00 to 1.30 and 0.98 to 1.09,
//   1500 1.15 to 1.65 and 1.16 to 1.49; 280 steps 0.93 to 1.02; 1.6 and 3.8 times as many chains, 600 steps 0.95 to 1.00
//   two (d = 600 and 1000 in binary32), 1.1 times as many: 360 steps 1.00 and 1.03, 600 1.10 to 1.20 and 1.02, 1500 1.24 to 1.33 and 1.31 to 1.38; more chains, 600
//   steps 0.86 to 1.03 and 0.99 to 1.08, 1500 0.97 to 1.13 and 1.00 to 1.13 (1.9 times as many, d = 700: after 256 1.10 times as fast as after 1024)
//   three (d = 60 in binary64, 140 in binary32), 600 steps: 0.70 to 0.84 and 1.00 to 1.02
unsigned turn_steps(const nuts_target* t, const nuts::DevSample& sa, long slots, int cus, unsigned steps)
{
    const long iters = sa.iter_end - sa.iter_begin;
    if (t->static_call || sa.n_chains <= slots || iters < 4) return 0;
    if (t->kind == NUTS_TARGET_STD_NORMAL) {
        const long rest = sa.n_chains % slots, waves = slots / (4L * cus);  // (of a SIMD)
        if (waves <= 2) steps = nuts::kTurnStepsEven;
        const bool few = waves <= 2 && rest <= (waves == 2 ? slots / 8 : slots / 2);
        if (rest == 0 || 4.5 * (double)iters < (few ? steps : nuts::kTurnSteps) * sa.eps) return 0;
    }
    return (iters - 1) * sa.leaf_steps * ((1l << sa.max_depth) - 1) >= (long)steps ? steps : 0;
}

// Workspace of the row kernels.  That of chains in turns adds eight vectors a slot (with a gradient sixteen) to the 4 max_depth + 9 that it has;
// a call that cannot have it does without turns.
int row_workspace(nuts_target* t, nuts::DevSample& sa, size_t slot, long slots, int kc, size_t elem, bool grad, unsigned steps, unsigned** turns)
{
    *turns = nullptr;
    const size_t base = slot * (size_t)slots;
    nuts::RowTurns plan{};
    size_t words = 0;
    bool has = false;
    int rc;
    if (steps) {
        const long n = std::min(sa.n_chains, nuts::kTurnChains * slots);
        unsigned ring = 1;
        while ((long)ring < n) ring *= 2;
        plan.mask = ring - 1;
        plan.row_bytes = (unsigned)nuts::row_turn_bytes(kc, elem, grad);
        plan.steps = t->turn_steps >= 0 ? (unsigned)t->turn_steps : steps;
        plan.first = sa.n_chains - n;
        words = ((nuts::kTurnRing + (size_t)ring) * sizeof(unsigned) + 255) & ~(size_t)255;
        rc = ensure_workspace_or(t, base, base + words + (size_t)plan.row_bytes * (size_t)n, &has);
    } else {
        rc = ensure_workspace(t, base);
    }
    if (rc) return rc;
    sa.workspace = t->ws_cur;
    sa.slot_bytes = slot;
    if (has) {
        *turns = reinterpret_cast<unsigned*>(t->ws_cur + base);
        plan.rows = t->ws_cur + base + words;
        hipLaunchKernelGGL(begin_turns_kernel, dim3(1), dim3(1024), 0, g_stream, *turns, plan);
        HIP_TRY(hipGetLastError(), NUTS_E_DEVICE);
        t->turns_cur = *turns;
    }
    return NUTS_OK;
}

template <typename T, int kC, bool kTurns = false>
int launch_elem_inst(nuts_target* t, nuts::DevSample sa, int variant, unsigned steps = 0)  // (steps: of turn_steps)
{
    const nuts::DevTarget<T> tg = dev_target<T>(t);
    size_t slot = (size_t)nuts::row_num_vectors(sa.max_depth) * 128 * kC * sizeof(T);
    slot = (slot + 255) & ~(size_t)255;
    const void* fn = reinterpret_cast<const void*>(nuts::nuts_elem_kernel<T, kC, kTurns>);
    HIP_TRY(hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes), NUTS_E_DEVICE);
    size_t lds_bytes = nuts::elem_lane_bytes<T, kC>() <= 32 ? 0 : 128 * kC * sizeof(T);
    int per_cu = 0, cus = 0;
    HIP_TRY(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (nuts::nuts_elem_kernel<T, kC, kTurns>), 256, lds_bytes), NUTS_E_DEVICE);
    HIP_TRY(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, t->device), NUTS_E_DEVICE);
    if (per_cu < 1) per_cu = 1;
    if constexpr (!kTurns && nuts::row_takes_turns<T, kC>())
        if (const unsigned n = turn_steps(t, sa, 4L * per_cu * cus, cus, nuts::kTurnSteps)) return launch_elem_inst<T, kC, true>(t, sa, variant, n);
    long blocks = (sa.n_chains + 3) / 4;
    if (blocks > (long)per_cu * cus) blocks = (long)per_cu * cus;
    if (t->static_call) {
        if (elem_eligible(t)) {
            // what an entry that cannot allocate takes: a slot's tree in 3 D + 7 vectors, for all that are resident at two or
            // (up to 1 KB of state) three workgroups per compute unit; it runs on as many as fit
            const size_t vec = (size_t)tg.dstride * sizeof(T), tree = ((size_t)(3 * sa.max_depth + 7) * vec + 255) & ~(size_t)255;
            const long most = (t->dim * (long)sizeof(T) <= 1024 ? 3L : 2L) * cus;
            int rc = ensure_workspace(t, tree * 4 * (size_t)std::min((long)((sa.n_chains + 3) / 4), most));
            if (rc) return rc;
        } else {
            int rc = static_check(t, sa);
            if (rc) return rc;
        }
        const long fit = (long)(((size_t)NUTS_STATIC_SCRATCH_BYTES - kStaticHeader) / (4 * slot));
        if (fit >= 1 && blocks > fit) blocks = fit;
    }
    const nuts::RowLds rl = row_lds(blocks, cus, lds_bytes, kC, sizeof(T), sa.max_depth, false);
    lds_bytes += (size_t)4 * (rl.n_first + rl.n_pool) * nuts::row_entry_bytes(kC, sizeof(T));
    unsigned* turns;
    int rc = row_workspace(t, sa, slot, blocks * 4, kC, sizeof(T), false, steps, &turns);
    if (rc) return rc;
    hipLaunchKernelGGL((nuts::nuts_elem_kernel<T, kC, kTurns>), dim3((unsigned)blocks), dim3(256), lds_bytes, g_stream, tg, sa, rl, turns);
    HIP_TRY(hipGetLastError(), NUTS_E_DEVICE);
    t->last_variant = variant;
    t->last_grid = (int)blocks;
    t->last_slots = blocks * 4 < sa.n_chains ? blocks * 4 : sa.n_chains;  // waves that get a chain
    return NUTS_OK;
}

template <typename T>
int launch_elem(nuts_target* t, const nuts::DevSample& sa, int variant)
{
    switch (row_chunks(t->dim)) {
    case 1: return launch_elem_inst<T, 1>(t, sa, variant);
    case 2: return launch_elem_inst<T, 2>(t, sa, variant);
    case 4: return launch_elem_inst<T, 4>(t, sa, variant);
    case 8: return launch_elem_inst<T, 8>(t, sa, variant);
    default: return launch_elem_inst<T, 16>(t, sa, variant);
    }
}

bool dense_eligible(const nuts_target* t)
{
    return t->kind == NUTS_TARGET_GAUSS_DENSE_PRECISION && t->dim <= nuts::kDenseMaxDim;
}

template <typename T, bool kBanded, bool kTurns = false>
int launch_dense_inst(nuts_target* t, nuts::DevSample sa, unsigned steps = 0)
{
    using namespace nuts;
    DevTarget<T> tg = dev_target<T>(t);
    const int threads = kDenseWaves * kWave;
    size_t lds_bytes = dense_base_elems(kBanded ? 0 : (int)t->dim) * sizeof(T);
    lds_bytes = (lds_bytes + 15) & ~(size_t)15;
    HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(nuts_dense_kernel<T, kBanded, kTurns>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes), NUTS_E_DEVICE);
    size_t slot = (size_t)row_num_vectors(sa.max_depth) * kDensePitch * sizeof(T);
    slot = (slot + 255) & ~(size_t)255;
    int per_cu = 0, cus = 0;
    HIP_TRY(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (nuts_dense_kernel<T, kBanded, kTurns>), threads, lds_bytes), NUTS_E_DEVICE);
    HIP_TRY(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, t->device), NUTS_E_DEVICE);
    if (per_cu < 1) per_cu = 1;
    if constexpr (!kTurns)
        if (const unsigned n = turn_steps(t, sa, (long)kDenseWaves * per_cu * cus, cus, kTurnStepsDense)) return launch_dense_inst<T, kBanded, true>(t, sa, n);
    long blocks = (sa.n_chains + kDenseWaves - 1) / kDenseWaves;
    const long resident = (long)per_cu * cus;
    if (blocks > resident) blocks = resident;
    const RowLds rl = row_lds(blocks, cus, lds_bytes, 1, sizeof(T), sa.max_depth, true);
    lds_bytes += (size_t)kDenseWaves * (rl.n_first + rl.n_pool) * row_entry_bytes(1, sizeof(T));
    unsigned* turns;
    int rc = row_workspace(t, sa, slot, blocks * kDenseWaves, 1, sizeof(T), true, steps, &turns);
    if (rc) return rc;
    hipLaunchKernelGGL((nuts_dense_kernel<T, kBanded, kTurns>), dim3((unsigned)blocks), dim3(threads), lds_bytes, g_stream, tg, sa, rl, turns);
    HIP_TRY(hipGetLastError(), NUTS_E_DEVICE);
    t->last_variant = NUTS_VARIANT_DENSE;
    t->last_grid = (int)blocks;
    t->last_slots = blocks * kDenseWaves < sa.n_chains ? blocks * kDenseWaves : sa.n_chains;
    return NUTS_OK;
}

template <typename T>
int launch_dense(nuts_target* t, const nuts::DevSample& sa)
{
    return t->dBand ? launch_dense_inst<T, true>(t, sa) : launch_dense_inst<T, false>(t, sa);
}

template <typename T, int kC>
int launch_band_inst(nuts_target* t, nuts::DevSample sa)
{
    const nuts::DevTarget<T> tg = dev_target<T>(t);
    size_t slot = (size_t)nuts::row_num_vectors(sa.max_depth) * 128 * kC * sizeof(T);
    slot = (slot + 255) & ~(size_t)255;
    const void* fn = reinterpret_cast<const void*>(nuts::nuts_band_kernel<T, kC>);
    HIP_TRY(hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes), NUTS_E_DEVICE);
    size_t lds_bytes = (size_t)4 * nuts::band_bcast(kC) * sizeof(T);
    int per_cu = 0, cus = 0;
    HIP_TRY(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (nuts::nuts_band_kernel<T, kC>), 256, lds_bytes), NUTS_E_DEVICE);
    HIP_TRY(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, t->device), NUTS_E_DEVICE);
    if (per_cu < 1) per_cu = 1;
    long blocks = (sa.n_chains + 3) / 4;
    if (blocks > (long)per_cu * cus) blocks = (long)per_cu * cus;
    if (t->static_call) {
        int rc = static_check(t, sa);
        if (rc) return rc;
        const long fit = (long)(((size_t)NUTS_STATIC_SCRATCH_BYTES - kStaticHeader) / (4 * slot));
        if (fit >= 1 && blocks > fit) blocks = fit;
    }
    const nuts::RowLds rl = row_lds(blocks, cus, lds_bytes, kC, sizeof(T), sa.max_depth, true);
    lds_bytes += (size_t)4 * (rl.n_first + rl.n_pool) * nuts::row_entry_bytes(kC, sizeof(T));
    int rc = ensure_workspace(t, slot * (size_t)blocks * 4);
    if (rc) return rc;
    sa.workspace = t->ws_cur;
    sa.slot_bytes = slot;
    hipLaunchKernelGGL((nuts::nuts_band_kernel<T, kC>), dim3((unsigned)blocks), dim3(256), lds_bytes, g_stream, tg,
                       static_cast<const T*>(t->dDiag), t->diag_present, sa, rl);
    HIP_TRY(hipGetLastError(), NUTS_E_DEVICE);
    t->last_variant = NUTS_VARIANT_WAVE;
    t->last_grid = (int)blocks;
    t->last_slots = blocks * 4 < sa.n_chains ? blocks * 4 : sa.n_chains;  // waves that get a chain
    return NUTS_OK;
}

// Chosen automatically only, as the block kernel below: one wavefront per chain, so they are reported as the wave variant
// that they stand in for.
bool band_eligible(const nuts_target* t) { return t->kind == NUTS_TARGET_GAUSS_DENSE_PRECISION && t->dDiag != nullptr; }

template <typename T>
int launch_band(nuts_target* t, const nuts::DevSample& sa)
{
    switch (row_chunks(t->dim)) {
    case 2: return launch_band_inst<T, 2>(t, sa);
    case 4: return launch_band_inst<T, 4>(t, sa);
    case 8: return launch_band_inst<T, 8>(t, sa);
    default: return launch_band_inst<T, 16>(t, sa);
    }
}

bool block_eligible(const nuts_target* t) { return t->kind == NUTS_TARGET_GAUSS_DENSE_PRECISION && t->block.ops != nullptr; }

template <typename T>
int launch_block(nuts_target* t, nuts::DevSample sa)
{
    int cus = 0;
    HIP_TRY(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, t->device), NUTS_E_DEVICE);
    nuts::BlockPlan bp;
    const int nc = nuts::block_chains_per_group((int)t->dim, sa.n_chains, cus);
    nuts::block_plan(t->block, sizeof(T), sa.n_chains, cus, sa.max_depth, nc, &bp);
    const size_t group_bytes = bp.slot_bytes * (size_t)bp.nc;
    if (t->static_call) {
        int rc = static_check(t, sa);
        if (rc) return rc;
        const long fit = (long)(((size_t)NUTS_STATIC_SCRATCH_BYTES - kStaticHeader) / group_bytes);
        if (fit >= 1 && bp.blocks > fit) bp.blocks = (int)fit;
    }
    int rc = ensure_workspace(t, group_bytes * (size_t)bp.blocks);
    if (rc) return rc;
    sa.workspace = t->ws_cur;
    sa.slot_bytes = bp.slot_bytes;
    HIP_TRY(nuts::block_launch<T>(t->block, sa, bp, g_stream), NUTS_E_DEVICE);
    t->last_variant = NUTS_VARIANT_WAVE;
    t->last_grid = bp.blocks;
    t->last_slots = 0;
    return NUTS_OK;
}

bool quad_eligible(const nuts_target* t, int max_depth)
{
    return t->kind == NUTS_TARGET_GAUSS_DENSE_PRECISION && t->dtype == NUTS_F64 && t->quad.ops != nullptr &&
           max_depth <= nuts::kQuadMaxDepth;
}

// Four chains per wavefront, four wavefronts per workgroup, one workgroup per compute unit (the matrix fills its LDS).
int launch_quad(nuts_target* t, nuts::DevSample sa)
{
    using namespace nuts;
    QuadArgs qa{t->quad.ops, t->quad.d, t->quad.n_r, t->quad.n_kb};
    size_t lds_bytes = quad_matrix_bytes(t->quad) + quad_stage_bytes();
    int cus = 0;
    HIP_TRY(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, t->device), NUTS_E_DEVICE);
    const int per_block = kQuadWaves * kQuadChains;
    long blocks = (sa.n_chains + per_block - 1) / per_block;
    if (blocks > cus) blocks = cus;  // further chains wait in the queue
    // spread few chains over the compute units first: a wave with one chain still runs whole matrix instructions
    size_t slot = (size_t)quad_num_vectors(sa.max_depth) * kQuadVecLen * sizeof(double);
    int rc = ensure_workspace(t, slot * (size_t)blocks * per_block);
    if (rc) return rc;
    sa.workspace = t->ws_cur;
    sa.slot_bytes = slot;
    HIP_TRY(quad_launch(qa, sa, (int)blocks, lds_bytes, g_stream), NUTS_E_DEVICE);
    t->last_variant = NUTS_VARIANT_QUAD;
    t->last_grid = (int)blocks;
    t->last_slots = 0;
    return NUTS_OK;
}

bool grid_eligible(const nuts_target* t)
{
    return t->kind == NUTS_TARGET_LOGISTIC_REGRESSION && t->dtype == NUTS_F32 && (t->grid.ops != nullptr || t->chip.x != nullptr);
}

// Rounds of (control, gradient) launches, enqueued in batches; the host waits for each batch
// and stops when every chain has halted, so this variant returns only when sampling is complete.
// Slots beyond the first 128 may run on up to three further streams, which the target owns.
int launch_grid(nuts_target* t, nuts::DevSample sa)
{
    using namespace nuts;
    typedef WaveChain<float> Chain;
    DevTarget<float> tg = dev_target<float>(t);
    // at most 1024 chains are resident; a slot whose chain has finished takes the next one from the queue
    const int n_slots = sa.n_chains >= kGridMaxChains ? kGridMaxChains : (int)((sa.n_chains + 3) / 4 * 4);
    const int n_sets = (n_slots + kGridSetChains - 1) / kGridSetChains;
    // consecutive sets share a stream: one control launch and one gradient launch serve them all
    const int most_streams = grid_streams(n_slots, t->n, (int)t->dim, (double)(sa.iter_end - sa.iter_begin) * (double)sa.n_chains);
    const int sets_per_stream = (n_sets + most_streams - 1) / most_streams;
    const int n_streams = (n_sets + sets_per_stream - 1) / sets_per_stream;
    int cus = 0;
    HIP_TRY(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, t->device), NUTS_E_DEVICE);
    GridArgs ga{};
    ga.ops = t->grid.ops;
    ga.d = t->grid.d;
    ga.ks1 = t->grid.ks1;
    ga.mt = t->grid.mt;
    ga.tail = t->grid.tail;
    ga.n_tiles = t->grid.n_tiles;
    ga.n_rows = t->grid.n_rows;
    // a slice per compute unit, but at least two row tiles per slice: a launch's fixed costs - operands of
    // Theta, first tile, partial results - weigh more than its width (+13 % at 10 000 rows and 1024 chains).
    // The split depends on the target only, never on the number of chains: a chain's results must not change
    // with the size of the batch it runs in.
    ga.n_slices = (ga.n_tiles + 1) / 2;
    if (ga.n_slices > cus) ga.n_slices = cus;
    if (ga.n_slices > kGridMaxSlices) ga.n_slices = kGridMaxSlices;
    ga.counters = sa.counters;
    ga.chain_stride = n_sets * kGridSetChains;
    {
        int rc = ensure_ftab(t);
        if (rc) return rc;
    }
    ga.ftab = static_cast<const double*>(t->dFtab);

    // carve the workspace
    size_t off = 0;
    auto take = [&](size_t bytes) { const size_t o = off; off = (off + bytes + 255) & ~(size_t)255; return o; };
    const size_t chain_ws = ((size_t)wave_num_vectors(sa.max_depth) * tg.dstride * sizeof(float) + 255) & ~(size_t)255;
    const size_t o_theta = take((size_t)kGridFeatPad * ga.chain_stride * sizeof(float));
    const size_t o_gpart = take((size_t)ga.n_slices * ga.chain_stride * kGridFeatPad * sizeof(float));
    const size_t o_llpart = take((size_t)ga.n_slices * ga.chain_stride * sizeof(double));
    const size_t o_active = take((size_t)kGridMaxStreams * kGridBatch * sizeof(int));
    const size_t o_column = take((size_t)ga.chain_stride * sizeof(int));
    const size_t o_halted = take((size_t)ga.chain_stride * sizeof(int));
    const size_t o_saved = take((size_t)ga.chain_stride * sizeof(Chain::Saved));
    const size_t o_chain = take(chain_ws * ga.chain_stride);
    int rc = ensure_workspace(t, off);
    if (rc) return rc;
    char* w = t->ws_cur;
    ga.b.theta_t = reinterpret_cast<float*>(w + o_theta);
    ga.b.g_part = reinterpret_cast<float*>(w + o_gpart);
    ga.b.ll_part = reinterpret_cast<double*>(w + o_llpart);
    ga.b.active_all = reinterpret_cast<int*>(w + o_active);
    ga.b.column = reinterpret_cast<int*>(w + o_column);
    ga.b.halted = reinterpret_cast<int*>(w + o_halted);
    ga.b.saved = w + o_saved;
    ga.b.chain_ws = w + o_chain;
    ga.b.chain_ws_bytes = chain_ws;

    // consecutive sets share a stream and its launches: same buffers (they own disjoint chain slots), own flags
    GridArgs span[kGridMaxStreams];
    hipStream_t stream[kGridMaxStreams] = {g_stream};
    for (int q = 0; q < n_streams; ++q) {
        span[q] = ga;
        span[q].stream = q;
        span[q].slot_base = q * sets_per_stream * kGridSetChains;
        const int left = n_slots - span[q].slot_base, full = sets_per_stream * kGridSetChains;
        span[q].n_span_slots = left < full ? left : full;
    }
    if (n_streams > 1 && !t->ev_fork) HIP_TRY(hipEventCreateWithFlags(&t->ev_fork, hipEventDisableTiming), NUTS_E_DEVICE);
    for (int q = 1; q < n_streams; ++q) {
        if (!t->side_stream[q - 1]) HIP_TRY(hipStreamCreateWithFlags(&t->side_stream[q - 1], hipStreamNonBlocking), NUTS_E_DEVICE);
        if (!t->ev_join[q - 1]) HIP_TRY(hipEventCreateWithFlags(&t->ev_join[q - 1], hipEventDisableTiming), NUTS_E_DEVICE);
        stream[q] = t->side_stream[q - 1];
    }

    hipLaunchKernelGGL(nuts_grid_fill_kernel, dim3(64), dim3(256), 0, g_stream, reinterpret_cast<int*>(ga.b.theta_t),
                       kGridFeatPad * ga.chain_stride, 0);
    hipLaunchKernelGGL(nuts_grid_fill_kernel, dim3(4), dim3(256), 0, g_stream, ga.b.halted, ga.chain_stride, 1);
    if (n_streams > 1) {  // the side streams start after everything enqueued so far
        HIP_TRY(hipEventRecord(t->ev_fork, g_stream), NUTS_E_DEVICE);
        for (int q = 1; q < n_streams; ++q) HIP_TRY(hipStreamWaitEvent(stream[q], t->ev_fork, 0), NUTS_E_DEVICE);
    }
    // (a guard against a run that never ends: every chain one after the other, every tree full)
    const unsigned long long max_rounds =
        (unsigned long long)sa.n_chains * (unsigned long long)(sa.iter_end - sa.iter_begin) *
            ((unsigned long long)sa.leaf_steps * (1ull << sa.max_depth) + 2) + 8;
    // Batches are enqueued one ahead of the host's look at the "halted" flags, so the GPU never waits for
    // the host; when the flags of batch k say that everybody has halted, batch k + 1 (already enqueued)
    // consists of launches that return at once.  Each set's flags are copied on its own stream: the
    // streams meet again only at the end.
    if (!t->halted_host) HIP_TRY(hipHostMalloc((void**)&t->halted_host, 2 * kGridMaxChains * sizeof(int)), NUTS_E_ALLOC);
    for (hipEvent_t& e : t->ev_batch)
        if (!e) HIP_TRY(hipEventCreateWithFlags(&e, hipEventDisableTiming), NUTS_E_DEVICE);
    unsigned long long rounds = 0;
    int first = 1;
    auto enqueue_batch = [&](int b) -> int {
        for (int q = 0; q < n_streams; ++q)
            hipLaunchKernelGGL(nuts_grid_fill_kernel, dim3(1), dim3(64), 0, stream[q],
                               ga.b.active_all + q * kGridBatch, kGridBatch, 0);
        for (int i = 0; i < kGridBatch; ++i) {
            for (int q = 0; q < n_streams; ++q) {
                hipLaunchKernelGGL(nuts_grid_control_kernel, dim3((unsigned)span[q].n_span_slots), dim3(256), 0, stream[q], tg, sa,
                                   span[q], i, first);
                grid_launch_grad_any(span[q], i, stream[q]);
            }
            first = 0;
            rounds += 1;
        }
        HIP_TRY(hipGetLastError(), NUTS_E_DEVICE);
        for (int q = 0; q < n_streams; ++q) {
            const int base = span[q].slot_base;
            const int count = ga.chain_stride - base < sets_per_stream * kGridSetChains ? ga.chain_stride - base : sets_per_stream * kGridSetChains;
            HIP_TRY(hipMemcpyAsync(t->halted_host + b * kGridMaxChains + base, ga.b.halted + base, count * sizeof(int),
                                   hipMemcpyDeviceToHost, stream[q]),
                    NUTS_E_DEVICE);
        }
        for (int q = 0; q < n_streams; ++q) HIP_TRY(hipEventRecord(t->ev_batch[kGridMaxStreams * b + q], stream[q]), NUTS_E_DEVICE);
        return NUTS_OK;
    };
    auto all_halted = [&](int b) -> int {  // 1 / 0, or a negative error code
        for (int q = 0; q < n_streams; ++q) HIP_TRY(hipEventSynchronize(t->ev_batch[kGridMaxStreams * b + q]), NUTS_E_DEVICE);
        for (int i = 0; i < n_sets * kGridSetChains; ++i)
            if (!t->halted_host[b * kGridMaxChains + i]) return 0;
        return 1;
    };
    rc = enqueue_batch(0);
    if (rc) return rc;
    for (int b = 0;; b ^= 1) {
        rc = enqueue_batch(b ^ 1);
        if (rc) return rc;
        const int done = all_halted(b);
        if (done < 0) return done;
        if (done) break;
        if (rounds > max_rounds + 2 * kGridBatch)
            return fail(NUTS_E_DEVICE, "grid sampler did not finish within %llu rounds", max_rounds);
    }
    for (int q = 1; q < n_streams; ++q) {  // the caller's stream continues after the side streams' last batch
        HIP_TRY(hipEventRecord(t->ev_join[q - 1], stream[q]), NUTS_E_DEVICE);
        HIP_TRY(hipStreamWaitEvent(g_stream, t->ev_join[q - 1], 0), NUTS_E_DEVICE);
    }
    hipLaunchKernelGGL(nuts_grid_finish_kernel, dim3(1), dim3(256), 0, g_stream, ga, sa, n_slots);
    HIP_TRY(hipGetLastError(), NUTS_E_DEVICE);
    t->last_variant = NUTS_VARIANT_GRID;
    t->last_grid = ga.n_slices;
    t->last_slots = 0;
    return NUTS_OK;
}

bool tile_eligible(const nuts_target* t, int max_depth)
{
    return t->kind == NUTS_TARGET_LOGISTIC_REGRESSION && t->dtype == NUTS_F64 && t->tile.base != nullptr &&
           t->dim <= nuts::kTileMaxDim && max_depth <= nuts::kTileMaxDepth;
}

// The lock-step kernel of nuts_wide.h: more features, binary32 targets with few rows, or four chains per workgroup.
bool wide_eligible(const nuts_target* t, int max_depth)
{
    return t->kind == NUTS_TARGET_LOGISTIC_REGRESSION && t->tile.base != nullptr && t->dim <= nuts::kWideMaxDim &&
           t->n <= 1000000 && max_depth <= nuts::kTileMaxDepth;
}

int launch_wide(nuts_target* t, nuts::DevSample sa, int nc, int cus)
{
    const size_t block = nuts::wide_block_bytes((int)t->dim, t->dtype == NUTS_F64 ? 8 : 4, nc, sa.max_depth);
    long blocks = (sa.n_chains + nc - 1) / nc;
    if (blocks > cus) blocks = cus;  // one workgroup per compute unit; further chains wait in the queue
    if (t->static_call) {
        int rc = tile_eligible(t, sa.max_depth) ? NUTS_OK : static_check(t, sa);
        if (rc) return rc;
        const long fit = (long)(((size_t)NUTS_STATIC_SCRATCH_BYTES - kStaticHeader) / block);
        if (fit >= 1 && blocks > fit) blocks = fit;
    }
    // Divided rows, if the workspace for twice as many workgroups can be had.  (nuts_sample_static has no words for pairs to meet at.)
    bool split = !t->static_call && nc == 4 && blocks <= nuts::kWideMaxPairs && nuts::wide_split_pays(sa.n_chains, cus, sa.iter_end - sa.iter_begin, t->n, t->tile.residual);
    const size_t slots = (block * (size_t)blocks * (split ? 2 : 1) + 255) & ~(size_t)255;
    int rc = split ? ensure_workspace_or(t, block * (size_t)blocks, slots + (size_t)blocks * 2 * nuts::wide_exchange_half(t->tile.mt), &split)
                   : ensure_workspace(t, slots);
    if (rc) return rc;
    const long pairs = split ? blocks : 0;
    if (split) blocks *= 2;
    sa.workspace = t->ws_cur;
    sa.slot_bytes = block;
    const nuts::WideArgs wa{nuts::tile_args(t->tile, 1.0 / (t->prior_scale * t->prior_scale)), t->tile.ks1, (int)pairs,
                            reinterpret_cast<unsigned*>(t->counters_cur + nuts::kCtrCount), t->ws_cur + slots, t->wide_apart};
    (t->dtype == NUTS_F64 ? nuts::wide_launch_f64 : nuts::wide_launch_f32)(wa, sa, nc, (int)blocks, g_stream);
    HIP_TRY(hipGetLastError(), NUTS_E_DEVICE);
    t->last_variant = NUTS_VARIANT_TILE;
    t->last_grid = (int)blocks;
    t->last_slots = 0;
    return NUTS_OK;
}

int launch_tile(nuts_target* t, nuts::DevSample sa)
{
    int cus = 0;
    HIP_TRY(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, t->device), NUTS_E_DEVICE);
    const int nc = nuts::wide_chains_per_block(sa.n_chains, cus, sa.iter_end - sa.iter_begin, t->n, (int)t->dim, t->tile.residual);
    if (!tile_eligible(t, sa.max_depth) || nc == 4) return launch_wide(t, sa, nc, cus);
    nuts::TileLaunch tl;
    nuts::tile_plan(t->tile, sa.n_chains, sa.max_depth, &tl);
    int rc = ensure_workspace(t, tl.workspace_bytes);
    if (rc) return rc;
    sa.workspace = t->ws_cur;
    sa.slot_bytes = tl.block_bytes;
    nuts::tile_launch(t->tile, sa, 1.0 / (t->prior_scale * t->prior_scale), tl, g_stream);
    HIP_TRY(hipGetLastError(), NUTS_E_DEVICE);
    t->last_variant = NUTS_VARIANT_TILE;
    t->last_grid = tl.blocks;
    t->last_slots = 0;
    return NUTS_OK;
}

// One launch of the chip kernel, which needs all its workgroups at once, one at a time on a device (two of them that each had a
// part of the chip would wait for each other).  A start that not all workgroups reach, because somebody else holds compute
// units, ends after half a second, before anything has been done.  The host then waits until a compute unit has room for a workgroup, as
// any launch would, and starts again; after three such starts with half as many workgroups, down to one, which waits for nobody.
// So a busy device or a stream that has a part of it delays a call and never fails it, and the outputs are the same bits (the
// rows are divided as for the whole chip).  As with the grid kernels, this returns only when sampling is complete.
std::mutex g_chip_mutex[kMaxDevices];

// Compute units that the call's stream may use (a stream can be created with a mask of them).
int stream_compute_units(int cus)
{
    uint32_t mask[32] = {};
    if (hipExtStreamGetCUMask(g_stream, 32, mask) != hipSuccess) {
        (void)hipGetLastError();
        return cus;
    }
    int n = 0;
    for (uint32_t m : mask) n += __builtin_popcount(m);
    return n >= 1 && n < cus ? n : cus;
}

__global__ void chip_room_kernel() {}

// Returns when a compute unit has had room for a workgroup, and a moment later: that of two processes whose workgroups shared
// the chip out among them one comes first.
int await_chip_room(size_t lds_bytes, int attempt)
{
    HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(chip_room_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes), NUTS_E_DEVICE);
    hipLaunchKernelGGL(chip_room_kernel, dim3(1), dim3(nuts::kChipThreads), lds_bytes, g_stream);
    HIP_TRY(hipGetLastError(), NUTS_E_DEVICE);
    HIP_TRY(hipStreamSynchronize(g_stream), NUTS_E_DEVICE);
    // (of the clock and this process's address space: no source of random numbers that could throw)
    const uint64_t seed = (uint64_t)std::chrono::steady_clock::now().time_since_epoch().count() ^ (uint64_t)reinterpret_cast<uintptr_t>(&g_stream);
    const unsigned span_us = 20000u << std::min(attempt, 5);
    std::this_thread::sleep_for(std::chrono::microseconds((seed * 0x9e3779b97f4a7c15ull >> 33) % span_us));
    return NUTS_OK;
}

int launch_chip(nuts_target* t, nuts::DevSample sa)
{
    using namespace nuts;
    int cus = 0;
    HIP_TRY(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, t->device), NUTS_E_DEVICE);
    const int mt = t->chip.mt;
    ChipPlan cp{};
    const int whole = cus < kChipMaxBlocks ? cus : kChipMaxBlocks;
    cp.blocks = std::min(whole, stream_compute_units(cus));
    if (t->chip_most > 0 && t->chip_most < cp.blocks) cp.blocks = t->chip_most;
    chip_lds(mt, sa.max_depth, &cp);
    ChipArgs ca{};
    ca.x = t->chip.x;
    ca.d = t->chip.d;
    ca.n_rows = t->chip.n_rows;
    ca.n_tiles = t->chip.n_tiles;
    ca.n_slices = chip_slices(ca.n_tiles, whole);
    const size_t most_slots = (size_t)std::min<long>(sa.n_chains, (long)cp.blocks * kChipOwners);
    ca.prior_prec = 1.0 / (t->prior_scale * t->prior_scale);
    ca.theta_bytes = (unsigned)((size_t)kChipColumns * 16 * mt * sizeof(float));
    ca.g_bytes = (unsigned)((size_t)ca.n_slices * ca.theta_bytes);
    size_t off = 0;
    auto take = [&](size_t bytes) { const size_t o = off; off = (off + bytes + 255) & ~(size_t)255; return o; };
    const size_t shared_words = (kChipCounters + 1) * kChipLine;
    const size_t o_shared = take(shared_words * sizeof(unsigned));
    const size_t o_theta = take(ca.theta_bytes), o_g = take(ca.g_bytes);
    const size_t o_ll = take((size_t)ca.n_slices * kChipColumns * sizeof(double));
    const size_t o_chains = take(cp.slot_bytes * most_slots);
    int rc = ensure_workspace(t, off);
    if (rc) return rc;
    ca.shared = reinterpret_cast<unsigned*>(t->ws_cur + o_shared);
    ca.theta = reinterpret_cast<float*>(t->ws_cur + o_theta);
    ca.g_part = reinterpret_cast<float*>(t->ws_cur + o_g);
    ca.ll_part = reinterpret_cast<double*>(t->ws_cur + o_ll);
    sa.workspace = t->ws_cur + o_chains;
    sa.slot_bytes = cp.slot_bytes;
    if (!t->chip_state) HIP_TRY(hipHostMalloc((void**)&t->chip_state, sizeof(unsigned)), NUTS_E_ALLOC);
    std::lock_guard<std::mutex> lock(g_chip_mutex[t->device]);
    for (int attempt = 0;; ++attempt) {
        ca.n_blocks = cp.blocks;
        ca.n_slots = (int)std::min<long>(sa.n_chains, (long)cp.blocks * kChipOwners);
        hipLaunchKernelGGL(fill_words_kernel, dim3(1), dim3(256), 0, g_stream, ca.shared, (int)shared_words, 0u);
        unsigned* const state = ca.shared + kChipCounters * kChipLine;
        if (t->chip_refuse > 0) {
            t->chip_refuse -= 1;
            hipLaunchKernelGGL(fill_words_kernel, dim3(1), dim3(64), 0, g_stream, state, 1, (unsigned)kChipNotStarted);
        }
        HIP_TRY(chip_launch(mt, ca, sa, cp, g_stream), NUTS_E_DEVICE);
        HIP_TRY(hipMemcpyAsync(t->chip_state, state, sizeof(unsigned), hipMemcpyDeviceToHost, g_stream), NUTS_E_DEVICE);
        HIP_TRY(hipStreamSynchronize(g_stream), NUTS_E_DEVICE);
        if (*t->chip_state == kChipRunning) break;
        if (*t->chip_state != kChipNotStarted) return fail(NUTS_E_DEVICE, "chip kernel: a workgroup did not reach a barrier in time");
        rc = await_chip_room(cp.lds_bytes, attempt);
        if (rc) return rc;
        if (attempt % 3 == 2) t->chip_most = cp.blocks = (cp.blocks + 1) / 2;  // (for the rest of the call)
    }
    t->last_variant = NUTS_VARIANT_GRID;
    t->last_grid = cp.blocks;
    t->last_slots = 0;
    return NUTS_OK;
}

}  // namespace

extern "C" {

const char* nuts_last_error(void) { return g_err; }

// For tests of what a busy device does to the chip kernel's runs on a target (not part of the interface): its next `refused` starts
// end as starts do that not all workgroups reach, and its calls take at most `most_blocks` workgroups (0: no bound).
int nuts_debug_chip_starts(nuts_target* t, int refused, int most_blocks)
{
    if (!t || refused < 0 || most_blocks < 0) return fail(NUTS_E_INVALID_ARG, "nuts_debug_chip_starts: bad argument");
    t->chip_refuse = refused;
    t->chip_bound = most_blocks;
    return NUTS_OK;
}

// For tests: 1: the wide kernel's pairs of workgroups do not meet, the first takes all rows; 2 or 3: the first or the second of them
// sends nothing from its third round on, and the other waits 0.2 ms for it; 0: as ever.
int nuts_debug_wide_apart(nuts_target* t, int apart)
{
    if (!t || apart < 0 || apart > 3) return fail(NUTS_E_INVALID_ARG, "nuts_debug_wide_apart: bad argument");
    t->wide_apart = apart;
    return NUTS_OK;
}

// For tests: how many steps a slot of the row kernels takes with a chain while others wait (less than 0: as ever).
int nuts_debug_turns(nuts_target* t, int steps)
{
    if (!t) return fail(NUTS_E_INVALID_ARG, "nuts_debug_turns: bad argument");
    t->turn_steps = steps;
    return NUTS_OK;
}

// For tests: allocations of more than `most` bytes of workspace are refused from now on (0: only those that the device refuses).
// *bytes: the workspace that there is; *refusals: how many have been refused.
int nuts_debug_workspace(nuts_target* t, unsigned long long most, unsigned long long* bytes, int* refusals)
{
    if (!t || !bytes || !refusals) return fail(NUTS_E_INVALID_ARG, "nuts_debug_workspace: bad argument");
    t->workspace_most = most == 0 ? SIZE_MAX : (size_t)most;
    *bytes = t->workspace_bytes;
    *refusals = t->workspace_refusals;
    return NUTS_OK;
}

// For tests, of the last call on a target: pairs of the wide kernel's workgroups that met, of these the ones of which one went on alone, and chains
// of the row kernels that were handed over.
int nuts_debug_counts(const nuts_target* t, unsigned long long* pairs_met, unsigned long long* pairs_lost, unsigned long long* turns)
{
    if (!t || !pairs_met || !pairs_lost || !turns || !t->has_run) return fail(NUTS_E_INVALID_ARG, "nuts_debug_counts: bad argument");
    HIP_TRY(hipEventSynchronize(t->ev_stop), NUTS_E_DEVICE);
    unsigned long long c[nuts::kCtrCount];
    HIP_TRY(hipMemcpy(c, t->counters_cur, sizeof(c), hipMemcpyDeviceToHost), NUTS_E_DEVICE);
    *pairs_met = c[nuts::kCtrPairsMet];
    *pairs_lost = c[nuts::kCtrPairsLost];
    *turns = c[nuts::kCtrTurns];
    return NUTS_OK;
}

int nuts_tile_pack(const double* X, const double* y, int64_t n, int64_t d, nuts_tile_layout* layout, double* operands,
                   int64_t capacity)
{
    if (!X || !y || !layout) return fail(NUTS_E_INVALID_ARG, "nuts_tile_pack: null argument");
    if (!nuts::tile_supports_shape(d, n)) return fail(NUTS_E_INVALID_ARG, "nuts_tile_pack: shape outside the tile variant's range");
    nuts::TileData td;
    std::vector<double> op, colsum;
    try {
        nuts::tile_pack_operands(X, y, n, d, false, &td, &op, &colsum);
    } catch (const std::bad_alloc&) {
        return fail(NUTS_E_ALLOC, "out of host memory");
    }
    layout->ks1 = td.ks1;
    layout->mt = td.mt;
    layout->n_tiles = td.n_tiles;
    layout->n_alloc_tiles = td.n_alloc_tiles;
    layout->const_col = td.z0_col;
    layout->reserved = 0;
    layout->const_val = td.z0_val;
    layout->n_pad = td.n_pad;
    layout->operand_doubles = (int64_t)op.size();
    if (operands) {
        if (capacity < (int64_t)op.size()) return fail(NUTS_E_INVALID_ARG, "nuts_tile_pack: operands buffer too small");
        std::memcpy(operands, op.data(), op.size() * sizeof(double));
    }
    return NUTS_OK;
}

int nuts_set_stream(void* hip_stream)
{
    g_stream = static_cast<hipStream_t>(hip_stream);
    return NUTS_OK;
}

int nuts_create_target(const nuts_target_desc* desc, nuts_target** out)
{
    if (!desc || !out) return fail(NUTS_E_INVALID_ARG, "desc and out must not be NULL");
    if (desc->dtype != NUTS_F32 && desc->dtype != NUTS_F64) return fail(NUTS_E_INVALID_ARG, "unknown dtype %d", desc->dtype);
    if (desc->kind < NUTS_TARGET_STD_NORMAL || desc->kind > NUTS_TARGET_LOGISTIC_REGRESSION)
        return fail(NUTS_E_INVALID_ARG, "unknown target kind %d", desc->kind);
    if (desc->dim < 1 || desc->dim > (1 << 24)) return fail(NUTS_E_INVALID_ARG, "dim must be in [1, 2^24]");
    if (desc->kind == NUTS_TARGET_GAUSS_DENSE_PRECISION && !desc->precision)
        return fail(NUTS_E_INVALID_ARG, "precision must not be NULL");
    if (desc->kind == NUTS_TARGET_GAUSS_DIAG && !desc->scales) return fail(NUTS_E_INVALID_ARG, "scales must not be NULL");
    if (desc->kind == NUTS_TARGET_LOGISTIC_REGRESSION) {
        if (!desc->X || !desc->y) return fail(NUTS_E_INVALID_ARG, "X and y must not be NULL");
        if (desc->n_data < 1 || desc->n_data > (1ll << 31) - 64) return fail(NUTS_E_INVALID_ARG, "n_data out of range");
        if (!(desc->prior_scale > 0.0) || !std::isfinite(desc->prior_scale))
            return fail(NUTS_E_INVALID_ARG, "prior_scale must be finite and > 0");
    }
    int rc = desc->dtype == NUTS_F64 ? check_values<double>(desc) : check_values<float>(desc);
    if (rc) return rc;

    nuts_target* t = new (std::nothrow) nuts_target();
    if (!t) return fail(NUTS_E_ALLOC, "out of host memory");
    t->kind = desc->kind;
    t->dtype = desc->dtype;
    t->dim = desc->dim;
    t->n = desc->kind == NUTS_TARGET_LOGISTIC_REGRESSION ? desc->n_data : 0;
    t->prior_scale = desc->kind == NUTS_TARGET_LOGISTIC_REGRESSION ? desc->prior_scale : 1.0;
    int n_dev = 0;
    const bool have_device = hipGetDeviceCount(&n_dev) == hipSuccess && n_dev >= 1;
    if (desc->kind != NUTS_TARGET_STD_NORMAL || have_device) {  // the standard normal has no data: it needs no device yet
        rc = ensure_device(t);
        try {  // (operand streams take up to twice the data's size on the host)
            if (!rc) rc = desc->dtype == NUTS_F64 ? build_device_data<double>(t, desc) : build_device_data<float>(t, desc);
            if (!rc && t->grid.ops) rc = ensure_ftab(t);
        } catch (const std::bad_alloc&) {
            rc = fail(NUTS_E_ALLOC, "out of host memory");
        }
        if (rc) {
            release(t);
            return rc;
        }
    }
    *out = t;
    return NUTS_OK;
}

int nuts_destroy_target(nuts_target* t)
{
    release(t);
    return NUTS_OK;
}

}  // extern "C"

namespace {

// Body of nuts_sample_ex and nuts_sample_static.  With use_static the call takes its workspace and counters from
// the device's static scratch array and refuses whatever would need an allocation.
int sample_impl(const nuts_target* target, int64_t n_chains, int64_t n_iters, double step_size,
                int32_t max_tree_depth, uint64_t seed, const nuts_sample_options* options, void* out_states,
                int32_t* out_tree_depths, int32_t* out_n_leapfrog, bool use_static)
{
    if (!target) return fail(NUTS_E_INVALID_ARG, "target must not be NULL");
    if (n_chains < 1 || n_chains > (1ll << 31) - 1) return fail(NUTS_E_INVALID_ARG, "n_chains must be in [1, 2^31)");
    if (n_iters < 1 || n_iters > (1ll << 31) - 1) return fail(NUTS_E_INVALID_ARG, "n_iters must be in [1, 2^31)");
    if (!(step_size > 0.0) || !std::isfinite(step_size)) return fail(NUTS_E_INVALID_ARG, "step_size must be finite and > 0");
    if (max_tree_depth < 1 || max_tree_depth > 20) return fail(NUTS_E_INVALID_ARG, "max_tree_depth must be in [1, 20]");
    nuts_sample_options opt{};
    if (options) opt = *options;
    if (opt.first_chain < 0 || opt.first_chain + n_chains > (1ll << 32))
        return fail(NUTS_E_INVALID_ARG, "chain ids must fit in 32 bits");
    if (opt.variant < NUTS_VARIANT_AUTO || opt.variant > NUTS_VARIANT_QUAD)
        return fail(NUTS_E_INVALID_ARG, "unknown variant %d", opt.variant);
    if (opt.schedule != NUTS_SCHEDULE_FREE && opt.schedule != NUTS_SCHEDULE_TRAJECTORY)
        return fail(NUTS_E_INVALID_ARG, "unknown schedule %d", opt.schedule);
    if (opt.sampler != NUTS_SAMPLER_MULTINOMIAL && opt.sampler != NUTS_SAMPLER_SLICE)
        return fail(NUTS_E_INVALID_ARG, "unknown sampler %d", opt.sampler);
    if (opt.leaf_steps < 0 || opt.leaf_steps > NUTS_MAX_LEAF_STEPS)
        return fail(NUTS_E_INVALID_ARG, "leaf_steps must be in [1, %d] (0 = 1)", NUTS_MAX_LEAF_STEPS);
    const int leaf_steps = opt.leaf_steps == 0 ? 1 : opt.leaf_steps;
    nuts_target* t = const_cast<nuts_target*>(target);  // the scratch cache is logically mutable
    if (opt.variant == NUTS_VARIANT_TILE && !tile_eligible(t, max_tree_depth))
        return fail(NUTS_E_UNSUPPORTED,
                    "the tile kernel needs binary64 logistic regression with dim <= %d and max_tree_depth <= %d",
                    nuts::kTileMaxDim, nuts::kTileMaxDepth);

    if (opt.variant == NUTS_VARIANT_ELEM && !elem_eligible(t))
        return fail(NUTS_E_UNSUPPORTED, "the element-wise kernel needs a standard-normal or diagonal-Gaussian target with dim <= %d",
                    elem_max_dim(t->dtype));

    if (opt.variant == NUTS_VARIANT_GRID && !grid_eligible(t))
        return fail(NUTS_E_UNSUPPORTED, "the grid kernels need binary32 logistic regression with dim <= %d", nuts::kGridMaxDim);

    if (opt.variant == NUTS_VARIANT_QUAD && !quad_eligible(t, max_tree_depth))
        return fail(NUTS_E_UNSUPPORTED, "the quad kernel needs a binary64 dense Gaussian target with dim <= %d and max_tree_depth <= %d",
                    nuts::kQuadMaxDim, nuts::kQuadMaxDepth);

    if (opt.variant == NUTS_VARIANT_DENSE && !dense_eligible(t))
        return fail(NUTS_E_UNSUPPORTED, "the dense-Gaussian register kernel needs a dense Gaussian target with dim <= %d",
                    nuts::kDenseMaxDim);

    const int elem_variant = elem_eligible(t) ? NUTS_VARIANT_ELEM : NUTS_VARIANT_WAVE;
    const bool use_elem = opt.variant == NUTS_VARIANT_ELEM ||
                          (opt.variant == NUTS_VARIANT_AUTO && t->dim <= kElemMaxDim &&
                           (t->kind == NUTS_TARGET_STD_NORMAL || t->kind == NUTS_TARGET_GAUSS_DIAG));
    const bool use_grid = opt.variant == NUTS_VARIANT_GRID ||
                          (opt.variant == NUTS_VARIANT_AUTO && grid_eligible(t) && grid_pays(t->n, t->dim));
    const bool use_tile = opt.variant == NUTS_VARIANT_TILE ||
                          (opt.variant == NUTS_VARIANT_AUTO && !use_grid &&
                           (tile_eligible(t, max_tree_depth) || wide_eligible(t, max_tree_depth)));
    // A precision matrix that is not banded goes to the matrix cores, four chains per wavefront, once there are
    // enough chains to give every compute unit several (below that the one-chain-per-wavefront kernel spreads
    // them over more SIMDs; measured crossover, see the profile summary of the quad kernel)
    const bool use_quad = opt.variant == NUTS_VARIANT_QUAD ||
                          (opt.variant == NUTS_VARIANT_AUTO && quad_eligible(t, max_tree_depth) && !t->dBand &&
                           n_chains >= nuts::kQuadAutoChains);
    const bool use_dense = !use_quad && (opt.variant == NUTS_VARIANT_DENSE || (opt.variant == NUTS_VARIANT_AUTO && dense_eligible(t)));

    const bool use_band = opt.variant == NUTS_VARIANT_AUTO && band_eligible(t);
    const bool use_block = opt.variant == NUTS_VARIANT_AUTO && block_eligible(t);

    int rc = NUTS_OK;
    if (use_static) {
        // nothing below may allocate: the target must already hold its device data, counters and events
        int dev = -1;
        if (hipGetDevice(&dev) != hipSuccess) return fail(NUTS_E_DEVICE, "no HIP device available (this library has no CPU path)");
        if (t->device < 0 || !t->counters || !t->ev_start || !t->ev_stop)
            return fail(NUTS_E_UNSUPPORTED, "the target was created without a GPU: nuts_sample_static cannot set it up");
        if (t->device != dev)
            return fail(NUTS_E_INVALID_ARG, "target was created on device %d, current device is %d", t->device, dev);
        if (!g_scratch_ptr[dev]) return fail(NUTS_E_DEVICE, "static scratch of device %d was not resolved", dev);
        if (use_grid && !use_dense && !use_tile)
            return fail(NUTS_E_UNSUPPORTED, "the grid kernels own streams and pinned host memory: not available without allocation");
        if (opt.schedule == NUTS_SCHEDULE_TRAJECTORY && !out_states)
            return fail(NUTS_E_UNSUPPORTED, "the trajectory schedule without out_states needs a carry buffer: pass out_states");
    } else {
        rc = ensure_device(t);
        if (rc) return rc;
    }
    t->static_call = use_static;
    t->chip_most = t->chip_bound;
    t->counters_cur = use_static ? reinterpret_cast<unsigned long long*>(g_scratch_ptr[t->device]) : t->counters;

    nuts::DevSample sa{};
    sa.n_chains = (long)n_chains;
    sa.first_chain = (long)opt.first_chain;
    sa.n_iters = (int)n_iters;
    sa.max_depth = max_tree_depth;
    sa.leaf_steps = leaf_steps;
    sa.sampler = opt.sampler;
    sa.eps = step_size;
    sa.key0 = (uint32_t)(seed & 0xffffffffu);
    sa.key1 = (uint32_t)(seed >> 32);
    sa.out_states = out_states;
    sa.out_depths = out_tree_depths;
    sa.out_nleap = out_n_leapfrog;
    sa.init_states = opt.init_states;
    sa.counters = t->counters_cur;

    const int pair_words = !use_static && use_tile ? nuts::kWideMaxPairs : 0;
    // the counters start at zero (a fill kernel, so that the call can sit inside a captured graph)
    hipLaunchKernelGGL(zero_counters_kernel, dim3(1), dim3(64), 0, g_stream, t->counters_cur, pair_words);
    HIP_TRY(hipGetLastError(), NUTS_E_DEVICE);

    auto launch = [&](const nuts::DevSample& s) -> int {
        int r;
        t->turns_cur = nullptr;
        if (use_quad)
            r = launch_quad(t, s);
        else if (use_dense)
            r = t->dtype == NUTS_F64 ? launch_dense<double>(t, s) : launch_dense<float>(t, s);
        else if (use_band)
            r = t->dtype == NUTS_F64 ? launch_band<double>(t, s) : launch_band<float>(t, s);
        else if (use_block)
            r = t->dtype == NUTS_F64 ? launch_block<double>(t, s) : launch_block<float>(t, s);
        else if (use_tile)
            r = launch_tile(t, s);
        else if (use_grid)
            r = t->chip.x ? launch_chip(t, s) : launch_grid(t, s);
        else if (use_elem)
            r = t->dtype == NUTS_F64 ? launch_elem<double>(t, s, elem_variant) : launch_elem<float>(t, s, elem_variant);
        else
            r = t->dtype == NUTS_F64 ? launch_wave<double>(t, s) : launch_wave<float>(t, s);
        if (r) return r;
        hipLaunchKernelGGL(close_launch_kernel, dim3(1), dim3(64), 0, g_stream, t->counters_cur, (unsigned long long)t->last_slots, pair_words, t->turns_cur);
        HIP_TRY(hipGetLastError(), NUTS_E_DEVICE);
        return NUTS_OK;
    };
    if (opt.schedule == NUTS_SCHEDULE_TRAJECTORY) {
        // every chain finishes iteration i before any chain starts iteration i + 1: one launch per
        // iteration; a launch starts from the states the one before wrote.  A caller that wants no
        // states still needs them for that: they go to a one-iteration carry buffer instead.
        const size_t carry_bytes = (size_t)n_chains * (size_t)t->dim * (t->dtype == NUTS_F64 ? 8 : 4);
        if (!use_static && !out_states && carry_bytes > t->carry_bytes) {
            if (t->carry) {
                HIP_TRY(hipDeviceSynchronize(), NUTS_E_DEVICE);
                (void)hipFree(t->carry);
                t->carry = nullptr;
                t->carry_bytes = 0;
            }
            HIP_TRY(hipMalloc(&t->carry, carry_bytes), NUTS_E_ALLOC);
            t->carry_bytes = carry_bytes;
        }
    }
    HIP_TRY(hipEventRecord(t->ev_start, g_stream), NUTS_E_DEVICE);
    if (opt.schedule == NUTS_SCHEDULE_TRAJECTORY) {
        const size_t row_bytes = (size_t)n_chains * (size_t)t->dim * (t->dtype == NUTS_F64 ? 8 : 4);
        for (int64_t i = 0; i < n_iters && !rc; ++i) {
            sa.iter_begin = (int)i;
            sa.iter_end = (int)i + 1;
            if (out_states) {
                if (i > 0) sa.init_states = static_cast<char*>(out_states) + (size_t)(i - 1) * row_bytes;
            } else {
                // the kernels address states as base + (iteration * n_chains + chain) * dim: shift the base so
                // that this iteration's row is the carry buffer (each chain reads its row before it writes it)
                sa.out_states = reinterpret_cast<void*>(reinterpret_cast<uintptr_t>(t->carry) - (uintptr_t)i * row_bytes);
                if (i > 0) sa.init_states = t->carry;
            }
            rc = launch(sa);
        }
    } else {
        sa.iter_begin = 0;
        sa.iter_end = (int)n_iters;
        rc = launch(sa);
    }
    if (rc) return rc;
    HIP_TRY(hipEventRecord(t->ev_stop, g_stream), NUTS_E_DEVICE);
    t->has_run = true;
    return NUTS_OK;
}

}  // namespace

extern "C" {

int nuts_sample_ex(const nuts_target* target, int64_t n_chains, int64_t n_iters, double step_size,
                   int32_t max_tree_depth, uint64_t seed, const nuts_sample_options* options, void* out_states,
                   int32_t* out_tree_depths, int32_t* out_n_leapfrog)
{
    return sample_impl(target, n_chains, n_iters, step_size, max_tree_depth, seed, options, out_states, out_tree_depths,
                       out_n_leapfrog, false);
}

int nuts_sample_static(const nuts_target* target, int64_t n_chains, int64_t n_iters, double step_size,
                       int32_t max_tree_depth, uint64_t seed, const nuts_sample_options* options, void* out_states,
                       int32_t* out_tree_depths, int32_t* out_n_leapfrog)
{
    return sample_impl(target, n_chains, n_iters, step_size, max_tree_depth, seed, options, out_states, out_tree_depths,
                       out_n_leapfrog, true);
}

int nuts_sample(const nuts_target* target, int64_t n_chains, int64_t n_iters, double step_size, int32_t max_tree_depth,
                uint64_t seed, void* out_states, int32_t* out_tree_depths, int32_t* out_n_leapfrog)
{
    return nuts_sample_ex(target, n_chains, n_iters, step_size, max_tree_depth, seed, nullptr, out_states,
                          out_tree_depths, out_n_leapfrog);
}

int nuts_get_stats(const nuts_target* target, nuts_stats* out)
{
    if (!target || !out) return fail(NUTS_E_INVALID_ARG, "target and out must not be NULL");
    if (!target->has_run) return fail(NUTS_E_INVALID_ARG, "no sampling call has been made on this target");
    HIP_TRY(hipEventSynchronize(target->ev_stop), NUTS_E_DEVICE);
    unsigned long long c[nuts::kCtrCount];
    HIP_TRY(hipMemcpy(c, target->counters_cur, sizeof(c), hipMemcpyDeviceToHost), NUTS_E_DEVICE);
    float ms = 0.f;
    HIP_TRY(hipEventElapsedTime(&ms, target->ev_start, target->ev_stop), NUTS_E_DEVICE);
    out->leaf_slots_issued = c[nuts::kCtrIssued];
    out->leaf_slots_useful = c[nuts::kCtrUseful];
    out->extra_grad_evals = c[nuts::kCtrExtra];
    out->rounds = c[nuts::kCtrRounds];
    out->kernel_ms = ms;
    out->phase_ticks[0] = c[nuts::kCtrCycControl];
    out->phase_ticks[1] = c[nuts::kCtrCycGrad];
    out->phase_ticks[2] = c[nuts::kCtrCycPost];
    out->variant = target->last_variant;
    out->grid_blocks = target->last_grid;
    return NUTS_OK;
}

}  // extern "C"
