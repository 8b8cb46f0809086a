// Host runtime of the frequency-Hough library: contexts, device-resident
// peakmaps, validation, tile planning, workspace management and the launch
// sequences behind the C ABI of include/fh.h.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <chrono>
#include <deque>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <tuple>
#include <vector>

#include "fh_internal.h"

using namespace fh;

// Scratch memory of fh_hough_map_i32_static (callers that cannot allocate):
// one copy of this array per GPU, held until the process ends.  Host code
// never passes the array's name to a kernel or a copy: the device address of
// each GPU's copy is taken once, with that device current, when the first
// context on it is created (scratch_init), and only that address is used.
constexpr size_t kStaticScratchBytes = (size_t)64 << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace {

thread_local std::string g_err = "no error";

// The status of a failed call.  HIP keeps the error of a failed call until it
// is asked for, whatever succeeds in between, and every launch asks for it: a
// call that fails takes its error along, or the next one would report it.
fh_status fail(fh_status s, const char *fmt, ...) {
    if (s == FH_E_DEVICE) (void)hipGetLastError();
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_err = buf;
    return s;
}

#define HIP_OK(expr)                                                                   \
    do {                                                                               \
        hipError_t e_ = (expr);                                                        \
        if (e_ != hipSuccess)                                                          \
            return fail(FH_E_DEVICE, "%s failed: %s", #expr, hipGetErrorString(e_));  \
    } while (0)

// Device address of each GPU's copy of `scratch` (nullptr until taken).
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices] = {};

// Take the address of the current device's copy of `scratch` (once per
// device).  Devices past kMaxDevices keep no address; the entry point that
// needs it then reports FH_E_UNSUPPORTED.
fh_status scratch_init(int device) {
    if (device < 0 || device >= kMaxDevices) return FH_OK;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (g_scratch_ptr[device]) return FH_OK;
    void *p = nullptr;
    hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p)
        return fail(FH_E_DEVICE, "hipGetSymbolAddress(scratch) on device %d: %s", device, hipGetErrorString(e));
    g_scratch_ptr[device] = p;
    return FH_OK;
}

// Device and pinned host memory, nullptr when there is none; the error of a
// failure goes no further (the caller may do without).
// *full: whether it failed for want of memory (and not, say, in a capture).
void *device_alloc(size_t n, bool *full = nullptr) {
    void *p = nullptr;
    const hipError_t e = hipMalloc(&p, n);
    if (full) *full = e == hipErrorOutOfMemory;
    if (e == hipSuccess) return p;
    (void)hipGetLastError();
    return nullptr;
}

void device_free(void *p) {
    if (p && hipFree(p) != hipSuccess) (void)hipGetLastError();
}

// Waits for the device's work as hipFree does, by freeing a small block (1.2 us
// when the device is idle): hipDeviceSynchronize() breaks every capture that is
// under way on the device, also in other threads, where hipFree is harmless.
// False when it cannot (this thread is capturing).
bool wait_as_free() {
    void *p = device_alloc(256);
    if (!p) return false;
    const bool ok = hipFree(p) == hipSuccess;
    if (!ok) (void)hipGetLastError();
    return ok;
}

void *pinned_alloc(size_t n) {
    void *p = nullptr;
    if (hipHostMalloc(&p, n, hipHostMallocDefault) == hipSuccess) return p;
    (void)hipGetLastError();
    return nullptr;
}

struct Spare;

// A device buffer that only grows.  Growing synchronises the stream first so
// that no enqueued kernel still uses the old allocation.
struct DevBuf {
    void *ptr = nullptr;
    size_t bytes = 0;
    Spare *spare = nullptr;  // given back when there is no room to grow
    bool allocate(size_t n);
    fh_status ensure(size_t want, hipStream_t st) {
        if (want <= bytes) return FH_OK;
        if (ptr) {
            hipError_t e = hipStreamSynchronize(st);
            if (e != hipSuccess) return fail(FH_E_DEVICE, "hipStreamSynchronize: %s", hipGetErrorString(e));
            (void)hipFree(ptr);
            ptr = nullptr;
            bytes = 0;
        }
        size_t n = std::max(want, (size_t)256);
        if (!allocate(n)) return fail(FH_E_NOMEM, "hipMalloc of %zu bytes failed", n);
        bytes = n;
        return FH_OK;
    }
    void release() {
        if (ptr) (void)hipFree(ptr);
        ptr = nullptr;
        bytes = 0;
    }
};

struct PinnedBuf {
    void *ptr = nullptr;
    size_t bytes = 0;
    fh_status ensure(size_t want, hipStream_t st) {
        if (want <= bytes) return FH_OK;
        if (ptr) {
            hipError_t e = hipStreamSynchronize(st);
            if (e != hipSuccess) return fail(FH_E_DEVICE, "hipStreamSynchronize: %s", hipGetErrorString(e));
            (void)hipHostFree(ptr);
            ptr = nullptr;
            bytes = 0;
        }
        size_t n = std::max(want, (size_t)4096);
        if (!(ptr = pinned_alloc(n))) return fail(FH_E_NOMEM, "hipHostMalloc of %zu bytes failed", n);
        bytes = n;
        return FH_OK;
    }
    void release() {
        if (ptr) (void)hipHostFree(ptr);
        ptr = nullptr;
        bytes = 0;
    }
};

// Device blocks of released peakmaps, kept for the next ones: building or
// filtering a peakmap otherwise spends several times its kernels' time in
// hipMalloc and hipFree (which maps and unmaps the pages): 700 us of calls
// around 70 us of kernels for a band of 2.1 M peaks.  At most kMaxBlocks
// blocks of kMaxBytes together; a block serves requests of half its size or
// more; given back when an allocation fails (Spare) and with the context.
// Locked: a peakmap may be released on another thread than the context's (a
// garbage collector's) while the context's is building one.
struct BlockPool {
    static constexpr size_t kMaxBlocks = 8;
    static constexpr size_t kMaxBytes = (size_t)256 << 20;
    struct Block { void *ptr; size_t bytes; };
    std::mutex mu;
    std::vector<Block> free_;
    size_t held = 0;
    BlockPool() { free_.reserve(kMaxBlocks + 1); }
    // the size that a request of n bytes is allocated with
    static size_t block_bytes(size_t n) { return (std::max(n, (size_t)1) + 4095) / 4096 * 4096; }
    // a kept block of at least n bytes and its size, or nullptr
    void *take(size_t n, size_t *bytes) {
        n = block_bytes(n);
        std::lock_guard<std::mutex> lock(mu);
        size_t at = free_.size();
        for (size_t k = 0; k < free_.size(); ++k)
            if (free_[k].bytes >= n && free_[k].bytes <= 2 * n &&
                (at == free_.size() || free_[k].bytes < free_[at].bytes))
                at = k;
        if (at == free_.size()) return nullptr;
        const Block b = free_[at];
        free_.erase(free_.begin() + (long)at);
        held -= b.bytes;
        *bytes = b.bytes;
        return b.ptr;
    }
    // no enqueued work uses the block any more
    void give(void *p, size_t bytes) {
        if (!p) return;
        if (bytes > kMaxBytes) {
            (void)hipFree(p);
            return;
        }
        std::lock_guard<std::mutex> lock(mu);
        free_.push_back({p, bytes});
        held += bytes;
        while (held > kMaxBytes || free_.size() > kMaxBlocks) {
            (void)hipFree(free_.front().ptr);
            held -= free_.front().bytes;
            free_.erase(free_.begin());
        }
    }
    // whether there was a block
    bool trim() {
        std::lock_guard<std::mutex> lock(mu);
        const bool any = !free_.empty();
        for (const Block &b : free_) (void)hipFree(b.ptr);
        free_.clear();
        held = 0;
        return any;
    }
};

// Device memory that a context keeps past a call only to save time: the blocks
// of released peakmaps, the row scratch of peakmap construction, partial tiles
// and rank tables.  Any allocation of the context that finds no room has it
// given back and is tried again.
struct Spare {
    BlockPool blocks;
    DevBuf *rows = nullptr;  // the row scratch, and
    bool rows_busy = false;  // whether a call is using it
    std::vector<DevBuf *> other;
    // frees it all (hipFree waits for the work that uses it); false: there was nothing
    bool give_back() {
        bool any = blocks.trim();
        auto drop = [&](DevBuf *b) {
            any = any || b->ptr;
            b->release();
        };
        if (!rows_busy) drop(rows);
        for (DevBuf *b : other) drop(b);
        return any;
    }
    void *allocate(size_t n) {
        bool full;
        void *p = device_alloc(n, &full);
        return p || !full || !give_back() ? p : device_alloc(n);
    }
    // a block of at least n bytes and its size, or nullptr
    void *block(size_t n, size_t *bytes) {
        if (void *p = blocks.take(n, bytes)) return p;
        *bytes = BlockPool::block_bytes(n);
        return allocate(*bytes);
    }
};

bool DevBuf::allocate(size_t n) { return (ptr = spare ? spare->allocate(n) : device_alloc(n)) != nullptr; }

// Number of a peakmap, never given twice in a process (a copy is another
// peakmap).  What a context keeps for a peakmap past a call is kept by it: a
// released peakmap's address is soon another one's.
struct Serial {
    uint64_t id = next();
    Serial() = default;
    Serial(const Serial &) {}
    Serial &operator=(const Serial &) = delete;
    static uint64_t next() {
        static std::atomic<uint64_t> n{0};
        return ++n;
    }
};

}  // namespace

struct fh_peakmap {
    Serial serial;
    int32_t n_fft = 0;
    int64_t n_peaks = 0;
    double t_fft = 0;
    double t_min = 0, t_max = 0;
    double v_max = 0;
    int32_t k_min = 0, k_max = 0;
    int32_t adjacent = 0;  // 1 if some FFT holds two peaks one natural bin apart
    int32_t max_per_fft = 0;
    // two device blocks: the head, t [N] | v [N][3] | offsets [N+1], and the bins
    void *head = nullptr;
    size_t head_bytes = 0, bins_bytes = 0;  // sizes of the two blocks
    int32_t device = 0;
    int64_t *d_offsets = nullptr;
    int32_t *d_bins = nullptr;
    double *d_t = nullptr;
    double *d_v = nullptr;
    int64_t bytes = 0;
};

// Device and pinned buffers of one in-flight search.  A context owns one;
// each serving lane owns another.
struct Workspace {
    DevBuf sht, Y, Y64, win, wsort, colmax, wq, ws, sky, qctr, part, rank;
    PinnedBuf h_sky;
    hipEvent_t staged = nullptr;  // last copy out of h_sky
    size_t device_bytes() const {
        size_t n = 0;
        for (const DevBuf *b : {&sht, &Y, &Y64, &win, &wsort, &colmax, &wq, &ws, &sky, &qctr, &part, &rank})
            n += b->bytes;
        return n;
    }
    void release() {
        for (DevBuf *b : {&sht, &Y, &Y64, &win, &wsort, &colmax, &wq, &ws, &sky, &qctr, &part, &rank})
            b->release();
        h_sky.release();
        if (staged) (void)hipEventDestroy(staged);
        staged = nullptr;
    }
};

struct fh_ctx {
    int32_t device = 0;
    int32_t n_cu = 256;
    Workspace main_ws;
    Workspace *cur = &main_ws;  // workspace used by the launch sequences
    int32_t window_method = 2;  // peak windows: 0 binary searches, 1 sweep, 2 fused front
    int32_t tile_parts = 0;     // workgroups per tile of small searches: 0 by rule (plan_parts)
    // Doppler correction: 0 exact per peak, 1 per-FFT shift at doppler_fref
    // (<= 0: each map's band centre)
    int32_t doppler_mode = 0;
    double doppler_fref = 0.0;
    DevBuf err;
    // refinement: sliced peakmap (volumes larger than the LDS) and per-call scratch
    DevBuf rf_offsets, rf_bins, rf_first, rf_counts, rf_cands, rf_aux;
    // cleaning: robust-statistic histogram and its rank sum
    DevBuf cl_hist, cl_s2;
    // peakmap construction: row scratch and peaks per FFT; pinned memory for
    // small results, which kernels write in place (a copy of their own cost
    // 8 us), and for staged times and velocities
    DevBuf pm_rows, pm_counts;
    PinnedBuf h_small, h_stage;
    Spare spare;
    // autotuned tile width per problem shape (shared by weighted and
    // unweighted searches: the two kernels differ only in the added value)
    std::map<std::tuple<int, int, int, int>, int> tuned;
    // width of a shape's last search where that was a small launch, which
    // chooses its own (reported by fh_plan_query)
    std::map<std::tuple<int, int, int, int>, int> used;
    // captured searches (fh_options.use_graph), keyed by the peakmap's serial
    // number and every argument and workspace pointer they bake in
    struct GraphEntry {
        std::vector<uint64_t> key;
        hipGraph_t graph = nullptr;
        hipGraphExec_t exec = nullptr;
    };
    std::vector<GraphEntry> graphs;
    // event-based timing (fh_ctx_profile)
    bool profiling = false;
    std::vector<hipEvent_t> ev_pool;
    size_t ev_used = 0;
    struct Span { hipEvent_t a, b; int kind; };
    std::vector<Span> spans;
    int64_t prof_updates = 0;

    fh_ctx() {
        spare.rows = &pm_rows;
        spare.other = {&main_ws.part, &main_ws.rank};
        for (DevBuf *b : {&main_ws.sht, &main_ws.Y, &main_ws.Y64, &main_ws.win, &main_ws.wsort, &main_ws.colmax,
                          &main_ws.wq, &main_ws.ws, &main_ws.sky, &main_ws.qctr, &err, &rf_offsets, &rf_bins,
                          &rf_first, &rf_counts, &rf_cands, &rf_aux, &cl_hist, &cl_s2, &pm_rows, &pm_counts})
            b->spare = &spare;
    }
};

namespace {

// nrb: row blocks the tiles run (the last one also takes `tail` rows past it
// when the grid's last 16-row block holds at most kTailRows rows); nrb_tab:
// every 16-row block of the grid (the shift records cover them all).
struct Plan {
    int W, nrb, nbb, nrbg;
    int nrb_tab, tail;
    int64_t tiles_per_sky;
};

// Spin-down shift tables of one search (see shift_tables), one buffer:
// gwin int64 [N][nrbg][2] | rec uint2 [nrb][N] | step u32 [N][16].
struct ShiftLayout {
    size_t gwin, rec, step, total;
};

ShiftLayout shift_layout(int64_t n_fft, int nrb, int nrbg) {
    auto al = [](size_t x) { return (x + 255) / 256 * 256; };
    ShiftLayout L;
    size_t o = 0;
    L.gwin = o; o += al((size_t)16 * n_fft * nrbg);
    L.rec = o;  o += al((size_t)8 * n_fft * nrb);
    L.step = o; o += al((size_t)4 * kTileRows * n_fft);
    L.total = o;
    return L;
}

// Rows of the grid's last 16-row block when the tiles of the block before
// it take them (at most kTailRows, and a block before it exists), else 0.
int tail_rows(const fh_grid &g) {
    const int nrb = (g.ns + kTileRows - 1) / kTileRows;
    const int r = g.ns - (nrb - 1) * kTileRows;
    return nrb >= 2 && r <= kTailRows ? r : 0;
}

Plan make_plan(const fh_grid &g, int W) {
    Plan p;
    p.W = W;
    p.nrb_tab = (g.ns + kTileRows - 1) / kTileRows;
    // the tail rows are folded only where the wider tile still fits the LDS
    p.tail = tail_rows(g);
    if (p.tail && tile_lds_bytes(W, g.kf, p.tail) > kLdsBytes - kLdsReserve) p.tail = 0;
    p.nrb = p.nrb_tab - (p.tail ? 1 : 0);
    p.nbb = (g.nf + W - 1) / W;
    p.nrbg = (p.nrb + kRowBlocksPerGroup - 1) / kRowBlocksPerGroup;
    p.tiles_per_sky = (int64_t)p.nrb * p.nbb;
    return p;
}

fh_status check_ctx(fh_ctx *ctx) {
    if (!ctx) return fail(FH_E_INVALID, "context is NULL");
    hipError_t e = hipSetDevice(ctx->device);
    if (e != hipSuccess) return fail(FH_E_DEVICE, "hipSetDevice(%d): %s", ctx->device, hipGetErrorString(e));
    return FH_OK;
}

// Checks the times and velocities of pm->n_fft FFTs and takes their extremes
// into pm: one pass without branches, and a second one that names the first
// bad FFT.
fh_status check_times(fh_peakmap *pm, const double *t, const double *v) {
    const int32_t N = pm->n_fft;
    double t_min = t[0], t_max = t[0], v2 = 0.0, sum = 0.0;
    for (int32_t i = 0; i < N; ++i) {
        const double *vi = v + 3 * (int64_t)i;
        const double n2 = vi[0] * vi[0] + vi[1] * vi[1] + vi[2] * vi[2];
        t_min = t[i] < t_min ? t[i] : t_min;
        t_max = t[i] > t_max ? t[i] : t_max;
        v2 = n2 > v2 ? n2 : v2;
        sum += 0.0 * t[i] + 0.0 * n2;  // NaN as soon as a value is not finite
    }
    pm->t_min = t_min;
    pm->t_max = t_max;
    pm->v_max = std::sqrt(v2);
    if (sum == 0.0 && pm->v_max < 1e-2) return FH_OK;
    for (int32_t i = 0; i < N; ++i) {
        if (!std::isfinite(t[i])) return fail(FH_E_INVALID, "t[%d] is not finite", i);
        const double *vi = v + 3 * (int64_t)i;
        if (!std::isfinite(vi[0]) || !std::isfinite(vi[1]) || !std::isfinite(vi[2]))
            return fail(FH_E_INVALID, "v[%d] is not finite", i);
        const double vn = std::sqrt(vi[0] * vi[0] + vi[1] * vi[1] + vi[2] * vi[2]);
        if (vn >= 1e-2) return fail(FH_E_INVALID, "|v[%d]| = %g >= 1e-2", i, vn);
    }
    return FH_OK;
}

// The head block of a peakmap of pm->n_fft FFTs.
bool alloc_head(fh_ctx *ctx, fh_peakmap *pm) {
    const size_t N = (size_t)pm->n_fft;
    pm->device = ctx->device;
    pm->head = ctx->spare.block(32 * N + 8 * (N + 1), &pm->head_bytes);
    if (!pm->head) return false;
    pm->d_t = (double *)pm->head;
    pm->d_v = pm->d_t + N;
    pm->d_offsets = (int64_t *)(pm->d_v + 3 * N);
    return true;
}

bool alloc_bins(fh_ctx *ctx, fh_peakmap *pm, int64_t n) {
    pm->d_bins = (int32_t *)ctx->spare.block(4 * (size_t)std::max<int64_t>(1, n), &pm->bins_bytes);
    return pm->d_bins != nullptr;
}

// A new peakmap with pm's FFTs (times, velocities, metadata) and no blocks.
fh_peakmap *like(const fh_peakmap *pm) {
    fh_peakmap *q = new fh_peakmap(*pm);
    q->head = nullptr;
    q->d_offsets = nullptr;
    q->d_bins = nullptr;
    q->d_t = q->d_v = nullptr;
    q->head_bytes = q->bins_bytes = 0;
    return q;
}

// Times and velocities of up to this many bytes (524 288 FFTs) are staged in
// pinned memory, which stays with the context; more are copied from the caller's.
constexpr size_t kMaxStage = (size_t)16 << 20;

// {total, largest} of a scan's counts, which the scan writes to pinned memory;
// waits for the stream.
hipError_t read_meta(fh_ctx *ctx, hipStream_t st, int64_t *total, int32_t *most) {
    const int64_t *h = (const int64_t *)ctx->h_small.ptr;
    const hipError_t e = hipStreamSynchronize(st);
    if (e == hipSuccess) {
        *total = h[0];
        *most = (int32_t)h[1];
    }
    return e;
}

// Largest spin-down step of one row, in fine bins: |dfdot tau| K_f T_FFT
// (Eq. sdstep) over the FFTs' reference-time offsets tau, plus rounding.
double row_step_bins(const fh_peakmap *pm, const fh_grid *g) {
    const double tau = std::max(std::fabs(pm->t_min - g->t0), std::fabs(pm->t_max - g->t0));
    return std::fabs(g->dfdot) * tau * ((double)g->kf * pm->t_fft) + 1e-6;
}

// Widest tile for the grid: its LDS also holds the tail rows when the grid
// has some, unless that leaves no tile of 64 bins (then they run as a row
// block of their own).
int tile_bins_limit(const fh_peakmap *pm, const fh_grid *g) {
    const int w = max_tile_bins(g->kf, row_step_bins(pm, g), kTileRows + tail_rows(*g));
    return w >= 64 ? w : max_tile_bins(g->kf, row_step_bins(pm, g), kTileRows);
}

fh_status check_grid(const fh_peakmap *pm, const fh_grid *g) {
    if (!pm) return fail(FH_E_INVALID, "peakmap is NULL");
    if (!g) return fail(FH_E_INVALID, "grid is NULL");
    if (g->kf < 1 || g->kf > 64) return fail(FH_E_INVALID, "kf=%d outside 1..64", g->kf);
    if (g->nf < 1 || g->nf > (1 << 22)) return fail(FH_E_INVALID, "nf=%d outside 1..2^22", g->nf);
    if (g->ns < 1 || g->ns > (1 << 15)) return fail(FH_E_INVALID, "ns=%d outside 1..2^15", g->ns);
    if (g->b0 < 0 || g->b0 >= ((int64_t)1 << 28)) return fail(FH_E_INVALID, "b0 outside [0, 2^28)");
    if (!std::isfinite(g->fdot0) || !std::isfinite(g->dfdot) || !std::isfinite(g->t0))
        return fail(FH_E_INVALID, "grid has a non-finite fdot0, dfdot or t0");
    // fixed-point range: |K_f k| < 2^28 and every shift far below 2^62
    if ((int64_t)pm->k_max * g->kf >= ((int64_t)1 << 28))
        return fail(FH_E_INVALID, "K_f * k reaches 2^28 (fixed-point range)");
    const double tau = std::max(std::fabs(pm->t_min - g->t0), std::fabs(pm->t_max - g->t0));
    const double S = (double)g->kf * pm->t_fft;
    const double gmax = (std::fabs(g->fdot0) + std::fabs(g->dfdot) * g->ns) * tau * S;
    if (!(gmax < 1e12)) return fail(FH_E_INVALID, "spin-down shifts exceed the fixed-point range");
    if (pm->max_per_fft >= 65536)
        return fail(FH_E_UNSUPPORTED, "an FFT holds %d peaks; at most 65535 are supported", pm->max_per_fft);
    // a window entry holds its FFT's place in a tile run in 15 bits, and the
    // tiles address a direction's stripe edges with 32-bit byte offsets
    if (wave_ffts(pm->n_fft) >= 32768)
        return fail(FH_E_UNSUPPORTED, "n_fft=%d: a tile run would hold more than 32767 FFTs", pm->n_fft);
    if (y_stride(pm->n_peaks, pm->n_fft) >= ((int64_t)1 << 30))
        return fail(FH_E_UNSUPPORTED, "n_peaks + 16 n_fft reaches 2^30");
    // the tiles address the shift records [row blocks][N] with 31-bit byte offsets
    const int64_t nrb = (int64_t)(g->ns + kTileRows - 1) / kTileRows;
    if ((int64_t)pm->n_fft * nrb >= ((int64_t)1 << 28))
        return fail(FH_E_UNSUPPORTED, "n_fft x row blocks = %lld reaches 2^28", (long long)pm->n_fft * nrb);
    if (max_tile_bins(g->kf, row_step_bins(pm, g), kTileRows) < 64)
        return fail(FH_E_UNSUPPORTED, "spin-down step of %.6g fine bins per row is too large for a tile",
                    row_step_bins(pm, g));
    return FH_OK;
}

fh_status check_sky(const double *n) {
    if (!n) return fail(FH_E_INVALID, "sky vector is NULL");
    for (int k = 0; k < 3; ++k)
        if (!std::isfinite(n[k])) return fail(FH_E_INVALID, "sky vector is not finite");
    const double r = std::sqrt(n[0] * n[0] + n[1] * n[1] + n[2] * n[2]);
    if (std::fabs(r - 1.0) > 1e-9) return fail(FH_E_INVALID, "sky vector is not a unit vector (|n| = %.17g)", r);
    return FH_OK;
}

std::tuple<int, int, int, int> tune_key(const fh_peakmap *pm, const fh_grid *g) {
    return std::make_tuple(pm->n_fft, g->nf, g->ns, g->kf);
}

// Tile width: the requested one (multiple of 64, at most what a 16-row tile
// holds; a width too wide for the tail rows runs them as a row block of
// their own), else the autotuned one, else the widest that also holds the
// tail rows.
int choose_tile_bins(const fh_ctx *ctx, const fh_peakmap *pm, const fh_grid *g, int requested) {
    const int wmax = tile_bins_limit(pm, g);
    if (requested > 0)
        return std::min(((requested + 63) / 64) * 64, max_tile_bins(g->kf, row_step_bins(pm, g), kTileRows));
    auto it = ctx->tuned.find(tune_key(pm, g));
    if (it != ctx->tuned.end()) return it->second;
    // a tile never needs to be wider than the map
    int w = std::min(wmax, ((g->nf + 63) / 64) * 64);
    return std::max(64, w);
}

// kinds of timed spans
enum { kSpanFront = 0, kSpanTiles = 1, kSpanSelect = 2, kSpanGraph = 3 };

hipEvent_t next_event(fh_ctx *ctx) {
    if (ctx->ev_used == ctx->ev_pool.size()) {
        hipEvent_t e;
        if (hipEventCreate(&e) != hipSuccess) return nullptr;
        ctx->ev_pool.push_back(e);
    }
    return ctx->ev_pool[ctx->ev_used++];
}

// Records an event before a group of launches and another after it.
// Profiling span.  A record that fails leaves an unrecorded event, which
// fh_ctx_profile_read then reports through hipEventElapsedTime.
struct Timed {
    fh_ctx *ctx;
    hipStream_t st;
    int kind;
    hipEvent_t a = nullptr;
    Timed(fh_ctx *c, hipStream_t s, int k) : ctx(c), st(s), kind(k) {
        if (ctx->profiling) {
            a = next_event(ctx);
            if (a) (void)hipEventRecord(a, st);
        }
    }
    ~Timed() {
        if (a) {
            hipEvent_t b = next_event(ctx);
            if (b) {
                (void)hipEventRecord(b, st);
                ctx->spans.push_back({a, b, kind});
            }
        }
    }
};

struct ChunkBufs {
    int64_t *gwin;   // spin-down shift tables (ShiftLayout)
    uint2 *rec;
    uint32_t *step, *base;
    uint32_t *Y;   // low words of the stripe edges (what the tiles read)
    int64_t *Y64;  // full stripe edges, only for the unfused window methods
    uint32_t *win;  // packed windows before the sort
    int2 *wsort;
    unsigned long long *colmax;
    uint32_t *wq;
    WeightStats *ws;
    double *sky;
    int32_t *qctr, *err;
    uint32_t *part = nullptr;  // partial tiles of searches with few tiles
    size_t part_bytes = 0;
    uint2 *rank = nullptr;  // peaks' rank table of a search of many directions
};

// Cost model of the tiles of small launches, in us, fitted to timed launches of
// one and five directions at T_FFT = 1024 .. 8192 s, W = 256 .. 2496 and 1 .. 16
// parts (single rounds).  Fitted to tiles whose blocks took more set-up; timed
// against the present ones it is within 40 % (20 % rms), and a refit to 6 % rms
// chose widths that moved calls by -2 to +3 % with no gain over all of them.
//   a tile's clearing, first loads and output: 4.2 + 2.5 per 1000 columns;
//   its FFTs: 3.05 ns each (a quarter of a block's window, term and pattern
//   set-up) and 0.43 ns per peak of the FFT's window, which is wider than the
//   tile by the rows' spread; a third more where the tile has tail rows.
double tile_fixed_us(int W) { return 4.2 + 2.5e-3 * W; }

double tile_accum_us(const fh_peakmap *pm, const fh_grid *g, const Plan &p) {
    const double density = (double)pm->n_peaks / pm->n_fft / ((double)g->kf * (pm->k_max - pm->k_min + 1));
    const double spread = 0.5 * row_step_bins(pm, g) * std::min(kTileRows * kRowBlocksPerGroup, g->ns);
    const double us = pm->n_fft * (3.05e-3 + 0.43e-3 * density * (p.W + g->kf + spread));
    return p.tail ? us * (1.0 + 0.33 / p.nrb) : us;
}

// n_tiles tiles, each shared by `parts` workgroups: rounds over the CUs, and
// the partial tiles written and read by the merge at 2.6 TB/s.
double tiles_us(const fh_ctx *ctx, const fh_peakmap *pm, const fh_grid *g, const Plan &p, int64_t n_tiles, int parts) {
    const double rounds = (double)((n_tiles * parts + ctx->n_cu - 1) / ctx->n_cu);
    const double us = rounds * (tile_fixed_us(p.W) + tile_accum_us(pm, g, p) / parts);
    return parts == 1 ? us
                      : us + 6.0 + 4.0e-6 * (double)part_words(p.W, g->kf, p.tail) * (double)(n_tiles * parts) / 2.6;
}

// "tile_parts" asks for at most this many rounds of workgroups over the CUs: it
// is for searches with few tiles, and a partial tile takes up to 160 KB (335 MB
// in all on 256 CUs).
constexpr int64_t kForcedRounds = 8;

// Workgroups that share each of n_tiles tiles (each accumulates every
// parts-th block of FFTs; a merge adds the partial tiles): more than one only
// where the launch leaves CUs idle and the model finds the shorter
// accumulation worth the partial tiles' way through memory.  One direction of
// 31 rows at T_FFT = 2048 s (32 tiles of 1280 bins): 84 us by one workgroup
// each, 29 us by eight.
int plan_parts(const fh_ctx *ctx, const fh_peakmap *pm, const fh_grid *g, const Plan &p, int64_t n_tiles) {
    // a part keeps one round of the ring of blocks for each of its waves
    const int64_t blocks = (int64_t)kTileWaves * (wave_ffts(pm->n_fft) / 4);
    const int64_t most = std::min<int64_t>(64, std::max<int64_t>(1, blocks / (3 * kTileWaves)));
    if (n_tiles < 1 || n_tiles > 65535) return 1;
    if (ctx->tile_parts > 0)
        return (int)std::max<int64_t>(1, std::min<int64_t>({ctx->tile_parts, most, kForcedRounds * ctx->n_cu / n_tiles}));
    int best = 1;
    double best_us = tiles_us(ctx, pm, g, p, n_tiles, 1);
    for (int64_t s = 2; s <= most && s * n_tiles <= 2 * ctx->n_cu; ++s) {
        const double us = tiles_us(ctx, pm, g, p, n_tiles, (int)s);
        if (us < best_us) {
            best_us = us;
            best = (int)s;
        }
    }
    return best;
}

// Launches of at most this many rounds of tiles over the CUs choose their
// width by the model: there the last, partly empty round and the parts decide
// (a width tuned on many directions left a map of 264 tiles two rounds of 66 us
// on 256 CUs).  Longer launches are tuned by timing.
constexpr int kSmallRounds = 6;

bool small_launch(const fh_ctx *ctx, const fh_peakmap *pm, const fh_grid *g, int n_dir) {
    const Plan p = make_plan(*g, std::max(64, std::min(tile_bins_limit(pm, g), ((g->nf + 63) / 64) * 64)));
    return p.tiles_per_sky * n_dir <= (int64_t)kSmallRounds * ctx->n_cu;
}

// Tile width of a small launch of n_dir directions: the band cut evenly into
// n blocks, for every n up to tiles of 192 bins; besides the tiles' cost, a
// window entry of the front and the window sort takes 12 ps.
int small_tile_bins(const fh_ctx *ctx, const fh_peakmap *pm, const fh_grid *g, int n_dir) {
    const int wmax = max_tile_bins(g->kf, row_step_bins(pm, g), kTileRows);
    int best_w = 0;
    double best_us = 0.0;
    for (int n = std::max(1, (g->nf + wmax - 1) / wmax); ; n += 1 + n / 16) {
        const int w = std::max(64, ((g->nf + n - 1) / n + 63) / 64 * 64);
        const Plan p = make_plan(*g, w);
        const int64_t n_tiles = p.tiles_per_sky * n_dir;
        const double us = tiles_us(ctx, pm, g, p, n_tiles, plan_parts(ctx, pm, g, p, n_tiles)) +
                          12e-6 * (double)p.nrbg * p.nbb * win_stride(pm->n_fft) * n_dir;
        if (best_w == 0 || us < best_us) {
            best_us = us;
            best_w = w;
        }
        if (w <= 192) break;
    }
    return best_w;
}

size_t parts_bytes(const fh_ctx *ctx, const fh_peakmap *pm, const fh_grid *g, const Plan &p, int slots) {
    const int64_t n_tiles = p.tiles_per_sky * slots;
    const int parts = plan_parts(ctx, pm, g, p, n_tiles);
    return parts > 1 ? (size_t)4 * part_words(p.W, g->kf, p.tail) * parts * n_tiles : 0;
}

// bytes for the partial tiles of every launch of n_sky directions in chunks
size_t search_parts_bytes(const fh_ctx *ctx, const fh_peakmap *pm, const fh_grid *g, const Plan &p, int chunk,
                          int n_sky) {
    const int last = n_sky % chunk;
    return std::max(n_sky >= chunk ? parts_bytes(ctx, pm, g, p, chunk) : 0,
                    last ? parts_bytes(ctx, pm, g, p, last) : 0);
}

// The parts of a launch of n_tiles tiles that fit the buffers it was given.
void set_parts(const fh_ctx *ctx, const fh_peakmap *pm, const fh_grid *g, const Plan &p, int64_t n_tiles,
               const ChunkBufs &b, TileArgs &a) {
    a.parts = plan_parts(ctx, pm, g, p, n_tiles);
    a.part_stride = part_words(p.W, g->kf, p.tail);
    a.part = b.part;
    if ((size_t)4 * a.part_stride * a.parts * n_tiles > b.part_bytes) a.parts = 1;
}

// Tile width of a launch sequence of n_dir directions.
int search_tile_bins(const fh_ctx *ctx, const fh_peakmap *pm, const fh_grid *g, int n_dir) {
    return small_launch(ctx, pm, g, n_dir) ? small_tile_bins(ctx, pm, g, n_dir) : choose_tile_bins(ctx, pm, g, 0);
}

// the unfused window methods (chosen, or forced when one FFT's edges do not
// fit the fused front's LDS) search the full 64-bit edges in device memory
bool needs_full_edges(const fh_ctx *ctx, const fh_peakmap *pm) {
    return !(ctx->window_method == 2 && front_ffts_per_block(pm->max_per_fft) > 0);
}

// Bytes of the rank table with which a launch of `slots` directions finds its
// windows (k_front_rank), 0 when it searches them (k_front): few directions do
// not repay the table, and wide, sparsely filled bands would make it larger
// than four directions' stripe edges.  Whole calls with tiles of 1280 bins,
// windows searched for -> from the table, in us: 6300 FFTs of 4096 s, 584 rows:
// 1 direction 317 -> 323, 2: 581 -> 575, 3: 726 -> 725, 8: 1790 -> 1771; 25 144
// of 1024 s, 17 rows: 1: 98 -> 109, 3: 117 -> 128, 8: 185 -> 191 (and 97: 463 ->
// 334 of front); 3143 of 8192 s, 118 rows: 1: 112 -> 121, 3: 222 -> 228, 8: 473
// -> 472.  Where the lines cross lies between 2 directions and some ten, by the
// rows; at 3 no shape loses more than 11 us.
constexpr int kRankMinDirs = 3;

// Row blocks up to which the tiles of such a launch compute the stripe edges
// from the natural bins instead of reading them.  Each peak's edge is then
// computed once per row block, and the front neither computes nor stores it:
// with few row blocks what the front saves (4 bytes per peak and direction
// written) is more than the tiles spend on ten FP64 instructions per block (17
// rows, 128 directions: front 793 -> 233 us, tiles 942 -> 949).  Whole calls of 128
// directions (97 of 17 rows, 64 of 147), edges read -> computed: 1 row block
// (17 rows) 1170 -> 815 us, weighted 1805 -> 1352; 2 (31 rows) 1654 -> 1418;
// 4 (60 rows) 2692 -> 2591; 8 (118 rows) 5218 -> 5353; 10 (147 rows) 3498 ->
// 3626.
constexpr int kTermRowBlocks = 4;

size_t rank_bytes(const fh_ctx *ctx, const fh_peakmap *pm, const Plan &p, int slots) {
    if (slots < kRankMinDirs || needs_full_edges(ctx, pm) || !rank_front_fits(pm->k_min, pm->k_max, p.nrbg)) return 0;
    const int64_t bytes = 8 * (int64_t)rank_words(pm->k_min, pm->k_max) * pm->n_fft;
    return bytes <= 16 * y_stride(pm->n_peaks, pm->n_fft) ? (size_t)bytes : 0;
}

// device bytes of the stripe edges of one direction
int64_t edge_bytes_per_sky(const fh_ctx *ctx, const fh_peakmap *pm) {
    return (needs_full_edges(ctx, pm) ? 12 : 4) * y_stride(pm->n_peaks, pm->n_fft);
}

// Calls that use the context's buffers are not captured by the caller: a
// later call may move the buffers under the graph (the static map is made
// for that).
fh_status refuse_capture(hipStream_t st) {
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    if (st && hipStreamIsCapturing(st, &cs) == hipSuccess && cs != hipStreamCaptureStatusNone)
        return fail(FH_E_DEVICE, "the stream is being captured");
    return FH_OK;
}

fh_status ensure_workspace(fh_ctx *ctx, const fh_peakmap *pm, const fh_grid *g, const Plan &p,
                           int slots, int n_sky, bool weighted, hipStream_t st, ChunkBufs &b) {
    const int64_t N = pm->n_fft;
    fh_status s;
    if ((s = refuse_capture(st))) return s;
    const ShiftLayout sl = shift_layout(N, p.nrb_tab, p.nrbg);
    if ((s = ctx->cur->sht.ensure(sl.total, st))) return s;
    if ((s = ctx->cur->Y.ensure((size_t)4 * y_stride(pm->n_peaks, pm->n_fft) * slots, st))) return s;
    if (needs_full_edges(ctx, pm) &&
        (s = ctx->cur->Y64.ensure((size_t)8 * y_stride(pm->n_peaks, pm->n_fft) * slots, st)))
        return s;
    const size_t n_win = (size_t)slots * p.nrbg * p.nbb * win_stride(N);
    if ((s = ctx->cur->win.ensure(4 * (n_win + win_stride(N)), st))) return s;
    if ((s = ctx->cur->wsort.ensure((size_t)8 * slots * p.nrbg * p.nbb * win_stride(N), st))) return s;
    if ((s = ctx->cur->colmax.ensure((size_t)8 * slots * g->nf, st))) return s;
    if ((s = ctx->cur->wq.ensure(weighted ? (size_t)4 * slots * N : 4, st))) return s;
    if ((s = ctx->cur->ws.ensure(sizeof(WeightStats) * (size_t)slots, st))) return s;
    if ((s = ctx->cur->sky.ensure((size_t)24 * n_sky, st))) return s;
    if ((s = ctx->cur->qctr.ensure(4 * kXcds, st))) return s;
    if ((s = ctx->err.ensure(4, st))) return s;
    // Partial tiles and the rank table only save time: where there is no room
    // for them, the tiles are not shared and the windows are searched for.
    const size_t pb = search_parts_bytes(ctx, pm, g, p, slots, n_sky);
    if (pb && (s = ctx->cur->part.ensure(pb, st)) && s != FH_E_NOMEM) return s;
    b.part = (uint32_t *)ctx->cur->part.ptr;
    b.part_bytes = ctx->cur->part.bytes;
    const size_t rb = rank_bytes(ctx, pm, p, slots);
    if (rb && (s = ctx->cur->rank.ensure(rb, st)) && s != FH_E_NOMEM) return s;
    b.rank = rb ? (uint2 *)ctx->cur->rank.ptr : nullptr;
    b.gwin = reinterpret_cast<int64_t *>((char *)ctx->cur->sht.ptr + sl.gwin);
    b.rec = reinterpret_cast<uint2 *>((char *)ctx->cur->sht.ptr + sl.rec);
    b.step = reinterpret_cast<uint32_t *>((char *)ctx->cur->sht.ptr + sl.step);
    b.Y = (uint32_t *)ctx->cur->Y.ptr;
    b.Y64 = (int64_t *)ctx->cur->Y64.ptr;
    b.win = (uint32_t *)ctx->cur->win.ptr;
    b.base = b.win + n_win;
    b.wsort = (int2 *)ctx->cur->wsort.ptr;
    b.colmax = (unsigned long long *)ctx->cur->colmax.ptr;
    b.wq = (uint32_t *)ctx->cur->wq.ptr;
    b.ws = (WeightStats *)ctx->cur->ws.ptr;
    b.sky = (double *)ctx->cur->sky.ptr;
    b.qctr = (int32_t *)ctx->cur->qctr.ptr;
    b.err = (int32_t *)ctx->err.ptr;
    return FH_OK;
}

TileArgs tile_args(const fh_peakmap *pm, const fh_grid *g, const Plan &p, int slots,
                   const ChunkBufs &b, bool weighted, int ws_stride) {
    TileArgs a{};
    a.n_fft = pm->n_fft;
    a.n_peaks = pm->n_peaks;
    a.kf = g->kf;
    a.nf = g->nf;
    a.ns = g->ns;
    a.W = p.W;
    a.nrb = p.nrb;
    a.tail = p.tail;
    a.nbb = p.nbb;
    a.nrbg = p.nrbg;
    a.n_slots = slots;
    a.Y = b.Y;
    a.win = b.wsort;
    a.rec = b.rec;
    a.step = b.step;
    a.wq = weighted ? b.wq : nullptr;
    a.ws = weighted ? b.ws : nullptr;
    a.ws_stride = ws_stride;
    a.colmax = b.colmax;
    a.queue_ctr = b.qctr;
    return a;
}

// The workspace's pinned staging buffer, grown to n bytes and free for reuse
// (the copy that last read it has run).
fh_status stage_buffer(Workspace *w, size_t n, hipStream_t st, char **out) {
    if (!w->staged && hipEventCreateWithFlags(&w->staged, hipEventDisableTiming) != hipSuccess) {
        w->staged = nullptr;
        return fail(FH_E_DEVICE, "hipEventCreate failed");
    }
    HIP_OK(hipEventSynchronize(w->staged));
    const fh_status s = w->h_sky.ensure(n, st);
    *out = (char *)w->h_sky.ptr;
    return s;
}

// Copy n staged bytes to the device.
fh_status stage_copy(Workspace *w, void *dst, size_t n, hipStream_t st) {
    HIP_OK(hipMemcpyAsync(dst, w->h_sky.ptr, n, hipMemcpyHostToDevice, st));
    HIP_OK(hipEventRecord(w->staged, st));
    return FH_OK;
}

// Directions of a call, handed to the launches: `arg` when few enough to
// travel as kernel arguments of the first setup, else already in device
// memory.
struct SkyDirs {
    const double *arg = nullptr;
    int n = 0;
};

// Directions of a call whose first launch is not a graph replay.
fh_status upload_sky(fh_ctx *ctx, const double *sky_host, int n_sky, const ChunkBufs &b, hipStream_t st,
                     SkyDirs *dirs) {
    *dirs = {};
    if (n_sky <= kArgSky) {
        dirs->arg = sky_host;
        dirs->n = n_sky;
        return FH_OK;
    }
    char *h;
    const fh_status s = stage_buffer(ctx->cur, (size_t)24 * n_sky, st, &h);
    if (s) return s;
    std::memcpy(h, sky_host, (size_t)24 * n_sky);
    return stage_copy(ctx->cur, b.sky, (size_t)24 * n_sky, st);
}

// Shared front half of every path: shifts, weights, stripe edges, windows.
// Reference of the per-FFT shift variant, in fine bins: (K_f T_FFT) f_ref.
double shift_reference_bins(const fh_ctx *ctx, const fh_peakmap *pm, const fh_grid *g) {
    const double f_ref = ctx->doppler_fref > 0
                             ? ctx->doppler_fref
                             : ((double)g->b0 + 0.5 * (double)g->nf) / ((double)g->kf * pm->t_fft);
    return ((double)g->kf * pm->t_fft) * f_ref;
}

fh_status enqueue_front(fh_ctx *ctx, const fh_peakmap *pm, const fh_grid *g, const Plan &p,
                        int slots, const double *d_sky, const SkyDirs &dirs, const float *d_w, int w_stride,
                        int64_t n_colmax, bool first, const ChunkBufs &b, hipStream_t st, bool terms_only = false) {
    Timed timed(ctx, st, kSpanFront);
    const bool weighted = d_w != nullptr;
    SetupArgs a{};
    a.n_fft = pm->n_fft;
    a.nrb = p.nrb_tab;
    a.nrb_run = p.nrb;
    a.ns = g->ns;
    a.t = pm->d_t;
    a.t0 = g->t0;
    a.S = ((double)g->kf * pm->t_fft) * 65536.0;
    a.fdot0 = g->fdot0;
    a.dfdot = g->dfdot;
    a.gwin = b.gwin;
    a.rec = b.rec;
    a.step = b.step;
    a.base = b.base;
    a.y_pad = terms_only ? 0 : kYPad;
    a.offsets = pm->d_offsets;
    a.err = b.err;
    a.n_vec = weighted ? (w_stride == 0 ? 1 : slots) : 0;
    a.w_stride = w_stride;
    a.mult = pm->adjacent ? 2 : 1;
    a.w = d_w;
    a.ws = b.ws;
    a.colmax = b.colmax;
    a.n_colmax = n_colmax;
    a.qctr = b.qctr;
    a.n_sky = dirs.n;
    a.sky = b.sky;
    if (dirs.n) std::memcpy(a.sky_arg, dirs.arg, (size_t)24 * dirs.n);
    const int F = ctx->window_method == 2 ? front_ffts_per_block(pm->max_per_fft) : 0;
    const int32_t sm = ctx->doppler_mode;
    const double q = sm ? shift_reference_bins(ctx, pm, g) : 0.0;
    const int ws_stride = w_stride == 0 ? 0 : 1;
    WeightArgs wa{};  // the front writes the fixed-point weights itself, or leaves them to the sort
    if (b.rank && rank_bytes(ctx, pm, p, slots) > 0) {
        // (the first chunk is the largest; later ones find its table)
        HIP_OK(launch_setup(a, pm->d_bins, pm->k_min, pm->k_max, first ? b.rank : nullptr, st));
        HIP_OK(launch_front_rank(pm->n_fft, pm->n_peaks, pm->d_offsets, pm->d_bins, pm->d_v, d_sky, slots, g->kf, g->b0,
                                 b.gwin, b.Y, d_w, w_stride, b.ws, ws_stride, b.wq, p.nrbg, p.nbb, p.W, pm->k_min,
                                 pm->k_max, b.rank, b.win, sm, q, terms_only, st));
    } else if (F > 0) {
        FrontArgs r{};
        r.n_peaks = pm->n_peaks;
        r.b0 = g->b0;
        r.bins = pm->d_bins;
        r.v = pm->d_v;
        r.sky = d_sky;
        r.n_slots = slots;
        r.kf = g->kf;
        r.nrbg = p.nrbg;
        r.nbb = p.nbb;
        r.W = p.W;
        r.F = F;
        r.shift_mode = sm;
        r.q = q;
        r.Y = b.Y;
        r.win = b.win;
        HIP_OK(launch_setup_front(a, r, pm->max_per_fft, st));
        if (weighted) wa = {d_w, b.ws, b.wq, w_stride, ws_stride};
    } else {
        HIP_OK(launch_setup(a, nullptr, 0, 0, nullptr, st));
        HIP_OK(launch_prep(pm->n_fft, pm->n_peaks, pm->d_offsets, pm->d_bins, pm->d_v, d_sky, slots, g->kf, g->b0, b.Y64,
                           d_w, w_stride, b.ws, ws_stride, b.wq, b.Y, sm, q, st));
        HIP_OK(launch_windows(pm->n_fft, pm->d_offsets, b.Y64, pm->n_peaks, b.gwin, p.nrbg, p.nbb, p.W, g->kf, slots,
                              b.win, ctx->window_method == 0 ? 0 : 1, st));
    }
    HIP_OK(launch_sort_windows(pm->n_fft, p.nrbg, p.nbb, slots, b.win, b.base, b.wsort, wa, st));
    return FH_OK;
}

fh_status enqueue_map(fh_ctx *ctx, const fh_peakmap *pm, const fh_grid *g, const Plan &p, const double *nhat,
                      const float *d_w, const ChunkBufs &b, void *out, hipStream_t st);

fh_status hough_map_common(fh_ctx *ctx, const fh_peakmap *pm, const double nhat[3],
                           const float *d_w, const fh_grid *g, void *out, void *stream) {
    fh_status s;
    if ((s = check_ctx(ctx))) return s;
    if ((s = check_grid(pm, g))) return s;
    if ((s = check_sky(nhat))) return s;
    if (!out) return fail(FH_E_INVALID, "output map pointer is NULL");
    hipStream_t st = (hipStream_t)stream;
    const bool weighted = d_w != nullptr;
    const Plan p = make_plan(*g, search_tile_bins(ctx, pm, g, 1));
    ChunkBufs b;
    if ((s = ensure_workspace(ctx, pm, g, p, 1, 1, weighted, st, b))) return s;
    return enqueue_map(ctx, pm, g, p, nhat, d_w, b, out, st);
}

// Front and tiles of one direction's map.
fh_status enqueue_map(fh_ctx *ctx, const fh_peakmap *pm, const fh_grid *g, const Plan &p, const double *nhat,
                      const float *d_w, const ChunkBufs &b, void *out, hipStream_t st) {
    fh_status s;
    const bool weighted = d_w != nullptr;
    if ((s = enqueue_front(ctx, pm, g, p, 1, b.sky, {nhat, 1}, d_w, 0, 0, true, b, st))) return s;
    TileArgs a = tile_args(pm, g, p, 1, b, weighted, 0);
    a.map_i32 = weighted ? nullptr : (int32_t *)out;
    a.map_f32 = weighted ? (float *)out : nullptr;
    a.tile_base = 0;
    {
        Timed timed(ctx, st, kSpanTiles);
        set_parts(ctx, pm, g, p, p.tiles_per_sky, b, a);
        HIP_OK(launch_tiles(a, weighted, true, false, (int32_t)p.tiles_per_sky, 0, st));
    }
    if (ctx->profiling) ctx->prof_updates += pm->n_peaks * (int64_t)g->ns;
    return FH_OK;
}

// chunk: as many directions as a 48 GiB workspace holds (a sixth of the
// MI355X's HBM), at most 4096: fewer launches, more tiles per persistent
// launch (the 256 Hz batch of 1024 directions, 27 GB, is one launch)
// Directions whose tiles one launch can number (tile ids are 32-bit).
int64_t chunk_by_tiles(const Plan &p) {
    return std::max<int64_t>(1, (((int64_t)1 << 31) - 1) / std::max<int64_t>(1, p.tiles_per_sky));
}

int default_chunk(const fh_ctx *ctx, const fh_peakmap *pm, const fh_grid *g, const Plan &p, int requested) {
    if (requested > 0) return (int)std::min<int64_t>(requested, chunk_by_tiles(p));
    const int64_t per_sky = edge_bytes_per_sky(ctx, pm) + 16 * (int64_t)p.nrbg * p.nbb * win_stride(pm->n_fft) + 8 * (int64_t)g->nf;
    const int64_t by_mem = std::max<int64_t>(1, ((int64_t)48 << 30) / std::max<int64_t>(1, per_sky));
    return (int)std::min<int64_t>(std::min<int64_t>(by_mem, 4096), chunk_by_tiles(p));
}

// Enqueue the search of n_sky directions (dirs, or already uploaded to b.sky)
// in chunks of `chunk`; sel == nullptr skips candidate selection.
// Optional per-bin column maxima of every direction, decoded: value [n_sky][nf]
// and smallest row holding it [n_sky][nf].
struct ColmaxOut {
    float *value = nullptr;
    int32_t *row = nullptr;
};

fh_status run_search(fh_ctx *ctx, const fh_peakmap *pm, const fh_grid *g, const Plan &p, int chunk,
                     int n_sky, const float *d_w, int w_stride, int schedule, const fh_select *sel,
                     fh_candidate *d_out, const ChunkBufs &b, hipStream_t st, const SkyDirs &dirs,
                     ColmaxOut cm_out = {}) {
    fh_status s;
    const bool weighted = d_w != nullptr;
    for (int32_t base = 0; base < n_sky; base += chunk) {
        const int slots = std::min(chunk, n_sky - base);
        const float *w = weighted ? d_w + (w_stride ? (int64_t)base * w_stride : 0) : nullptr;
        TileArgs a = tile_args(pm, g, p, slots, b, weighted, w_stride == 0 ? 0 : 1);
        const int64_t n_tiles = p.tiles_per_sky * slots;
        set_parts(ctx, pm, g, p, n_tiles, b, a);
        // A single round of tiles is dispatched by the hardware: a persistent
        // workgroup claims its next tile when it starts one, so early ones
        // would take two tiles and late ones none (240 tiles of a 4096 s band:
        // 165 us, against 90 us).
        const bool persistent = schedule == FH_SCHED_PERSISTENT && a.parts == 1 && n_tiles > ctx->n_cu;
        const bool terms_only = persistent && p.nrb <= kTermRowBlocks && b.rank &&
                                rank_bytes(ctx, pm, p, slots) > 0 && pm->n_peaks < ((int64_t)1 << 29);
        if (terms_only) a.bins = pm->d_bins;
        if ((s = enqueue_front(ctx, pm, g, p, slots, b.sky + 3 * (int64_t)base, base == 0 ? dirs : SkyDirs{}, w,
                               w_stride, (int64_t)slots * g->nf, base == 0, b, st, terms_only)))
            return s;
        {
            const int grid_blocks = (int)std::min<int64_t>(ctx->n_cu, n_tiles);
            Timed timed(ctx, st, kSpanTiles);
            HIP_OK(launch_tiles(a, weighted, false, persistent, (int32_t)n_tiles, grid_blocks, st));
        }
        if (ctx->profiling) ctx->prof_updates += pm->n_peaks * (int64_t)g->ns * slots;
        if (cm_out.value)
            HIP_OK(launch_colmax_decode(b.colmax, g->nf, slots, weighted ? b.ws : nullptr,
                                        weighted ? (w_stride == 0 ? 0 : 1) : 0,
                                        cm_out.value + (int64_t)base * g->nf, cm_out.row + (int64_t)base * g->nf,
                                        st));
        if (sel) {
            Timed timed_sel(ctx, st, kSpanSelect);
            HIP_OK(launch_select(b.colmax, g->nf, slots, *sel, base, pm->n_fft, weighted ? b.ws : nullptr,
                                 weighted ? (w_stride == 0 ? 0 : 1) : 0, d_out, st));
        }
    }
    return FH_OK;
}

// Tile-width autotuner: times the persistent search of a sample of the
// directions for each candidate width (multiples of 64 up to what the LDS
// holds) and keeps the fastest per problem shape and weighting.  With tail
// rows, the widest 16-row tile (too wide to hold them, so they run as a row
// block of their own) is a candidate too.
fh_status autotune(fh_ctx *ctx, const fh_peakmap *pm, const fh_grid *g, int n_sky,
                   const double *sky, const float *d_w, int w_stride, hipStream_t st) {
    const bool weighted = d_w != nullptr;
    const int wmax = tile_bins_limit(pm, g);
    const int wmap = std::max(64, ((g->nf + 63) / 64) * 64);  // a tile never needs to be wider than the map
    const int wcap = std::min(wmax, wmap);
    std::vector<int> cands;
    for (int w : {512, 832, 1280, 1792, 2176})
        if (w < wcap) cands.push_back(w);
    cands.push_back(wcap);
    const int w16 = std::min(max_tile_bins(g->kf, row_step_bins(pm, g), kTileRows), wmap);
    if (w16 > wcap) cands.push_back(w16);
    const int sample = std::min(n_sky, 128);
    // (the width outlives the "tile_parts" option: it is tuned without)
    struct Options {
        fh_ctx *ctx;
        const int32_t parts;
        ~Options() { ctx->tile_parts = parts; }
    } options{ctx, ctx->tile_parts};
    ctx->tile_parts = 0;
    const bool was = ctx->profiling;
    ctx->profiling = false;
    hipEvent_t e0, e1;
    HIP_OK(hipEventCreate(&e0));
    HIP_OK(hipEventCreate(&e1));
    int best_w = wcap;
    float best_ms = 0.f;
    fh_status s = FH_OK;
    for (int w : cands) {
        const Plan p = make_plan(*g, w);
        ChunkBufs b;
        if ((s = ensure_workspace(ctx, pm, g, p, sample, n_sky, weighted, st, b))) break;
        SkyDirs dirs;
        if ((s = upload_sky(ctx, sky, sample, b, st, &dirs))) break;
        float ms = 0.f;
        for (int rep = 0; rep < 2 && s == FH_OK; ++rep) {
            if (hipEventRecord(e0, st) != hipSuccess) { s = fail(FH_E_DEVICE, "hipEventRecord"); break; }
            s = run_search(ctx, pm, g, p, sample, sample, d_w, w_stride, FH_SCHED_PERSISTENT, nullptr,
                           nullptr, b, st, dirs);
            if (s) break;
            if (hipEventRecord(e1, st) != hipSuccess || hipEventSynchronize(e1) != hipSuccess ||
                hipEventElapsedTime(&ms, e0, e1) != hipSuccess) {
                s = fail(FH_E_DEVICE, "autotune timing failed");
                break;
            }
        }
        if (s) break;
        if (best_ms == 0.f || ms < best_ms) {
            best_ms = ms;
            best_w = w;
        }
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    ctx->profiling = was;
    if (s) return s;
    ctx->tuned[tune_key(pm, g)] = best_w;
    return FH_OK;
}

// Tile width of a search: the requested one, by the model where a launch has
// few tiles, else the autotuned one (tuning it first if need be).
fh_status plan_width(fh_ctx *ctx, const fh_peakmap *pm, const fh_grid *g, int n_sky, const double *sky,
                     const float *d_w, int w_stride, const fh_options &o, hipStream_t st, int *width) {
    if (o.tile_bins > 0) {
        *width = choose_tile_bins(ctx, pm, g, o.tile_bins);
        return FH_OK;
    }
    // directions per launch (a plain schedule runs them one by one)
    const int dirs = o.schedule == FH_SCHED_PLAIN ? 1 : o.sky_chunk > 0 ? std::min(o.sky_chunk, n_sky) : n_sky;
    if (small_launch(ctx, pm, g, dirs)) {
        *width = small_tile_bins(ctx, pm, g, dirs);
        ctx->used[tune_key(pm, g)] = *width;
        return FH_OK;
    }
    fh_status s = FH_OK;
    if (ctx->tuned.find(tune_key(pm, g)) == ctx->tuned.end())
        s = autotune(ctx, pm, g, n_sky, sky, d_w, w_stride, st);
    *width = choose_tile_bins(ctx, pm, g, 0);
    ctx->used.erase(tune_key(pm, g));
    return s;
}

}  // namespace

// peakmap cleaning helpers
namespace {

fh_status check_gross(const fh_gross *geo) {
    if (!geo) return fail(FH_E_INVALID, "gross geometry is NULL");
    if (!(geo->dt_h > 0) || !(geo->df_h > 0) || !std::isfinite(geo->dt_h) || !std::isfinite(geo->df_h) ||
        !std::isfinite(geo->t_origin))
        return fail(FH_E_INVALID, "gross cells need finite dt_h > 0, df_h > 0 and t_origin");
    if (geo->n_t < 1 || geo->n_f < 1 || (int64_t)geo->n_t * geo->n_f > ((int64_t)1 << 31))
        return fail(FH_E_INVALID, "gross histogram of %d x %d cells", geo->n_t, geo->n_f);
    return FH_OK;
}

// A new peakmap holding the peaks of pm that `spec` keeps.
fh_status filter_peakmap(fh_ctx *ctx, const fh_peakmap *pm, const FilterSpec &spec, hipStream_t st,
                         fh_peakmap **out) {
    fh_status s;
    const int32_t N = pm->n_fft;
    if ((s = ctx->rf_counts.ensure(4 * (size_t)std::max(1, N), st))) return s;
    fh_peakmap *q = like(pm);
    if (!alloc_head(ctx, q)) {
        fh_peakmap_release(ctx, q);
        return fail(FH_E_NOMEM, "device allocation for the cleaned peakmap failed");
    }
    // (the count also copies the times and velocities)
    hipError_t e = launch_filter(N, pm->d_offsets, pm->d_bins, spec, pm->d_t, q->d_t, (int32_t *)ctx->rf_counts.ptr,
                                 q->d_offsets, nullptr, 0, (int64_t *)ctx->h_small.ptr, st);
    int64_t P = 0;
    if (e == hipSuccess) e = read_meta(ctx, st, &P, &q->max_per_fft);
    if (e == hipSuccess && !alloc_bins(ctx, q, P)) e = hipErrorOutOfMemory;
    if (e == hipSuccess)
        e = launch_filter(N, pm->d_offsets, pm->d_bins, spec, nullptr, nullptr, nullptr, q->d_offsets, q->d_bins, 1,
                          nullptr, st);
    if (e != hipSuccess) {
        fh_peakmap_release(ctx, q);
        return fail(e == hipErrorOutOfMemory ? FH_E_NOMEM : FH_E_DEVICE, "filtering the peakmap failed: %s",
                    hipGetErrorString(e));
    }
    q->n_peaks = P;
    q->bytes = (int64_t)(8 * (size_t)(N + 1) + 4 * (size_t)std::max<int64_t>(1, P) + 32 * (size_t)N);
    *out = q;
    return FH_OK;
}

}  // namespace

extern "C" {

const char *fh_version(void) { return "fh-mi355x 0.1 (gfx950)"; }

const char *fh_last_error(void) { return g_err.c_str(); }

fh_status fh_ctx_create(int32_t device, fh_ctx **out) {
    if (!out) return fail(FH_E_INVALID, "out is NULL");
    *out = nullptr;
    int n = 0;
    hipError_t e = hipGetDeviceCount(&n);
    if (e != hipSuccess || n == 0) return fail(FH_E_DEVICE, "no HIP device available");
    if (device < 0 || device >= n) return fail(FH_E_INVALID, "device %d not in [0, %d)", device, n);
    HIP_OK(hipSetDevice(device));
    hipDeviceProp_t prop;
    HIP_OK(hipGetDeviceProperties(&prop, device));
    if (std::strncmp(prop.gcnArchName, "gfx950", 6) != 0)
        return fail(FH_E_UNSUPPORTED, "device %d is %s; this library is built for gfx950", device, prop.gcnArchName);
    HIP_OK(init_kernel_attributes());
    fh_status ss = scratch_init(device);
    if (ss) return ss;
    fh_ctx *c = new fh_ctx();
    c->device = device;
    c->n_cu = prop.multiProcessorCount;
    fh_status s = c->err.ensure(4, nullptr);
    if (!s) s = c->h_small.ensure(256, nullptr);
    if (s) {
        c->err.release();
        delete c;
        return s;
    }
    if (hipMemset(c->err.ptr, 0, 4) != hipSuccess) {
        c->err.release();
        c->h_small.release();
        delete c;
        return fail(FH_E_DEVICE, "hipMemset failed");
    }
    *out = c;
    return FH_OK;
}

void fh_ctx_destroy(fh_ctx *ctx) {
    if (!ctx) return;
    (void)hipSetDevice(ctx->device);
    (void)hipDeviceSynchronize();
    for (auto &e : ctx->graphs) {
        (void)hipGraphExecDestroy(e.exec);
        (void)hipGraphDestroy(e.graph);
    }
    ctx->graphs.clear();
    ctx->main_ws.release();
    ctx->err.release();
    for (DevBuf *b : {&ctx->rf_offsets, &ctx->rf_bins, &ctx->rf_first, &ctx->rf_counts,
                      &ctx->rf_cands, &ctx->rf_aux, &ctx->cl_hist, &ctx->cl_s2, &ctx->pm_rows, &ctx->pm_counts})
        b->release();
    ctx->h_small.release();
    ctx->h_stage.release();
    ctx->spare.blocks.trim();
    for (hipEvent_t e : ctx->ev_pool) (void)hipEventDestroy(e);
    delete ctx;
}

fh_status fh_ctx_set_doppler(fh_ctx *ctx, int32_t mode, double f_ref) {
    fh_status s;
    if ((s = check_ctx(ctx))) return s;
    if (mode != 0 && mode != 1) return fail(FH_E_INVALID, "Doppler mode must be 0 (exact) or 1 (per-FFT shift)");
    if (!std::isfinite(f_ref)) return fail(FH_E_INVALID, "reference frequency is not finite");
    ctx->doppler_mode = mode;
    ctx->doppler_fref = f_ref;
    return FH_OK;
}

fh_status fh_ctx_set_option(fh_ctx *ctx, const char *name, int64_t value) {
    fh_status s;
    if ((s = check_ctx(ctx))) return s;
    if (!name) return fail(FH_E_INVALID, "option name is NULL");
    if (std::strcmp(name, "window_method") == 0) {
        if (value < 0 || value > 2) return fail(FH_E_INVALID, "window_method must be 0, 1 or 2");
        ctx->window_method = (int32_t)value;
        return FH_OK;
    }
    if (std::strcmp(name, "tile_parts") == 0) {
        if (value < 0 || value > 64) return fail(FH_E_INVALID, "tile_parts must be 0 .. 64");
        ctx->tile_parts = (int32_t)value;
        return FH_OK;
    }
    return fail(FH_E_INVALID, "unknown option '%s'", name);
}

fh_status fh_ctx_check(fh_ctx *ctx, void *stream) {
    fh_status s;
    if ((s = check_ctx(ctx))) return s;
    hipStream_t st = (hipStream_t)stream;
    HIP_OK(hipStreamSynchronize(st));
    int32_t flag = 0;
    HIP_OK(hipMemcpy(&flag, ctx->err.ptr, 4, hipMemcpyDeviceToHost));
    HIP_OK(hipMemset(ctx->err.ptr, 0, 4));
    if (flag & 2) return fail(FH_E_DEVICE, "internal: a spin-down residual code left its 2-bit range");
    if (flag) return fail(FH_E_INVALID, "a weight vector held a value that is not finite or outside (0, 65536), or whose sum is too large");
    return FH_OK;
}

fh_status fh_peakmap_upload(fh_ctx *ctx, const fh_peakmap_desc *d, void *stream, fh_peakmap **out) {
    fh_status s;
    if (!out) return fail(FH_E_INVALID, "out is NULL");
    *out = nullptr;
    if ((s = check_ctx(ctx))) return s;
    if (!d) return fail(FH_E_INVALID, "descriptor is NULL");
    const int32_t N = d->n_fft;
    if (N < 1) return fail(FH_E_INVALID, "n_fft=%d < 1", N);
    if (!d->offsets || !d->t || !d->v || (d->n_peaks > 0 && !d->bins))
        return fail(FH_E_INVALID, "a peakmap array is NULL");
    if (!(d->t_fft > 0) || !std::isfinite(d->t_fft)) return fail(FH_E_INVALID, "t_fft must be finite and > 0");
    if (d->offsets[0] != 0) return fail(FH_E_INVALID, "offsets[0] != 0");
    if (d->offsets[N] != d->n_peaks) return fail(FH_E_INVALID, "offsets[N] != n_peaks");
    if (d->n_peaks < 0 || d->n_peaks >= ((int64_t)1 << 31)) return fail(FH_E_INVALID, "n_peaks outside [0, 2^31)");
    fh_peakmap *pm = new fh_peakmap();
    pm->n_fft = N;
    pm->n_peaks = d->n_peaks;
    pm->t_fft = d->t_fft;
    if ((s = check_times(pm, d->t, d->v))) {
        delete pm;
        return s;
    }
    pm->k_min = 0x7fffffff;
    pm->k_max = 0;
    for (int32_t i = 0; i < N; ++i) {
        const int64_t a = d->offsets[i], e = d->offsets[i + 1];
        if (e < a) { delete pm; return fail(FH_E_INVALID, "offsets decrease at FFT %d", i); }
        pm->max_per_fft = std::max<int32_t>(pm->max_per_fft, (int32_t)(e - a));
        if (e == a) continue;
        // ascending bins: the first is the least, the last the largest
        const int32_t *k = d->bins + a;
        int32_t bad = 0, adjacent = 0;
        for (int64_t p = 1; p < e - a; ++p) {
            bad |= k[p] <= k[p - 1];
            adjacent |= (int64_t)k[p] == (int64_t)k[p - 1] + 1;
        }
        if (k[0] < 0) bad = 1;
        for (int64_t p = 0; bad && p < e - a; ++p) {  // name the first bad peak
            if (k[p] < 0) { delete pm; return fail(FH_E_INVALID, "negative bin at peak %lld", (long long)(a + p)); }
            if (p > 0 && k[p] <= k[p - 1]) {
                delete pm;
                return fail(FH_E_INVALID, "bins not strictly ascending in FFT %d", i);
            }
        }
        pm->adjacent |= adjacent;
        pm->k_min = std::min(pm->k_min, k[0]);
        pm->k_max = std::max(pm->k_max, k[e - a - 1]);
    }
    if (pm->n_peaks == 0) pm->k_min = pm->k_max = 0;
    hipStream_t st = (hipStream_t)stream;
    const size_t b_off = 8 * (size_t)(N + 1), b_bins = 4 * (size_t)std::max<int64_t>(1, d->n_peaks);
    const size_t b_t = 8 * (size_t)N, b_v = 24 * (size_t)N;
    if (!alloc_head(ctx, pm) || !alloc_bins(ctx, pm, d->n_peaks)) {
        fh_peakmap_release(ctx, pm);
        return fail(FH_E_NOMEM, "device allocation for the peakmap failed");
    }
    pm->bytes = (int64_t)(b_off + b_bins + b_t + b_v);
    hipError_t e = hipMemcpyAsync(pm->d_offsets, d->offsets, b_off, hipMemcpyHostToDevice, st);
    if (e == hipSuccess && d->n_peaks > 0)
        e = hipMemcpyAsync(pm->d_bins, d->bins, 4 * (size_t)d->n_peaks, hipMemcpyHostToDevice, st);
    if (e == hipSuccess) e = hipMemcpyAsync(pm->d_t, d->t, b_t, hipMemcpyHostToDevice, st);
    if (e == hipSuccess) e = hipMemcpyAsync(pm->d_v, d->v, b_v, hipMemcpyHostToDevice, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) {
        fh_peakmap_release(ctx, pm);
        return fail(FH_E_DEVICE, "peakmap upload failed: %s", hipGetErrorString(e));
    }
    *out = pm;
    return FH_OK;
}

fh_status fh_peakmap_from_spectra(fh_ctx *ctx, int32_t n_fft, int32_t n_bins, int64_t ld,
                                  const float *d_sp, const float *d_sar, int32_t k0, float theta,
                                  const double *t, const double *v, double t_fft, void *stream,
                                  fh_peakmap **out) {
    fh_status s;
    if (!out) return fail(FH_E_INVALID, "out is NULL");
    *out = nullptr;
    if ((s = check_ctx(ctx))) return s;
    if (n_fft < 1 || n_fft > (1 << 24)) return fail(FH_E_INVALID, "n_fft=%d outside 1..2^24", n_fft);
    if (n_bins < 3 || ld < n_bins) return fail(FH_E_INVALID, "need n_bins >= 3 and ld >= n_bins");
    if (!d_sp || !t || !v) return fail(FH_E_INVALID, "a spectrum or time/velocity array is NULL");
    if (k0 < 0 || (int64_t)k0 + n_bins >= ((int64_t)1 << 31)) return fail(FH_E_INVALID, "k0 out of range");
    if (!std::isfinite(theta)) return fail(FH_E_INVALID, "theta is not finite");
    if (!(t_fft > 0) || !std::isfinite(t_fft)) return fail(FH_E_INVALID, "t_fft must be finite and > 0");
    fh_peakmap *pm = new fh_peakmap();
    pm->n_fft = n_fft;
    pm->t_fft = t_fft;
    if ((s = check_times(pm, t, v))) {
        delete pm;
        return s;
    }
    hipStream_t st = (hipStream_t)stream;
    const int32_t cap = n_bins / 2 + 1;  // strict local maxima are never adjacent
    const size_t b_off = 8 * (size_t)(n_fft + 1), b_t = 8 * (size_t)n_fft, b_v = 24 * (size_t)n_fft;
    struct Busy {  // the rows stay while this call uses them
        bool &f;
        ~Busy() { f = false; }
    } busy{ctx->spare.rows_busy};
    if ((s = ctx->pm_counts.ensure(4 * (size_t)n_fft, st)) ||
        (s = ctx->pm_rows.ensure(4 * (size_t)n_fft * cap, st))) {
        delete pm;
        return s;
    }
    ctx->spare.rows_busy = true;
    if (!alloc_head(ctx, pm)) {
        fh_peakmap_release(ctx, pm);
        return fail(FH_E_NOMEM, "device allocation for the peakmap failed");
    }
    // (every use of the staging buffer ends with a wait for its copy)
    const bool staged = b_t + b_v <= kMaxStage && ctx->h_stage.ensure(b_t + b_v, st) == FH_OK;
    if (staged) {
        std::memcpy(ctx->h_stage.ptr, t, b_t);
        std::memcpy((char *)ctx->h_stage.ptr + b_t, v, b_v);
    }
    int32_t *rows_buf = (int32_t *)ctx->pm_rows.ptr, *counts = (int32_t *)ctx->pm_counts.ptr;
    int64_t P = 0;
    hipError_t e = launch_pm_rows(n_fft, n_bins, ld, d_sp, d_sar, k0, theta, cap, rows_buf, counts, st);
    if (e == hipSuccess) e = launch_pm_scan(n_fft, counts, pm->d_offsets, (int64_t *)ctx->h_small.ptr, st);
    if (e == hipSuccess)
        e = staged ? hipMemcpyAsync(pm->d_t, ctx->h_stage.ptr, b_t + b_v, hipMemcpyHostToDevice, st)
                   : hipMemcpyAsync(pm->d_t, t, b_t, hipMemcpyHostToDevice, st);
    if (e == hipSuccess && !staged) e = hipMemcpyAsync(pm->d_v, v, b_v, hipMemcpyHostToDevice, st);
    const hipError_t e2 = read_meta(ctx, st, &P, &pm->max_per_fft);
    if (e == hipSuccess) e = e2;
    if (e == hipSuccess && !alloc_bins(ctx, pm, P)) e = hipErrorOutOfMemory;
    if (e == hipSuccess) e = launch_pm_pack(n_fft, cap, rows_buf, pm->d_offsets, pm->d_bins, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    // the scratch of a usual band stays; that of a large one (14 MB per 1000
    // FFTs x 7000 bins) goes back
    if (ctx->pm_rows.bytes > BlockPool::kMaxBytes) {
        if (e != hipSuccess) (void)hipStreamSynchronize(st);
        ctx->pm_rows.release();
    }
    if (e != hipSuccess) {
        fh_peakmap_release(ctx, pm);
        return fail(e == hipErrorOutOfMemory ? FH_E_NOMEM : FH_E_DEVICE, "peakmap construction failed: %s",
                    hipGetErrorString(e));
    }
    pm->n_peaks = P;
    pm->k_min = k0 + 1;
    pm->k_max = k0 + n_bins - 2;
    pm->adjacent = 0;
    pm->bytes = (int64_t)(b_off + 4 * (size_t)std::max<int64_t>(1, P) + b_t + b_v);
    *out = pm;
    return FH_OK;
}

fh_status fh_peakmap_download(fh_ctx *ctx, const fh_peakmap *pm, int64_t *offsets, int32_t *bins) {
    fh_status s;
    if ((s = check_ctx(ctx))) return s;
    if (!pm) return fail(FH_E_INVALID, "peakmap is NULL");
    if (offsets) HIP_OK(hipMemcpy(offsets, pm->d_offsets, 8 * (size_t)(pm->n_fft + 1), hipMemcpyDeviceToHost));
    if (bins && pm->n_peaks > 0)
        HIP_OK(hipMemcpy(bins, pm->d_bins, 4 * (size_t)pm->n_peaks, hipMemcpyDeviceToHost));
    return FH_OK;
}

fh_status fh_peakmap_shape(const fh_peakmap *pm, int32_t *n_fft, int64_t *n_peaks) {
    if (!pm) return fail(FH_E_INVALID, "peakmap is NULL");
    if (n_fft) *n_fft = pm->n_fft;
    if (n_peaks) *n_peaks = pm->n_peaks;
    return FH_OK;
}

void fh_peakmap_release(fh_ctx *ctx, fh_peakmap *pm) {
    if (!pm) return;
    if (ctx) (void)hipSetDevice(ctx->device);
    // no block is handed on while the device may use it
    if (ctx && ctx->device == pm->device && (pm->head || pm->d_bins) && wait_as_free()) {
        ctx->spare.blocks.give(pm->head, pm->head_bytes);
        ctx->spare.blocks.give(pm->d_bins, pm->bins_bytes);
    } else {
        device_free(pm->head);
        device_free(pm->d_bins);
    }
    delete pm;
}

int64_t fh_peakmap_bytes(const fh_peakmap *pm) { return pm ? pm->bytes : 0; }

fh_status fh_peakmap_slice(fh_ctx *ctx, const fh_peakmap *pm, int32_t k_lo, int32_t k_hi, void *stream,
                           fh_peakmap **out) {
    fh_status s;
    if (!out) return fail(FH_E_INVALID, "out is NULL");
    *out = nullptr;
    if ((s = check_ctx(ctx))) return s;
    if (!pm) return fail(FH_E_INVALID, "peakmap is NULL");
    if (k_lo < 0 || k_hi <= k_lo) return fail(FH_E_INVALID, "need 0 <= k_lo < k_hi");
    hipStream_t st = (hipStream_t)stream;
    const int32_t N = pm->n_fft;
    const int64_t cap = std::min<int64_t>((int64_t)N * (k_hi - k_lo), pm->n_peaks);
    if ((s = ctx->rf_first.ensure(8 * (size_t)N, st)) || (s = ctx->rf_counts.ensure(4 * (size_t)N, st)))
        return s;
    fh_peakmap *q = like(pm);
    q->k_min = k_lo;
    q->k_max = k_hi - 1;
    const size_t b_off = 8 * (size_t)(N + 1), b_bins = 4 * (size_t)std::max<int64_t>(1, cap);
    if (!alloc_head(ctx, q) || !alloc_bins(ctx, q, cap)) {
        fh_peakmap_release(ctx, q);
        return fail(FH_E_NOMEM, "device allocation for the sliced peakmap failed");
    }
    q->bytes = (int64_t)(b_off + b_bins + 32 * (size_t)N);
    hipError_t e = launch_slice(N, pm->d_offsets, pm->d_bins, k_lo, k_hi, pm->d_t, q->d_t, (int64_t *)ctx->rf_first.ptr,
                                (int32_t *)ctx->rf_counts.ptr, q->d_offsets, q->d_bins, (int64_t *)ctx->h_small.ptr,
                                st);
    // exact peak count and longest FFT of the slice (the allocation keeps the bound)
    if (e == hipSuccess) e = read_meta(ctx, st, &q->n_peaks, &q->max_per_fft);
    if (e != hipSuccess) {
        fh_peakmap_release(ctx, q);
        return fail(FH_E_DEVICE, "slicing the peakmap failed: %s", hipGetErrorString(e));
    }
    *out = q;
    return FH_OK;
}

fh_status fh_refine(fh_ctx *ctx, const fh_peakmap *pm, int32_t n_cand, const fh_coarse_cand *cands,
                    const fh_refine_opts *o, const float *d_w, fh_refined *d_out, void *stream) {
    fh_status s;
    if ((s = check_ctx(ctx))) return s;
    if (!pm || !o) return fail(FH_E_INVALID, "peakmap or options is NULL");
    if (n_cand < 0 || (n_cand > 0 && (!cands || !d_out))) return fail(FH_E_INVALID, "bad candidate arrays");
    if (o->kf < 1 || o->kf > 64 || o->k_fdot < 1 || o->k_sky < 1 || o->k_sky % 2 == 0 || o->k_sky > 63)
        return fail(FH_E_INVALID, "refine options need 1 <= kf <= 64, k_fdot >= 1, odd 1 <= k_sky <= 63");
    if (!(o->dfdot > 0) || !std::isfinite(o->dfdot) || !std::isfinite(o->t0) || !(o->theta > 0))
        return fail(FH_E_INVALID, "refine options need dfdot > 0, finite t0 and theta > 0");
    if (n_cand == 0) return FH_OK;
    hipStream_t st = (hipStream_t)stream;
    if ((s = refuse_capture(st))) return s;
    const int kf = o->kf, ks = o->k_sky, n_dir = ks * ks, L = (ks - 1) / 2;
    const int ns = 4 * o->k_fdot, nf = 2 * kf + 1;
    const double T = pm->t_fft, dfd = o->dfdot / o->k_fdot;
    const double tau = std::max(std::fabs(pm->t_min - o->t0), std::fabs(pm->t_max - o->t0));
    const double ce = std::cos(23.44 * M_PI / 180.0), se = std::sin(23.44 * M_PI / 180.0);
    std::vector<fh_grid> grids((size_t)n_cand);
    std::vector<int32_t> klo((size_t)n_cand), khi((size_t)n_cand);
    std::vector<double> sky((size_t)n_cand * n_dir * 3), aux((size_t)n_cand * (4 + 2 * n_dir));
    double *prm = aux.data(), *lamb = aux.data() + 4 * (size_t)n_cand;
    int32_t width = 1, kmin = 0x7fffffff, kmax = 0;
    for (int c = 0; c < n_cand; ++c) {
        const fh_coarse_cand &q = cands[c];
        if (!std::isfinite(q.f0) || !(q.f0 > 0) || !std::isfinite(q.fdot) || !std::isfinite(q.lambda) ||
            !std::isfinite(q.beta) || !std::isfinite(q.dlambda) || !std::isfinite(q.dbeta))
            return fail(FH_E_INVALID, "candidate %d is not finite", c);
        fh_grid &g = grids[c];
        g.kf = kf;
        g.b0 = (int64_t)std::llround(q.f0 * kf * T) - kf;
        g.nf = nf;
        g.ns = ns;
        g.fdot0 = q.fdot - 2.0 * o->dfdot;
        g.dfdot = dfd;
        g.t0 = o->t0;
        if (g.b0 < 0) return fail(FH_E_INVALID, "candidate %d lies below the first fine bin", c);
        prm[4 * c + 0] = (double)g.b0 / (kf * T);
        prm[4 * c + 1] = 1.0 / (kf * T);
        prm[4 * c + 2] = g.fdot0;
        prm[4 * c + 3] = dfd;
        // peaks whose stripes can reach the refined bins: Doppler and
        // spin-down drift over the observation, plus one bin each side
        const double f_lo = (double)g.b0 / (kf * T), f_hi = (double)(g.b0 + nf) / (kf * T);
        const double fd_max = std::max(std::fabs(g.fdot0), std::fabs(g.fdot0 + (ns - 1) * dfd));
        const int64_t margin = (int64_t)std::ceil((f_hi * pm->v_max * 1.01 + fd_max * tau) * T) + 2;
        klo[c] = (int32_t)std::max<int64_t>(0, (int64_t)std::floor(f_lo * T) - margin);
        khi[c] = (int32_t)std::min<int64_t>((int64_t)1 << 30, (int64_t)std::ceil(f_hi * T) + margin + 1);
        width = std::max(width, khi[c] - klo[c]);
        kmin = std::min(kmin, klo[c]);
        kmax = std::max(kmax, khi[c] - 1);
        // longitudes (as they are, and turned by pi for latitudes over a pole)
        // and their sines and cosines, once per column of the refined sky
        struct Angle { double a, c, s; };
        Angle lams[2][63];
        bool turned = false;
        auto longitudes = [&](int over) {
            for (int i = -L; i <= L; ++i) {
                double lam = q.lambda + i * (q.dlambda / ks);
                if (over) lam += M_PI;
                lam = std::fmod(lam, 2.0 * M_PI);
                if (lam < 0) lam += 2.0 * M_PI;
                lams[over][i + L] = {lam, std::cos(lam), std::sin(lam)};
            }
        };
        longitudes(0);
        for (int j = -L; j <= L; ++j) {
            double bet = q.beta + j * (q.dbeta / ks);
            const bool over = std::fabs(bet) > 0.5 * M_PI;  // over a pole
            if (over) {
                if (!turned) longitudes(1);
                turned = true;
                bet = (bet > 0 ? M_PI : -M_PI) - bet;
            }
            const double cb = std::cos(bet), ze = std::sin(bet);
            for (int i = -L; i <= L; ++i) {
                const int d = (j + L) * ks + (i + L);
                const Angle &lam = lams[over ? 1 : 0][i + L];
                lamb[2 * ((size_t)c * n_dir + d)] = lam.a;
                lamb[2 * ((size_t)c * n_dir + d) + 1] = bet;
                const double x = cb * lam.c, ye = cb * lam.s;
                double n[3] = {x, ye * ce - ze * se, ye * se + ze * ce};
                const double r = std::sqrt(n[0] * n[0] + n[1] * n[1] + n[2] * n[2]);
                for (int k = 0; k < 3; ++k) sky[3 * ((size_t)c * n_dir + d) + k] = n[k] / r;
            }
        }
    }
    const int32_t N = pm->n_fft;
    const int64_t cap = std::min<int64_t>((int64_t)N * width, pm->n_peaks);
    fh_peakmap sub(*pm);  // the widest candidate's part of the peakmap
    sub.n_peaks = cap;
    sub.k_min = kmin;
    sub.k_max = kmax;
    sub.max_per_fft = std::min<int32_t>(pm->max_per_fft, width);
    for (int c = 0; c < n_cand; ++c)
        if ((s = check_grid(&sub, &grids[c]))) return s;
    const bool weighted = d_w != nullptr;
    // one upload: parameters and sky points of the pick, refined directions,
    // and the candidates' grids
    std::vector<RefineCand> rc((size_t)n_cand);
    for (int c = 0; c < n_cand; ++c) {
        double far2 = 0.0;  // squared distance of the farthest direction from the middle one
        const double *n = sky.data() + 3 * (size_t)c * n_dir, *m = n + 3 * (n_dir / 2);
        for (int d = 0; d < n_dir; ++d) {
            double x2 = 0.0;
            for (int k = 0; k < 3; ++k) x2 += (n[3 * d + k] - m[k]) * (n[3 * d + k] - m[k]);
            far2 = std::max(far2, x2);
        }
        rc[c] = {grids[c].b0, grids[c].fdot0, ctx->doppler_mode ? shift_reference_bins(ctx, &sub, &grids[c]) : 0.0,
                 std::sqrt(far2), klo[c], khi[c]};
    }
    const size_t b_aux = 8 * aux.size(), b_sky = 8 * sky.size(), b_rc = sizeof(RefineCand) * rc.size();
    if ((s = ctx->rf_cands.ensure(sizeof(fh_candidate) * 2 * (size_t)n_cand * n_dir, st)) ||
        (s = ctx->rf_aux.ensure(b_aux + b_sky + b_rc, st)))
        return s;
    char *h;
    if ((s = stage_buffer(ctx->cur, b_aux + b_sky + b_rc, st, &h))) return s;
    std::memcpy(h, aux.data(), b_aux);
    std::memcpy(h + b_aux, sky.data(), b_sky);
    std::memcpy(h + b_aux + b_sky, rc.data(), b_rc);
    if ((s = stage_copy(ctx->cur, ctx->rf_aux.ptr, b_aux + b_sky + b_rc, st))) return s;
    const double *daux = (const double *)ctx->rf_aux.ptr;
    double *d_sky = (double *)((char *)ctx->rf_aux.ptr + b_aux);
    const RefineCand *d_rc = (const RefineCand *)((char *)ctx->rf_aux.ptr + b_aux + b_sky);
    fh_candidate *dc = (fh_candidate *)ctx->rf_cands.ptr;
    if (refine_cell_bytes(kf, nf, ns) > 0) {
        // a volume that fits the LDS: all candidates at once (in chunks whose
        // peak runs take at most 64 MiB)
        const int chunk = (int)std::min<int64_t>(std::min(n_cand, 65535),
                                                 std::max<int64_t>(1, ((int64_t)64 << 20) / (24 * (int64_t)N)));
        if ((s = ctx->rf_first.ensure(24 * (size_t)chunk * N, st)) ||
            (s = ctx->cur->ws.ensure(sizeof(WeightStats), st)))
            return s;
        WeightStats *ws = weighted ? (WeightStats *)ctx->cur->ws.ptr : nullptr;
        Timed timed(ctx, st, kSpanTiles);
        if (weighted)
            HIP_OK(launch_weight_stats(N, d_w, pm->adjacent ? 2 : 1, ws, (int32_t *)ctx->err.ptr, st));
        for (int c = 0; c < n_cand; c += chunk) {
            const int nc = std::min(chunk, n_cand - c);
            int4 *firsts = (int4 *)ctx->rf_first.ptr;
            HIP_OK(launch_refine_cells(N, pm->d_offsets, pm->d_bins, pm->d_t, pm->d_v, nc, n_dir,
                                       d_sky + 3 * (size_t)c * n_dir, d_rc + c, (int2 *)(firsts + (size_t)chunk * N),
                                       firsts, kf, nf, ns, dfd, o->t0, T, o->theta, d_w, ws, ctx->doppler_mode,
                                       dc + 2 * (size_t)c * n_dir, st));
        }
        if (ctx->profiling) ctx->prof_updates += cap * (int64_t)ns * n_dir * n_cand;
    } else {
        // a larger one: candidate by candidate, the sliced peakmap (context-owned
        // arrays) searched with the tiles
        if ((s = ctx->rf_offsets.ensure(8 * (size_t)(N + 1), st)) || (s = ctx->rf_bins.ensure(4 * (size_t)cap + 4, st)) ||
            (s = ctx->rf_first.ensure(8 * (size_t)N, st)) || (s = ctx->rf_counts.ensure(4 * (size_t)N, st)))
            return s;
        sub.d_offsets = (int64_t *)ctx->rf_offsets.ptr;
        sub.d_bins = (int32_t *)ctx->rf_bins.ptr;
        const Plan p = make_plan(grids[0], choose_tile_bins(ctx, &sub, &grids[0], 0));
        ChunkBufs b;
        if ((s = ensure_workspace(ctx, &sub, &grids[0], p, n_dir, 1, weighted, st, b))) return s;
        fh_select sel{nf, nf, -1, o->theta};
        for (int c = 0; c < n_cand; ++c) {
            HIP_OK(launch_slice(N, pm->d_offsets, pm->d_bins, klo[c], khi[c], nullptr, nullptr, (int64_t *)ctx->rf_first.ptr,
                                (int32_t *)ctx->rf_counts.ptr, sub.d_offsets, sub.d_bins, nullptr, st));
            ChunkBufs bc = b;
            bc.sky = d_sky + 3 * (size_t)c * n_dir;
            if ((s = run_search(ctx, &sub, &grids[c], p, n_dir, n_dir, d_w, 0, FH_SCHED_PERSISTENT, &sel,
                                dc + 2 * (int64_t)c * n_dir, bc, st, {})))
                return s;
        }
    }
    HIP_OK(launch_refine_pick(n_cand, n_dir, dc, daux, daux + 4 * (size_t)n_cand, d_out, st));
    return FH_OK;
}


// ---- peakmap cleaning ----

fh_status fh_gross_histogram(fh_ctx *ctx, const fh_peakmap *pm, const fh_gross *geo, int32_t *d_hist,
                             void *stream) {
    fh_status s;
    if ((s = check_ctx(ctx))) return s;
    if (!pm) return fail(FH_E_INVALID, "peakmap is NULL");
    if ((s = check_gross(geo))) return s;
    if (!d_hist) return fail(FH_E_INVALID, "histogram pointer is NULL");
    HIP_OK(launch_gross_hist(pm->n_fft, pm->d_offsets, pm->d_bins, pm->d_t, pm->t_fft, *geo, d_hist,
                             (hipStream_t)stream));
    return FH_OK;
}

fh_status fh_clean_gross(fh_ctx *ctx, const fh_peakmap *pm, const fh_gross *geo, double threshold,
                         int32_t *d_hist, void *stream, fh_peakmap **out) {
    fh_status s;
    if (!out) return fail(FH_E_INVALID, "out is NULL");
    *out = nullptr;
    if (std::isnan(threshold)) return fail(FH_E_INVALID, "threshold is NaN");
    if ((s = fh_gross_histogram(ctx, pm, geo, d_hist, stream))) return s;
    FilterSpec f{};
    f.mode = 0;
    f.t = pm->d_t;
    f.t_fft = pm->t_fft;
    f.geo = *geo;
    f.hist = d_hist;
    f.thr = threshold;
    return filter_peakmap(ctx, pm, f, (hipStream_t)stream, out);
}

fh_status fh_bin_counts(fh_ctx *ctx, const fh_peakmap *pm, int32_t k_lo, int32_t k_hi, int32_t *d_counts,
                        void *stream) {
    fh_status s;
    if ((s = check_ctx(ctx))) return s;
    if (!pm) return fail(FH_E_INVALID, "peakmap is NULL");
    if (k_lo < 0 || k_hi <= k_lo) return fail(FH_E_INVALID, "need 0 <= k_lo < k_hi");
    if (!d_counts) return fail(FH_E_INVALID, "counts pointer is NULL");
    HIP_OK(launch_bin_counts(pm->n_fft, pm->n_peaks, pm->d_offsets, pm->d_bins, k_lo, k_hi, d_counts,
                             (hipStream_t)stream));
    return FH_OK;
}

fh_status fh_robust_stats(fh_ctx *ctx, const int32_t *d_x, int32_t n, int32_t x_max, double out[2],
                          void *stream) {
    fh_status s;
    if ((s = check_ctx(ctx))) return s;
    if (!d_x || !out) return fail(FH_E_INVALID, "data or output pointer is NULL");
    if (n < 1) return fail(FH_E_INVALID, "robust statistic of %d values", n);
    if (x_max < 0 || x_max > (1 << 28)) return fail(FH_E_INVALID, "x_max=%d outside 0..2^28", x_max);
    hipStream_t st = (hipStream_t)stream;
    if ((s = ctx->cl_hist.ensure(4 * (2 * (size_t)x_max + 1), st)) || (s = ctx->cl_s2.ensure(8, st)) ||
        (s = ctx->err.ensure(4, st)))
        return s;
    double *h = (double *)ctx->h_small.ptr;  // m1, m2, error flag
    HIP_OK(launch_robust(d_x, n, x_max, (int32_t *)ctx->cl_hist.ptr, (int64_t *)ctx->cl_s2.ptr, h,
                         (int32_t *)ctx->err.ptr, st));
    HIP_OK(hipStreamSynchronize(st));
    if (h[2] != 0.0) return fail(FH_E_INVALID, "a value lies outside [0, x_max=%d]", x_max);
    out[0] = h[0];
    out[1] = h[1];
    return FH_OK;
}

fh_status fh_line_counts(fh_ctx *ctx, const fh_peakmap *pm, const fh_grid *g, int32_t *d_out, void *stream) {
    fh_status s;
    if ((s = check_ctx(ctx))) return s;
    if ((s = check_grid(pm, g))) return s;
    if (!d_out) return fail(FH_E_INVALID, "output pointer is NULL");
    hipStream_t st = (hipStream_t)stream;
    const Plan p = make_plan(*g, search_tile_bins(ctx, pm, g, 1));
    ChunkBufs b;
    if ((s = ensure_workspace(ctx, pm, g, p, 1, 1, false, st, b))) return s;
    const double zero[3] = {0.0, 0.0, 0.0};  // v . n = 0: no Doppler correction
    if ((s = run_search(ctx, pm, g, p, 1, 1, nullptr, 0, FH_SCHED_PERSISTENT, nullptr, nullptr, b, st, {zero, 1})))
        return s;
    HIP_OK(launch_colmax_values(b.colmax, g->nf, d_out, st));
    return FH_OK;
}

fh_status fh_veto_bins(fh_ctx *ctx, const fh_peakmap *pm, int32_t k_lo, int32_t k_hi, const int32_t *d_x,
                       int64_t n_x, int32_t step, int64_t offset, double threshold, void *stream,
                       fh_peakmap **out) {
    fh_status s;
    if (!out) return fail(FH_E_INVALID, "out is NULL");
    *out = nullptr;
    if ((s = check_ctx(ctx))) return s;
    if (!pm) return fail(FH_E_INVALID, "peakmap is NULL");
    if (k_lo < 0 || k_hi <= k_lo) return fail(FH_E_INVALID, "need 0 <= k_lo < k_hi");
    if (!d_x || n_x < 1) return fail(FH_E_INVALID, "statistic array is NULL or empty");
    if (std::isnan(threshold)) return fail(FH_E_INVALID, "threshold is NaN");
    FilterSpec f{};
    f.mode = 1;
    f.k_lo = k_lo;
    f.k_hi = k_hi;
    f.step = step;
    f.offset = offset;
    f.n_x = n_x;
    f.x = d_x;
    f.thr = threshold;
    return filter_peakmap(ctx, pm, f, (hipStream_t)stream, out);
}

fh_status fh_plan_query(fh_ctx *ctx, const fh_peakmap *pm, const fh_grid *g, int32_t tile_bins,
                        fh_plan_info *out) {
    fh_status s;
    if ((s = check_ctx(ctx))) return s;
    if ((s = check_grid(pm, g))) return s;
    if (!out) return fail(FH_E_INVALID, "out is NULL");
    if (tile_bins < 0) return fail(FH_E_INVALID, "tile_bins < 0");
    int width = choose_tile_bins(ctx, pm, g, tile_bins);
    const auto used = ctx->used.find(tune_key(pm, g));
    if (tile_bins == 0 && used != ctx->used.end()) width = used->second;
    const Plan p = make_plan(*g, width);
    out->tile_rows = kTileRows;
    out->tile_bins = p.W;
    out->n_row_blocks = p.nrb;
    out->n_bin_blocks = p.nbb;
    out->workspace_bytes = edge_bytes_per_sky(ctx, pm) + 16 * (int64_t)p.nrbg * p.nbb * win_stride(pm->n_fft) +
                           8 * (int64_t)g->nf + 4 * (int64_t)pm->n_fft + 4 * p.tiles_per_sky +
                           (int64_t)shift_layout(pm->n_fft, p.nrb_tab, p.nrbg).total;
    out->cell_updates = pm->n_peaks * (int64_t)g->ns;
    return FH_OK;
}

fh_status fh_hough_map_i32(fh_ctx *ctx, const fh_peakmap *pm, const double nhat[3],
                           const fh_grid *grid, int32_t *d_map, void *stream) {
    return hough_map_common(ctx, pm, nhat, nullptr, grid, d_map, stream);
}

fh_status fh_hough_map_f32(fh_ctx *ctx, const fh_peakmap *pm, const double nhat[3],
                           const float *d_w, const fh_grid *grid, float *d_map, void *stream) {
    if (!d_w) return fail(FH_E_INVALID, "weights pointer is NULL");
    return hough_map_common(ctx, pm, nhat, d_w, grid, d_map, stream);
}

}  // extern "C"

namespace {

// Pieces of the unweighted map path carved out of `scratch` (256-byte aligned
// byte offsets).  Every piece a kernel reads is written earlier in the same
// call (edges, every window entry including the padding FFTs,
// the shift table and the direction), so nothing has to start at zero; the
// error flag and the queue counters are only read on paths this call does not
// take (weights, the persistent schedule).
struct StaticLayout {
    size_t sky, err, qctr, sht, y, y64, win, n_win, wsort, total;
    ShiftLayout shl;
};

StaticLayout static_layout(const fh_ctx *ctx, const fh_peakmap *pm, const Plan &p) {
    auto al = [](size_t x) { return (x + 255) / 256 * 256; };
    const size_t ys = (size_t)y_stride(pm->n_peaks, pm->n_fft);
    // 8 bytes per window as reserved for the unsorted ones: they take 4, and
    // the FFTs' first edges lie behind them
    const size_t wins = (size_t)8 * p.nrbg * p.nbb * win_stride(pm->n_fft);
    StaticLayout L{};
    size_t o = 0;
    L.sky = o;   o += al(24);
    L.err = o;   o += al(4);
    L.qctr = o;  o += al(4 * kXcds);
    L.shl = shift_layout(pm->n_fft, p.nrb_tab, p.nrbg);
    L.sht = o;   o += L.shl.total;
    L.y = o;     o += al(4 * ys);
    L.y64 = o;   if (needs_full_edges(ctx, pm)) o += al(8 * ys);
    L.win = o;   o += al(wins);
    L.n_win = wins / 8;
    L.wsort = o; o += al(wins);
    L.total = o;
    return L;
}

}  // namespace

extern "C" {

fh_status fh_hough_map_i32_static(fh_ctx *ctx, const fh_peakmap *pm, const double nhat[3],
                                  const fh_grid *g, int32_t *d_map, void *stream) {
    fh_status s;
    if ((s = check_ctx(ctx))) return s;
    if ((s = check_grid(pm, g))) return s;
    if ((s = check_sky(nhat))) return s;
    if (!d_map) return fail(FH_E_INVALID, "output map pointer is NULL");
    hipStream_t st = (hipStream_t)stream;
    Plan p = make_plan(*g, search_tile_bins(ctx, pm, g, 1));
    StaticLayout L = static_layout(ctx, pm, p);
    if (L.total > kStaticScratchBytes) {  // wider tiles need fewer windows
        p = make_plan(*g, choose_tile_bins(ctx, pm, g, 0));
        L = static_layout(ctx, pm, p);
    }
    if (L.total > kStaticScratchBytes)
        return fail(FH_E_UNSUPPORTED, "this map needs %zu bytes of scratch; the static scratch holds %zu",
                    L.total, kStaticScratchBytes);
    void *base = ctx->device < kMaxDevices ? g_scratch_ptr[ctx->device] : nullptr;
    if (!base) return fail(FH_E_UNSUPPORTED, "no static scratch on device %d", ctx->device);
    char *c = static_cast<char *>(base);
    ChunkBufs b{};
    b.sky = reinterpret_cast<double *>(c + L.sky);
    b.err = reinterpret_cast<int32_t *>(c + L.err);
    b.qctr = reinterpret_cast<int32_t *>(c + L.qctr);
    b.colmax = reinterpret_cast<unsigned long long *>(c + L.qctr);  // not written by the map path
    b.gwin = reinterpret_cast<int64_t *>(c + L.sht + L.shl.gwin);
    b.rec = reinterpret_cast<uint2 *>(c + L.sht + L.shl.rec);
    b.step = reinterpret_cast<uint32_t *>(c + L.sht + L.shl.step);
    b.Y = reinterpret_cast<uint32_t *>(c + L.y);
    b.Y64 = reinterpret_cast<int64_t *>(c + L.y64);
    b.win = reinterpret_cast<uint32_t *>(c + L.win);
    b.base = b.win + L.n_win;
    b.wsort = reinterpret_cast<int2 *>(c + L.wsort);
    b.part = reinterpret_cast<uint32_t *>(c + L.total);  // what is left holds partial tiles
    b.part_bytes = kStaticScratchBytes - L.total;
    // no profiling spans here: recording one can create an event
    const bool was = ctx->profiling;
    ctx->profiling = false;
    s = enqueue_map(ctx, pm, g, p, nhat, nullptr, b, d_map, st);
    ctx->profiling = was;
    return s;
}

fh_status fh_hough_candidates(fh_ctx *ctx, const fh_peakmap *pm, int32_t n_sky, const double *sky,
                              const float *d_w, int32_t w_stride, const fh_grid *g,
                              const fh_select *sel, const fh_options *opts, fh_candidate *d_out,
                              void *stream) {
    fh_status s;
    if ((s = check_ctx(ctx))) return s;
    if ((s = check_grid(pm, g))) return s;
    if (n_sky < 1) return fail(FH_E_INVALID, "n_sky=%d < 1", n_sky);
    if (!sky) return fail(FH_E_INVALID, "sky is NULL");
    for (int32_t k = 0; k < n_sky; ++k)
        if ((s = check_sky(sky + 3 * (int64_t)k))) return s;
    if (!sel || sel->width < 1 || sel->excl < 0 || !std::isfinite(sel->theta) || !(sel->theta > 0))
        return fail(FH_E_INVALID, "selection needs width >= 1, excl >= 0, theta > 0");
    if (!d_out) return fail(FH_E_INVALID, "output pointer is NULL");
    if (d_w && w_stride != 0 && w_stride != pm->n_fft)
        return fail(FH_E_INVALID, "w_stride must be 0 or n_fft");
    fh_options o{FH_SCHED_PERSISTENT, 0, 0, 0};
    if (opts) o = *opts;
    if (o.schedule != FH_SCHED_PLAIN && o.schedule != FH_SCHED_PERSISTENT)
        return fail(FH_E_INVALID, "unknown schedule %d", o.schedule);
    if (o.tile_bins < 0 || o.sky_chunk < 0) return fail(FH_E_INVALID, "negative option");
    hipStream_t st = (hipStream_t)stream;
    const bool weighted = d_w != nullptr;
    int width = 0;
    if ((s = plan_width(ctx, pm, g, n_sky, sky, d_w, w_stride, o, st, &width))) return s;
    const Plan p = make_plan(*g, width);
    int chunk = o.schedule == FH_SCHED_PLAIN ? 1 : default_chunk(ctx, pm, g, p, o.sky_chunk);
    chunk = std::min(chunk, n_sky);
    ChunkBufs b;
    if ((s = ensure_workspace(ctx, pm, g, p, chunk, n_sky, weighted, st, b))) return s;
    SkyDirs dirs;
    if ((s = upload_sky(ctx, sky, n_sky, b, st, &dirs))) return s;
    if (!o.use_graph)
        return run_search(ctx, pm, g, p, chunk, n_sky, d_w, w_stride, o.schedule, sel, d_out, b, st, dirs);
    if (st == nullptr) return fail(FH_E_INVALID, "use_graph needs a created stream, not the default stream");
    if (dirs.n) {  // the graph reads its directions from memory
        SkyArg arg;
        std::memcpy(arg.v, dirs.arg, (size_t)24 * dirs.n);
        HIP_OK(launch_set_sky(arg, dirs.n, b.sky, st));
    }

    // hipGraph: capture the whole search once, replay it while the peakmap and
    // every argument and workspace pointer it bakes in is unchanged (sky vectors
    // and weights are read from device memory at replay time, so their contents
    // may change).
    auto bits = [](double x) { uint64_t u; std::memcpy(&u, &x, 8); return u; };
    std::vector<uint64_t> key = {
        pm->serial.id, (uint64_t)g->kf, (uint64_t)g->b0, (uint64_t)g->nf, (uint64_t)g->ns,
        bits(g->fdot0), bits(g->dfdot), bits(g->t0), (uint64_t)sel->width, (uint64_t)(uint32_t)sel->excl,
        (uint64_t)(uint32_t)sel->sep, bits(sel->theta), (uint64_t)o.schedule, (uint64_t)p.W,
        (uint64_t)chunk, (uint64_t)n_sky, (uint64_t)(uintptr_t)d_w, (uint64_t)(uint32_t)w_stride,
        (uint64_t)(uintptr_t)d_out, (uint64_t)(uintptr_t)st, (uint64_t)(uintptr_t)b.Y,
        (uint64_t)(uintptr_t)b.win, (uint64_t)(uintptr_t)b.wsort, (uint64_t)(uintptr_t)b.colmax, (uint64_t)(uintptr_t)b.wq,
        (uint64_t)(uintptr_t)b.ws, (uint64_t)(uintptr_t)b.sky,
        (uint64_t)(uintptr_t)b.gwin,
        (uint64_t)(uintptr_t)b.qctr, (uint64_t)(uintptr_t)b.Y64, (uint64_t)ctx->window_method,
        (uint64_t)ctx->tile_parts, (uint64_t)(uintptr_t)b.part, (uint64_t)b.part_bytes,
        (uint64_t)(uintptr_t)b.rank,
        (uint64_t)ctx->doppler_mode, bits(ctx->doppler_fref)};
    fh_ctx::GraphEntry *ge = nullptr;
    for (auto &e : ctx->graphs)
        if (e.key == key) ge = &e;
    if (!ge) {
        const bool was = ctx->profiling;
        ctx->profiling = false;  // no event records inside the capture
        HIP_OK(hipStreamBeginCapture(st, hipStreamCaptureModeThreadLocal));
        s = run_search(ctx, pm, g, p, chunk, n_sky, d_w, w_stride, o.schedule, sel, d_out, b, st, {});
        hipGraph_t graph = nullptr;
        hipError_t e = hipStreamEndCapture(st, &graph);
        ctx->profiling = was;
        if (s) {
            if (graph) (void)hipGraphDestroy(graph);
            return s;
        }
        if (e != hipSuccess) return fail(FH_E_DEVICE, "hipStreamEndCapture: %s", hipGetErrorString(e));
        hipGraphExec_t exec = nullptr;
        e = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
        if (e != hipSuccess) {
            (void)hipGraphDestroy(graph);
            return fail(FH_E_DEVICE, "hipGraphInstantiate: %s", hipGetErrorString(e));
        }
        if (ctx->graphs.size() >= 16) {
            (void)hipGraphExecDestroy(ctx->graphs.front().exec);
            (void)hipGraphDestroy(ctx->graphs.front().graph);
            ctx->graphs.erase(ctx->graphs.begin());
        }
        ctx->graphs.push_back({key, graph, exec});
        ge = &ctx->graphs.back();
    }
    {
        Timed timed(ctx, st, kSpanGraph);
        HIP_OK(hipGraphLaunch(ge->exec, st));
    }
    if (ctx->profiling) ctx->prof_updates += pm->n_peaks * (int64_t)g->ns * n_sky;
    return FH_OK;
}

fh_status fh_hough_colmax(fh_ctx *ctx, const fh_peakmap *pm, int32_t n_sky, const double *sky, const float *d_w,
                          int32_t w_stride, const fh_grid *g, const fh_options *opts, float *d_value,
                          int32_t *d_row, void *stream) {
    fh_status s;
    if ((s = check_ctx(ctx))) return s;
    if ((s = check_grid(pm, g))) return s;
    if (n_sky < 1) return fail(FH_E_INVALID, "n_sky=%d < 1", n_sky);
    if (!sky) return fail(FH_E_INVALID, "sky is NULL");
    for (int32_t k = 0; k < n_sky; ++k)
        if ((s = check_sky(sky + 3 * (int64_t)k))) return s;
    if (!d_value || !d_row) return fail(FH_E_INVALID, "output pointer is NULL");
    if (d_w && w_stride != 0 && w_stride != pm->n_fft)
        return fail(FH_E_INVALID, "w_stride must be 0 or n_fft");
    fh_options o{FH_SCHED_PERSISTENT, 0, 0, 0};
    if (opts) o = *opts;
    if (o.schedule != FH_SCHED_PLAIN && o.schedule != FH_SCHED_PERSISTENT)
        return fail(FH_E_INVALID, "unknown schedule %d", o.schedule);
    if (o.tile_bins < 0 || o.sky_chunk < 0) return fail(FH_E_INVALID, "negative option");
    hipStream_t st = (hipStream_t)stream;
    const bool weighted = d_w != nullptr;
    int width = 0;
    if ((s = plan_width(ctx, pm, g, n_sky, sky, d_w, w_stride, o, st, &width))) return s;
    const Plan p = make_plan(*g, width);
    int chunk = o.schedule == FH_SCHED_PLAIN ? 1 : default_chunk(ctx, pm, g, p, o.sky_chunk);
    chunk = std::min(chunk, n_sky);
    ChunkBufs b;
    if ((s = ensure_workspace(ctx, pm, g, p, chunk, n_sky, weighted, st, b))) return s;
    SkyDirs dirs;
    if ((s = upload_sky(ctx, sky, n_sky, b, st, &dirs))) return s;
    ColmaxOut cm;
    cm.value = d_value;
    cm.row = d_row;
    return run_search(ctx, pm, g, p, chunk, n_sky, d_w, w_stride, o.schedule, nullptr, nullptr, b, st, dirs, cm);
}

fh_status fh_ctx_profile(fh_ctx *ctx, int32_t enable) {
    fh_status s;
    if ((s = check_ctx(ctx))) return s;
    if (enable) {
        HIP_OK(hipDeviceSynchronize());
        ctx->spans.clear();
        ctx->ev_used = 0;
        ctx->prof_updates = 0;
    }
    ctx->profiling = enable != 0;
    return FH_OK;
}

fh_status fh_ctx_profile_read(fh_ctx *ctx, fh_profile *out) {
    fh_status s;
    if ((s = check_ctx(ctx))) return s;
    if (!out) return fail(FH_E_INVALID, "out is NULL");
    HIP_OK(hipDeviceSynchronize());
    fh_profile p{};
    for (const auto &sp : ctx->spans) {
        float ms = 0.f;
        HIP_OK(hipEventElapsedTime(&ms, sp.a, sp.b));
        if (sp.kind == kSpanTiles) { p.tiles_ms += ms; p.tiles_launches++; }
        else if (sp.kind == kSpanFront) { p.front_ms += ms; p.front_launches++; }
        else if (sp.kind == kSpanGraph) { p.graph_ms += ms; p.graph_launches++; }
        else { p.select_ms += ms; p.select_launches++; }
    }
    p.cell_updates = ctx->prof_updates;
    *out = p;
    return FH_OK;
}

}  // extern "C"

// ---------------------------------------------------------------------------
// continuous-batching server

namespace {

using Clock = std::chrono::steady_clock;

double ms_between(Clock::time_point a, Clock::time_point b) {
    return std::chrono::duration<double, std::milli>(b - a).count();
}

// Byte layout of one search's workspace inside a block of the server's
// arena: the same buffers ensure_workspace provides, 256-byte aligned.
struct SearchLayout {
    size_t sht = 0, y = 0, y64 = 0, win = 0, wsort = 0, colmax = 0, wq = 0, ws = 0, sky = 0, qctr = 0, part = 0, total = 0;
    size_t n_win = 0, rank = 0, rank_size = 0, part_bytes = 0;
    ShiftLayout shl{};
};

// (with_rank: room for the rank table, which only saves time)
SearchLayout search_layout(const fh_ctx *ctx, const fh_peakmap *pm, const fh_grid *g, const Plan &p, int chunk,
                           int n_sky, bool weighted, bool with_rank = true) {
    auto al = [](size_t x) { return (x + 255) / 256 * 256; };
    const size_t N = (size_t)pm->n_fft, c = (size_t)chunk;
    const size_t ys = (size_t)y_stride(pm->n_peaks, pm->n_fft);
    const size_t wins = (size_t)8 * c * p.nrbg * p.nbb * win_stride(pm->n_fft);  // (as static_layout)
    SearchLayout L;
    size_t o = 0;
    L.shl = shift_layout((int64_t)N, p.nrb_tab, p.nrbg);
    L.sht = o;    o += L.shl.total;
    L.y = o;      o += al(4 * ys * c);
    L.y64 = o;    if (needs_full_edges(ctx, pm)) o += al(8 * ys * c);
    L.win = o;    o += al(wins);
    L.n_win = wins / 8;
    L.wsort = o;  o += al(wins);
    L.colmax = o; o += al(8 * c * (size_t)g->nf);
    L.wq = o;     o += al(weighted ? 4 * c * N : 4);
    L.ws = o;     o += al(sizeof(WeightStats) * c);
    L.sky = o;    o += al(24 * (size_t)n_sky);
    L.qctr = o;   o += al(4 * kXcds);
    L.rank_size = with_rank ? rank_bytes(ctx, pm, p, chunk) : 0;
    L.rank = o;   o += al(L.rank_size);
    L.total = o;
    return L;
}

ChunkBufs carve(char *base, const SearchLayout &L, int32_t *err) {
    ChunkBufs b{};
    b.part = reinterpret_cast<uint32_t *>(base + L.part);
    b.part_bytes = L.part_bytes;
    b.rank = L.rank_size ? reinterpret_cast<uint2 *>(base + L.rank) : nullptr;
    b.gwin = reinterpret_cast<int64_t *>(base + L.sht + L.shl.gwin);
    b.rec = reinterpret_cast<uint2 *>(base + L.sht + L.shl.rec);
    b.step = reinterpret_cast<uint32_t *>(base + L.sht + L.shl.step);
    b.Y = reinterpret_cast<uint32_t *>(base + L.y);
    b.Y64 = reinterpret_cast<int64_t *>(base + L.y64);
    b.win = reinterpret_cast<uint32_t *>(base + L.win);
    b.base = b.win + L.n_win;
    b.wsort = reinterpret_cast<int2 *>(base + L.wsort);
    b.colmax = reinterpret_cast<unsigned long long *>(base + L.colmax);
    b.wq = reinterpret_cast<uint32_t *>(base + L.wq);
    b.ws = reinterpret_cast<WeightStats *>(base + L.ws);
    b.sky = reinterpret_cast<double *>(base + L.sky);
    b.qctr = reinterpret_cast<int32_t *>(base + L.qctr);
    b.err = err;
    return b;
}

// First-fit allocator over the server's device arena (host bookkeeping
// only; block sizes are multiples of 256 bytes).
struct Arena {
    char *base = nullptr;
    size_t bytes = 0;
    std::map<size_t, size_t> free_;  // offset -> size, never adjacent
    void reset(char *p, size_t n) {
        base = p;
        bytes = n;
        free_.clear();
        if (n) free_[0] = n;
    }
    bool alloc(size_t n, size_t *off) {
        for (auto it = free_.begin(); it != free_.end(); ++it) {
            if (it->second < n) continue;
            *off = it->first;
            const size_t rest = it->second - n, o2 = it->first + n;
            free_.erase(it);
            if (rest) free_[o2] = rest;
            return true;
        }
        return false;
    }
    void release(size_t off, size_t n) {
        auto nx = free_.lower_bound(off);
        if (nx != free_.end() && off + n == nx->first) {  // merge with the next block
            n += nx->second;
            nx = free_.erase(nx);
        }
        if (nx != free_.begin()) {
            auto pv = std::prev(nx);
            if (pv->first + pv->second == off) {  // merge with the previous block
                pv->second += n;
                return;
            }
        }
        free_[off] = n;
    }
};

struct ServerRequest {
    uint64_t id = 0;
    fh_request r{};
    std::vector<double> sky;
    Clock::time_point t_submit, t_admit;
    SearchLayout layout;
    int64_t footprint = 0;  // bytes that the search needs; its block holds layout.total
    size_t arena_off = 0;
    int32_t chunk = 1;
    int32_t W = 64;
    int32_t window_method = 2;  // the context's, for which the block is laid out
    int32_t lane = -1;
    int32_t status = FH_OK;
    double device_ms = 0.0, latency_ms = 0.0, queue_ms = 0.0;
};

struct Lane {
    hipStream_t st = nullptr;
    hipEvent_t ev_start = nullptr, ev_done = nullptr;
    uint64_t req = 0;  // 0 = idle
};

}  // namespace

struct fh_server {
    fh_ctx *ctx = nullptr;
    int64_t budget = 0;
    Arena arena;  // budget bytes of device memory, allocated once at creation
    int32_t max_queue = 0;
    std::vector<Lane> lanes;
    std::deque<uint64_t> queue;
    std::map<uint64_t, ServerRequest> reqs;  // queued, running, finished-unreported
    std::deque<uint64_t> finished;
    uint64_t next_id = 1;
    int64_t in_flight = 0;
};

namespace {

void retire_lanes(fh_server *srv) {
    for (size_t li = 0; li < srv->lanes.size(); ++li) {
        Lane &L = srv->lanes[li];
        if (!L.req) continue;
        hipError_t q = hipEventQuery(L.ev_done);
        if (q == hipErrorNotReady) continue;
        ServerRequest &R = srv->reqs[L.req];
        const Clock::time_point now = Clock::now();
        if (q != hipSuccess) {
            R.status = FH_E_DEVICE;
        } else {
            float ms = 0.f;
            if (hipEventElapsedTime(&ms, L.ev_start, L.ev_done) == hipSuccess) R.device_ms = ms;
        }
        R.latency_ms = ms_between(R.t_submit, now);
        srv->arena.release(R.arena_off, R.layout.total);
        srv->in_flight -= (int64_t)R.layout.total;
        srv->finished.push_back(R.id);
        L.req = 0;
    }
}

void admit(fh_server *srv) {
    fh_ctx *ctx = srv->ctx;
    while (!srv->queue.empty()) {
        const uint64_t id = srv->queue.front();
        ServerRequest &R = srv->reqs[id];
        int li = -1;
        for (size_t k = 0; k < srv->lanes.size(); ++k)
            if (!srv->lanes[k].req) { li = (int)k; break; }
        if (li < 0) break;  // wait for a lane
        // arrival order: the head waits until a block for its workspace is free
        size_t off = 0;
        if (!srv->arena.alloc(R.layout.total, &off)) break;
        srv->queue.pop_front();
        Lane &L = srv->lanes[li];
        R.lane = li;
        R.arena_off = off;
        R.t_admit = Clock::now();
        R.queue_ms = ms_between(R.t_submit, R.t_admit);
        const fh_request &q = R.r;
        const Plan p = make_plan(q.grid, R.W);
        // the workspace is the arena block: nothing is allocated or freed here
        ChunkBufs b = carve(srv->arena.base + off, R.layout, (int32_t *)ctx->err.ptr);
        fh_status s = FH_OK;
        SkyDirs dirs;
        if (q.n_sky <= kArgSky)
            dirs = {R.sky.data(), q.n_sky};
        else if (hipMemcpyAsync(b.sky, R.sky.data(), (size_t)24 * q.n_sky, hipMemcpyHostToDevice, L.st) != hipSuccess)
            s = fail(FH_E_DEVICE, "copying the request's sky vectors failed");
        if (!s && hipEventRecord(L.ev_start, L.st) != hipSuccess) s = fail(FH_E_DEVICE, "hipEventRecord");
        const int32_t method = ctx->window_method;
        ctx->window_method = R.window_method;
        if (!s)
            s = run_search(ctx, q.pm, &q.grid, p, R.chunk, q.n_sky, q.d_w, q.w_stride,
                           FH_SCHED_PERSISTENT, &q.sel, q.d_out, b, L.st, dirs);
        ctx->window_method = method;
        if (hipEventRecord(L.ev_done, L.st) != hipSuccess && !s) s = fail(FH_E_DEVICE, "hipEventRecord");
        R.status = s;
        srv->in_flight += (int64_t)R.layout.total;
        L.req = id;
    }
}

}  // namespace

extern "C" {

fh_status fh_server_create(fh_ctx *ctx, int64_t hbm_budget, int32_t lanes, int32_t max_queue,
                           fh_server **out) {
    fh_status s;
    if (!out) return fail(FH_E_INVALID, "out is NULL");
    *out = nullptr;
    if ((s = check_ctx(ctx))) return s;
    if (hbm_budget <= 0) return fail(FH_E_INVALID, "hbm_budget must be > 0");
    if (lanes < 1 || lanes > 16) return fail(FH_E_INVALID, "lanes=%d outside 1..16", lanes);
    if (max_queue < 1) return fail(FH_E_INVALID, "max_queue must be >= 1");
    // the arena is carved in 256-byte pieces
    const int64_t budget = hbm_budget / 256 * 256;
    if (budget <= 0) return fail(FH_E_INVALID, "hbm_budget must be at least 256 bytes");
    void *mem = ctx->spare.allocate((size_t)budget);
    if (!mem) return fail(FH_E_NOMEM, "allocating the server's %lld-byte arena failed", (long long)budget);
    fh_server *srv = new fh_server();
    srv->ctx = ctx;
    srv->budget = budget;
    srv->arena.reset(static_cast<char *>(mem), (size_t)budget);
    srv->max_queue = max_queue;
    srv->lanes.resize(lanes);
    for (Lane &L : srv->lanes) {
        if (hipStreamCreateWithFlags(&L.st, hipStreamNonBlocking) != hipSuccess ||
            hipEventCreate(&L.ev_start) != hipSuccess || hipEventCreate(&L.ev_done) != hipSuccess) {
            fh_server_destroy(srv);
            return fail(FH_E_DEVICE, "creating the server's streams failed");
        }
    }
    *out = srv;
    return FH_OK;
}

fh_status fh_server_submit(fh_server *srv, const fh_request *req, uint64_t *id) {
    fh_status s;
    if (!srv) return fail(FH_E_INVALID, "server is NULL");
    if (!req || !id) return fail(FH_E_INVALID, "request or id is NULL");
    fh_ctx *ctx = srv->ctx;
    if ((s = check_ctx(ctx))) return s;
    if ((s = check_grid(req->pm, &req->grid))) return s;
    if (req->n_sky < 1 || !req->sky) return fail(FH_E_INVALID, "request needs n_sky >= 1 and sky");
    for (int32_t k = 0; k < req->n_sky; ++k)
        if ((s = check_sky(req->sky + 3 * (int64_t)k))) return s;
    const fh_select &sel = req->sel;
    if (sel.width < 1 || sel.excl < 0 || !std::isfinite(sel.theta) || !(sel.theta > 0))
        return fail(FH_E_INVALID, "selection needs width >= 1, excl >= 0, theta > 0");
    if (!req->d_out) return fail(FH_E_INVALID, "output pointer is NULL");
    if (req->d_w && req->w_stride != 0 && req->w_stride != req->pm->n_fft)
        return fail(FH_E_INVALID, "w_stride must be 0 or n_fft");
    if ((int32_t)srv->queue.size() >= srv->max_queue) return fail(FH_E_BUSY, "request queue is full");
    ServerRequest R;
    R.id = srv->next_id++;
    R.r = *req;
    R.sky.assign(req->sky, req->sky + 3 * (int64_t)req->n_sky);
    R.r.sky = nullptr;
    R.window_method = ctx->window_method;
    R.t_submit = Clock::now();
    // the largest chunk whose search fits one lane's share of the budget, with
    // the default tile width and without what only saves time
    const bool weighted = req->d_w != nullptr;
    const int64_t share = srv->budget / (int64_t)srv->lanes.size();
    auto plan = [&](int chunk, int width, bool parts, bool rank) {
        const Plan p = make_plan(req->grid, width);
        R.W = width;
        R.chunk = (int)std::min<int64_t>(chunk, chunk_by_tiles(p));
        R.layout = search_layout(ctx, req->pm, &req->grid, p, R.chunk, req->n_sky, weighted, rank);
        if (parts) {
            R.layout.part = R.layout.total;
            R.layout.part_bytes =
                (search_parts_bytes(ctx, req->pm, &req->grid, p, R.chunk, req->n_sky) + 255) / 256 * 256;
            R.layout.total += R.layout.part_bytes;
        }
        return (int64_t)R.layout.total;
    };
    const int wide = choose_tile_bins(ctx, req->pm, &req->grid, 0);
    for (int chunk = std::min<int>(req->n_sky, 256); plan(chunk, wide, false, false) > share && R.chunk > 1;)
        chunk = (R.chunk + 1) / 2;
    R.footprint = (int64_t)R.layout.total;
    if (R.footprint > srv->budget) {
        srv->next_id--;
        return fail(FH_E_UNSUPPORTED, "request needs %lld workspace bytes, over the %lld-byte budget",
                    (long long)R.footprint, (long long)srv->budget);
    }
    // and of what saves time, as much as the share has room for: the tile width
    // of a launch of that many directions (more windows), the rank table and
    // partial tiles
    const int chunk = R.chunk, narrow = search_tile_bins(ctx, req->pm, &req->grid, chunk);
    auto fits = [&](int width, bool parts, bool rank) { return plan(chunk, width, parts, rank) <= share && R.chunk == chunk; };
    if (!fits(narrow, true, true) && !fits(narrow, false, true) && !fits(narrow, false, false) && !fits(wide, false, true))
        plan(chunk, wide, false, false);
    *id = R.id;
    srv->reqs[R.id] = std::move(R);
    srv->queue.push_back(*id);
    return FH_OK;
}

fh_status fh_server_poll(fh_server *srv, fh_completion *out, int32_t max, int32_t *n) {
    fh_status s;
    if (!srv || !n) return fail(FH_E_INVALID, "server or n is NULL");
    *n = 0;
    if (max > 0 && !out) return fail(FH_E_INVALID, "out is NULL");
    if ((s = check_ctx(srv->ctx))) return s;
    retire_lanes(srv);
    admit(srv);
    int32_t k = 0;
    while (k < max && !srv->finished.empty()) {
        const uint64_t id = srv->finished.front();
        srv->finished.pop_front();
        const ServerRequest &R = srv->reqs[id];
        fh_completion c{};
        c.id = R.id;
        c.tag = R.r.tag;
        c.status = R.status;
        c.lane = R.lane;
        c.queue_ms = R.queue_ms;
        c.latency_ms = R.latency_ms;
        c.device_ms = R.device_ms;
        c.footprint = R.footprint;
        c.cell_updates = R.r.pm->n_peaks * (int64_t)R.r.grid.ns * R.r.n_sky;
        out[k++] = c;
        srv->reqs.erase(id);
    }
    *n = k;
    return FH_OK;
}

fh_status fh_server_cancel(fh_server *srv, uint64_t id) {
    if (!srv) return fail(FH_E_INVALID, "server is NULL");
    auto it = srv->reqs.find(id);
    if (it == srv->reqs.end()) return fail(FH_E_INVALID, "unknown request id %llu", (unsigned long long)id);
    for (auto q = srv->queue.begin(); q != srv->queue.end(); ++q) {
        if (*q == id) {
            srv->queue.erase(q);
            it->second.status = FH_E_CANCELLED;
            it->second.latency_ms = ms_between(it->second.t_submit, Clock::now());
            srv->finished.push_back(id);
            return FH_OK;
        }
    }
    for (const Lane &L : srv->lanes)
        if (L.req == id) return fail(FH_E_BUSY, "request %llu is running", (unsigned long long)id);
    return fail(FH_E_INVALID, "request %llu has finished", (unsigned long long)id);
}

fh_status fh_server_stats(const fh_server *srv, int32_t *queued, int32_t *running, int32_t *finished,
                          int64_t *bytes_in_flight) {
    if (!srv) return fail(FH_E_INVALID, "server is NULL");
    int32_t r = 0;
    for (const Lane &L : srv->lanes) r += L.req ? 1 : 0;
    if (queued) *queued = (int32_t)srv->queue.size();
    if (running) *running = r;
    if (finished) *finished = (int32_t)srv->finished.size();
    if (bytes_in_flight) *bytes_in_flight = srv->in_flight;
    return FH_OK;
}

fh_status fh_server_drain(fh_server *srv) {
    fh_status s;
    if (!srv) return fail(FH_E_INVALID, "server is NULL");
    if ((s = check_ctx(srv->ctx))) return s;
    // admit and run everything accepted; completions stay for fh_server_poll
    for (;;) {
        retire_lanes(srv);
        admit(srv);
        bool busy = !srv->queue.empty();
        for (const Lane &L : srv->lanes) busy = busy || L.req != 0;
        if (!busy) return FH_OK;
        for (const Lane &L : srv->lanes)
            if (L.req) HIP_OK(hipEventSynchronize(L.ev_done));
    }
}

void fh_server_destroy(fh_server *srv) {
    if (!srv) return;
    if (srv->ctx) (void)hipSetDevice(srv->ctx->device);
    // run everything that was accepted, then release
    fh_server_drain(srv);
    for (Lane &L : srv->lanes) {
        if (L.st) (void)hipStreamSynchronize(L.st);
        if (L.ev_start) (void)hipEventDestroy(L.ev_start);
        if (L.ev_done) (void)hipEventDestroy(L.ev_done);
        if (L.st) (void)hipStreamDestroy(L.st);
    }
    if (srv->arena.base) (void)hipFree(srv->arena.base);
    delete srv;
}

}  // extern "C"
