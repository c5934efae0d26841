// Host side of the C ABI declared in include/gv.h: argument validation,
// workspace layout, launch sequencing, HIP graph capture and tunables.
#include <math.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <limits>
#include <mutex>
#include <new>

#include "gv_internal.h"

namespace gv {

// launchers defined next to their kernels
hipError_t launch_fill_u32(uint32_t* p, uint32_t value, int64_t count, hipStream_t stream);
hipError_t launch_project(const Args& a, hipStream_t stream);
hipError_t launch_scatter(const Args& a, hipStream_t stream);
hipError_t launch_export_records(const Args& a, float* records, int32_t* counts, hipStream_t stream);
hipError_t launch_tile_sort(const Args& a, int64_t segments, hipStream_t stream);
hipError_t launch_composite_fwd(const Args& a, hipStream_t stream);
hipError_t launch_vis_count(const Args& a, uint32_t* counts, hipStream_t stream);
hipError_t launch_loss_finalize(const Args& a, hipStream_t stream);
hipError_t launch_composite_bwd(const Args& a, hipStream_t stream);
hipError_t launch_project_bwd(const Args& a, hipStream_t stream);
int64_t project_bwd_blocks(int64_t n);
int64_t bin_blocks(int64_t n);
int64_t scan_blocks(int64_t count);
hipError_t launch_tile_scan(const Args& a, unsigned long long* tmp, hipStream_t stream);

static thread_local int32_t g_last_hip = 0;
static std::mutex g_tune_mu;
// the autotuner's choice on the 960x540 benchmark clip
constexpr Tuning DEFAULT_TUNE = {128, 1024, 64, 52, std::numeric_limits<int64_t>::max()};
static Tuning g_tune = DEFAULT_TUNE;
static Tuning g_autotuned = DEFAULT_TUNE;  // the last setting that gv_autotune installed

Tuning current_tuning() {
    std::lock_guard<std::mutex> lk(g_tune_mu);
    return g_tune;
}

void install_tuning(const Tuning& t) {
    std::lock_guard<std::mutex> lk(g_tune_mu);
    g_tune = t;
}

static bool same_kernels(const Tuning& a, const Tuning& b) {
    return a.batch == b.batch && a.sort_cap == b.sort_cap && a.bwd_batch == b.bwd_batch && a.compact == b.compact;
}

// The setting that gv_set_tuning's four values stand for: the defaults and the
// last autotuned setting with the launches they adapt to, so that saving and
// restoring them changes nothing, any other as it is.
static void install_values(Tuning t) {
    std::lock_guard<std::mutex> lk(g_tune_mu);
    t.adapt_below = same_kernels(t, DEFAULT_TUNE)  ? DEFAULT_TUNE.adapt_below
                    : same_kernels(t, g_autotuned) ? g_autotuned.adapt_below
                                                   : 0;
    g_tune = t;
}

// Installs the setting measured fastest on launches of `tiles` tiles; on
// those, and larger ones, it runs as it was measured.  Where it has the values
// of the defaults, and they would run other kernels there, it is named by
// another bwd_batch: the one-wave adjoint runs batches of 64 whatever that says.
static Tuning install_autotuned(Tuning t, int64_t tiles) {
    if (same_kernels(t, DEFAULT_TUNE) && tiles <= FWD_QUADRANT_ITEMS) t.bwd_batch = 128;
    t.adapt_below = tiles;
    std::lock_guard<std::mutex> lk(g_tune_mu);
    g_tune = g_autotuned = t;
    return t;
}

static inline size_t align_up(size_t x) { return (x + 255) & ~static_cast<size_t>(255); }

constexpr int64_t K_LIMIT = 0x7fffffffLL;        // positions are u32; keep one bit spare
constexpr size_t PER_ENTRY_BYTES = 16 + 4 + 4 + 36 + 16;  // kv, sgid, sslot, part, tkv

Layout make_layout(const gv_camera& cam, int64_t n, int frames, int64_t k_cap) {
    Layout L{};
    L.n = n;
    L.frames = frames;
    L.width = cam.width;
    L.height = cam.height;
    L.tiles_x = (cam.width + TILE - 1) / TILE;
    L.tiles_y = (cam.height + TILE - 1) / TILE;
    L.tiles = L.tiles_x * L.tiles_y;
    L.pixels = static_cast<int64_t>(cam.width) * cam.height;
    L.k_cap = k_cap;
    const int64_t FN = static_cast<int64_t>(frames) * n;
    const int64_t FT = static_cast<int64_t>(frames) * L.tiles;
    L.pose_blocks = project_bwd_blocks(n);
    L.bin_blocks = L.tiles <= LDS_TILE_LIMIT ? bin_blocks(n) : 0;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t o = off;
        off = align_up(off + bytes);
        return o;
    };
    L.status = take(ST_WORDS * sizeof(uint32_t));
    L.col4 = take(sizeof(ColorOp) * static_cast<size_t>(FN));  // per frame: view-dependent colour
    L.rec = take(sizeof(Record) * static_cast<size_t>(FN));
    L.dkey = take(4 * static_cast<size_t>(FN));
    L.tmask = take(8 * static_cast<size_t>(FN));
    L.rect = take(sizeof(uint2) * static_cast<size_t>(FN));
    L.gcnt = take(4 * static_cast<size_t>(FN));
    L.goff = take(4 * static_cast<size_t>(FN));
    L.tcnt = take(4 * static_cast<size_t>(FT));
    L.toff = take(4 * static_cast<size_t>(FT + 1));
    L.tcur = take(4 * static_cast<size_t>(FT));
    L.bhist = take(4 * static_cast<size_t>(FT) * static_cast<size_t>(L.bin_blocks));
    L.scan_tmp = take(8 * static_cast<size_t>(scan_blocks(FT) + 1));
    L.tfin = take(4 * static_cast<size_t>(frames) * L.pixels);
    L.nlast = take(4 * static_cast<size_t>(frames) * L.pixels);
    L.loss_part = take(4 * static_cast<size_t>(FT));
    L.shapes = take(sizeof(ShapeD) * static_cast<size_t>(n));
    L.pose_part = take(8 * 12 * static_cast<size_t>(L.pose_blocks) * frames);
    L.intr_part = take(8 * 4 * static_cast<size_t>(L.pose_blocks));
    L.vis = take((static_cast<size_t>(FN) + 3) / 4 * 4);
    const size_t K = static_cast<size_t>(k_cap);
    L.kv = take(sizeof(KeySlot) * K);
    L.sgid = take(4 * K);
    L.sslot = take(4 * K);
    L.part = take(4 * PART * K);
    L.pused = take(4 * (K / 32 + 2));
    L.tkv = take(sizeof(KeySlot) * K);
    L.total = off;
    return L;
}

// Largest k with make_layout(k).total <= ws_bytes (0 if even k = 0 does not fit).
static int64_t capacity_for(const gv_camera& cam, int64_t n, int frames, size_t ws_bytes) {
    const size_t fixed = make_layout(cam, n, frames, 0).total;
    if (ws_bytes < fixed) return 0;
    int64_t lo = 0;
    int64_t hi = std::min<int64_t>(K_LIMIT, static_cast<int64_t>((ws_bytes - fixed) / PER_ENTRY_BYTES) + 1);
    while (lo < hi) {
        const int64_t mid = lo + (hi - lo + 1) / 2;
        if (make_layout(cam, n, frames, mid).total <= ws_bytes) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

static bool camera_ok(const gv_camera* c) {
    if (!c) return false;
    if (c->width < 1 || c->height < 1 || c->width > 16384 || c->height > 16384) return false;
    const float v[] = {c->fx, c->fy, c->cx, c->cy, c->near_plane, c->dilation, c->bg[0], c->bg[1], c->bg[2]};
    for (float x : v)
        if (!isfinite(x)) return false;
    return c->fx > 0.f && c->fy > 0.f && c->near_plane > 0.f && c->dilation >= 0.f;
}

static bool scene_ok(const gv_scene* s) {
    if (!s) return false;
    if (s->n < 0 || s->n > K_LIMIT) return false;
    if (s->dtype != GV_F32 && s->dtype != GV_BF16) return false;
    if (s->n_ctrl != 0 && (s->n_ctrl < 4 || s->n_ctrl > GV_MAX_CTRL || !s->ctrl || s->mean_coeffs)) return false;
    if (s->n_ctrl == 0 && s->ctrl) return false;
    if (s->sh_degree < 0 || s->sh_degree > GV_MAX_SH_DEGREE || (s->sh_degree > 0) != (s->sh != nullptr)) return false;
    const bool means_ok = s->means || s->n_ctrl > 0;
    if (s->n > 0 && (!means_ok || !s->log_scales || !s->quats || !s->opacity_logits || !s->colors)) return false;
    return true;
}

static void set_grads(Args& a, const gv_grads* g) {
    a.g_means = g->means;
    a.g_log_scales = g->log_scales;
    a.g_quats = g->quats;
    a.g_opacity = g->opacity_logits;
    a.g_colors = g->colors;
    a.g_coeffs = g->mean_coeffs;
    a.g_ctrl = g->ctrl;
    a.g_scale_coeffs = g->scale_coeffs;
    a.g_quat_coeffs = g->quat_coeffs;
    a.g_sh = g->sh;
    a.g_intr = g->intrinsics;
}

static gv_status hip_status(hipError_t e) {
    if (e == hipSuccess) return GV_OK;
    g_last_hip = static_cast<int32_t>(e);
    return GV_ERR_HIP;
}

#define GV_TRY(expr)                                  \
    do {                                              \
        const hipError_t e_ = (expr);                 \
        if (e_ != hipSuccess) return hip_status(e_);  \
    } while (0)

// Fill the kernel argument block for `frames` frames over workspace `ws`.
static gv_status make_args(const gv_scene* s, const gv_camera* c, int frames, const float* poses, const float* times,
                           void* ws, size_t ws_bytes, Args& a, Layout& L) {
    if (!scene_ok(s) || !camera_ok(c) || frames < 1 || frames > 65535 || !poses) return GV_ERR_INVALID_ARG;
    if (!ws || (reinterpret_cast<uintptr_t>(ws) & 255u) != 0u) return GV_ERR_WORKSPACE;
    const int64_t k = capacity_for(*c, s->n, frames, ws_bytes);
    L = make_layout(*c, s->n, frames, k);
    if (L.total > ws_bytes) return GV_ERR_WORKSPACE;
    memset(&a, 0, sizeof(a));
    a.n = s->n;
    a.dtype = s->dtype;
    a.means = s->means;
    a.log_scales = s->log_scales;
    a.quats = s->quats;
    a.opacity_logits = s->opacity_logits;
    a.colors = s->colors;
    a.mean_coeffs = s->mean_coeffs;
    a.n_ctrl = s->n_ctrl;
    a.ctrl = s->ctrl;
    a.scale_coeffs = s->scale_coeffs;
    a.quat_coeffs = s->quat_coeffs;
    a.sh_degree = s->sh_degree;
    a.sh = s->sh;
    a.width = c->width;
    a.height = c->height;
    a.tiles_x = L.tiles_x;
    a.tiles_y = L.tiles_y;
    a.tiles = L.tiles;
    a.fx = c->fx; a.fy = c->fy; a.cx = c->cx; a.cy = c->cy;
    a.near_plane = c->near_plane;
    a.dilation = c->dilation;
    for (int i = 0; i < 3; ++i) a.bg[i] = c->bg[i];
    a.frames = frames;
    a.poses = poses;
    a.times = times;
    char* b = static_cast<char*>(ws);
    a.status = reinterpret_cast<uint32_t*>(b + L.status);
    a.col4 = reinterpret_cast<ColorOp*>(b + L.col4);
    a.col_stride = s->sh_degree > 0 ? s->n : 0;
    a.rec = reinterpret_cast<Record*>(b + L.rec);
    a.dkey = reinterpret_cast<float*>(b + L.dkey);
    a.rect = reinterpret_cast<uint2*>(b + L.rect);
    a.tmask = reinterpret_cast<uint64_t*>(b + L.tmask);
    a.gcnt = reinterpret_cast<uint32_t*>(b + L.gcnt);
    a.goff = reinterpret_cast<uint32_t*>(b + L.goff);
    a.tcnt = reinterpret_cast<uint32_t*>(b + L.tcnt);
    a.toff = reinterpret_cast<uint32_t*>(b + L.toff);
    a.tcur = reinterpret_cast<uint32_t*>(b + L.tcur);
    a.bhist = L.bin_blocks > 0 ? reinterpret_cast<uint32_t*>(b + L.bhist) : nullptr;
    a.bin_blocks = static_cast<int>(L.bin_blocks);
    a.bin_rounds = BIN_GROUP / 256;
    a.tfin = reinterpret_cast<float*>(b + L.tfin);
    a.nlast = reinterpret_cast<uint32_t*>(b + L.nlast);
    a.loss_part = reinterpret_cast<float*>(b + L.loss_part);
    a.shapes = reinterpret_cast<ShapeD*>(b + L.shapes);
    a.pose_part = reinterpret_cast<double*>(b + L.pose_part);
    a.intr_part = reinterpret_cast<double*>(b + L.intr_part);
    a.kv = reinterpret_cast<KeySlot*>(b + L.kv);
    a.sgid = reinterpret_cast<uint32_t*>(b + L.sgid);
    a.sslot = reinterpret_cast<uint32_t*>(b + L.sslot);
    a.part = reinterpret_cast<float*>(b + L.part);
    a.pused = reinterpret_cast<uint32_t*>(b + L.pused);
    a.tkv = reinterpret_cast<KeySlot*>(b + L.tkv);
    a.k_cap = L.k_cap;
    // Binning workgroups of 256 Gaussians where those of BIN_GROUP would leave
    // CUs idle, if their histograms (four times as many) fit in the sort's merge
    // scratch, which nothing uses before the sort.  Projection and scatter with
    // the larger and the smaller ones, by number of the larger: 2 (2k Gaussians,
    // 64 tiles) 26 + 12 against 15 + 8 us, 20 (20k, 300 tiles) 26 + 12 against
    // 16 + 9, 98 (100k, 2,040 tiles) 39 + 21 against 28 + 20; 392 (four such frames)
    // 43 + 52 against 58 + 59, as every workgroup stores a count for every tile.
    constexpr int64_t BIN_FEW = 128;
    const int64_t fine = (s->n + 255) / 256;
    if (L.bin_blocks > 0 && L.bin_blocks * frames < BIN_FEW &&
        4 * fine * frames * L.tiles <= static_cast<int64_t>(sizeof(KeySlot)) * L.k_cap) {
        a.bhist = reinterpret_cast<uint32_t*>(a.tkv);
        a.bin_blocks = static_cast<int>(fine);
        a.bin_rounds = 1;
    }
    a.tune = current_tuning();
    return GV_OK;
}

static unsigned long long* scan_tmp(const Args& a, const Layout& L) {
    return reinterpret_cast<unsigned long long*>(reinterpret_cast<char*>(a.status) - L.status + L.scan_tmp);
}

// Scratch of gv_render_fwd_noalloc: a fixed device array, one copy per GPU
// (each device holds its own at its own address until the process ends).
// Host code never uses the array's name as an address: the address is taken
// once per device with hipGetSymbolAddress, with that device current, and
// kept in g_scratch_ptr.
constexpr size_t NOALLOC_SCRATCH_BYTES = GV_NOALLOC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[NOALLOC_SCRATCH_BYTES];
constexpr int MAX_DEVICES = 64;
static std::mutex g_scratch_mu;
static void* g_scratch_ptr[MAX_DEVICES] = {};

static gv_status scratch_of_current_device(void** out) {
    int dev = -1;
    GV_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= MAX_DEVICES) return GV_ERR_UNSUPPORTED;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        GV_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p || (reinterpret_cast<uintptr_t>(p) & 255u) != 0u) return GV_ERR_HIP;
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return GV_OK;
}

// Optional HIP events between the stages of a launch sequence (GV_STAGES).
struct StageTimer {
    hipEvent_t ev[GV_STAGES + 1];
    hipStream_t st;
    void mark(int i) {
        if (i >= 0 && i <= GV_STAGES) hipEventRecord(ev[i], st);
    }
};

static inline void mark(StageTimer* tm, int i) {
    if (tm) tm->mark(i);
}

// Words of host memory through which a frame's intersection count reaches the
// host while the kernels behind the scan run: one page for the process, taken
// on first use and kept, a word per call in flight.  With the count copied to
// the host before the scatter was launched, the GPU idled through the copy, the
// host's wake-up and the next launch: forward and backward of one 128x128 frame
// 112 against 79 us, of one 960x540 frame of 100k Gaussians 280 against 246.
class TotalSlots {
  public:
    // A word, zero, or nullptr if all are in use or there is no host memory.
    unsigned long long* take() {
        std::lock_guard<std::mutex> lk(mu_);
        if (!page_ && !failed_) {
            void* p = nullptr;
            // another thread may be capturing a graph
            hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
            const bool relaxed = hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess;
            failed_ = hipHostMalloc(&p, COUNT * STRIDE * sizeof(unsigned long long),
                                    hipHostMallocPortable | hipHostMallocMapped | hipHostMallocCoherent) != hipSuccess;
            if (relaxed) static_cast<void>(hipThreadExchangeStreamCaptureMode(&mode));
            if (failed_) static_cast<void>(hipGetLastError());
            else page_ = static_cast<unsigned long long*>(p);
        }
        if (!page_ || !free_) return nullptr;
        const int k = __builtin_ctzll(free_);
        free_ &= free_ - 1;
        __atomic_store_n(page_ + k * STRIDE, 0ull, __ATOMIC_RELEASE);
        return page_ + k * STRIDE;
    }
    void give_back(unsigned long long* p) {
        std::lock_guard<std::mutex> lk(mu_);
        free_ |= 1ull << ((p - page_) / STRIDE);
    }

  private:
    static constexpr int COUNT = 64, STRIDE = 8;  // a cache line each
    std::mutex mu_;
    unsigned long long* page_ = nullptr;
    bool failed_ = false;
    uint64_t free_ = ~0ull;
};
static TotalSlots g_totals;

// Waits for the scan to write *word; GV_ERR_CAPACITY beyond k_cap.  Ends with
// the stream's work at the latest.  Only a written word may be used again.
static gv_status wait_for_total(unsigned long long* word, int64_t k_cap, hipStream_t st) {
    unsigned long long v = 0;
    for (uint32_t spin = 1; !(v = __atomic_load_n(word, __ATOMIC_ACQUIRE)); ++spin) {
        __builtin_ia32_pause();
        if (spin % 8192u) continue;
        const hipError_t e = hipStreamQuery(st);
        if (e == hipErrorNotReady) continue;
        v = __atomic_load_n(word, __ATOMIC_ACQUIRE);
        if (!v) return e == hipSuccess ? GV_ERR_HIP : hip_status(e);
        break;
    }
    g_totals.give_back(word);
    return v - 1 > static_cast<unsigned long long>(k_cap) ? GV_ERR_CAPACITY : GV_OK;
}

// Projection, binning and scans; optionally reads the intersection count back.
static gv_status enqueue_binning(const Args& a, const Layout& L, hipStream_t st, bool readback,
                                 StageTimer* tm = nullptr) {
    const int64_t FT = static_cast<int64_t>(a.frames) * a.tiles;
    mark(tm, 0);
    GV_TRY(launch_project(a, st));
    mark(tm, 1);
    GV_TRY(launch_tile_scan(a, scan_tmp(a, L), st));
    mark(tm, 2);
    if (readback) {
        uint32_t k2[2] = {0, 0};
        GV_TRY(hipMemcpyAsync(k2, a.status + ST_K_LO, sizeof(k2), hipMemcpyDeviceToHost, st));
        GV_TRY(hipStreamSynchronize(st));
        const uint64_t K = static_cast<uint64_t>(k2[0]) | (static_cast<uint64_t>(k2[1]) << 32);
        if (K > static_cast<uint64_t>(a.k_cap)) return GV_ERR_CAPACITY;
    }
    GV_TRY(launch_scatter(a, st));
    mark(tm, 3);
    GV_TRY(launch_tile_sort(a, FT, st));
    mark(tm, 4);
    return GV_OK;
}

static gv_status enqueue_batch(const gv_scene* scene, const gv_camera* cam, const float* poses, const float* times,
                               int32_t frames, const float* targets, const float* dL_dimages, uint32_t flags,
                               float* images, float* loss, gv_grads* grads, float* dL_dposes, void* ws,
                               size_t ws_bytes, hipStream_t st, StageTimer* tm = nullptr) {
    if ((flags & ~(GV_FWD | GV_BWD | GV_LOSS_L2 | GV_ACCUMULATE)) != 0u || !(flags & (GV_FWD | GV_BWD)))
        return GV_ERR_INVALID_ARG;
    if (!images) return GV_ERR_INVALID_ARG;
    if ((flags & GV_LOSS_L2) && !targets) return GV_ERR_INVALID_ARG;
    if ((flags & GV_BWD) && !(flags & GV_LOSS_L2) && !dL_dimages) return GV_ERR_INVALID_ARG;
    if ((flags & GV_BWD) && !grads) return GV_ERR_INVALID_ARG;
    Args a;
    Layout L;
    gv_status s = make_args(scene, cam, frames, poses, times, ws, ws_bytes, a, L);
    if (s != GV_OK) return s;
    a.images = images;
    const double denom = 3.0 * static_cast<double>(L.pixels) * frames;
    if (flags & GV_LOSS_L2) {
        a.targets = targets;
        a.loss = loss;
        a.loss_norm = static_cast<float>(1.0 / denom);
        a.loss_scale = static_cast<float>(2.0 / denom);
    }
    a.dl_dimages = (flags & GV_LOSS_L2) ? nullptr : dL_dimages;
    if (grads) set_grads(a, grads);
    a.g_poses = dL_dposes;
    a.accumulate = (flags & GV_ACCUMULATE) ? 1 : 0;
    if (flags & GV_FWD) {
        s = enqueue_binning(a, L, st, false, tm);
        if (s != GV_OK) return s;
        GV_TRY(launch_composite_fwd(a, st));
        mark(tm, 5);
        if (a.loss) GV_TRY(launch_loss_finalize(a, st));
        mark(tm, 6);
    } else {
        for (int i = 0; i <= 6; ++i) mark(tm, i);
    }
    if (flags & GV_BWD) {
        GV_TRY(launch_composite_bwd(a, st));
        mark(tm, 7);
        GV_TRY(launch_project_bwd(a, st));
        mark(tm, 8);
    } else {
        mark(tm, 7);
        mark(tm, 8);
    }
    return GV_OK;
}

}  // namespace gv

using namespace gv;

struct gv_graph {
    hipGraph_t graph;
    hipGraphExec_t exec;
};


static gv_status render_fwd(const gv_scene* scene, const gv_camera* cam, const float* pose7, float t, float* image,
                            float* T_final, void* ws, size_t ws_bytes, void* stream, bool host_word) {
    if (!image) return GV_ERR_INVALID_ARG;
    Args a;
    Layout L;
    gv_status s = make_args(scene, cam, 1, pose7, nullptr, ws, ws_bytes, a, L);
    if (s != GV_OK) return s;
    hipStream_t st = static_cast<hipStream_t>(stream);
    a.t0 = t;
    a.images = image;
    a.tfin_out = T_final;
    // a capturing stream cannot be waited for: there the copy reports the error
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (host_word && hipStreamIsCapturing(st, &capture) != hipSuccess) {
        static_cast<void>(hipGetLastError());
        host_word = false;
    }
    a.total_out = host_word && capture == hipStreamCaptureStatusNone ? g_totals.take() : nullptr;
    s = enqueue_binning(a, L, st, !a.total_out);
    if (s != GV_OK) return s;
    GV_TRY(launch_composite_fwd(a, st));
    return a.total_out ? wait_for_total(a.total_out, a.k_cap, st) : GV_OK;
}

extern "C" {

gv_status gv_workspace_bytes(const gv_camera* cam, int64_t n, int32_t frames, int64_t k_capacity, size_t* out) {
    if (!camera_ok(cam) || n < 0 || n > K_LIMIT || frames < 1 || frames > 65535 || k_capacity < 0 ||
        k_capacity > K_LIMIT || !out)
        return GV_ERR_INVALID_ARG;
    *out = make_layout(*cam, n, frames, k_capacity).total;
    return GV_OK;
}

gv_status gv_workspace_capacity(const gv_camera* cam, int64_t n, int32_t frames, size_t ws_bytes, int64_t* out) {
    if (!camera_ok(cam) || n < 0 || n > K_LIMIT || frames < 1 || frames > 65535 || !out) return GV_ERR_INVALID_ARG;
    *out = capacity_for(*cam, n, frames, ws_bytes);
    return GV_OK;
}

gv_status gv_project_fwd(const gv_scene* scene, const gv_camera* cam, const float* pose7, float t, float* records,
                         int32_t* tile_counts, void* ws, size_t ws_bytes, void* stream) {
    if (!records || !tile_counts) return GV_ERR_INVALID_ARG;
    Args a;
    Layout L;
    gv_status s = make_args(scene, cam, 1, pose7, nullptr, ws, ws_bytes, a, L);
    if (s != GV_OK) return s;
    hipStream_t st = static_cast<hipStream_t>(stream);
    a.t0 = t;
    // the slots of a forward on this workspace stay (the count pass hands them
    // out in another order every time), so that its backward still finds them
    a.goff = nullptr;
    a.pused = nullptr;
    GV_TRY(launch_project(a, st));
    GV_TRY(launch_export_records(a, records, tile_counts, st));
    return GV_OK;
}

gv_status gv_render_fwd(const gv_scene* scene, const gv_camera* cam, const float* pose7, float t, float* image,
                        float* T_final, void* ws, size_t ws_bytes, void* stream) {
    return render_fwd(scene, cam, pose7, t, image, T_final, ws, ws_bytes, stream, true);
}

gv_status gv_render_fwd_noalloc(const gv_scene* scene, const gv_camera* cam, const float* pose7, float t,
                                float* image, float* T_final, void* stream) {
    if (!image || !pose7 || !scene_ok(scene) || !camera_ok(cam)) return GV_ERR_INVALID_ARG;
    // the frame's fixed arrays must fit before the device is touched
    if (make_layout(*cam, scene->n, 1, 0).total > NOALLOC_SCRATCH_BYTES) return GV_ERR_WORKSPACE;
    void* ws = nullptr;
    const gv_status s = scratch_of_current_device(&ws);
    if (s != GV_OK) return s;
    return render_fwd(scene, cam, pose7, t, image, T_final, ws, NOALLOC_SCRATCH_BYTES, stream, false);
}

gv_status gv_render_bwd(const gv_scene* scene, const gv_camera* cam, const float* pose7, float t, const float* image,
                        const float* dL_dimage, const float* target, float loss_scale, uint32_t flags, gv_grads* grads,
                        float* dL_dpose7, void* ws, size_t ws_bytes, void* stream) {
    if ((flags & ~(GV_LOSS_L2 | GV_ACCUMULATE | GV_BWD | GV_FWD)) != 0u || !grads || !image) return GV_ERR_INVALID_ARG;
    if ((flags & GV_LOSS_L2) ? !target : !dL_dimage) return GV_ERR_INVALID_ARG;
    if (!isfinite(loss_scale)) return GV_ERR_INVALID_ARG;
    Args a;
    Layout L;
    gv_status s = make_args(scene, cam, 1, pose7, nullptr, ws, ws_bytes, a, L);
    if (s != GV_OK) return s;
    hipStream_t st = static_cast<hipStream_t>(stream);
    a.t0 = t;
    a.images = const_cast<float*>(image);
    if (flags & GV_LOSS_L2) {
        a.targets = target;
        a.loss_scale = loss_scale;
    } else {
        a.dl_dimages = dL_dimage;
    }
    set_grads(a, grads);
    a.g_poses = dL_dpose7;
    a.accumulate = (flags & GV_ACCUMULATE) ? 1 : 0;
    GV_TRY(launch_composite_bwd(a, st));
    GV_TRY(launch_project_bwd(a, st));
    return GV_OK;
}

gv_status gv_render_batch(const gv_scene* scene, const gv_camera* cam, const float* poses, const float* times,
                          int32_t frames, const float* targets, const float* dL_dimages, uint32_t flags, float* images,
                          float* loss, gv_grads* grads, float* dL_dposes, void* ws, size_t ws_bytes, void* stream) {
    return enqueue_batch(scene, cam, poses, times, frames, targets, dL_dimages, flags, images, loss, grads, dL_dposes,
                         ws, ws_bytes, static_cast<hipStream_t>(stream));
}

gv_status gv_visibility_counts(const gv_scene* scene, const gv_camera* cam, const float* poses, const float* times,
                               int32_t frames, float* images, uint32_t* counts, void* ws, size_t ws_bytes,
                               void* stream) {
    if (!counts || !images) return GV_ERR_INVALID_ARG;
    Args a;
    Layout L;
    gv_status s = make_args(scene, cam, frames, poses, times, ws, ws_bytes, a, L);
    if (s != GV_OK) return s;
    hipStream_t st = static_cast<hipStream_t>(stream);
    a.images = images;
    a.vis = reinterpret_cast<uint8_t*>(static_cast<char*>(ws) + L.vis);
    const int64_t FN = static_cast<int64_t>(frames) * a.n;
    GV_TRY(launch_fill_u32(reinterpret_cast<uint32_t*>(a.vis), 0u, (FN + 3) / 4, st));
    s = enqueue_binning(a, L, st, false, nullptr);
    if (s != GV_OK) return s;
    GV_TRY(launch_composite_fwd(a, st));
    GV_TRY(launch_vis_count(a, counts, st));
    return GV_OK;
}

gv_status gv_render_batch_timed(const gv_scene* scene, const gv_camera* cam, const float* poses, const float* times,
                                int32_t frames, const float* targets, const float* dL_dimages, uint32_t flags,
                                float* images, float* loss, gv_grads* grads, float* dL_dposes, void* ws,
                                size_t ws_bytes, void* stream, float* stage_ms) {
    if (!stage_ms) return GV_ERR_INVALID_ARG;
    StageTimer tm;
    tm.st = static_cast<hipStream_t>(stream);
    int made = 0;
    hipError_t e = hipSuccess;
    for (; made <= GV_STAGES && e == hipSuccess; ++made) e = hipEventCreate(&tm.ev[made]);
    gv_status s = (e == hipSuccess) ? GV_OK : hip_status(e);
    if (s == GV_OK)
        s = enqueue_batch(scene, cam, poses, times, frames, targets, dL_dimages, flags, images, loss, grads, dL_dposes,
                          ws, ws_bytes, tm.st, &tm);
    if (s == GV_OK) {
        e = hipEventSynchronize(tm.ev[GV_STAGES]);
        if (e != hipSuccess) s = hip_status(e);
    }
    for (int i = 0; i < GV_STAGES; ++i) {
        float ms = 0.f;
        if (s == GV_OK) hipEventElapsedTime(&ms, tm.ev[i], tm.ev[i + 1]);
        stage_ms[i] = ms;
    }
    for (int i = 0; i < made && i <= GV_STAGES; ++i) hipEventDestroy(tm.ev[i]);
    return s;
}

// Instantiate a captured graph and hand it out; every failure path releases
// what was made (no exception crosses the C ABI).
static gv_status finish_graph(gv_status s, hipError_t capture_err, hipGraph_t graph, gv_graph** out) {
    if (s == GV_OK && capture_err != hipSuccess) s = hip_status(capture_err);
    if (s != GV_OK) {
        if (graph) hipGraphDestroy(graph);
        return s;
    }
    hipGraphExec_t exec = nullptr;
    const hipError_t e = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
    if (e != hipSuccess) {
        hipGraphDestroy(graph);
        return hip_status(e);
    }
    gv_graph* g = new (std::nothrow) gv_graph;
    if (!g) {
        hipGraphExecDestroy(exec);
        hipGraphDestroy(graph);
        return GV_ERR_HIP;
    }
    g->graph = graph;
    g->exec = exec;
    *out = g;
    return GV_OK;
}

gv_status gv_batch_graph_create(const gv_scene* scene, const gv_camera* cam, const float* poses, const float* times,
                                int32_t frames, const float* targets, const float* dL_dimages, uint32_t flags,
                                float* images, float* loss, gv_grads* grads, float* dL_dposes, void* ws,
                                size_t ws_bytes, gv_graph** out) {
    if (!out) return GV_ERR_INVALID_ARG;
    *out = nullptr;
    hipStream_t cs;
    GV_TRY(hipStreamCreateWithFlags(&cs, hipStreamNonBlocking));
    hipError_t e = hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal);
    if (e != hipSuccess) {
        hipStreamDestroy(cs);
        return hip_status(e);
    }
    const gv_status s = enqueue_batch(scene, cam, poses, times, frames, targets, dL_dimages, flags, images, loss, grads,
                                      dL_dposes, ws, ws_bytes, cs);
    hipGraph_t graph = nullptr;
    e = hipStreamEndCapture(cs, &graph);
    hipStreamDestroy(cs);
    return finish_graph(s, e, graph, out);
}

gv_status gv_fit_graph_create(const gv_scene* scene, const gv_camera* cam, const float* theta, const float* z0,
                              int32_t substeps, void* ode_ws, size_t ode_ws_bytes, const float* times, int32_t frames,
                              const float* targets, const float* dL_dimages, float* poses, float* images, float* loss,
                              gv_grads* grads, float* dL_dposes, float* dtheta, float* dz0, void* ws, size_t ws_bytes,
                              gv_graph** out) {
    if (!out || !theta || !z0 || !poses || !dL_dposes || !dtheta || !dz0 || !grads) return GV_ERR_INVALID_ARG;
    if ((targets == nullptr) == (dL_dimages == nullptr)) return GV_ERR_INVALID_ARG;
    *out = nullptr;
    const uint32_t flags = GV_FWD | GV_BWD | (targets ? GV_LOSS_L2 : 0u);
    hipStream_t cs;
    GV_TRY(hipStreamCreateWithFlags(&cs, hipStreamNonBlocking));
    hipError_t e = hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal);
    if (e != hipSuccess) {
        hipStreamDestroy(cs);
        return hip_status(e);
    }
    gv_status s = gv_camera_ode_fwd(theta, z0, frames, substeps, poses, ode_ws, ode_ws_bytes, cs);
    if (s == GV_OK)
        s = enqueue_batch(scene, cam, poses, times, frames, targets, dL_dimages, flags, images, loss, grads, dL_dposes,
                          ws, ws_bytes, cs);
    if (s == GV_OK)
        s = gv_camera_ode_bwd(theta, z0, frames, substeps, dL_dposes, dtheta, dz0, ode_ws, ode_ws_bytes, cs);
    hipGraph_t graph = nullptr;
    e = hipStreamEndCapture(cs, &graph);
    hipStreamDestroy(cs);
    return finish_graph(s, e, graph, out);
}

gv_status gv_batch_graph_launch(gv_graph* graph, void* stream) {
    if (!graph) return GV_ERR_INVALID_ARG;
    GV_TRY(hipGraphLaunch(graph->exec, static_cast<hipStream_t>(stream)));
    return GV_OK;
}

gv_status gv_batch_graph_destroy(gv_graph* graph) {
    if (!graph) return GV_ERR_INVALID_ARG;
    hipGraphExecDestroy(graph->exec);
    hipGraphDestroy(graph->graph);
    delete graph;
    return GV_OK;
}

gv_status gv_get_tuning(gv_tuning* out) {
    if (!out) return GV_ERR_INVALID_ARG;
    const Tuning t = current_tuning();
    memset(out, 0, sizeof(*out));
    out->batch = t.batch;
    out->sort_cap = t.sort_cap;
    out->compact = t.compact;
    out->bwd_batch = t.bwd_batch;
    return GV_OK;
}

static bool batch_ok(int b) { return b == 64 || b == 128 || b == 256; }

gv_status gv_set_tuning(const gv_tuning* t) {
    if (!t) return GV_ERR_INVALID_ARG;
    if (!batch_ok(t->batch)) return GV_ERR_INVALID_ARG;
    if (t->bwd_batch != 0 && !batch_ok(t->bwd_batch)) return GV_ERR_INVALID_ARG;
    if (t->sort_cap != 512 && t->sort_cap != 1024 && t->sort_cap != 2048 && t->sort_cap != 4096)
        return GV_ERR_INVALID_ARG;
    if (t->compact < 0 || t->compact > 63) return GV_ERR_INVALID_ARG;
    Tuning n = current_tuning();
    n.batch = t->batch;
    n.bwd_batch = t->bwd_batch ? t->bwd_batch : t->batch;
    n.sort_cap = t->sort_cap;
    n.compact = t->compact;
    install_values(n);
    return GV_OK;
}

// Key of a tuning-cache line: the settings of one problem shape.
struct TuneKey {
    char arch[32];
    int width, height, n_bucket, frames, dtype, dynamics, sh_degree;
};

static bool same_key(const TuneKey& a, const TuneKey& b) {
    return strcmp(a.arch, b.arch) == 0 && a.width == b.width && a.height == b.height && a.n_bucket == b.n_bucket &&
           a.frames == b.frames && a.dtype == b.dtype && a.dynamics == b.dynamics && a.sh_degree == b.sh_degree;
}

static const char* TUNE_LINE =
    "{\"arch\": \"%31[^\"]\", \"width\": %d, \"height\": %d, \"n_bucket\": %d, \"frames\": %d, \"dtype\": %d, "
    "\"dynamics\": %d, \"sh_degree\": %d, \"batch\": %d, \"bwd_batch\": %d, \"sort_cap\": %d, \"compact\": %d}";

// The first line of the cache file with this key, if any.
static bool cached_tuning(const char* path, const TuneKey& key, Tuning& out) {
    FILE* fp = fopen(path, "r");
    if (!fp) return false;
    char line[512];
    bool found = false;
    while (!found && fgets(line, sizeof(line), fp)) {
        TuneKey k{};
        Tuning t = current_tuning();
        if (sscanf(line, TUNE_LINE, k.arch, &k.width, &k.height, &k.n_bucket, &k.frames, &k.dtype, &k.dynamics,
                   &k.sh_degree, &t.batch, &t.bwd_batch, &t.sort_cap, &t.compact) == 12 &&
            same_key(k, key)) {
            out = t;
            found = true;
        }
    }
    fclose(fp);
    return found;
}

static bool tuning_valid(const Tuning& t) {
    return batch_ok(t.batch) && batch_ok(t.bwd_batch) &&
           (t.sort_cap == 512 || t.sort_cap == 1024 || t.sort_cap == 2048 || t.sort_cap == 4096) && t.compact >= 0 &&
           t.compact <= 63;
}

gv_status gv_autotune(const gv_scene* scene, const gv_camera* cam, const float* poses, const float* times,
                      int32_t frames, const float* targets, float* images, float* loss, gv_grads* grads,
                      float* dL_dposes, void* ws, size_t ws_bytes, const char* cache_path, gv_tuning* chosen) {
    if (!targets || !images || !grads || !scene_ok(scene) || !camera_ok(cam)) return GV_ERR_INVALID_ARG;
    TuneKey key{};
    {
        int dev = 0;
        hipDeviceProp_t prop;
        if (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&prop, dev) == hipSuccess) {
            const char* c = strchr(prop.gcnArchName, ':');  // drop feature suffixes (":sramecc+:xnack-")
            const size_t len = c ? static_cast<size_t>(c - prop.gcnArchName) : strlen(prop.gcnArchName);
            memcpy(key.arch, prop.gcnArchName, len < sizeof(key.arch) - 1 ? len : sizeof(key.arch) - 1);
        }
        if (!key.arch[0]) strcpy(key.arch, "unknown");
        key.width = cam->width;
        key.height = cam->height;
        key.n_bucket = scene->n > 0 ? static_cast<int>(floor(4.0 * log2(static_cast<double>(scene->n)))) : -1;
        key.frames = frames;
        key.dtype = scene->dtype;
        key.dynamics = (scene->mean_coeffs ? 1 : 0) | (scene->n_ctrl > 0 ? 2 : 0) |
                       (scene->scale_coeffs || scene->quat_coeffs ? 4 : 0);
        key.sh_degree = scene->sh_degree;
    }
    Tuning best = current_tuning();
    const int64_t tiles = static_cast<int64_t>((cam->width + TILE - 1) / TILE) * ((cam->height + TILE - 1) / TILE) * frames;
    if (cache_path && cached_tuning(cache_path, key, best) && tuning_valid(best)) {
        best = install_autotuned(best, tiles);
        if (chosen) {
            memset(chosen, 0, sizeof(*chosen));
            chosen->batch = best.batch;
            chosen->sort_cap = best.sort_cap;
            chosen->compact = best.compact;
            chosen->bwd_batch = best.bwd_batch;
        }
        return GV_OK;
    }
    const uint32_t flags = GV_FWD | GV_BWD | GV_LOSS_L2;
    hipStream_t st;
    GV_TRY(hipStreamCreateWithFlags(&st, hipStreamNonBlocking));
    StageTimer tm;
    tm.st = st;
    int made = 0;
    hipError_t he = hipSuccess;
    for (; made <= GV_STAGES && he == hipSuccess; ++made) he = hipEventCreate(&tm.ev[made]);
    const Tuning saved = current_tuning();
    gv_status result = (he == hipSuccess) ? GV_OK : hip_status(he);
    // The stages are independent (no stage's output depends on another
    // stage's kernel variant), so every stage keeps its own fastest option,
    // timed on every run that used it.  Options: forward kernel (4x4-block,
    // quadrant, compacted, or one wave per tile) x LDS batch (64, 128, 256);
    // backward kernel
    // (one quadrant per wave at batch 64, 128, 256; two quadrants per wave at
    // batch 64, 128; four quadrants per wave at batch 64); sort capacity
    // (512 ... 4096).  Run c takes forward option c, backward option c mod 6
    // and sort option c mod 4, so twelve runs per round try every option of
    // every stage.  The compacted backward (LDS atomics per lane)
    // measured ten times slower than the quadrant backward on every clip
    // tried and is left to gv_set_tuning.
    constexpr int NF = 12, NB = 6, NS = 4;
    const int f_kernel[4] = {0, 4, 1, 36};
    const int batches[3] = {64, 128, 256};
    const int b_batch[NB] = {64, 128, 256, 64, 128, 64};
    const int b_pair[NB] = {0, 0, 0, 8, 8, 16};
    const int caps[NS] = {512, 1024, 2048, 4096};
    float fwd_ms[NF] = {}, bwd_ms[NB] = {}, sort_ms[NS] = {};
    int fwd_n[NF] = {}, bwd_n[NB] = {}, sort_n[NS] = {};
    // Round-robin over the runs, so that clock or cache drift during the
    // measurement affects all options alike; the first pass warms up.
    constexpr int REPS = 3;
    for (int r = 0; r <= REPS && result == GV_OK; ++r) {
        for (int c = 0; c < NF && result == GV_OK; ++c) {
            Tuning t = saved;
            const int fc = c;
            t.compact = f_kernel[fc / 3] | b_pair[c % NB];
            t.batch = batches[fc % 3];
            t.bwd_batch = b_batch[c % NB];
            t.sort_cap = caps[c % NS];
            t.adapt_below = 0;  // time the kernel named
            install_tuning(t);
            gv_status s = enqueue_batch(scene, cam, poses, times, frames, targets, nullptr, flags, images, loss,
                                        grads, dL_dposes, ws, ws_bytes, st, &tm);
            if (s == GV_OK && hipEventSynchronize(tm.ev[GV_STAGES]) != hipSuccess) s = GV_ERR_HIP;
            uint32_t w[1] = {0};
            if (s == GV_OK && hipMemcpy(w, ws, sizeof(w), hipMemcpyDeviceToHost) != hipSuccess) s = GV_ERR_HIP;
            if (s == GV_OK && w[0]) s = GV_ERR_CAPACITY;
            if (s != GV_OK) {
                result = s;
                break;
            }
            if (r == 0) continue;
            float ms[GV_STAGES];
            for (int i = 0; i < GV_STAGES; ++i) hipEventElapsedTime(&ms[i], tm.ev[i], tm.ev[i + 1]);
            fwd_ms[c] += ms[4];
            fwd_n[c] += 1;
            bwd_ms[c % NB] += ms[6];
            bwd_n[c % NB] += 1;
            sort_ms[c % NS] += ms[3];
            sort_n[c % NS] += 1;
        }
    }
    best = saved;
    if (result == GV_OK) {
        int bf = 0, bb = 0, bs = 0;
        for (int c = 1; c < NF; ++c)
            if (fwd_ms[c] / fwd_n[c] < fwd_ms[bf] / fwd_n[bf]) bf = c;
        for (int c = 1; c < NB; ++c)
            if (bwd_ms[c] / bwd_n[c] < bwd_ms[bb] / bwd_n[bb]) bb = c;
        for (int c = 1; c < NS; ++c)
            if (sort_ms[c] / sort_n[c] < sort_ms[bs] / sort_n[bs]) bs = c;
        best.compact = f_kernel[bf / 3] | b_pair[bb];
        best.batch = batches[bf % 3];
        best.bwd_batch = b_batch[bb];
        best.sort_cap = caps[bs];
    }
    if (result == GV_OK) best = install_autotuned(best, tiles);
    else install_tuning(saved);
    for (int i = 0; i < made && i <= GV_STAGES; ++i) hipEventDestroy(tm.ev[i]);
    hipStreamDestroy(st);
    if (result != GV_OK) return result;
    if (chosen) {
        memset(chosen, 0, sizeof(*chosen));
        chosen->batch = best.batch;
        chosen->sort_cap = best.sort_cap;
        chosen->compact = best.compact;
        chosen->bwd_batch = best.bwd_batch;
    }
    if (cache_path) {
        FILE* fp = fopen(cache_path, "a");
        if (fp) {
            fprintf(fp,
                    "{\"arch\": \"%s\", \"width\": %d, \"height\": %d, \"n_bucket\": %d, \"frames\": %d, "
                    "\"dtype\": %d, \"dynamics\": %d, \"sh_degree\": %d, \"batch\": %d, \"bwd_batch\": %d, "
                    "\"sort_cap\": %d, \"compact\": %d}\n",
                    key.arch, key.width, key.height, key.n_bucket, key.frames, key.dtype, key.dynamics,
                    key.sh_degree, best.batch, best.bwd_batch, best.sort_cap, best.compact);
            fclose(fp);
        }
    }
    return GV_OK;
}

gv_status gv_device_status(const void* ws, uint32_t out[4]) {
    if (!ws || !out) return GV_ERR_INVALID_ARG;
    GV_TRY(hipDeviceSynchronize());
    uint32_t w[4];
    GV_TRY(hipMemcpy(w, ws, sizeof(w), hipMemcpyDeviceToHost));
    out[0] = w[ST_OVERFLOW];
    out[1] = w[ST_NONFINITE];
    out[2] = w[ST_K_LO];
    out[3] = w[ST_K_HI];
    return GV_OK;
}

const char* gv_status_str(gv_status s) {
    switch (s) {
        case GV_OK: return "ok";
        case GV_ERR_INVALID_ARG: return "invalid argument";
        case GV_ERR_WORKSPACE: return "workspace too small or misaligned";
        case GV_ERR_CAPACITY: return "intersection capacity exceeded";
        case GV_ERR_HIP: return "HIP runtime error";
        case GV_ERR_UNSUPPORTED: return "unsupported";
    }
    return "unknown status";
}

int32_t gv_last_hip_error(void) { return g_last_hip; }

int32_t gv_abi_version(void) { return 5; }

}  // extern "C"
