// C ABI of libfdgs: argument validation, scratch management and the order in
// which the kernels of one render are enqueued.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <new>
#include <string>
#include <vector>

#include "fdgs_internal.h"

using namespace fdgs;

namespace {

thread_local std::string g_err;
thread_local hipError_t g_hip_error = hipSuccess;   // what the last FDGS_ERR_HIP of HIP_TRY was

constexpr int kMaskMaxFrames = 256;   // frame times of one keyframe window
constexpr int kMaskMaxViews = 64;     // mask cameras

fdgs_status fail(fdgs_status code, const char *fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_err = buf;
    return code;
}

#define HIP_TRY(expr)                                                                      \
    do {                                                                                   \
        hipError_t e_ = (expr);                                                            \
        if (e_ != hipSuccess) {                                                            \
            g_hip_error = e_;                                                              \
            return fail(FDGS_ERR_HIP, "%s failed: %s", #expr, hipGetErrorString(e_));      \
        }                                                                                  \
    } while (0)

struct Buf {
    void *p = nullptr;
    size_t cap = 0;
    template <typename T>
    T *as() const { return static_cast<T *>(p); }
};

// Blocks replaced by a larger one.  Kernels enqueued before the growth (on
// whatever stream the caller gave) may still read the old block, so it is not
// freed at once: it waits here until a device-wide synchronisation that
// starts after its retirement -- fdgs_destroy, a growth that finds more than
// kRetiredLimit bytes waiting, or an allocation that runs out of memory -- so
// that a growth does not stall every stream of the process.  Growth is geometric (1.5x), so a buffer retires a
// few blocks at most.
std::mutex g_retired_mu;
std::vector<std::pair<int, void *>> g_retired;   // (device, block)
size_t g_retired_bytes = 0;
constexpr size_t kRetiredLimit = size_t(1) << 30;

hipError_t free_retired() {
    std::vector<std::pair<int, void *>> mine;
    {
        std::lock_guard<std::mutex> lk(g_retired_mu);
        mine.swap(g_retired);
        g_retired_bytes = 0;
    }
    if (mine.empty()) return hipSuccess;
    int cur = 0;
    hipError_t e = hipGetDevice(&cur);
    // every block taken here was retired before this synchronisation started
    std::vector<int> devs;
    for (const auto &r : mine)
        if (std::find(devs.begin(), devs.end(), r.first) == devs.end()) devs.push_back(r.first);
    for (int d : devs) {
        const hipError_t f = hipSetDevice(d) == hipSuccess ? hipDeviceSynchronize() : hipErrorInvalidDevice;
        if (e == hipSuccess) e = f;
    }
    for (const auto &r : mine) {
        (void)hipSetDevice(r.first);
        const hipError_t f = hipFree(r.second);
        if (e == hipSuccess) e = f;
    }
    (void)hipSetDevice(cur);
    return e;
}

bool retire_all_spares();   // whether there were any

hipError_t ensure(Buf &b, size_t bytes) {
    bytes = std::max<size_t>(bytes, 256);
    if (bytes <= b.cap) return hipSuccess;
    const size_t want = std::max(bytes, b.cap + b.cap / 2);
    if (b.p) {
        bool flush = false;
        int dev = 0;
        const hipError_t de = hipGetDevice(&dev);
        if (de != hipSuccess) return de;
        {
            std::lock_guard<std::mutex> lk(g_retired_mu);
            g_retired.emplace_back(dev, b.p);
            g_retired_bytes += b.cap;
            flush = g_retired_bytes > kRetiredLimit;
        }
        b.p = nullptr;
        b.cap = 0;
        if (flush) {
            const hipError_t e = free_retired();
            if (e != hipSuccess) return e;
        }
    }
    size_t got = want;
    hipError_t e = hipMalloc(&b.p, got);
    if (e == hipErrorOutOfMemory) {
        // out of memory: free the retired blocks and the released states' (a device
        // synchronisation), then try again, at the exact size if the geometric one
        // still does not fit
        (void)hipGetLastError();
        bool waiting = retire_all_spares();
        {
            std::lock_guard<std::mutex> lk(g_retired_mu);
            waiting = waiting || !g_retired.empty();
        }
        e = waiting ? free_retired() : hipErrorOutOfMemory;
        if (e == hipSuccess) e = hipMalloc(&b.p, got);
        if (e == hipErrorOutOfMemory && want > bytes) {
            (void)hipGetLastError();
            got = bytes;
            e = hipMalloc(&b.p, got);
        }
    }
    if (e != hipSuccess) {
        b.p = nullptr;
        return e;
    }
    b.cap = got;
    return hipSuccess;
}

void release(Buf &b) {
    if (b.p) (void)hipFree(b.p);
    b.p = nullptr;
    b.cap = 0;
}

constexpr int32_t kDefaultPpt = 2;
// Largest processed count of a view ordered by buckets, of which there are at most
// 4096: a bucket's ranking grows with its square.  Order of one view, all visible,
// by buckets and by the radix sort: 200k 45 and 74 us, 500k 77 and 86, 700k 106 and
// 100, 1M 156 and 115, 1.5M 280 and 153; four batched views of 300k 104 and 181, of
// 800k 325 and 358.  Up to the bound more than 4096 equal depths are in order, too,
// which the radix path reports as an error.  With a device count (a mask) the bound
// is the model's size, since a mask may keep all of it (3M, 27% kept: 128 and 153
// us; 60%: 367 and 186; all: 760 and 239).
constexpr int64_t kBucketMaxN = int64_t(1) << 20;

// Several views of one forward pass: device copies of their descriptions and of
// the view of each chunk of entries, the largest processed count and their sum
// (without the padding of the chunks).
struct ViewTable {
    const ViewDesc *views = nullptr;
    const uint32_t *chunk_view = nullptr;
    int32_t V = 1;
    int64_t max_n = 0;
    int64_t n_proc = 0;
};

bool valid_tile(int w, int h) {
    return (w == 8 && h == 8) || (w == 16 && h == 16) || (w == 32 && (h == 8 || h == 16 || h == 32));
}

int bits_for(int64_t v) {   // bits needed to represent values in [0, v)
    int b = 0;
    while (b < 63 && (int64_t(1) << b) < v) ++b;
    return b;
}

}  // namespace

struct fdgs_state {
    fdgs_state *handle = nullptr;   // what the caller holds (new_handle)
    fdgs_ctx *owner = nullptr;
    bool has_forward = false;
    bool has_g2d = false;   // a backward's first phase ran since the last forward
    bool g2d_wide = true;   // the form it left its sums in
    bool ordered = false;   // sched holds the last forward's tiles longest list first
    // per processed Gaussian
    Buf rec, depth_key, rect, tiles, visible, vis_pos, order_k, order_v, order_k2, order_v2, offsets;
    Buf bucket;        // depth buckets (BucketWork)
    Buf vis_count;     // per preprocess workgroup: sampled keys, key ranges, numbers of visible entries
    // per instance
    Buf tkeys, tids, tkeys2, tids2;
    // per tile / pixel
    Buf ranges, T_final, n_contrib;
    Buf sched;         // uint32[V x tiles]: the compositor's longest-first item order
    Buf counts;        // int64[4]: n_vis, n_inst
    Buf g2d;
    Buf scratch;
    // what the forward used
    fdgs_model model{};
    const uint32_t *idx = nullptr;
    const int64_t *n_idx_dev = nullptr;
    KCam cam{};
    double t = 0.0;
    RenderParams rp{};
    int32_t batch = 128;
    int32_t ppt = 2;   // pixels per thread of the forward (the adjoint takes 4 when it did, else 2)
    int64_t n_max = 0;
    int64_t capacity = 0;
    uint32_t *sorted_ids = nullptr;   // points into tids or tids2
    uint32_t *vis_list = nullptr;     // visible positions in ascending order (vis_pos), for the adjoint
    uint32_t *sorted_keys = nullptr;
    int32_t W = 0, H = 0;
    // Whether work on another stream than the null stream may use the buffers:
    // a pass ran on one, or the caller holds their addresses (fdgs_state_binning).
    bool beyond_null_stream = false;
    int32_t device = 0;     // of a released state that waits for reuse

    template <typename F>
    void each(F f) {
        for (Buf *b : {&rec, &depth_key, &rect, &tiles, &visible, &vis_pos, &order_k, &order_v, &order_k2,
                       &order_v2, &offsets, &bucket, &vis_count, &tkeys, &tids, &tkeys2, &tids2, &ranges, &sched,
                       &T_final, &n_contrib, &counts, &g2d, &scratch})
            f(*b);
    }
    void free_all() { each([](Buf &b) { release(b); }); }
    size_t bytes() {
        size_t n = 0;
        each([&](Buf &b) { n += b.cap; });
        return n;
    }
};

namespace {

// Released states whose buffers wait for their context's next new state: a
// training loop that keeps a state for each step's adjoint and releases it
// would otherwise allocate and free two dozen buffers a step, behind a
// device-wide synchronisation (fine-tuning step of 200k Gaussians 2.5 -> 0.95 ms,
// autograd step of 60k 0.71 -> 0.34 ms).  Only states whose whole life was on
// the null stream wait here, and only a pass on the null stream takes them:
// its order is then the only one there is to keep.  At most kSpareStates and
// kSpareLimit bytes over all contexts; given back by fdgs_destroy and by an
// allocation that runs out of memory.
// The caller's name of a state: a number that comes once per process, so that a
// released name stays unknown whichever state its buffers serve next.
fdgs_state *new_handle() {
    static std::atomic<uintptr_t> next{64};
    return reinterpret_cast<fdgs_state *>(next.fetch_add(16));
}

std::mutex g_spare_mu;
constexpr int kSpareStates = 8;
fdgs_state *g_spare[kSpareStates];   // oldest first
int g_n_spare = 0;
constexpr size_t kSpareLimit = size_t(1) << 30;

// Keeps the state, which then belongs to whoever takes it; false when there is no room for it.
bool keep_spare(fdgs_state *s, int32_t device) {
    std::lock_guard<std::mutex> lk(g_spare_mu);
    size_t total = s->bytes();
    for (int k = 0; k < g_n_spare; ++k) total += g_spare[k]->bytes();
    if (g_n_spare == kSpareStates || total > kSpareLimit) return false;
    s->device = device;
    s->has_forward = false;
    g_spare[g_n_spare++] = s;
    return true;
}

// The context's most recently released spare (of any context: null), or null.
fdgs_state *take_spare(const fdgs_ctx *owner) {
    std::lock_guard<std::mutex> lk(g_spare_mu);
    for (int k = g_n_spare - 1; k >= 0; --k)
        if (!owner || g_spare[k]->owner == owner) {
            fdgs_state *s = g_spare[k];
            std::copy(g_spare + k + 1, g_spare + g_n_spare, g_spare + k);
            --g_n_spare;
            return s;
        }
    return nullptr;
}

// Turns the spares of one context (of all: null) into retired blocks; whether there were any.
bool retire_spares(const fdgs_ctx *owner) {
    bool any = false;
    while (fdgs_state *s = take_spare(owner)) {
        any = true;
        std::lock_guard<std::mutex> lk(g_retired_mu);
        s->each([&](Buf &b) {
            if (!b.p) return;
            g_retired.emplace_back(s->device, b.p);
            g_retired_bytes += b.cap;
        });
        delete s;
    }
    return any;
}

bool retire_all_spares() { return retire_spares(nullptr); }

}  // namespace

struct PendingStage {
    int stage;
    hipEvent_t e0, e1;
};

struct fdgs_ctx {
    int32_t device = 0;
    fdgs_state scratch_state;
    std::vector<fdgs_state *> states;
    Buf overflow;                  // int32 device flag
    Buf mask_frames, mask_views, mask_scratch;
    Buf mask_flags;                // contributed-mode visibility bytes
    Buf prune_a, prune_b, prune_c, prune_d, prune_e, prune_times;   // score / prune work
    Buf vq_scratch;                // k-means keys, values, cluster ranges, radix scratch
    int64_t *host_counts = nullptr;  // pinned
    // profiling
    int prof = 0;                  // 0 off, 1 stage events and counts, 2 also evaluated pairs
    Buf prof_acc;                  // uint64[5]: processed, visible, instances, pairs, blended pairs
    std::vector<hipEvent_t> free_events;
    std::vector<PendingStage> pending;
    double ms[FDGS_NUM_STAGES] = {};
    int64_t calls[FDGS_NUM_STAGES] = {};
    bool capturing = false;        // inside hipStreamBeginCapture / EndCapture
    // batched rendering
    fdgs_state batch_state;
    std::vector<Buf> batch_tables;
    hipGraph_t graph = nullptr;
    hipGraphExec_t graph_exec = nullptr;
    hipStream_t capture_stream = nullptr;   // graphs are captured here (the caller's may be the null stream)
    std::vector<unsigned char> graph_key;
    Buf tune_ref, tune_img, tune_diff;
    Buf probe_sink;                // fdgs_measure_peaks
    Buf side_table;                // view table of a visibility or score pass

    hipEvent_t get_event() {
        if (!free_events.empty()) {
            hipEvent_t e = free_events.back();
            free_events.pop_back();
            return e;
        }
        hipEvent_t e = nullptr;
        if (hipEventCreate(&e) != hipSuccess) return nullptr;
        return e;
    }
};

namespace {

// Records HIP events around one stage when profiling is on.
struct StageTimer {
    fdgs_ctx *c;
    int stage;
    hipStream_t s;
    hipEvent_t e0 = nullptr;
    StageTimer(fdgs_ctx *c_, int stage_, hipStream_t s_) : c(c_), stage(stage_), s(s_) {
        if (c->prof && !c->capturing && (e0 = c->get_event())) (void)hipEventRecord(e0, s);
    }
    ~StageTimer() {
        if (!c->prof || c->capturing || !e0) return;
        hipEvent_t e1 = c->get_event();
        if (!e1) return;
        (void)hipEventRecord(e1, s);
        c->pending.push_back(PendingStage{stage, e0, e1});
    }
};

}  // namespace

extern "C" {

const char *fdgs_last_error(void) { return g_err.c_str(); }

const char *fdgs_version(void) { return "fdgs 0.1 (gfx950)"; }

void fdgs_render_cfg_default(fdgs_render_cfg *cfg) {
    if (!cfg) return;
    std::memset(cfg, 0, sizeof *cfg);
    cfg->tile_w = 16;
    cfg->tile_h = 16;
    cfg->batch = 128;
    cfg->alpha_min = 1.0f / 255.0f;
    cfg->alpha_max = 0.99f;
    cfg->t_min = 1e-4f;
    cfg->dilation = 0.3f;
    cfg->temporal_cull = 1;
    cfg->tile_cull = 1;
    cfg->schedule = 1;
    cfg->instance_capacity = 0;
}

fdgs_status fdgs_create(fdgs_ctx **out, int32_t device) {
    if (!out) return fail(FDGS_ERR_INVALID_ARG, "fdgs_create: out is NULL");
    *out = nullptr;
    int count = 0;
    HIP_TRY(hipGetDeviceCount(&count));
    if (device < 0 || device >= count)
        return fail(FDGS_ERR_INVALID_ARG, "fdgs_create: device %d not in [0, %d)", device, count);
    HIP_TRY(hipSetDevice(device));
    fdgs_ctx *c = new (std::nothrow) fdgs_ctx();
    if (!c) return fail(FDGS_ERR_HIP, "fdgs_create: out of host memory");
    c->device = device;
    c->scratch_state.owner = c;
    c->batch_state.owner = c;
    hipError_t e = ensure(c->overflow, sizeof(int32_t));
    if (e == hipSuccess) e = hipMemset(c->overflow.p, 0, sizeof(int32_t));
    if (e == hipSuccess) e = hipHostMalloc((void **)&c->host_counts, 4 * sizeof(int64_t), hipHostMallocDefault);
    if (e != hipSuccess) {
        release(c->overflow);
        delete c;
        return fail(FDGS_ERR_HIP, "fdgs_create: %s", hipGetErrorString(e));
    }
    *out = c;
    return FDGS_OK;
}

fdgs_status fdgs_destroy(fdgs_ctx *ctx) {
    if (!ctx) return FDGS_OK;
    (void)hipSetDevice(ctx->device);
    (void)hipDeviceSynchronize();
    retire_spares(ctx);
    (void)free_retired();
    for (fdgs_state *s : ctx->states) {
        s->free_all();
        delete s;
    }
    ctx->scratch_state.free_all();
    ctx->batch_state.free_all();
    for (Buf &b : ctx->batch_tables) release(b);
    if (ctx->graph_exec) (void)hipGraphExecDestroy(ctx->graph_exec);
    if (ctx->graph) (void)hipGraphDestroy(ctx->graph);
    if (ctx->capture_stream) (void)hipStreamDestroy(ctx->capture_stream);
    release(ctx->tune_ref);
    release(ctx->tune_img);
    release(ctx->tune_diff);
    release(ctx->overflow);
    release(ctx->mask_frames);
    release(ctx->mask_views);
    release(ctx->mask_scratch);
    release(ctx->mask_flags);
    release(ctx->probe_sink);
    release(ctx->side_table);
    for (Buf *b : {&ctx->prune_a, &ctx->prune_b, &ctx->prune_c, &ctx->prune_d, &ctx->prune_e, &ctx->prune_times,
                   &ctx->vq_scratch})
        release(*b);
    release(ctx->prof_acc);
    for (auto &p : ctx->pending) {
        (void)hipEventDestroy(p.e0);
        (void)hipEventDestroy(p.e1);
    }
    for (hipEvent_t e : ctx->free_events) (void)hipEventDestroy(e);
    if (ctx->host_counts) (void)hipHostFree(ctx->host_counts);
    delete ctx;
    return FDGS_OK;
}

}  // extern "C"

namespace {

fdgs_status check_model(const fdgs_model *m, const char *fn) {
    if (!m) return fail(FDGS_ERR_INVALID_ARG, "%s: model is NULL", fn);
    if (m->n < 0 || m->n >= (int64_t(1) << 31))
        return fail(FDGS_ERR_INVALID_ARG, "%s: model n=%lld out of range", fn, (long long)m->n);
    if (m->sh_degree < 0 || m->sh_degree > 3)
        return fail(FDGS_ERR_INVALID_ARG, "%s: sh_degree %d not in 0..3", fn, m->sh_degree);
    if (m->n > 0 && (!m->mean || !m->log_scale || !m->q_left || !m->q_right || !m->opacity_logit ||
                     (!m->sh && !m->sh_index)))
        return fail(FDGS_ERR_INVALID_ARG, "%s: a model pointer is NULL", fn);
    if (m->sh_index) {
        if (!m->sh_codebook || m->sh_codebook_size < 1)
            return fail(FDGS_ERR_INVALID_ARG, "%s: sh_index needs sh_codebook and sh_codebook_size >= 1", fn);
        if (reinterpret_cast<uintptr_t>(m->sh_codebook) % 16 != 0)
            return fail(FDGS_ERR_INVALID_ARG, "%s: sh_codebook must be 16-byte aligned", fn);
    }
    return FDGS_OK;
}

fdgs_status check_camera(const fdgs_camera *c, const char *fn) {
    if (!c) return fail(FDGS_ERR_INVALID_ARG, "%s: camera is NULL", fn);
    if (c->width < 1 || c->height < 1 || c->width > 16384 || c->height > 16384)
        return fail(FDGS_ERR_INVALID_ARG, "%s: image %dx%d out of range", fn, c->width, c->height);
    if (!(c->znear > 0.0) || !std::isfinite(c->znear))
        return fail(FDGS_ERR_INVALID_ARG, "%s: znear must be > 0", fn);
    const double v[] = {c->fx, c->fy, c->cx, c->cy};
    for (double x : v)
        if (!std::isfinite(x)) return fail(FDGS_ERR_INVALID_ARG, "%s: non-finite intrinsics", fn);
    for (int k = 0; k < 9; ++k)
        if (!std::isfinite(c->R[k])) return fail(FDGS_ERR_INVALID_ARG, "%s: non-finite R", fn);
    for (int k = 0; k < 3; ++k)
        if (!std::isfinite(c->tvec[k])) return fail(FDGS_ERR_INVALID_ARG, "%s: non-finite tvec", fn);
    if (!(c->fx > 0.0) || !(c->fy > 0.0)) return fail(FDGS_ERR_INVALID_ARG, "%s: focal must be > 0", fn);
    return FDGS_OK;
}

fdgs_status check_cfg(const fdgs_render_cfg *cfg, const char *fn) {
    if (!cfg) return fail(FDGS_ERR_INVALID_ARG, "%s: cfg is NULL", fn);
    if (!valid_tile(cfg->tile_w, cfg->tile_h))
        return fail(FDGS_ERR_INVALID_ARG, "%s: tile %dx%d not one of 8x8, 16x16, 32x8, 32x16, 32x32", fn, cfg->tile_w,
                    cfg->tile_h);
    if (cfg->batch != 64 && cfg->batch != 128 && cfg->batch != 256 &&
        !((cfg->batch == 512 || cfg->batch == 1024) && cfg->tile_w == 32 && cfg->tile_h == 32))
        return fail(FDGS_ERR_INVALID_ARG, "%s: batch %d not one of 64, 128, 256 (or 512 with 32x32 tiles)", fn,
                    cfg->batch);
    if (cfg->schedule != 0 && cfg->schedule != 1)
        return fail(FDGS_ERR_INVALID_ARG, "%s: schedule %d not one of 0, 1", fn, cfg->schedule);
    if (cfg->pixels_per_thread != 0 && cfg->pixels_per_thread != 1 && cfg->pixels_per_thread != 2 &&
        cfg->pixels_per_thread != 4)
        return fail(FDGS_ERR_INVALID_ARG, "%s: pixels_per_thread %d not one of 0, 1, 2, 4", fn,
                    cfg->pixels_per_thread);
    if (!(cfg->alpha_min > 0.0f) || !(cfg->alpha_max > cfg->alpha_min) || !(cfg->alpha_max < 1.0f))
        return fail(FDGS_ERR_INVALID_ARG, "%s: need 0 < alpha_min < alpha_max < 1", fn);
    if (!(cfg->t_min > 0.0f) || !(cfg->t_min < 1.0f))
        return fail(FDGS_ERR_INVALID_ARG, "%s: need 0 < t_min < 1", fn);
    if (!(cfg->dilation >= 0.0f) || !std::isfinite(cfg->dilation))
        return fail(FDGS_ERR_INVALID_ARG, "%s: dilation must be finite and >= 0", fn);
    for (int k = 0; k < 3; ++k)
        if (!std::isfinite(cfg->bg[k])) return fail(FDGS_ERR_INVALID_ARG, "%s: non-finite bg", fn);
    if (cfg->instance_capacity < 0 || cfg->instance_capacity > 0xffffffffll)
        return fail(FDGS_ERR_INVALID_ARG, "%s: instance_capacity out of range", fn);
    return FDGS_OK;
}

KModel kmodel(const fdgs_model *m) {
    return KModel{m->mean,  m->log_scale, m->q_left,   m->q_right,     m->opacity_logit,
                  m->sh,    m->n,         m->sh_degree, m->sh_index,   m->sh_codebook,
                  m->sh_index ? m->sh_codebook_size : 0};
}

KCam kcam(const fdgs_camera *c) {
    KCam k;
    std::memcpy(k.R, c->R, sizeof k.R);
    std::memcpy(k.t, c->tvec, sizeof k.t);
    k.fx = c->fx;
    k.fy = c->fy;
    k.cx = c->cx;
    k.cy = c->cy;
    k.znear = c->znear;
    k.W = c->width;
    k.H = c->height;
    return k;
}

fdgs_state *find_state(fdgs_ctx *ctx, fdgs_state *handle) {
    for (fdgs_state *x : ctx->states)
        if (x->handle == handle) return x;
    return nullptr;
}

// Entries a view takes in the concatenated buffers: whole chunks, at least one.
int64_t padded_entries(int64_t n) { return std::max<int64_t>((n + kViewChunk - 1) / kViewChunk, 1) * kViewChunk; }

// What a ViewTable points to: the views, then the view of each of the n_total / kViewChunk chunks.
std::vector<unsigned char> view_table_bytes(const std::vector<ViewDesc> &table, int64_t n_total) {
    std::vector<unsigned char> bytes(sizeof(ViewDesc) * table.size() + sizeof(uint32_t) * (size_t)(n_total / kViewChunk));
    std::memcpy(bytes.data(), table.data(), sizeof(ViewDesc) * table.size());
    uint32_t *chunk = reinterpret_cast<uint32_t *>(bytes.data() + sizeof(ViewDesc) * table.size());
    for (size_t v = 0; v < table.size(); ++v)
        for (int64_t c = 0; c < padded_entries(table[v].n_proc) / kViewChunk; ++c) *chunk++ = (uint32_t)v;
    return bytes;
}

// Visibility or score pass over views of the whole model: the forward of every
// (camera, time), marking contrib or adding to weight (one of them) per
// Gaussian.  Views of one image size share launches, up to kSideEntries entries
// each, so that the front end's short launches and the read-back of the
// instance count come once per launch (20 views of 200k at two keyframes:
// 9.8 -> 4.0 ms; pruning scores of 1M Gaussians over 8 views, 4 per launch: 3.6
// -> 2.4 ms).  cfg null: the defaults, with 32x32 tiles where that leaves enough
// of them -- marks and weights don't depend on the tiling, and larger tiles
// make fewer instances.  Views that don't fit into memory together run one by one.
constexpr int64_t kSideEntries = int64_t(1) << 22;
constexpr int64_t kSideTiles = 2048;
// Tiles of the views of one launch (12 bytes of lists and order each): enough that
// only images past 8192 x 8192 pixels in 16x16 tiles are alone for it.
constexpr int64_t kSideMostTiles = int64_t(1) << 22;
struct SidePass {
    const fdgs_camera *cams;
    int32_t n_cams;
    const double *times;     // one per camera; with every_time, every camera at each of n_times
    int32_t n_times;
    bool every_time;
    int64_t size() const { return every_time ? (int64_t)n_cams * n_times : n_cams; }
    const fdgs_camera &cam(int64_t p) const { return cams[p % n_cams]; }
    double time(int64_t p) const { return times[every_time ? p / n_cams : p]; }
};
fdgs_status run_side_views(fdgs_ctx *ctx, const fdgs_model *model, const SidePass &pass, const fdgs_render_cfg *cfg,
                           const fdgs_render_cfg &defaults, uint8_t *contrib, float *weight, hipStream_t stream);

fdgs_status run_forward(fdgs_ctx *ctx, fdgs_state *S, const ViewDesc *one, const ViewTable &vt,
                        const int64_t *n_dev, int64_t n_total, int32_t W, int32_t H, const fdgs_render_cfg *cfg,
                        float *out_rgb, float *out_T, bool need_state, hipStream_t stream,
                        uint8_t *contrib = nullptr, float *weight = nullptr);

}  // namespace

extern "C" {

fdgs_status fdgs_slice_4d(fdgs_ctx *ctx, const fdgs_model *model, double t, const uint32_t *idx, int64_t m,
                          float *out_mean3, float *out_cov3, float *out_p, hipStream_t stream) {
    if (!ctx) return fail(FDGS_ERR_INVALID_ARG, "fdgs_slice_4d: ctx is NULL");
    if (fdgs_status st = check_model(model, "fdgs_slice_4d")) return st;
    if (!std::isfinite(t)) return fail(FDGS_ERR_INVALID_ARG, "fdgs_slice_4d: t is not finite");
    if (m < 0 || m >= (int64_t(1) << 31)) return fail(FDGS_ERR_INVALID_ARG, "fdgs_slice_4d: m out of range");
    if (!idx && m > model->n) return fail(FDGS_ERR_INVALID_ARG, "fdgs_slice_4d: m > n without idx");
    if (m > 0 && (!out_mean3 || !out_cov3 || !out_p))
        return fail(FDGS_ERR_INVALID_ARG, "fdgs_slice_4d: an output pointer is NULL");
    if (m > 0 && idx && model->n == 0) return fail(FDGS_ERR_INVALID_ARG, "fdgs_slice_4d: idx into empty model");
    HIP_TRY(hipSetDevice(ctx->device));
    HIP_TRY(launch_slice(kmodel(model), t, idx, m, out_mean3, out_cov3, out_p, stream));
    return FDGS_OK;
}

}  // extern "C"

namespace {

// Validation shared by the mask entry points; fills the effective alpha_min
// and dilation.
fdgs_status check_mask_args(const fdgs_model *model, const fdgs_mask_spec *spec, const uint32_t *out_bits,
                            const uint32_t *out_idx, const int64_t *out_count, float *amin_out, float *dil_out,
                            const char *fn) {
    if (fdgs_status st = check_model(model, fn)) return st;
    if (!spec) return fail(FDGS_ERR_INVALID_ARG, "%s: spec is NULL", fn);
    if (spec->mode != FDGS_MASK_TEMPORAL && spec->mode != FDGS_MASK_TEMPORAL_AND_TILE &&
        spec->mode != FDGS_MASK_CONTRIBUTED)
        return fail(FDGS_ERR_INVALID_ARG, "%s: unknown mode %d", fn, spec->mode);
    if (spec->mode != FDGS_MASK_CONTRIBUTED) {
        if (spec->n_frames < 1 || spec->n_frames > kMaskMaxFrames || !spec->frame_times)
            return fail(FDGS_ERR_INVALID_ARG, "%s: need 1..%d frame times", fn, kMaskMaxFrames);
        for (int f = 0; f < spec->n_frames; ++f)
            if (!std::isfinite(spec->frame_times[f]))
                return fail(FDGS_ERR_INVALID_ARG, "%s: non-finite frame time", fn);
    }
    if (spec->mode != FDGS_MASK_TEMPORAL) {
        if (spec->n_views < 1 || spec->n_views > kMaskMaxViews || !spec->views)
            return fail(FDGS_ERR_INVALID_ARG, "%s: modes 1 and 2 need 1..%d views", fn, kMaskMaxViews);
        for (int v = 0; v < spec->n_views; ++v)
            if (fdgs_status st = check_camera(&spec->views[v], fn)) return st;
        if (!std::isfinite(spec->key_lo) || !std::isfinite(spec->key_hi))
            return fail(FDGS_ERR_INVALID_ARG, "%s: non-finite keyframe time", fn);
    }
    if (!out_bits || !out_idx || !out_count) return fail(FDGS_ERR_INVALID_ARG, "%s: an output is NULL", fn);
    const float amin = spec->alpha_min > 0.0f ? spec->alpha_min : 1.0f / 255.0f;
    if (!(amin < 1.0f)) return fail(FDGS_ERR_INVALID_ARG, "%s: alpha_min must be < 1", fn);
    *amin_out = amin;
    *dil_out = spec->dilation >= 0.0f ? spec->dilation : 0.3f;
    return FDGS_OK;
}

// Modes TEMPORAL and TEMPORAL_AND_TILE: copies the window's frame times and
// mask cameras into frames_dev / views_dev (device, room for the spec's
// counts), runs the predicate and compacts the bits with compact_scratch
// (compact_scratch_bytes(n)); synchronises the stream, since the host arrays
// are copied asynchronously.
fdgs_status enqueue_window_mask(const fdgs_model *model, const fdgs_mask_spec *spec, float amin, float dil,
                                double *frames_dev, KCam *views_dev, void *compact_scratch, uint32_t *out_bits,
                                uint32_t *out_idx, int64_t *out_count, hipStream_t stream) {
    HIP_TRY(hipMemcpyAsync(frames_dev, spec->frame_times, sizeof(double) * spec->n_frames, hipMemcpyHostToDevice,
                           stream));
    KCam views[kMaskMaxViews];
    const int32_t n_views = spec->mode == FDGS_MASK_TEMPORAL_AND_TILE ? spec->n_views : 0;
    for (int v = 0; v < n_views; ++v) views[v] = kcam(&spec->views[v]);
    if (n_views > 0)
        HIP_TRY(hipMemcpyAsync(views_dev, views, sizeof(KCam) * n_views, hipMemcpyHostToDevice, stream));
    MaskArgs a;
    a.frames = frames_dev;
    a.n_frames = spec->n_frames;
    a.views = views_dev;
    a.n_views = n_views;
    a.key_lo = spec->key_lo;
    a.key_hi = spec->key_hi;
    a.mode = spec->mode;
    a.level = 2.0 * std::log(1.0 / (double)amin);
    a.rect_level = a.level * (1.0 + 1e-4) + 1e-4;
    a.dilation = dil;
    HIP_TRY(launch_mask_bits(kmodel(model), a, out_bits, stream));
    HIP_TRY(compact_bits(out_bits, model->n, out_idx, out_count, compact_scratch, stream));
    // the host arrays were copied asynchronously: finish before returning
    HIP_TRY(hipStreamSynchronize(stream));
    return FDGS_OK;
}

}  // namespace

extern "C" {

fdgs_status fdgs_build_active_mask(fdgs_ctx *ctx, const fdgs_model *model, const fdgs_mask_spec *spec,
                                   uint32_t *out_bits, uint32_t *out_idx, int64_t *out_count,
                                   hipStream_t stream) {
    const char *fn = "fdgs_build_active_mask";
    if (!ctx) return fail(FDGS_ERR_INVALID_ARG, "%s: ctx is NULL", fn);
    float amin = 0.0f, dil = 0.0f;
    if (fdgs_status st = check_mask_args(model, spec, out_bits, out_idx, out_count, &amin, &dil, fn)) return st;
    HIP_TRY(hipSetDevice(ctx->device));
    const int64_t n = model->n;
    if (spec->mode == FDGS_MASK_CONTRIBUTED) {
        // the union over views and both keyframes of the Gaussians some pixel blends
        fdgs_render_cfg cfg;
        fdgs_render_cfg_default(&cfg);
        cfg.alpha_min = amin;
        cfg.dilation = dil;
        cfg.pixels_per_thread = 2;
        HIP_TRY(ensure(ctx->mask_flags, (size_t)((n + 3) / 4) * 4 + 4));
        HIP_TRY(launch_fill_u32(ctx->mask_flags.as<uint32_t>(), (n + 3) / 4, 0u, stream));
        const double keys[2] = {spec->key_lo, spec->key_hi};
        const SidePass pass{spec->views, spec->n_views, keys, spec->key_hi == spec->key_lo ? 1 : 2, true};
        if (fdgs_status st = run_side_views(ctx, model, pass, nullptr, cfg, ctx->mask_flags.as<uint8_t>(), nullptr, stream))
            return st;
        HIP_TRY(launch_flags_to_bits(ctx->mask_flags.as<uint8_t>(), n, out_bits, stream));
        HIP_TRY(ensure(ctx->mask_scratch, compact_scratch_bytes(n)));
        HIP_TRY(compact_bits(out_bits, n, out_idx, out_count, ctx->mask_scratch.p, stream));
        HIP_TRY(hipStreamSynchronize(stream));
        return FDGS_OK;
    }
    HIP_TRY(ensure(ctx->mask_frames, sizeof(double) * spec->n_frames));
    if (spec->mode == FDGS_MASK_TEMPORAL_AND_TILE) HIP_TRY(ensure(ctx->mask_views, sizeof(KCam) * spec->n_views));
    HIP_TRY(ensure(ctx->mask_scratch, compact_scratch_bytes(n)));
    return enqueue_window_mask(model, spec, amin, dil, ctx->mask_frames.as<double>(), ctx->mask_views.as<KCam>(),
                               ctx->mask_scratch.p, out_bits, out_idx, out_count, stream);
}

}  // extern "C"

namespace {

// Scratch of fdgs_build_active_mask_noalloc: one array per GPU, held until the
// process ends.  Host code never passes `scratch` itself (in host code the
// name is a stand-in, not a device address): it uses the address that
// hipGetSymbolAddress returns for the current device.
//   [0, 2 KiB)        frame times (double[256])
//   [2 KiB, 12 KiB)   mask cameras (KCam[64], 144 B each)
//   [12 KiB, 2 MiB)   per-chunk counts of the compaction (compact_scratch_bytes(n): 8 B per
//                     1024 Gaussians, 1 MiB at the maximum of 2^27)
constexpr size_t kNoAllocFrames = 0;
constexpr size_t kNoAllocViews = 2048;
constexpr size_t kNoAllocCompact = 12288;
constexpr size_t kNoAllocBytes = size_t(2) << 20;
static_assert(sizeof(double) * kMaskMaxFrames <= kNoAllocViews - kNoAllocFrames, "frame times fit");
static_assert(sizeof(KCam) * kMaskMaxViews <= kNoAllocCompact - kNoAllocViews, "mask cameras fit");
static __device__ __align__(256) unsigned char scratch[kNoAllocBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices] = {};

// Device address of `scratch` on the current device (looked up once per device).
fdgs_status noalloc_scratch(void **out, const char *fn) {
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return fail(FDGS_ERR_UNSUPPORTED, "%s: device %d out of range", fn, dev);
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p) return fail(FDGS_ERR_HIP, "%s: no device address for the scratch array", fn);
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return FDGS_OK;
}

}  // namespace

extern "C" {

fdgs_status fdgs_measure_peaks(fdgs_ctx *ctx, double *out, hipStream_t stream) {
    const char *fn = "fdgs_measure_peaks";
    if (!ctx) return fail(FDGS_ERR_INVALID_ARG, "%s: ctx is NULL", fn);
    if (!out) return fail(FDGS_ERR_INVALID_ARG, "%s: out is NULL", fn);
    HIP_TRY(hipSetDevice(ctx->device));
    int cus = 0;
    HIP_TRY(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, ctx->device));
    HIP_TRY(ensure(ctx->probe_sink, sizeof(float) * 8 * (size_t)std::max(cus, 1)));
    HIP_TRY(measure_peaks(ctx->probe_sink.as<float>(), out, stream));
    return FDGS_OK;
}

fdgs_status fdgs_mask_overlap(const uint32_t *bits_a, const uint32_t *bits_b, int64_t n, int64_t *out,
                              hipStream_t stream) {
    const char *fn = "fdgs_mask_overlap";
    if (n < 0 || n >= (int64_t(1) << 31)) return fail(FDGS_ERR_INVALID_ARG, "%s: n out of range", fn);
    if (!out || (n > 0 && (!bits_a || !bits_b))) return fail(FDGS_ERR_INVALID_ARG, "%s: a pointer is NULL", fn);
    HIP_TRY(launch_mask_overlap(bits_a, bits_b, n, out, stream));
    return FDGS_OK;
}

fdgs_status fdgs_build_active_mask_noalloc(const fdgs_model *model, const fdgs_mask_spec *spec,
                                           uint32_t *out_bits, uint32_t *out_idx, int64_t *out_count,
                                           hipStream_t stream) {
    const char *fn = "fdgs_build_active_mask_noalloc";
    float amin = 0.0f, dil = 0.0f;
    if (fdgs_status st = check_mask_args(model, spec, out_bits, out_idx, out_count, &amin, &dil, fn)) return st;
    if (spec->mode == FDGS_MASK_CONTRIBUTED)
        return fail(FDGS_ERR_UNSUPPORTED, "%s: mode FDGS_MASK_CONTRIBUTED renders views and needs allocations", fn);
    if (model->n > FDGS_NOALLOC_MAX_GAUSSIANS || compact_scratch_bytes(model->n) > kNoAllocBytes - kNoAllocCompact)
        return fail(FDGS_ERR_INVALID_ARG, "%s: n = %lld exceeds the maximum of %lld Gaussians", fn,
                    (long long)model->n, (long long)FDGS_NOALLOC_MAX_GAUSSIANS);
    unsigned char *base = nullptr;
    if (fdgs_status st = noalloc_scratch(reinterpret_cast<void **>(&base), fn)) return st;
    return enqueue_window_mask(model, spec, amin, dil, reinterpret_cast<double *>(base + kNoAllocFrames),
                               reinterpret_cast<KCam *>(base + kNoAllocViews), base + kNoAllocCompact, out_bits,
                               out_idx, out_count, stream);
}

}  // extern "C"

namespace {

RenderParams make_params(const fdgs_render_cfg *cfg, int32_t W, int32_t H) {
    RenderParams rp;
    rp.tile_w = cfg->tile_w;
    rp.tile_h = cfg->tile_h;
    rp.tiles_x = (W + cfg->tile_w - 1) / cfg->tile_w;
    rp.tiles_y = (H + cfg->tile_h - 1) / cfg->tile_h;
    for (int k = 0; k < 3; ++k) rp.bg[k] = cfg->bg[k];
    rp.alpha_min = cfg->alpha_min;
    rp.alpha_max = cfg->alpha_max;
    rp.t_min = cfg->t_min;
    rp.dilation = cfg->dilation;
    rp.temporal_cull = cfg->temporal_cull ? 1 : 0;
    rp.tile_cull = cfg->tile_cull ? 1 : 0;
    rp.colour = 1;
    rp.vanilla_level = 2.0 * std::log(1.0 / (double)cfg->alpha_min) * (1.0 + 1e-4) + 1e-4;
    return rp;
}

// The forward pipeline for V views of one resolution.  V == 1: `one` by value,
// processed count optionally on the device (n_dev).  Otherwise `vt` holds the
// views, with host-known counts, and n_total covers their padded chunks.
// With capture set nothing may synchronise or allocate: the caller guarantees
// buffers are already large enough and a fixed instance capacity is given.
fdgs_status run_forward(fdgs_ctx *ctx, fdgs_state *S, const ViewDesc *one, const ViewTable &vt,
                        const int64_t *n_dev, int64_t n_total, int32_t W, int32_t H, const fdgs_render_cfg *cfg,
                        float *out_rgb, float *out_T, bool need_state, hipStream_t stream, uint8_t *contrib,
                        float *weight) {
    const char *fn = "fdgs_render";
    const int32_t V = vt.V;
    RenderParams rp = make_params(cfg, W, H);
    rp.colour = !contrib && !weight;
    const int64_t tiles_per_view = (int64_t)rp.tiles_x * rp.tiles_y;
    const int64_t n_keys = tiles_per_view * V;
    if (n_keys >= (int64_t(1) << 31)) return fail(FDGS_ERR_INVALID_ARG, "%s: too many tiles x views", fn);
    const int32_t ppt = cfg->pixels_per_thread ? cfg->pixels_per_thread : kDefaultPpt;
    const int64_t n_max = n_total;
    const int64_t npx = (int64_t)W * H;

    HIP_TRY(ensure(S->rec, sizeof(Rec2D) * n_max));
    HIP_TRY(ensure(S->depth_key, sizeof(uint64_t) * n_max));
    HIP_TRY(ensure(S->rect, sizeof(int32_t) * 4 * n_max));
    HIP_TRY(ensure(S->tiles, sizeof(uint32_t) * n_max));
    HIP_TRY(ensure(S->visible, n_max));
    HIP_TRY(ensure(S->order_k, sizeof(uint32_t) * n_max));
    HIP_TRY(ensure(S->order_v, sizeof(uint32_t) * n_max));
    HIP_TRY(ensure(S->order_k2, sizeof(uint32_t) * n_max));
    HIP_TRY(ensure(S->order_v2, sizeof(uint32_t) * n_max));
    HIP_TRY(ensure(S->offsets, sizeof(uint64_t) * n_max));
    // views of not too many processed Gaussians: depth order and offsets by buckets (three launches)
    const int64_t n_view_max = vt.views ? vt.max_n : n_max;
    const bool by_buckets = n_max > 0 && n_view_max <= kBucketMaxN &&
                            n_view_max * tiles_per_view < (int64_t(1) << kBucketTileBits);
    size_t bucket_words = 0, bucket_clear = 0;
    if (by_buckets) {
        (void)bucket_work(nullptr, n_view_max, V, &bucket_words, &bucket_clear);
        HIP_TRY(ensure(S->bucket, sizeof(uint32_t) * bucket_words));
    }
    HIP_TRY(ensure(S->counts, sizeof(int64_t) * 4));
    HIP_TRY(ensure(S->ranges, sizeof(uint32_t) * 2 * n_keys));
    if (cfg->schedule) HIP_TRY(ensure(S->sched, sizeof(uint32_t) * n_keys));
    if (need_state) {
        HIP_TRY(ensure(S->T_final, sizeof(float) * npx));
        HIP_TRY(ensure(S->n_contrib, sizeof(uint32_t) * npx));
    }
    const size_t scratch = std::max(scan_scratch_bytes(n_max), sort_scratch_bytes(n_max));
    HIP_TRY(ensure(S->scratch, scratch));
    int64_t *counts = S->counts.as<int64_t>();

    const int64_t pre_blocks = (n_total + kPreprocessBlock - 1) / kPreprocessBlock;
    const size_t sample_words = (size_t)V * kSampleBlocks * 4;
    HIP_TRY(ensure(S->vis_count, sizeof(uint32_t) * (sample_words + 3 * (size_t)pre_blocks)));
    uint32_t *samples = S->vis_count.as<uint32_t>(), *block_range = samples + sample_words;
    uint32_t *vis_count = block_range + 2 * pre_blocks;
    PreprocOut po{S->rec.as<Rec2D>(), S->depth_key.as<uint64_t>(), S->rect.as<int32_t>(), S->tiles.as<uint32_t>(),
                  S->visible.as<uint8_t>(), vis_count, block_range, samples, S->bucket.as<uint32_t>(),
                  by_buckets ? (int64_t)bucket_clear : 0};
    {
        StageTimer tm(ctx, FDGS_STAGE_PREPROCESS, stream);
        HIP_TRY(launch_preprocess(one, vt.views, vt.chunk_view, V, n_dev, n_total, rp, po, stream));
    }
    // the compacted list of visible entries: the radix sort's input, and the adjoint's
    if (!by_buckets || need_state) {
        StageTimer tm(ctx, FDGS_STAGE_COMPACT, stream);
        if (need_state) HIP_TRY(ensure(S->vis_pos, sizeof(uint32_t) * n_max));
        HIP_TRY(compact_visible(S->visible.as<uint8_t>(), S->depth_key.as<uint64_t>(), n_dev, n_max, counts + 0,
                                by_buckets ? nullptr : S->order_k.as<uint32_t>(),
                                by_buckets ? nullptr : S->order_v.as<uint32_t>(),
                                need_state ? S->vis_pos.as<uint32_t>() : nullptr, nullptr, 0, nullptr, S->scratch.p,
                                stream, vis_count));
    }
    uint32_t *ov = nullptr;
    if (by_buckets) {
        StageTimer tm(ctx, FDGS_STAGE_DEPTH_SORT, stream);
        ov = S->order_v2.as<uint32_t>();
        HIP_TRY(depth_order_views(S->visible.as<uint8_t>(), S->depth_key.as<uint64_t>(), S->tiles.as<uint32_t>(),
                                  block_range, n_dev, n_max, vt.views, vt.chunk_view, V, n_view_max,
                                  S->bucket.as<uint32_t>(), S->order_v.as<uint32_t>(), S->order_k2.as<uint32_t>(), ov,
                                  S->offsets.as<uint64_t>(), counts, stream, samples));
    } else {
        StageTimer tm(ctx, FDGS_STAGE_DEPTH_SORT, stream);
        int alt = 0;
        HIP_TRY(radix_sort_u32(S->order_k.as<uint32_t>(), S->order_v.as<uint32_t>(), S->order_k2.as<uint32_t>(),
                               S->order_v2.as<uint32_t>(), counts + 0, n_max, 0, 32, S->scratch.p, &alt, stream));
        uint32_t *ok = alt ? S->order_k2.as<uint32_t>() : S->order_k.as<uint32_t>();
        ov = alt ? S->order_v2.as<uint32_t>() : S->order_v.as<uint32_t>();
        HIP_TRY(launch_fix_depth_ties(ok, ov, S->depth_key.as<uint64_t>(), counts + 0, n_max,
                                      ctx->overflow.as<int32_t>(), stream));
        if (V > 1) {
            // group by view, keeping the depth order inside each view (stable)
            uint32_t *kv = alt ? S->order_k.as<uint32_t>() : S->order_k2.as<uint32_t>();
            uint32_t *vv = alt ? S->order_v.as<uint32_t>() : S->order_v2.as<uint32_t>();
            HIP_TRY(launch_gather_view(vt.chunk_view, ov, ok, counts + 0, n_max, stream));
            int alt_v = 0;
            HIP_TRY(radix_sort_u32(ok, ov, kv, vv, counts + 0, n_max, 0, std::max(1, bits_for(V)), S->scratch.p,
                                   &alt_v, stream));
            if (alt_v) ov = vv;
        }
    }
    S->vis_list = need_state ? S->vis_pos.as<uint32_t>() : nullptr;
    if (!by_buckets) {
        StageTimer tm(ctx, FDGS_STAGE_OFFSETS, stream);
        HIP_TRY(scan_u32_to_u64(S->tiles.as<uint32_t>(), ov, S->offsets.as<uint64_t>(), counts + 0, n_max,
                                counts + 1, S->scratch.p, stream));
    }
    int64_t capacity = cfg->instance_capacity;
    if (capacity == 0) {
        HIP_TRY(hipMemcpyAsync(ctx->host_counts, counts, 2 * sizeof(int64_t), hipMemcpyDeviceToHost, stream));
        HIP_TRY(hipStreamSynchronize(stream));
        capacity = ctx->host_counts[1];
        if (capacity > 0xffffffffll)
            return fail(FDGS_ERR_CAPACITY, "%s: %lld tile instances exceed 2^32", fn, (long long)capacity);
    }
    HIP_TRY(ensure(S->tkeys, sizeof(uint32_t) * capacity));
    HIP_TRY(ensure(S->tids, sizeof(uint32_t) * capacity));
    HIP_TRY(ensure(S->tkeys2, sizeof(uint32_t) * capacity));
    HIP_TRY(ensure(S->tids2, sizeof(uint32_t) * capacity));
    // the duplicate writes the tile sort's first-digit histogram when its windows tile the sort's blocks
    const int tile_bits = std::max(1, bits_for(n_keys));
    const int sort_chunk = radix_chunk(capacity);
    const int64_t hist_cols = (capacity > 0 && sort_chunk % duplicate_window(capacity) == 0)
                                  ? (capacity + sort_chunk - 1) / sort_chunk * (sort_chunk / duplicate_window(capacity))
                                  : 0;
    HIP_TRY(ensure(S->scratch, std::max(scratch, sort_scratch_bytes(capacity, hist_cols))));
    {
        StageTimer tm(ctx, FDGS_STAGE_DUPLICATE, stream);
        HIP_TRY(launch_duplicate(ov, S->offsets.as<uint64_t>(), S->rect.as<int32_t>(), S->rec.as<Rec2D>(), vt.chunk_view, counts + 0, n_max, rp,
                                 S->tkeys.as<uint32_t>(), S->tids.as<uint32_t>(), counts + 1, capacity,
                                 ctx->overflow.as<int32_t>(), hist_cols ? S->scratch.as<uint32_t>() : nullptr,
                                 radix_first_bits(0, tile_bits), hist_cols, stream));
    }
    {
        StageTimer tm(ctx, FDGS_STAGE_TILE_SORT, stream);
        int alt2 = 0;
        HIP_TRY(radix_sort_u32(S->tkeys.as<uint32_t>(), S->tids.as<uint32_t>(), S->tkeys2.as<uint32_t>(),
                               S->tids2.as<uint32_t>(), counts + 1, capacity, 0, tile_bits, S->scratch.p, &alt2, stream,
                               hist_cols));
        S->sorted_keys = alt2 ? S->tkeys2.as<uint32_t>() : S->tkeys.as<uint32_t>();
        S->sorted_ids = alt2 ? S->tids2.as<uint32_t>() : S->tids.as<uint32_t>();
    }
    {
        StageTimer tm(ctx, FDGS_STAGE_RANGES, stream);
        HIP_TRY(launch_tile_ranges(S->sorted_keys, counts + 1, capacity, (int32_t)n_keys, S->ranges.as<uint32_t>(),
                                   stream));
        // the longest-first schedule's item order, from the ranges
        if (cfg->schedule == 1)
            HIP_TRY(launch_tile_order(S->ranges.as<uint32_t>(), (int32_t)n_keys, S->sched.as<uint32_t>(), stream));
    }
    float *T_out = need_state ? S->T_final.as<float>() : out_T;
    uint64_t *acc = nullptr;
    if (ctx->prof && !ctx->capturing) {
        HIP_TRY(ensure(ctx->prof_acc, 5 * sizeof(uint64_t)));
        acc = ctx->prof_acc.as<uint64_t>();
        HIP_TRY(launch_accumulate_counts(n_dev, vt.views ? vt.n_proc : n_total, counts, capacity, acc, stream));
    }
    {
        StageTimer tm(ctx, FDGS_STAGE_COMPOSITE, stream);
        HIP_TRY(launch_composite(rp, W, H, V, cfg->batch, S->ranges.as<uint32_t>(), S->sorted_ids, S->rec.as<Rec2D>(),
                                 out_rgb, T_out, need_state ? S->n_contrib.as<uint32_t>() : nullptr,
                                 acc && ctx->prof == 2 ? acc + 3 : nullptr,
                                 ppt,
                                 cfg->schedule ? S->sched.as<uint32_t>() : nullptr, contrib, weight,
                                 V > 1 ? padded_entries(n_view_max) : 0, stream));
    }
    if (need_state && out_T)
        HIP_TRY(hipMemcpyAsync(out_T, S->T_final.p, sizeof(float) * npx, hipMemcpyDeviceToDevice, stream));
    S->rp = rp;
    S->batch = cfg->batch;
    S->ppt = ppt;
    S->ordered = cfg->schedule == 1;   // its compositor ordered the tiles into sched
    S->capacity = capacity;
    S->W = W;
    S->H = H;
    return FDGS_OK;
}

}  // namespace

extern "C" {

fdgs_status fdgs_render_forward(fdgs_ctx *ctx, const fdgs_model *model, const uint32_t *idx,
                                const int64_t *n_idx_dev, const fdgs_camera *cam, double t,
                                const fdgs_render_cfg *cfg, float *out_rgb, float *out_T,
                                fdgs_state **keep_state, hipStream_t stream) {
    const char *fn = "fdgs_render_forward";
    if (!ctx) return fail(FDGS_ERR_INVALID_ARG, "%s: ctx is NULL", fn);
    if (fdgs_status st = check_model(model, fn)) return st;
    if (fdgs_status st = check_camera(cam, fn)) return st;
    if (fdgs_status st = check_cfg(cfg, fn)) return st;
    if (!std::isfinite(t)) return fail(FDGS_ERR_INVALID_ARG, "%s: t is not finite", fn);
    if (idx && !n_idx_dev) return fail(FDGS_ERR_INVALID_ARG, "%s: idx given without n_idx_dev", fn);
    if (!out_rgb) return fail(FDGS_ERR_INVALID_ARG, "%s: out_rgb is NULL", fn);
    fdgs_state *S = &ctx->scratch_state;
    if (keep_state) {
        if (*keep_state) {
            S = find_state(ctx, *keep_state);
            if (!S) return fail(FDGS_ERR_STATE, "%s: *keep_state does not belong to this context", fn);
        } else {
            S = stream == nullptr ? take_spare(ctx) : nullptr;
            if (!S) S = new (std::nothrow) fdgs_state();
            if (!S) return fail(FDGS_ERR_HIP, "%s: out of host memory", fn);
            S->owner = ctx;
            S->handle = new_handle();
            ctx->states.push_back(S);
            *keep_state = S->handle;
        }
    }
    HIP_TRY(hipSetDevice(ctx->device));
    S->has_forward = false;
    if (stream != nullptr) S->beyond_null_stream = true;
    ViewDesc one;
    one.m = kmodel(model);
    one.cam = kcam(cam);
    one.t = t;
    one.idx = idx;
    one.p_off = 0;
    one.n_proc = model->n;
    const int64_t *n_dev = idx ? n_idx_dev : nullptr;
    if (fdgs_status st = run_forward(ctx, S, &one, ViewTable(), n_dev, model->n, cam->width, cam->height, cfg,
                                     out_rgb, out_T, keep_state != nullptr, stream))
        return st;
    S->model = *model;
    S->idx = idx;
    S->n_idx_dev = n_idx_dev;
    S->cam = one.cam;
    S->t = t;
    S->n_max = model->n;
    S->has_forward = true;
    S->has_g2d = false;
    return FDGS_OK;
}

}  // extern "C"

namespace {

fdgs_status check_batch(const fdgs_model *scenes, int32_t n_scenes, const fdgs_view *views, int32_t n_views,
                        const char *fn) {
    if (n_scenes < 1 || !scenes) return fail(FDGS_ERR_INVALID_ARG, "%s: need at least one scene", fn);
    if (n_views < 1 || !views) return fail(FDGS_ERR_INVALID_ARG, "%s: need at least one view", fn);
    for (int k = 0; k < n_scenes; ++k)
        if (fdgs_status st = check_model(&scenes[k], fn)) return st;
    for (int v = 0; v < n_views; ++v) {
        const fdgs_view &w = views[v];
        if (w.scene < 0 || w.scene >= n_scenes)
            return fail(FDGS_ERR_INVALID_ARG, "%s: view %d names scene %d of %d", fn, v, w.scene, n_scenes);
        if (fdgs_status st = check_camera(&w.cam, fn)) return st;
        if (w.cam.width != views[0].cam.width || w.cam.height != views[0].cam.height)
            return fail(FDGS_ERR_INVALID_ARG, "%s: views differ in image size", fn);
        if (!std::isfinite(w.t)) return fail(FDGS_ERR_INVALID_ARG, "%s: view %d time not finite", fn, v);
        if (w.idx && (w.n_idx < 0 || w.n_idx > scenes[w.scene].n))
            return fail(FDGS_ERR_INVALID_ARG, "%s: view %d n_idx out of range", fn, v);
    }
    return FDGS_OK;
}

fdgs_status run_side_views(fdgs_ctx *ctx, const fdgs_model *model, const SidePass &pass, const fdgs_render_cfg *cfg,
                           const fdgs_render_cfg &defaults, uint8_t *contrib, float *weight, hipStream_t stream) try {
    const int64_t n = model->n, stride = padded_entries(n);
    auto desc = [&](int64_t p, int64_t at) {
        ViewDesc d;
        d.m = kmodel(model);
        d.cam = kcam(&pass.cam(p));
        d.t = pass.time(p);
        d.idx = nullptr;
        d.p_off = at * stride;
        d.n_proc = n;
        return d;
    };
    auto tiles = [&](int64_t p) {
        const int32_t tw = (cfg ? cfg : &defaults)->tile_w, th = (cfg ? cfg : &defaults)->tile_h;
        return (int64_t)((pass.cam(p).width + tw - 1) / tw) * ((pass.cam(p).height + th - 1) / th);
    };
    // the groups that share a launch, and their view tables one after another
    struct Group {
        int64_t p0;
        int32_t V;
        size_t table;
    };
    std::vector<Group> groups;
    std::vector<unsigned char> bytes;
    for (int64_t p = 0; p < pass.size();) {
        const int64_t most = std::max<int64_t>(std::min(kSideEntries / stride, kSideMostTiles / tiles(p)), 1);
        Group g{p, 0, bytes.size()};
        std::vector<ViewDesc> table;
        for (; p < pass.size() && g.V < most && pass.cam(p).width == pass.cam(g.p0).width &&
               pass.cam(p).height == pass.cam(g.p0).height; ++p)
            table.push_back(desc(p, g.V++));
        if (g.V > 1) {
            const std::vector<unsigned char> t = view_table_bytes(table, stride * g.V);
            bytes.insert(bytes.end(), t.begin(), t.end());
            bytes.resize((bytes.size() + 15) / 16 * 16);
        }
        groups.push_back(g);
    }
    bool together = true;
    if (!bytes.empty()) {
        const hipError_t e = ensure(ctx->side_table, bytes.size());
        if (e == hipErrorOutOfMemory) {
            (void)hipGetLastError();
            together = false;
        } else {
            HIP_TRY(e);
            HIP_TRY(hipMemcpyAsync(ctx->side_table.p, bytes.data(), bytes.size(), hipMemcpyHostToDevice, stream));
            HIP_TRY(hipStreamSynchronize(stream));   // `bytes` may go
        }
    }
    for (const Group &g : groups) {
        const int32_t W = pass.cam(g.p0).width, H = pass.cam(g.p0).height;
        auto cfg_for = [&](int32_t V) {
            fdgs_render_cfg c = cfg ? *cfg : defaults;
            if (!cfg && (int64_t)((W + 31) / 32) * ((H + 31) / 32) * V >= kSideTiles) {
                c.tile_w = c.tile_h = 32;
                c.batch = 256;
            }
            return c;
        };
        if (g.V > 1 && together) {
            ViewTable vt;
            vt.views = reinterpret_cast<const ViewDesc *>(ctx->side_table.as<unsigned char>() + g.table);
            vt.chunk_view = reinterpret_cast<const uint32_t *>(vt.views + g.V);
            vt.V = g.V;
            vt.max_n = n;
            vt.n_proc = n * g.V;
            const fdgs_render_cfg c = cfg_for(g.V);
            const fdgs_status st = run_forward(ctx, &ctx->scratch_state, nullptr, vt, nullptr, stride * g.V, W, H, &c,
                                               nullptr, nullptr, false, stream, contrib, weight);
            if (st == FDGS_OK) continue;
            // no room for the views' buffers or instances together: one at a time from here on
            // (both are found out before the compositor, which marks and adds, is enqueued)
            if (st != FDGS_ERR_CAPACITY && !(st == FDGS_ERR_HIP && g_hip_error == hipErrorOutOfMemory)) return st;
            (void)hipGetLastError();
            together = false;
        }
        for (int64_t p = g.p0; p < g.p0 + g.V; ++p) {
            const ViewDesc one = desc(p, 0);
            const fdgs_render_cfg c = cfg_for(1);
            if (fdgs_status st = run_forward(ctx, &ctx->scratch_state, &one, ViewTable(), nullptr, n, W, H, &c, nullptr,
                                             nullptr, false, stream, contrib, weight))
                return st;
        }
    }
    return FDGS_OK;
} catch (const std::bad_alloc &) {
    return fail(FDGS_ERR_HIP, "fdgs_render: out of host memory");
}

// Views per launch of a batch: as asked, but no more than share one usefully.  A
// view takes whole chunks of entries and the buckets that the largest one needs,
// each a workgroup: tens of thousands of tiny views in one launch would take
// gigabytes of padding, and beside a large one more workgroups than a grid holds.
constexpr int32_t kBatchMostViews = 1024;
int32_t views_in_launch(int32_t asked, int32_t n_views) {
    return std::min({asked > 0 ? asked : n_views, n_views, kBatchMostViews});
}

// Enqueue every launch of a batch (no graph handling).
fdgs_status enqueue_batch(fdgs_ctx *ctx, const fdgs_model *scenes, const fdgs_view *views, int32_t n_views,
                          const fdgs_render_cfg *cfg, int32_t per_launch, bool upload, float *out_rgb,
                          hipStream_t stream) {
    const int32_t W = views[0].cam.width, H = views[0].cam.height;
    const int64_t img = 3ll * W * H;
    const int32_t n_launch = (n_views + per_launch - 1) / per_launch;
    if (upload && (int32_t)ctx->batch_tables.size() < n_launch) ctx->batch_tables.resize(n_launch);
    // kernels of an earlier batch on this stream may still read the tables
    // about to be overwritten (the upload below is ordered on no stream)
    if (upload) HIP_TRY(hipStreamSynchronize(stream));
    for (int32_t c = 0; c < n_launch; ++c) {
        const int32_t v0 = c * per_launch, V = std::min(per_launch, n_views - v0);
        std::vector<ViewDesc> table(V);
        int64_t off = 0, max_n = 0, sum_n = 0;
        for (int32_t k = 0; k < V; ++k) {
            const fdgs_view &w = views[v0 + k];
            ViewDesc &d = table[k];
            d.m = kmodel(&scenes[w.scene]);
            d.cam = kcam(&w.cam);
            d.t = w.t;
            d.idx = w.idx;
            d.n_proc = w.idx ? w.n_idx : scenes[w.scene].n;
            d.p_off = off;
            off += padded_entries(d.n_proc);
            max_n = std::max(max_n, d.n_proc);
            sum_n += d.n_proc;
        }
        if (off >= (int64_t(1) << 32))
            return fail(FDGS_ERR_CAPACITY, "fdgs_render_batch: %lld Gaussians in one launch exceed 2^32",
                        (long long)off);
        Buf &tb = ctx->batch_tables[c];
        if (upload) {
            const std::vector<unsigned char> bytes = view_table_bytes(table, off);
            HIP_TRY(ensure(tb, bytes.size()));
            HIP_TRY(hipMemcpy(tb.p, bytes.data(), bytes.size(), hipMemcpyHostToDevice));
        }
        if (V == 1) {
            if (fdgs_status st = run_forward(ctx, &ctx->batch_state, &table[0], ViewTable(), nullptr, table[0].n_proc, W, H, cfg,
                                             out_rgb + v0 * img, nullptr, false, stream))
                return st;
        } else {
            ViewTable vt;
            vt.views = tb.as<ViewDesc>();
            vt.chunk_view = reinterpret_cast<const uint32_t *>(vt.views + V);
            vt.V = V;
            vt.max_n = max_n;
            vt.n_proc = sum_n;
            if (fdgs_status st = run_forward(ctx, &ctx->batch_state, nullptr, vt, nullptr, off, W, H, cfg,
                                             out_rgb + v0 * img, nullptr, false, stream))
                return st;
        }
    }
    return FDGS_OK;
}

// A captured graph holds the addresses of the batch buffers and view tables;
// any other use of them (which may re-upload or regrow them) retires it.
void drop_graph(fdgs_ctx *ctx) {
    if (ctx->graph_exec) (void)hipGraphExecDestroy(ctx->graph_exec);
    if (ctx->graph) (void)hipGraphDestroy(ctx->graph);
    ctx->graph_exec = nullptr;
    ctx->graph = nullptr;
    ctx->graph_key.clear();
}

template <typename T>
void append_bytes(std::vector<unsigned char> &k, const T *p, size_t n) {
    const unsigned char *b = reinterpret_cast<const unsigned char *>(p);
    k.insert(k.end(), b, b + sizeof(T) * n);
}

}  // namespace

extern "C" {

fdgs_status fdgs_render_batch(fdgs_ctx *ctx, const fdgs_model *scenes, int32_t n_scenes, const fdgs_view *views,
                              int32_t n_views, const fdgs_render_cfg *cfg, int32_t views_per_launch,
                              int32_t use_graph, float *out_rgb, hipStream_t stream) {
    const char *fn = "fdgs_render_batch";
    if (!ctx) return fail(FDGS_ERR_INVALID_ARG, "%s: ctx is NULL", fn);
    if (fdgs_status st = check_batch(scenes, n_scenes, views, n_views, fn)) return st;
    if (fdgs_status st = check_cfg(cfg, fn)) return st;
    if (!out_rgb) return fail(FDGS_ERR_INVALID_ARG, "%s: out_rgb is NULL", fn);
    if (views_per_launch < 0) return fail(FDGS_ERR_INVALID_ARG, "%s: views_per_launch < 0", fn);
    if (use_graph && cfg->instance_capacity <= 0)
        return fail(FDGS_ERR_INVALID_ARG, "%s: use_graph needs a fixed instance_capacity", fn);
    const int32_t per = views_in_launch(views_per_launch, n_views);
    HIP_TRY(hipSetDevice(ctx->device));
    if (!use_graph) {
        drop_graph(ctx);
        return enqueue_batch(ctx, scenes, views, n_views, cfg, per, true, out_rgb, stream);
    }

    std::vector<unsigned char> key;
    append_bytes(key, scenes, n_scenes);
    append_bytes(key, views, n_views);
    append_bytes(key, cfg, 1);
    append_bytes(key, &per, 1);
    append_bytes(key, &out_rgb, 1);
    if (ctx->graph_exec && key == ctx->graph_key) {
        HIP_TRY(hipGraphLaunch(ctx->graph_exec, stream));
        return FDGS_OK;
    }
    drop_graph(ctx);
    // eager run: uploads the view tables and sizes every buffer
    if (fdgs_status st = enqueue_batch(ctx, scenes, views, n_views, cfg, per, true, out_rgb, stream)) return st;
    HIP_TRY(hipStreamSynchronize(stream));
    if (!ctx->capture_stream) HIP_TRY(hipStreamCreateWithFlags(&ctx->capture_stream, hipStreamNonBlocking));
    hipStream_t cs = ctx->capture_stream;
    HIP_TRY(hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal));
    ctx->capturing = true;
    fdgs_status st = enqueue_batch(ctx, scenes, views, n_views, cfg, per, false, out_rgb, cs);
    ctx->capturing = false;
    hipGraph_t g = nullptr;
    hipError_t e = hipStreamEndCapture(cs, &g);
    if (st != FDGS_OK) {
        if (g) (void)hipGraphDestroy(g);
        return st;
    }
    if (e != hipSuccess) return fail(FDGS_ERR_HIP, "%s: capture failed: %s", fn, hipGetErrorString(e));
    hipGraphExec_t ex = nullptr;
    e = hipGraphInstantiate(&ex, g, nullptr, nullptr, 0);
    if (e != hipSuccess) {
        (void)hipGraphDestroy(g);
        return fail(FDGS_ERR_HIP, "%s: graph instantiation failed: %s", fn, hipGetErrorString(e));
    }
    ctx->graph = g;
    ctx->graph_exec = ex;
    ctx->graph_key = key;
    HIP_TRY(hipGraphLaunch(ctx->graph_exec, stream));
    return FDGS_OK;
}

fdgs_status fdgs_autotune(fdgs_ctx *ctx, const fdgs_model *scenes, int32_t n_scenes, const fdgs_view *views,
                          int32_t n_views, int32_t views_per_launch, int32_t repeats, fdgs_render_cfg *inout_cfg,
                          fdgs_tune_result *results, int32_t max_results, int32_t *n_results, hipStream_t stream) {
    const char *fn = "fdgs_autotune";
    if (!ctx || !inout_cfg) return fail(FDGS_ERR_INVALID_ARG, "%s: ctx or cfg is NULL", fn);
    if (fdgs_status st = check_batch(scenes, n_scenes, views, n_views, fn)) return st;
    if (fdgs_status st = check_cfg(inout_cfg, fn)) return st;
    if (repeats < 1) repeats = 1;
    const int32_t per = views_in_launch(views_per_launch, n_views);
    HIP_TRY(hipSetDevice(ctx->device));
    drop_graph(ctx);
    const size_t img_bytes = sizeof(float) * 3ull * views[0].cam.width * views[0].cam.height * n_views;
    HIP_TRY(ensure(ctx->tune_ref, img_bytes));
    HIP_TRY(ensure(ctx->tune_img, img_bytes));
    HIP_TRY(ensure(ctx->tune_diff, sizeof(unsigned long long)));
    struct Cand { int tw, th, b, ppt, sched; };
    std::vector<Cand> cands;
    const int shapes[5][2] = {{16, 16}, {8, 8}, {32, 8}, {32, 16}, {32, 32}};
    for (int sched : {1, 0})
        for (auto &sh : shapes)
            for (int b : {64, 128, 256, 512, 1024})
                for (int ppt : {1, 2, 4})
                    if ((sh[0] * sh[1] > 64 || ppt == 1) && (b <= 256 || sh[0] * sh[1] == 1024))
                        cands.push_back({sh[0], sh[1], b, ppt, sched});
    hipEvent_t e0 = ctx->get_event(), e1 = ctx->get_event();
    if (!e0 || !e1) return fail(FDGS_ERR_HIP, "%s: event creation failed", fn);
    double best = 1e300;
    int best_i = -1;
    bool all_same = true;
    int32_t tried = 0;
    for (size_t i = 0; i < cands.size(); ++i) {
        fdgs_render_cfg c = *inout_cfg;
        c.tile_w = cands[i].tw;
        c.tile_h = cands[i].th;
        c.batch = cands[i].b;
        c.pixels_per_thread = cands[i].ppt;
        c.schedule = cands[i].sched;
        c.instance_capacity = 0;   // exact sizing: tile counts change with the tile shape
        float *dst = (i == 0 ? ctx->tune_ref : ctx->tune_img).as<float>();
        if (fdgs_status st = enqueue_batch(ctx, scenes, views, n_views, &c, per, true, dst, stream)) return st;
        double ms_best = 1e300;
        for (int r = 0; r < repeats; ++r) {
            HIP_TRY(hipEventRecord(e0, stream));
            if (fdgs_status st = enqueue_batch(ctx, scenes, views, n_views, &c, per, false, dst, stream)) return st;
            HIP_TRY(hipEventRecord(e1, stream));
            HIP_TRY(hipEventSynchronize(e1));
            float ms = 0.f;
            HIP_TRY(hipEventElapsedTime(&ms, e0, e1));
            ms_best = std::min(ms_best, (double)ms);
        }
        bool same = true;
        if (i > 0) {
            unsigned long long diff = 0;
            HIP_TRY(launch_count_diff(ctx->tune_ref.as<uint32_t>(), ctx->tune_img.as<uint32_t>(),
                                      (int64_t)(img_bytes / 4), ctx->tune_diff.as<unsigned long long>(), stream));
            HIP_TRY(hipMemcpyAsync(&diff, ctx->tune_diff.p, sizeof diff, hipMemcpyDeviceToHost, stream));
            HIP_TRY(hipStreamSynchronize(stream));
            same = diff == 0;
        }
        all_same = all_same && same;
        if (results && tried < max_results)
            results[tried] = fdgs_tune_result{c.tile_w, c.tile_h, c.batch, c.pixels_per_thread, c.schedule, ms_best,
                                              same ? 1 : 0};
        ++tried;
        if (same && ms_best < best) {
            best = ms_best;
            best_i = (int)i;
        }
    }
    ctx->free_events.push_back(e0);
    ctx->free_events.push_back(e1);
    if (n_results) *n_results = tried;
    if (best_i >= 0) {
        inout_cfg->tile_w = cands[best_i].tw;
        inout_cfg->tile_h = cands[best_i].th;
        inout_cfg->batch = cands[best_i].b;
        inout_cfg->pixels_per_thread = cands[best_i].ppt;
        inout_cfg->schedule = cands[best_i].sched;
    }
    if (!all_same) return fail(FDGS_ERR_STATE, "%s: a configuration rendered different images", fn);
    return FDGS_OK;
}

}  // extern "C"

namespace {

// The state a backward phase may use, or an error.
fdgs_status backward_state(fdgs_ctx *ctx, fdgs_state *state, const char *fn, fdgs_state **out) {
    if (!ctx) return fail(FDGS_ERR_INVALID_ARG, "%s: ctx is NULL", fn);
    fdgs_state *S = state ? find_state(ctx, state) : nullptr;
    if (!S) return fail(FDGS_ERR_STATE, "%s: state is not a live state of this context", fn);
    if (!S->has_forward) return fail(FDGS_ERR_STATE, "%s: state holds no forward pass", fn);
    if (S->model.sh_index)
        return fail(FDGS_ERR_UNSUPPORTED, "%s: the forward used vector-quantised SH (no adjoint)", fn);
    *out = S;
    return FDGS_OK;
}

fdgs_status check_grads(const fdgs_state *S, const fdgs_grads *grads, const char *fn) {
    if (!grads) return fail(FDGS_ERR_INVALID_ARG, "%s: grads is NULL", fn);
    if (S->model.n > 0 && (!grads->mean || !grads->log_scale || !grads->q_left || !grads->q_right ||
                           !grads->opacity_logit || !grads->sh))
        return fail(FDGS_ERR_INVALID_ARG, "%s: a gradient pointer is NULL", fn);
    return FDGS_OK;
}

// Phase 1: adjoint compositor into the state's per-Gaussian 2D gradients.
fdgs_status enqueue_backward_2d(fdgs_ctx *ctx, fdgs_state *S, const float *dL_drgb, hipStream_t stream) {
    if (stream != nullptr) S->beyond_null_stream = true;
    HIP_TRY(hipSetDevice(ctx->device));
    // float64 lines, or float32 (28% of their memory) where those do not fit; a state that found
    // no room for them does not ask again while its block is large enough for the small form
    const int64_t n_g2d = std::max<int64_t>(S->n_max, 1);
    const size_t lines = G2d::bytes(n_g2d, true), small = G2d::bytes(n_g2d, false);
    S->g2d_wide = S->g2d_wide || S->g2d.cap < small || S->g2d.cap >= lines;
    if (S->g2d_wide) {
        const hipError_t e = ensure(S->g2d, lines);
        if (e == hipErrorOutOfMemory) {
            (void)hipGetLastError();
            S->g2d_wide = false;
        } else {
            HIP_TRY(e);
        }
    }
    if (!S->g2d_wide) HIP_TRY(ensure(S->g2d, small));
    const G2d g2d{S->g2d.p, S->g2d_wide};
    StageTimer tm(ctx, FDGS_STAGE_BWD_COMPOSITE, stream);
    HIP_TRY(launch_clear_g2d(S->vis_list, S->counts.as<int64_t>(), S->n_max, g2d, stream));
    // the adjoint takes the tiles longest list first: the forward's order when it
    // made one, else one made here
    const int32_t n_tiles = S->rp.tiles_x * S->rp.tiles_y;
    if (!S->ordered) {
        HIP_TRY(ensure(S->sched, sizeof(uint32_t) * std::max<int32_t>(n_tiles, 1)));
        HIP_TRY(launch_tile_order(S->ranges.as<uint32_t>(), n_tiles, S->sched.as<uint32_t>(), stream));
        S->ordered = true;
    }
    HIP_TRY(launch_composite_backward(S->rp, S->W, S->H, S->batch, S->ppt, S->ranges.as<uint32_t>(), S->sorted_ids,
                                      S->rec.as<Rec2D>(), S->T_final.as<float>(), S->n_contrib.as<uint32_t>(),
                                      dL_drgb, g2d, S->n_max, S->sched.as<uint32_t>(), stream));
    S->has_g2d = true;
    return FDGS_OK;
}

// Phase 2: the 2D gradients through projection, slicing and activations into grads.
fdgs_status enqueue_backward_params(fdgs_ctx *ctx, fdgs_state *S, const fdgs_grads *grads, hipStream_t stream) {
    if (stream != nullptr) S->beyond_null_stream = true;
    HIP_TRY(hipSetDevice(ctx->device));
    StageTimer tm(ctx, FDGS_STAGE_BWD_PREPROCESS, stream);
    const int64_t *n_proc_dev = S->idx ? S->n_idx_dev : nullptr;
    HIP_TRY(launch_preprocess_backward(kmodel(&S->model), S->idx, n_proc_dev, S->n_max, S->cam, S->t, S->rp,
                                       S->vis_list, S->counts.as<int64_t>(), G2d{S->g2d.p, S->g2d_wide}, *grads, stream));
    return FDGS_OK;
}

}  // namespace

extern "C" {

fdgs_status fdgs_render_backward(fdgs_ctx *ctx, fdgs_state *state, const float *dL_drgb, const fdgs_grads *grads,
                                 hipStream_t stream) {
    const char *fn = "fdgs_render_backward";
    fdgs_state *S = nullptr;
    if (fdgs_status st = backward_state(ctx, state, fn, &S)) return st;
    if (!dL_drgb) return fail(FDGS_ERR_INVALID_ARG, "%s: dL_drgb is NULL", fn);
    if (fdgs_status st = check_grads(S, grads, fn)) return st;
    if (fdgs_status st = enqueue_backward_2d(ctx, S, dL_drgb, stream)) return st;
    return enqueue_backward_params(ctx, S, grads, stream);
}

fdgs_status fdgs_render_backward_2d(fdgs_ctx *ctx, fdgs_state *state, const float *dL_drgb, hipStream_t stream) {
    const char *fn = "fdgs_render_backward_2d";
    fdgs_state *S = nullptr;
    if (fdgs_status st = backward_state(ctx, state, fn, &S)) return st;
    if (!dL_drgb) return fail(FDGS_ERR_INVALID_ARG, "%s: dL_drgb is NULL", fn);
    return enqueue_backward_2d(ctx, S, dL_drgb, stream);
}

fdgs_status fdgs_render_backward_params(fdgs_ctx *ctx, fdgs_state *state, const fdgs_grads *grads,
                                        hipStream_t stream) {
    const char *fn = "fdgs_render_backward_params";
    fdgs_state *S = nullptr;
    if (fdgs_status st = backward_state(ctx, state, fn, &S)) return st;
    if (!S->has_g2d)
        return fail(FDGS_ERR_STATE, "%s: no fdgs_render_backward_2d since the state's last forward", fn);
    if (fdgs_status st = check_grads(S, grads, fn)) return st;
    return enqueue_backward_params(ctx, S, grads, stream);
}

fdgs_status fdgs_state_release(fdgs_ctx *ctx, fdgs_state *state) {
    if (!ctx) return fail(FDGS_ERR_INVALID_ARG, "fdgs_state_release: ctx is NULL");
    if (!state) return FDGS_OK;
    fdgs_state *S = find_state(ctx, state);
    if (!S) return fail(FDGS_ERR_STATE, "fdgs_state_release: unknown state");
    ctx->states.erase(std::find(ctx->states.begin(), ctx->states.end(), S));
    if (!S->beyond_null_stream && keep_spare(S, ctx->device)) return FDGS_OK;
    (void)hipSetDevice(ctx->device);
    (void)hipDeviceSynchronize();
    S->free_all();
    delete S;
    return FDGS_OK;
}

fdgs_status fdgs_state_binning(fdgs_ctx *ctx, fdgs_state *state, fdgs_binning *out, hipStream_t stream) {
    const char *fn = "fdgs_state_binning";
    if (!ctx || !out) return fail(FDGS_ERR_INVALID_ARG, "%s: ctx or out is NULL", fn);
    fdgs_state *S = state ? find_state(ctx, state) : nullptr;
    if (!S || !S->has_forward) return fail(FDGS_ERR_STATE, "%s: no forward pass in state", fn);
    HIP_TRY(hipSetDevice(ctx->device));
    S->beyond_null_stream = true;   // the caller may read the buffers on any stream
    HIP_TRY(hipMemcpyAsync(ctx->host_counts, S->counts.p, 2 * sizeof(int64_t), hipMemcpyDeviceToHost, stream));
    int64_t nproc = S->n_max;
    if (S->idx) HIP_TRY(hipMemcpyAsync(ctx->host_counts + 2, S->n_idx_dev, sizeof(int64_t), hipMemcpyDeviceToHost, stream));
    HIP_TRY(hipStreamSynchronize(stream));
    if (S->idx) nproc = std::min(ctx->host_counts[2], S->n_max);
    out->sorted_ids = S->sorted_ids;
    out->tile_ranges = S->ranges.as<uint32_t>();
    out->rects = S->rect.as<int32_t>();
    out->depth = reinterpret_cast<const double *>(S->depth_key.p);
    out->visible = S->visible.as<uint8_t>();
    out->n_vis = ctx->host_counts[0];
    out->n_inst = std::min(ctx->host_counts[1], S->capacity);
    out->n_proc = nproc;
    out->n_tiles = S->rp.tiles_x * S->rp.tiles_y;
    out->tiles_x = S->rp.tiles_x;
    out->tiles_y = S->rp.tiles_y;
    return FDGS_OK;
}

fdgs_status fdgs_profile_enable(fdgs_ctx *ctx, int32_t enable) {
    if (!ctx) return fail(FDGS_ERR_INVALID_ARG, "fdgs_profile_enable: ctx is NULL");
    HIP_TRY(hipSetDevice(ctx->device));
    if (enable && !ctx->prof_acc.p) {
        HIP_TRY(ensure(ctx->prof_acc, 5 * sizeof(uint64_t)));
        HIP_TRY(hipMemset(ctx->prof_acc.p, 0, 5 * sizeof(uint64_t)));
    }
    ctx->prof = enable <= 0 ? 0 : (enable >= 2 ? 2 : 1);
    return FDGS_OK;
}

fdgs_status fdgs_profile_read(fdgs_ctx *ctx, fdgs_profile *out, int32_t reset) {
    if (!ctx || !out) return fail(FDGS_ERR_INVALID_ARG, "fdgs_profile_read: ctx or out is NULL");
    HIP_TRY(hipSetDevice(ctx->device));
    HIP_TRY(hipDeviceSynchronize());
    for (auto &p : ctx->pending) {
        float ms = 0.f;
        HIP_TRY(hipEventElapsedTime(&ms, p.e0, p.e1));
        ctx->ms[p.stage] += ms;
        ctx->calls[p.stage] += 1;
        ctx->free_events.push_back(p.e0);
        ctx->free_events.push_back(p.e1);
    }
    ctx->pending.clear();
    std::memset(out, 0, sizeof *out);
    for (int k = 0; k < FDGS_NUM_STAGES; ++k) {
        out->ms[k] = ctx->ms[k];
        out->calls[k] = ctx->calls[k];
    }
    if (ctx->prof_acc.p) {
        uint64_t acc[5];
        HIP_TRY(hipMemcpy(acc, ctx->prof_acc.p, sizeof acc, hipMemcpyDeviceToHost));
        out->processed = (int64_t)acc[0];
        out->visible = (int64_t)acc[1];
        out->instances = (int64_t)acc[2];
        out->pairs = acc[3];
        out->blended = acc[4];
        if (reset) HIP_TRY(hipMemset(ctx->prof_acc.p, 0, sizeof acc));
    }
    if (reset) {
        for (int k = 0; k < FDGS_NUM_STAGES; ++k) {
            ctx->ms[k] = 0.0;
            ctx->calls[k] = 0;
        }
    }
    return FDGS_OK;
}

fdgs_status fdgs_spatial_score(fdgs_ctx *ctx, const fdgs_model *model, const fdgs_camera *cams, const double *times,
                               int32_t n_views, const fdgs_render_cfg *cfg, float *inout_score, hipStream_t stream) {
    const char *fn = "fdgs_spatial_score";
    if (!ctx) return fail(FDGS_ERR_INVALID_ARG, "%s: ctx is NULL", fn);
    if (fdgs_status st = check_model(model, fn)) return st;
    if (n_views < 0 || (n_views > 0 && (!cams || !times)))
        return fail(FDGS_ERR_INVALID_ARG, "%s: need n_views >= 0 cameras and times", fn);
    fdgs_render_cfg c;
    if (cfg) {
        if (fdgs_status st = check_cfg(cfg, fn)) return st;
        c = *cfg;
    } else {
        fdgs_render_cfg_default(&c);
        c.pixels_per_thread = 2;
    }
    c.instance_capacity = 0;
    if (c.tile_w * c.tile_h == 64) c.pixels_per_thread = 1;
    if (model->n > 0 && !inout_score) return fail(FDGS_ERR_INVALID_ARG, "%s: inout_score is NULL", fn);
    for (int v = 0; v < n_views; ++v) {
        if (fdgs_status st = check_camera(&cams[v], fn)) return st;
        if (!std::isfinite(times[v])) return fail(FDGS_ERR_INVALID_ARG, "%s: view %d time not finite", fn, v);
    }
    HIP_TRY(hipSetDevice(ctx->device));
    const SidePass pass{cams, n_views, times, n_views, false};
    if (fdgs_status st = run_side_views(ctx, model, pass, cfg ? &c : nullptr, c, nullptr, inout_score, stream)) return st;
    HIP_TRY(hipStreamSynchronize(stream));
    return FDGS_OK;
}

fdgs_status fdgs_variation_score(fdgs_ctx *ctx, const fdgs_model *model, const double *times, int32_t n_times,
                                 const float *spatial, float *out_score, hipStream_t stream) {
    const char *fn = "fdgs_variation_score";
    if (!ctx) return fail(FDGS_ERR_INVALID_ARG, "%s: ctx is NULL", fn);
    if (fdgs_status st = check_model(model, fn)) return st;
    if (n_times < 0 || (n_times > 0 && !times)) return fail(FDGS_ERR_INVALID_ARG, "%s: bad times", fn);
    for (int f = 0; f < n_times; ++f)
        if (!std::isfinite(times[f])) return fail(FDGS_ERR_INVALID_ARG, "%s: non-finite time", fn);
    const int64_t n = model->n;
    if (n > 0 && (!spatial || !out_score)) return fail(FDGS_ERR_INVALID_ARG, "%s: a score pointer is NULL", fn);
    if (n == 0) return FDGS_OK;
    if (n >= (int64_t(1) << 32)) return fail(FDGS_ERR_INVALID_ARG, "%s: n too large", fn);
    HIP_TRY(hipSetDevice(ctx->device));
    HIP_TRY(ensure(ctx->prune_times, sizeof(double) * std::max(1, n_times)));
    if (n_times > 0)
        HIP_TRY(hipMemcpyAsync(ctx->prune_times.p, times, sizeof(double) * n_times, hipMemcpyHostToDevice, stream));
    HIP_TRY(ensure(ctx->prune_a, sizeof(float) * n));      // S^TV
    HIP_TRY(ensure(ctx->prune_b, sizeof(uint32_t) * n));   // volume keys
    HIP_TRY(ensure(ctx->prune_c, sizeof(uint32_t) * n));   // values
    HIP_TRY(ensure(ctx->prune_d, sizeof(uint32_t) * 3 * n));   // sort ping-pong (keys, values) and a copy
    HIP_TRY(ensure(ctx->prune_e, sort_scratch_bytes(n)));
    uint32_t *vk = ctx->prune_b.as<uint32_t>(), *vv = ctx->prune_c.as<uint32_t>();
    uint32_t *k2 = ctx->prune_d.as<uint32_t>(), *v2 = k2 + n, *keep_keys = v2 + n;
    HIP_TRY(launch_temporal_volume(kmodel(model), ctx->prune_times.as<double>(), n_times, ctx->prune_a.as<float>(),
                                   vk, vv, stream));
    HIP_TRY(hipMemcpyAsync(keep_keys, vk, sizeof(uint32_t) * n, hipMemcpyDeviceToDevice, stream));
    int alt = 0;
    HIP_TRY(radix_sort_u32(vk, vv, k2, v2, nullptr, n, 0, 32, ctx->prune_e.p, &alt, stream));
    const uint32_t *sorted = alt ? k2 : vk;
    const int64_t q = (int64_t)std::floor(0.9 * (double)(n - 1));
    HIP_TRY(launch_variation_score(ctx->prune_a.as<float>(), keep_keys, sorted, n, q, spatial, out_score, stream));
    HIP_TRY(hipStreamSynchronize(stream));
    return FDGS_OK;
}

fdgs_status fdgs_prune(fdgs_ctx *ctx, const float *score, int64_t n, int64_t n_keep, uint32_t *out_bits,
                       uint32_t *out_idx, int64_t *out_count, hipStream_t stream) {
    const char *fn = "fdgs_prune";
    if (!ctx) return fail(FDGS_ERR_INVALID_ARG, "%s: ctx is NULL", fn);
    if (n < 0 || n >= (int64_t(1) << 32)) return fail(FDGS_ERR_INVALID_ARG, "%s: n out of range", fn);
    if (n_keep < 0 || n_keep > n) return fail(FDGS_ERR_INVALID_ARG, "%s: n_keep out of range", fn);
    if (!out_bits || !out_idx || !out_count || (n > 0 && !score))
        return fail(FDGS_ERR_INVALID_ARG, "%s: a pointer is NULL", fn);
    HIP_TRY(hipSetDevice(ctx->device));
    HIP_TRY(ensure(ctx->prune_b, sizeof(uint32_t) * std::max<int64_t>(n, 1)));
    HIP_TRY(ensure(ctx->prune_c, sizeof(uint32_t) * std::max<int64_t>(n, 1)));
    HIP_TRY(ensure(ctx->prune_d, sizeof(uint32_t) * 3 * std::max<int64_t>(n, 1)));
    HIP_TRY(ensure(ctx->prune_e, std::max(sort_scratch_bytes(n), compact_scratch_bytes(n))));
    HIP_TRY(ensure(ctx->mask_flags, (size_t)((n + 3) / 4) * 4 + 4));
    uint32_t *keys = ctx->prune_b.as<uint32_t>(), *vals = ctx->prune_c.as<uint32_t>();
    uint32_t *k2 = ctx->prune_d.as<uint32_t>(), *v2 = k2 + n;
    HIP_TRY(launch_fill_u32(ctx->mask_flags.as<uint32_t>(), (n + 3) / 4, 0u, stream));
    HIP_TRY(launch_prune_keys(score, n, keys, vals, stream));
    int alt = 0;
    HIP_TRY(radix_sort_u32(keys, vals, k2, v2, nullptr, n, 0, 32, ctx->prune_e.p, &alt, stream));
    HIP_TRY(launch_mark_first(alt ? v2 : vals, n_keep, ctx->mask_flags.as<uint8_t>(), stream));
    HIP_TRY(launch_flags_to_bits(ctx->mask_flags.as<uint8_t>(), n, out_bits, stream));
    HIP_TRY(compact_bits(out_bits, n, out_idx, out_count, ctx->prune_e.p, stream));
    HIP_TRY(hipStreamSynchronize(stream));
    return FDGS_OK;
}

fdgs_status fdgs_sh_kmeans(fdgs_ctx *ctx, const fdgs_model *model, const uint32_t *init_index, int64_t k,
                           int32_t iterations, float *codebook, uint32_t *assignment, hipStream_t stream) {
    const char *fn = "fdgs_sh_kmeans";
    if (!ctx) return fail(FDGS_ERR_INVALID_ARG, "%s: ctx is NULL", fn);
    if (fdgs_status st = check_model(model, fn)) return st;
    if (!model->sh) return fail(FDGS_ERR_INVALID_ARG, "%s: model->sh is NULL (nothing to quantise)", fn);
    if (k < 1 || k > (int64_t(1) << 24)) return fail(FDGS_ERR_INVALID_ARG, "%s: k=%lld not in [1, 2^24]", fn, (long long)k);
    if (iterations < 0 || iterations > 1000)
        return fail(FDGS_ERR_INVALID_ARG, "%s: iterations=%d not in [0, 1000]", fn, iterations);
    if (!init_index || !codebook || !assignment)
        return fail(FDGS_ERR_INVALID_ARG, "%s: init_index, codebook or assignment is NULL", fn);
    if (reinterpret_cast<uintptr_t>(codebook) % 16 != 0)
        return fail(FDGS_ERR_INVALID_ARG, "%s: codebook must be 16-byte aligned", fn);
    if (model->n == 0) return FDGS_OK;
    HIP_TRY(hipSetDevice(ctx->device));
    bool lean = false;   // no room for the screening's arrays: the search alone, in a tenth of the memory
    hipError_t e = ensure(ctx->vq_scratch, vq_scratch_bytes(model->n, k, lean));
    if (e == hipErrorOutOfMemory) {
        (void)hipGetLastError();
        lean = true;
        e = ensure(ctx->vq_scratch, vq_scratch_bytes(model->n, k, lean));
    }
    HIP_TRY(e);
    HIP_TRY(vq_kmeans(model->sh, model->n, init_index, k, iterations, codebook, assignment, ctx->vq_scratch.p, lean,
                      stream));
    return FDGS_OK;
}

fdgs_status fdgs_adam_step(fdgs_ctx *ctx, float *param, const float *grad, float *m, float *v, int64_t n, float lr,
                           float beta1, float beta2, float eps, int32_t step, hipStream_t stream) {
    const char *fn = "fdgs_adam_step";
    if (!ctx) return fail(FDGS_ERR_INVALID_ARG, "%s: ctx is NULL", fn);
    if (n < 0) return fail(FDGS_ERR_INVALID_ARG, "%s: n < 0", fn);
    if (n > 0 && (!param || !grad || !m || !v)) return fail(FDGS_ERR_INVALID_ARG, "%s: a pointer is NULL", fn);
    if (step < 1) return fail(FDGS_ERR_INVALID_ARG, "%s: step must be >= 1", fn);
    if (!(beta1 >= 0.0f && beta1 < 1.0f) || !(beta2 >= 0.0f && beta2 < 1.0f) || !(eps > 0.0f) ||
        !std::isfinite(lr))
        return fail(FDGS_ERR_INVALID_ARG, "%s: need 0 <= beta < 1, eps > 0, finite lr", fn);
    HIP_TRY(hipSetDevice(ctx->device));
    HIP_TRY(launch_adam(param, grad, m, v, n, lr, beta1, beta2, eps, step, stream));
    return FDGS_OK;
}

fdgs_status fdgs_check_overflow(fdgs_ctx *ctx, hipStream_t stream) {
    if (!ctx) return fail(FDGS_ERR_INVALID_ARG, "fdgs_check_overflow: ctx is NULL");
    HIP_TRY(hipSetDevice(ctx->device));
    int32_t flag = 0;
    HIP_TRY(hipMemcpyAsync(&flag, ctx->overflow.p, sizeof flag, hipMemcpyDeviceToHost, stream));
    HIP_TRY(hipStreamSynchronize(stream));
    if (flag) {
        HIP_TRY(hipMemsetAsync(ctx->overflow.p, 0, sizeof flag, stream));
        HIP_TRY(hipStreamSynchronize(stream));
        if (flag & 1)
            return fail(FDGS_ERR_CAPACITY, "fdgs_check_overflow: a forward pass exceeded its instance capacity");
        return fail(FDGS_ERR_UNSUPPORTED,
                    "fdgs_check_overflow: more than 4096 Gaussians shared one float32 depth; "
                    "their order fell back to processing order");
    }
    return FDGS_OK;
}

}  // extern "C"
