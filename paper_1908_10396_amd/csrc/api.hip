// C ABI of libavq (declared in include/avq.h): argument checking, the index
// object, device buffers and the sequence of kernel launches of each call.
#include <stdarg.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <mutex>
#include <new>

#include "avq_internal.h"
#include <cmath>

namespace avq {

static thread_local char g_err[512] = "";

void set_error(const char *fmt, ...)
{
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof(g_err), fmt, ap);
    va_end(ap);
}

int DevBuf::reserve(size_t bytes)
{
    if (bytes <= cap) return AVQ_OK;
    if (p) { (void)hipFree(p); p = nullptr; cap = 0; }
    if (limit != 0 && bytes > limit) { set_error("%zu bytes of scratch exceed the limit", bytes); return AVQ_ENOMEM; }
    hipError_t e = hipMalloc(&p, bytes);
    if (e != hipSuccess) {
        p = nullptr;
        (void)hipGetLastError();
        set_error("hipMalloc(%zu) failed: %s", bytes, hipGetErrorString(e));
        return e == hipErrorOutOfMemory ? AVQ_ENOMEM : AVQ_EHIP;
    }
    cap = bytes;
    return AVQ_OK;
}

void DevBuf::release()
{
    if (p) (void)hipFree(p);
    p = nullptr;
    cap = 0;
}

} // namespace avq

using namespace avq;

struct avq_index {
    avq_config cfg;
    int kc = 0, ds = 0, NB = 0;
    bool have_codebooks = false, have_centers = false;
    DevBuf codebooks, centers, centers_t;
    // database
    int64_t n = 0, n_slots = 0, n_blocks = 0, max_leaf_blocks = 0;
    const float *x = nullptr;
    DevBuf x_own, codes_logical, codes_blocked, assign, perm, leaf_blk;
    // per-call scratch
    DevBuf lut, lut8, scale, bias, partial, cand, leaf_ids, leaf_ip, tmp, thr;
    int tune_target_wgs = 0, tune_waves = 0, tune_qt = 0, tune_small_batch = -1, tune_small_impl = 0, tune_select_split = 0, tune_rerank_split = 0, tune_bound_bits = 0;
    int tune_stream_loads = 0; // single-query scan of the code array: 0 = nontemporal loads when the array exceeds the Infinity Cache, 1 = never, 2 = always
    int tune_mfma = 0; // 0 = use the matrix-core scan where it applies, 1 = never
    int tune_prefilter = 0; // 0 = fp32-table batches go through the 8-bit-table scan where it applies, 1 = never,
                            // 2 = as 0 but odd queries always take the plain scan afterwards (exercises that branch)
    int tune_bound_leaves = 0; // leaves per query that supply the bound of the grouped scan over leaves, 0 = built-in
    int tune_group_min = 0; // (query, leaf) pairs from which a batch on a partitioned index is regrouped by leaf; 0 = built in
    int tune_product = 0; // 0 = flat batches through the product of queries and decoded points where it applies, 1 = never, 2 = wherever it can
    int tune_sample = 0; // 0 = batches guess the candidate scan's bounds from a sample where possible, 1 = never, 2 = from a sample scanned with lists
    int tune_prefilter_cap = 0; // candidate keys per (query, chunk) of that scan, 0 = built-in
    DevBuf block_max, lists, refined, lut_fail, fail, cand_keys, groups, kept, fail_rows, product;
    DevBuf exact_ws; // exact search: operands, norms, block maxima of a launch's queries (exact_scratch)
    // training and encoding: points by coordinate and the sums of an iteration, undecided points, tables (ScratchKeeper)
    DevBuf train_ws;
    // optional per-stage timing with HIP events recorded on the caller's stream
    bool prof_on = false;
    std::vector<hipEvent_t> prof_pool;
    size_t prof_used = 0;
    struct ProfRec { int stage; hipEvent_t a, b; };
    std::vector<ProfRec> prof_recs;
};

// Records an event pair around one stage's launches while profiling is on.
struct StageTimer {
    avq_index *idx;
    hipStream_t st;
    hipEvent_t a = nullptr, b = nullptr;
    int stage;
    StageTimer(avq_index *i, int stage_, hipStream_t s, bool enabled = true) : idx(i), st(s), stage(stage_)
    {
        if (!idx->prof_on || !enabled) return; // (creating an event allocates)
        while (idx->prof_pool.size() < idx->prof_used + 2) {
            hipEvent_t e;
            if (hipEventCreate(&e) != hipSuccess) return;
            idx->prof_pool.push_back(e);
        }
        a = idx->prof_pool[idx->prof_used++];
        b = idx->prof_pool[idx->prof_used++];
        (void)hipEventRecord(a, st);
    }
    ~StageTimer()
    {
        if (!a) return;
        (void)hipEventRecord(b, st);
        idx->prof_recs.push_back({stage, a, b});
    }
};

// Scratch that an index keeps between calls of one kind; what a larger training or encoding needs is given back at its end
// (both synchronise there anyway).
constexpr size_t kKeepScratch = (size_t)256 << 20;
struct ScratchKeeper {
    DevBuf *ws;
    ~ScratchKeeper() { if (ws->cap > kKeepScratch) ws->release(); }
};

// Exact search does not synchronise, so what it takes it keeps: at most as much as the points themselves (kKeepScratch
// where they are few, 2 GiB where they are many). Fewer queries a launch cost: with 256 MB, 10,000,000 x 128 points and
// 1,000 queries took 6.8 instead of 4.5 ms, 1,183,514 x 100 and 4,000 queries 2.13 instead of 1.94.
static size_t exact_scratch(int64_t n, int d)
{
    return std::min<size_t>((size_t)2 << 30, std::max(kKeepScratch, sizeof(float) * (size_t)n * d));
}

static int check_index(const avq_index *idx)
{
    if (!idx) { set_error("index is NULL"); return AVQ_EINVAL; }
    return AVQ_OK;
}

extern "C" const char *avq_last_error(void) { return g_err; }
extern "C" const char *avq_version(void) { return "avq 0.1 (gfx950)"; }

extern "C" double avq_eta(int32_t d, double T, double norm, int32_t eta_mode)
{
    if (eta_mode != AVQ_ETA_LIMIT && eta_mode != AVQ_ETA_EXACT) return -1.0;
    return eta_host(d, T, norm, eta_mode);
}

extern "C" int avq_create(const avq_config *cfg, avq_index **out)
{
    if (!cfg || !out) { set_error("avq_create: NULL argument"); return AVQ_EINVAL; }
    *out = nullptr;
    if (cfg->d < 2 || cfg->M < 1 || cfg->d % cfg->M != 0) {
        set_error("avq_create: need d >= 2, M >= 1, d %% M == 0 (d=%d M=%d)", cfg->d, cfg->M);
        return AVQ_EINVAL;
    }
    if (cfg->bits != 4 && cfg->bits != 8) { set_error("avq_create: bits must be 4 or 8"); return AVQ_EINVAL; }
    if (!(cfg->T >= 0.0f)) { set_error("avq_create: T must be >= 0"); return AVQ_EINVAL; }
    if (cfg->eta_mode < 0 || cfg->eta_mode > 2) { set_error("avq_create: bad eta_mode"); return AVQ_EINVAL; }
    if (cfg->eta_mode == AVQ_ETA_EXPLICIT && !(cfg->eta_explicit >= 1.0f)) {
        set_error("avq_create: eta_explicit must be >= 1");
        return AVQ_EINVAL;
    }
    if (cfg->kmeans_iters < 0 || cfg->encode_passes < 0 || cfg->n_leaves < 0 || cfg->leaf_kmeans_iters < 0 ||
        cfg->leaf_aniso_iters < 0) {
        set_error("avq_create: negative count");
        return AVQ_EINVAL;
    }
    if (cfg->M > 256) { set_error("avq_create: M > 256 not supported"); return AVQ_EINVAL; }
    avq_index *idx = new (std::nothrow) avq_index();
    if (!idx) { set_error("avq_create: out of host memory"); return AVQ_ENOMEM; }
    idx->cfg = *cfg;
    idx->kc = 1 << cfg->bits;
    idx->ds = cfg->d / cfg->M;
    idx->NB = (cfg->M * cfg->bits + 7) / 8;
    int rc = idx->codebooks.reserve(sizeof(float) * (size_t)cfg->M * idx->kc * idx->ds);
    if (rc == AVQ_OK && cfg->n_leaves > 0) {
        rc = idx->centers.reserve(sizeof(float) * (size_t)cfg->n_leaves * cfg->d);
        if (rc == AVQ_OK) rc = idx->centers_t.reserve(sizeof(float) * (size_t)cfg->n_leaves * cfg->d);
    }
    if (rc != AVQ_OK) { avq_destroy(idx); return rc; }
    *out = idx;
    return AVQ_OK;
}

extern "C" void avq_destroy(avq_index *idx)
{
    if (!idx) return;
    DevBuf *all[] = {&idx->exact_ws, &idx->codebooks, &idx->centers, &idx->centers_t, &idx->x_own, &idx->codes_logical,
                     &idx->codes_blocked, &idx->assign, &idx->perm, &idx->leaf_blk, &idx->lut, &idx->lut8,
                     &idx->scale, &idx->bias, &idx->partial, &idx->cand, &idx->leaf_ids, &idx->leaf_ip,
                     &idx->tmp, &idx->block_max, &idx->lists, &idx->thr, &idx->refined, &idx->lut_fail,
                     &idx->fail, &idx->cand_keys, &idx->groups, &idx->kept, &idx->fail_rows, &idx->product, &idx->train_ws};
    for (DevBuf *b : all) b->release();
    for (hipEvent_t e : idx->prof_pool) (void)hipEventDestroy(e);
    delete idx;
}

extern "C" int64_t avq_size(const avq_index *idx) { return idx ? idx->n : 0; }

extern "C" int avq_set_tuning(avq_index *idx, const char *name, int32_t value)
{
    AVQ_TRY(check_index(idx));
    if (!name || value < 0) { set_error("avq_set_tuning: bad argument"); return AVQ_EINVAL; }
    if (!strcmp(name, "scan_target_wgs")) idx->tune_target_wgs = value;
    else if (!strcmp(name, "scan_waves")) idx->tune_waves = value;
    else if (!strcmp(name, "scan_qt")) idx->tune_qt = value;
    else if (!strcmp(name, "small_batch_max")) idx->tune_small_batch = value - 1; // 0 = built-in
    else if (!strcmp(name, "small_batch_impl")) idx->tune_small_impl = value;
    else if (!strcmp(name, "scan_mfma")) idx->tune_mfma = value;
    else if (!strcmp(name, "scan_prefilter")) idx->tune_prefilter = value;
    else if (!strcmp(name, "prefilter_cap")) idx->tune_prefilter_cap = value;
    else if (!strcmp(name, "scan_product")) idx->tune_product = value;
    else if (!strcmp(name, "scan_sample")) idx->tune_sample = value;
    else if (!strcmp(name, "group_min_pairs")) idx->tune_group_min = value;
    else if (!strcmp(name, "bound_leaves")) idx->tune_bound_leaves = value;
    else if (!strcmp(name, "select_split")) idx->tune_select_split = value;
    else if (!strcmp(name, "rerank_split")) idx->tune_rerank_split = value;
    else if (!strcmp(name, "bound_bits")) idx->tune_bound_bits = value;
    else if (!strcmp(name, "stream_loads")) idx->tune_stream_loads = value;
    else if (!strcmp(name, "scratch_limit_kb")) {
        idx->train_ws.limit = idx->exact_ws.limit = idx->product.limit = (size_t)value * 1024;
        if (value > 0 && idx->train_ws.cap > idx->train_ws.limit) idx->train_ws.release();
        if (value > 0 && idx->exact_ws.cap > idx->exact_ws.limit) idx->exact_ws.release();
        if (value > 0 && idx->product.cap > idx->product.limit) idx->product.release();
    }
    else { set_error("avq_set_tuning: unknown name '%s'", name); return AVQ_EINVAL; }
    return AVQ_OK;
}

extern "C" int avq_profile_enable(avq_index *idx, int32_t on)
{
    AVQ_TRY(check_index(idx));
    idx->prof_on = on != 0;
    return AVQ_OK;
}

extern "C" int avq_profile_read(avq_index *idx, double *ms_out, int64_t *launches_out, int32_t reset)
{
    AVQ_TRY(check_index(idx));
    if (!ms_out || !launches_out) { set_error("avq_profile_read: NULL output"); return AVQ_EINVAL; }
    for (int s = 0; s < AVQ_N_STAGES; ++s) { ms_out[s] = 0.0; launches_out[s] = 0; }
    for (const avq_index::ProfRec &r : idx->prof_recs) {
        AVQ_HIP(hipEventSynchronize(r.b));
        float ms = 0.0f;
        AVQ_HIP(hipEventElapsedTime(&ms, r.a, r.b));
        ms_out[r.stage] += (double)ms;
        launches_out[r.stage] += 1;
    }
    if (reset) { idx->prof_recs.clear(); idx->prof_used = 0; }
    return AVQ_OK;
}

// ---- dictionaries and leaf centers -------------------------------------------------

extern "C" int avq_set_codebooks(avq_index *idx, const float *codebooks)
{
    AVQ_TRY(check_index(idx));
    if (!codebooks) { set_error("avq_set_codebooks: NULL"); return AVQ_EINVAL; }
    AVQ_HIP(hipMemcpy(idx->codebooks.p, codebooks, sizeof(float) * (size_t)idx->cfg.M * idx->kc * idx->ds,
                      hipMemcpyDefault));
    idx->have_codebooks = true;
    return AVQ_OK;
}

extern "C" int avq_get_codebooks(avq_index *idx, float *out)
{
    AVQ_TRY(check_index(idx));
    if (!out) { set_error("avq_get_codebooks: NULL"); return AVQ_EINVAL; }
    if (!idx->have_codebooks) { set_error("avq_get_codebooks: no dictionaries yet"); return AVQ_ESTATE; }
    AVQ_HIP(hipMemcpy(out, idx->codebooks.p, sizeof(float) * (size_t)idx->cfg.M * idx->kc * idx->ds,
                      hipMemcpyDefault));
    return AVQ_OK;
}

static int refresh_centers_t(avq_index *idx, hipStream_t st)
{
    AVQ_TRY(launch_transpose(idx->centers.as<float>(), idx->cfg.n_leaves, idx->cfg.d,
                             idx->centers_t.as<float>(), st));
    AVQ_HIP(hipStreamSynchronize(st));
    return AVQ_OK;
}

extern "C" int avq_set_leaf_centers(avq_index *idx, const float *centers)
{
    AVQ_TRY(check_index(idx));
    if (idx->cfg.n_leaves <= 0) { set_error("avq_set_leaf_centers: flat index"); return AVQ_ESTATE; }
    if (!centers) { set_error("avq_set_leaf_centers: NULL"); return AVQ_EINVAL; }
    AVQ_HIP(hipMemcpy(idx->centers.p, centers, sizeof(float) * (size_t)idx->cfg.n_leaves * idx->cfg.d,
                      hipMemcpyDefault));
    AVQ_TRY(refresh_centers_t(idx, nullptr));
    idx->have_centers = true;
    return AVQ_OK;
}

extern "C" int avq_get_leaf_centers(avq_index *idx, float *out)
{
    AVQ_TRY(check_index(idx));
    if (idx->cfg.n_leaves <= 0 || !idx->have_centers) {
        set_error("avq_get_leaf_centers: no leaf centers");
        return AVQ_ESTATE;
    }
    if (!out) { set_error("avq_get_leaf_centers: NULL"); return AVQ_EINVAL; }
    AVQ_HIP(hipMemcpy(out, idx->centers.p, sizeof(float) * (size_t)idx->cfg.n_leaves * idx->cfg.d,
                      hipMemcpyDefault));
    return AVQ_OK;
}

// Assignment of rows to leaves: nearest center, or smallest anisotropic loss when the index learns its
// leaves as an anisotropic vector quantizer (cfg.leaf_aniso_iters > 0).
static int assign_to_leaves(avq_index *idx, const float *x, int64_t n, int32_t *assign, hipStream_t st)
{
    const avq_config &c = idx->cfg;
    if (c.leaf_aniso_iters > 0)
        return launch_assign_aniso(x, n, c.d, idx->centers.as<float>(), c.n_leaves, c.eta_mode, (double)c.T,
                                   (double)c.eta_explicit, assign, st);
    // Few points and centers: one launch of fp64 distances instead of four (one avq_encode, us, four / one): 1,000 and 16,384
    // points: 8 x 32 about 147 / 118 and 162 / 137, 32 x 32 136 / 127 and 159 / 149, 64 x 32 136 / 156 and 159 / 174.
    const bool few = n <= 16384 && (int64_t)c.n_leaves * c.d <= 1024;
    if (few || !nearest_supported(c.d, c.n_leaves))
        return launch_assign_nearest(x, n, c.d, idx->centers.as<float>(), c.n_leaves, assign, st);
    // The lists of undecided points take 20 bytes a point: 84 MB for 4,194,304 rows at a time (a launch of so many fills the
    // chip; the centers are packed again for each, some 10 us).
    const int64_t rows = std::min<int64_t>(n, (int64_t)1 << 22);
    const int rc = idx->train_ws.reserve(nearest_ws_bytes(rows, c.d, c.n_leaves, 1));
    if (rc == AVQ_ENOMEM) return launch_assign_nearest(x, n, c.d, idx->centers.as<float>(), c.n_leaves, assign, st); // needs no scratch
    AVQ_TRY(rc);
    for (int64_t i = 0; i < n; i += rows)
        AVQ_TRY(launch_nearest(x + (size_t)i * c.d, std::min(rows, n - i), c.d, idx->centers.as<float>(), idx->centers_t.as<float>(),
                               c.n_leaves, idx->train_ws.p, assign + i, nullptr, 1, nullptr, st));
    return AVQ_OK;
}

// Theorem 4.2 for every leaf at once: the leaf centers are the codewords of a one-dictionary quantizer whose
// codes are the leaf assignments, so the joint update of Appendix 7.5 with M = 1 is the theorem's closed form.
static int update_leaf_centers(avq_index *idx, const float *x, int64_t n, const int32_t *assign, int max_iters, double tol,
                               int *iters, double *rel, hipStream_t st)
{
    const avq_config &c = idx->cfg;
    const int D = c.n_leaves * c.d;
    DevBuf scratch;
    int rc = scratch.reserve(pq_update_scratch_bytes(n, D, c.n_leaves));
    if (rc == AVQ_OK)
        rc = pq_joint_update_device(x, n, c.d, 1, c.n_leaves, 32, (const uint8_t *)assign, nullptr, nullptr, c.eta_mode,
                                    (double)c.T, (double)c.eta_explicit, idx->centers.as<float>(), scratch.p, max_iters, tol,
                                    iters, rel, st);
    if (rc == AVQ_OK && hipStreamSynchronize(st) != hipSuccess) { set_error("leaf center update: stream error"); rc = AVQ_EHIP; }
    scratch.release();
    if (rc == AVQ_OK) rc = refresh_centers_t(idx, st);
    return rc;
}

extern "C" int avq_train(avq_index *idx, const float *x, int64_t n_train, void *hip_stream)
{
    AVQ_TRY(check_index(idx));
    hipStream_t st = (hipStream_t)hip_stream;
    const avq_config &c = idx->cfg;
    if (!x || n_train < idx->kc || n_train < c.n_leaves || n_train > 0x7fffffff) {
        set_error("avq_train: need a device pointer and max(k_c, n_leaves) <= n_train < 2^31");
        return AVQ_EINVAL;
    }
    const ScratchKeeper keep{&idx->train_ws};
    const int32_t *assign = nullptr;
    if (c.n_leaves > 0) {
        // leaf centers from at most 256 rows per leaf, then every training row to its leaf
        const int64_t n_leaf_train = std::min<int64_t>(n_train, (int64_t)256 * c.n_leaves);
        int rc = AVQ_ENOMEM;
        if (nearest_supported(c.d, c.n_leaves))
            rc = kmeans_leaves_device(x, n_leaf_train, c.d, c.n_leaves, c.leaf_kmeans_iters, c.seed, idx->centers.as<float>(),
                                      idx->centers_t.as<float>(), &idx->train_ws, st);
        if (rc != AVQ_ENOMEM) {
            AVQ_TRY(rc);
        } else { // another dimension, or no room for its scratch (which it asks for before anything else)
            AVQ_TRY(kmeans_device(x, n_leaf_train, c.d, c.n_leaves, c.leaf_kmeans_iters, c.seed, idx->centers.as<float>(), st));
            AVQ_TRY(refresh_centers_t(idx, st));
        }
        idx->have_centers = true;
        AVQ_TRY(idx->tmp.reserve(sizeof(int32_t) * (size_t)n_train));
        // Section 4 with the leaf centers as codewords: alternate the assignment under the anisotropic loss
        // (Definition 4.1) and Theorem 4.2's update, starting from the l2 centers
        for (int it = 0; it < c.leaf_aniso_iters; ++it) {
            AVQ_TRY(launch_assign_aniso(x, n_leaf_train, c.d, idx->centers.as<float>(), c.n_leaves, c.eta_mode, (double)c.T,
                                        (double)c.eta_explicit, idx->tmp.as<int32_t>(), st));
            AVQ_TRY(update_leaf_centers(idx, x, n_leaf_train, idx->tmp.as<int32_t>(), 500, 1e-10, nullptr, nullptr, st));
        }
        AVQ_TRY(assign_to_leaves(idx, x, n_train, idx->tmp.as<int32_t>(), st));
        assign = idx->tmp.as<int32_t>();
    }
    AVQ_TRY(pq_kmeans_device(x, n_train, c.d, c.M, idx->kc, c.kmeans_iters, c.seed, assign ? idx->centers.as<float>() : nullptr,
                             assign, idx->codebooks.as<float>(), &idx->train_ws, st));
    AVQ_HIP(hipStreamSynchronize(st));
    idx->have_codebooks = true;
    return AVQ_OK;
}

// ---- database ------------------------------------------------------------------------

// The points of a partitioned index grouped by the leaves in idx->assign: perm, leaf_blk and the number of blocks.
static int group_by_leaves(avq_index *idx, int64_t n, hipStream_t st)
{
    // ascending id inside a leaf, each leaf padded to whole blocks
    const avq_config &c = idx->cfg;
    const size_t b_ws = (leaf_layout_ws_bytes(n, c.n_leaves) + 255) & ~(size_t)255;
    AVQ_TRY(idx->tmp.reserve(b_ws + sizeof(LeafLayoutInfo)));
    AVQ_TRY(idx->leaf_blk.reserve(sizeof(int32_t) * (size_t)(c.n_leaves + 1)));
    LeafLayoutInfo *info_dev = (LeafLayoutInfo *)(idx->tmp.as<unsigned char>() + b_ws), info;
    const int32_t *assign = idx->assign.as<int32_t>();
    AVQ_TRY(launch_leaf_counts(assign, n, c.n_leaves, idx->tmp.p, idx->leaf_blk.as<int32_t>(), info_dev, st));
    AVQ_HIP(hipMemcpyAsync(&info, info_dev, sizeof(info), hipMemcpyDeviceToHost, st));
    AVQ_HIP(hipStreamSynchronize(st));
    if (info.first_bad < n) {
        int32_t leaf = 0;
        AVQ_HIP(hipMemcpy(&leaf, assign + info.first_bad, sizeof(leaf), hipMemcpyDeviceToHost));
        set_error("leaf assignment %d of point %lld out of range", leaf, (long long)info.first_bad);
        return AVQ_EINVAL;
    }
    if (info.n_blocks * kBlockPoints > 0x7fffffff) { set_error("index too large"); return AVQ_EINVAL; }
    idx->max_leaf_blocks = info.max_leaf_blocks;
    idx->n_blocks = info.n_blocks;
    idx->n_slots = info.n_blocks * kBlockPoints;
    AVQ_TRY(idx->perm.reserve(sizeof(int32_t) * (size_t)idx->n_slots));
    return launch_leaf_places(assign, n, c.n_leaves, idx->tmp.p, idx->leaf_blk.as<int32_t>(), idx->perm.as<int32_t>(), idx->n_slots, st);
}

// codes_logical (and, if partitioned, the points grouped by leaf) are on the device; builds the blocked layout.
static int install_database(avq_index *idx, const float *x, int64_t n, hipStream_t st)
{
    const avq_config &c = idx->cfg;
    if (x && !c.borrow_x) {
        AVQ_TRY(idx->x_own.reserve(sizeof(float) * (size_t)n * c.d));
        AVQ_HIP(hipMemcpyAsync(idx->x_own.p, x, sizeof(float) * (size_t)n * c.d, hipMemcpyDeviceToDevice, st));
        idx->x = idx->x_own.as<float>();
    } else {
        idx->x = x;
    }
    if (c.n_leaves <= 0) {
        idx->n_blocks = (n + kBlockPoints - 1) / kBlockPoints;
        idx->n_slots = idx->n_blocks * kBlockPoints;
    }
    AVQ_TRY(idx->codes_blocked.reserve((size_t)idx->n_slots * idx->NB));
    AVQ_TRY(launch_to_blocked(idx->codes_logical.as<uint8_t>(), n, idx->NB, c.n_leaves > 0 ? idx->perm.as<int32_t>() : nullptr,
                              idx->codes_blocked.as<uint8_t>(), idx->n_blocks, st));
    AVQ_HIP(hipStreamSynchronize(st));
    idx->n = n;
    return AVQ_OK;
}

static int check_n(int64_t n)
{
    if (n < 1 || n >= 0x7fffffffll - 512) { set_error("n = %lld out of range", (long long)n); return AVQ_EINVAL; }
    return AVQ_OK;
}

extern "C" int avq_set_database(avq_index *idx, const float *x, const uint8_t *packed,
                                const int32_t *leaf_assign, int64_t n, void *hip_stream)
{
    AVQ_TRY(check_index(idx));
    AVQ_TRY(check_n(n));
    hipStream_t st = (hipStream_t)hip_stream;
    const avq_config &c = idx->cfg;
    if (!packed) { set_error("avq_set_database: packed is NULL"); return AVQ_EINVAL; }
    if ((c.n_leaves > 0) != (leaf_assign != nullptr)) {
        set_error("avq_set_database: leaf_assign must be given exactly for a partitioned index");
        return AVQ_EINVAL;
    }
    if (c.n_leaves > 0 && !idx->have_centers) { set_error("avq_set_database: no leaf centers yet"); return AVQ_ESTATE; }
    AVQ_TRY(idx->codes_logical.reserve((size_t)n * idx->NB + 16)); // rows are read in whole words, and a word ahead
    AVQ_HIP(hipMemcpyAsync(idx->codes_logical.p, packed, (size_t)n * idx->NB, hipMemcpyDefault, st));
    if (leaf_assign) {
        AVQ_TRY(idx->assign.reserve(sizeof(int32_t) * (size_t)n));
        AVQ_HIP(hipMemcpyAsync(idx->assign.p, leaf_assign, sizeof(int32_t) * (size_t)n, hipMemcpyDefault, st));
    }
    AVQ_HIP(hipStreamSynchronize(st));
    idx->n = 0;
    if (leaf_assign) AVQ_TRY(group_by_leaves(idx, n, st));
    return install_database(idx, x, n, st);
}

extern "C" int avq_encode(avq_index *idx, const float *x, int64_t n, void *hip_stream)
{
    AVQ_TRY(check_index(idx));
    AVQ_TRY(check_n(n));
    hipStream_t st = (hipStream_t)hip_stream;
    const avq_config &c = idx->cfg;
    if (!x) { set_error("avq_encode: x is NULL"); return AVQ_EINVAL; }
    if (!idx->have_codebooks) { set_error("avq_encode: no dictionaries yet (avq_train first)"); return AVQ_ESTATE; }
    if (c.n_leaves > 0 && !idx->have_centers) { set_error("avq_encode: no leaf centers yet"); return AVQ_ESTATE; }
    if (c.n_leaves > 0) AVQ_TRY(check_assign(c.d, c.n_leaves, c.leaf_aniso_iters > 0)); // refused: the database stays
    idx->n = 0;
    const ScratchKeeper keep{&idx->train_ws};
    AVQ_TRY(idx->codes_logical.reserve((size_t)n * idx->NB + 16)); // rows are read in whole words, and a word ahead
    const int32_t *assign = nullptr;
    if (c.n_leaves > 0) {
        AVQ_TRY(idx->assign.reserve(sizeof(int32_t) * (size_t)n));
        AVQ_TRY(assign_to_leaves(idx, x, n, idx->assign.as<int32_t>(), st));
        assign = idx->assign.as<int32_t>();
        AVQ_TRY(group_by_leaves(idx, n, st));
    }
    AVQ_TRY(launch_encode(x, n, c.d, c.M, idx->kc, c.bits, idx->codebooks.as<float>(), assign ? idx->centers.as<float>() : nullptr,
                          assign, assign ? idx->perm.as<int32_t>() : nullptr, idx->n_slots, c.eta_mode, (double)c.T,
                          (double)c.eta_explicit, c.encode_passes, idx->codes_logical.as<uint8_t>(), &idx->train_ws, st));
    return install_database(idx, x, n, st);
}

extern "C" int avq_update_codebooks(avq_index *idx, const float *x, int64_t n, int32_t max_iters, double tol,
                                    int32_t *iters_out, double *rel_residual_out, void *hip_stream)
{
    AVQ_TRY(check_index(idx));
    hipStream_t st = (hipStream_t)hip_stream;
    const avq_config &c = idx->cfg;
    if (!x) { set_error("avq_update_codebooks: x is NULL"); return AVQ_EINVAL; }
    if (idx->n <= 0) { set_error("avq_update_codebooks: no codes yet (avq_encode first)"); return AVQ_ESTATE; }
    if (n != idx->n) {
        set_error("avq_update_codebooks: n = %lld but the codes are of %lld points", (long long)n, (long long)idx->n);
        return AVQ_EINVAL;
    }
    if (max_iters < 1 || !(tol >= 0.0)) { set_error("avq_update_codebooks: max_iters < 1 or tol < 0"); return AVQ_EINVAL; }
    const int ds = c.d / c.M, D = c.M * idx->kc * ds;
    DevBuf scratch;
    int iters = 0;
    double rel = 0.0;
    int rc = scratch.reserve(pq_update_scratch_bytes(n, D, c.M * idx->kc));
    if (rc == AVQ_OK)
        rc = pq_joint_update_device(x, n, c.d, c.M, idx->kc, c.bits, idx->codes_logical.as<uint8_t>(),
                                    c.n_leaves > 0 ? idx->centers.as<float>() : nullptr,
                                    c.n_leaves > 0 ? idx->assign.as<int32_t>() : nullptr, c.eta_mode,
                                    (double)c.T, (double)c.eta_explicit, idx->codebooks.as<float>(), scratch.p,
                                    max_iters, tol, &iters, &rel, st);
    if (rc == AVQ_OK && hipStreamSynchronize(st) != hipSuccess) { set_error("avq_update_codebooks: stream error"); rc = AVQ_EHIP; }
    scratch.release();
    if (rc != AVQ_OK) return rc;
    if (iters_out) *iters_out = iters;
    if (rel_residual_out) *rel_residual_out = rel;
    return AVQ_OK;
}

extern "C" int avq_update_leaf_centers(avq_index *idx, const float *x, int64_t n, int32_t max_iters, double tol,
                                       int32_t *iters_out, double *rel_residual_out, void *hip_stream)
{
    AVQ_TRY(check_index(idx));
    hipStream_t st = (hipStream_t)hip_stream;
    const avq_config &c = idx->cfg;
    if (!x) { set_error("avq_update_leaf_centers: x is NULL"); return AVQ_EINVAL; }
    if (c.n_leaves <= 0) { set_error("avq_update_leaf_centers: flat index"); return AVQ_EINVAL; }
    if (idx->n <= 0) { set_error("avq_update_leaf_centers: no database yet (avq_encode first)"); return AVQ_ESTATE; }
    if (n != idx->n) {
        set_error("avq_update_leaf_centers: n = %lld but the stored assignment is of %lld points", (long long)n, (long long)idx->n);
        return AVQ_EINVAL;
    }
    if (max_iters < 1 || !(tol >= 0.0)) { set_error("avq_update_leaf_centers: max_iters < 1 or tol < 0"); return AVQ_EINVAL; }
    int iters = 0;
    double rel = 0.0;
    AVQ_TRY(update_leaf_centers(idx, x, n, idx->assign.as<int32_t>(), max_iters, tol, &iters, &rel, st));
    if (iters_out) *iters_out = iters;
    if (rel_residual_out) *rel_residual_out = rel;
    return AVQ_OK;
}

extern "C" int avq_get_codes(avq_index *idx, uint8_t *out)
{
    AVQ_TRY(check_index(idx));
    if (idx->n <= 0) { set_error("avq_get_codes: no database"); return AVQ_ESTATE; }
    if (!out) { set_error("avq_get_codes: NULL"); return AVQ_EINVAL; }
    AVQ_HIP(hipMemcpy(out, idx->codes_logical.p, (size_t)idx->n * idx->NB, hipMemcpyDefault));
    return AVQ_OK;
}

extern "C" int avq_get_leaf_assign(avq_index *idx, int32_t *out)
{
    AVQ_TRY(check_index(idx));
    if (idx->n <= 0 || idx->cfg.n_leaves <= 0) { set_error("avq_get_leaf_assign: no partitioned database"); return AVQ_ESTATE; }
    if (!out) { set_error("avq_get_leaf_assign: NULL"); return AVQ_EINVAL; }
    AVQ_HIP(hipMemcpy(out, idx->assign.p, sizeof(int32_t) * (size_t)idx->n, hipMemcpyDefault));
    return AVQ_OK;
}

// ---- query path ----------------------------------------------------------------------

static int build_tables(avq_index *idx, const float *queries, int nq, int lut_mode, hipStream_t st)
{
    const avq_config &c = idx->cfg;
    const size_t entries = (size_t)nq * c.M * idx->kc;
    AVQ_TRY(idx->lut.reserve(entries * sizeof(float)));
    if (lut_mode == AVQ_LUT_U8) {
        AVQ_TRY(idx->lut8.reserve(entries));
        AVQ_TRY(idx->scale.reserve(sizeof(float) * (size_t)nq));
        AVQ_TRY(idx->bias.reserve(sizeof(float) * (size_t)nq));
    }
    return launch_lut(queries, nq, idx->codebooks.as<float>(), c.d, c.M, idx->kc, idx->lut.as<float>(),
                      lut_mode == AVQ_LUT_U8 ? idx->lut8.as<uint8_t>() : nullptr, idx->scale.as<float>(),
                      idx->bias.as<float>(), st);
}

// The scan of the whole code array for one or a few queries reads an array that does not fit the 256 MB Infinity
// Cache once per query: nontemporal loads and a wave per block then (block_bound_stream_kernel). Measured per call,
// plain against streamed: 320 MB 80 / 73 us for one query, 127 / 118 for two, equal at four, 614 / 766 at sixteen
// (the queries of a call share what the caches hold when few workgroups per query walk the array together);
// 1.6 GB 326 / 262, 606 / 494, 1139 / 967, 2220 / 1899 (eight queries), 3291 / 3765 (sixteen). An array that fits
// the cache stays resident between calls and is loaded the plain way.
static bool stream_loads_nontemporal(const avq_index *idx, int nq)
{
    if (idx->tune_stream_loads == 1) return false;
    if (idx->tune_stream_loads == 2) return true;
    const size_t bytes = (size_t)idx->n_blocks * 256 * (size_t)idx->NB;
    return bytes > ((size_t)256 << 20) && (nq <= 2 || (nq <= 8 && bytes > ((size_t)1 << 30)));
}

static void fill_scan_params(const avq_index *idx, int nq, int R, int ns, ScanParams *p)
{
    memset(p, 0, sizeof(*p));
    p->codes = idx->codes_blocked.as<uint8_t>();
    p->n_blocks = idx->n_blocks;
    p->n_valid = (int32_t)idx->n;
    p->lut = idx->lut.as<float>();
    p->lut8 = idx->lut8.as<uint8_t>();
    p->scale = idx->scale.as<float>();
    p->bias = idx->bias.as<float>();
    p->B = nq;
    p->M = idx->cfg.M;
    p->bits = idx->cfg.bits;
    p->NB = idx->NB;
    p->R = R;
    p->ns = ns;
}

// Chooses the flat scan's grid: query tiles x chunks of the block range.
static void plan_flat(const avq_index *idx, const ScanShape &s, int nq, ScanParams *p)
{
    p->n_tiles = (nq + s.qt - 1) / s.qt;
    // one resident set of workgroups: the fp32 tile of 8 runs two workgroups per compute unit
    const int builtin = (s.qt == 8 && s.lists_global && idx->cfg.bits == 4) ? 512 : 1024;
    const int target = idx->tune_target_wgs > 0 ? idx->tune_target_wgs : builtin;
    int64_t chunks = (target + p->n_tiles - 1) / p->n_tiles;
    if (idx->tune_target_wgs <= 0 && p->n_tiles > target) {
        // more tiles than fit at once: a few chunks per tile so that the last round of workgroups
        // is nearly full (each extra chunk costs about 2 % in list handling)
        double best = 0.0;
        for (int c = 1; c <= 4; ++c) {
            const double rounds = (double)p->n_tiles * c / target;
            const double score = rounds / std::ceil(rounds) * (1.0 - 0.02 * (c - 1));
            if (score > best) { best = score; chunks = c; }
        }
    }
    const int64_t max_chunks = std::max<int64_t>(1, idx->n_blocks / s.waves);
    chunks = std::max<int64_t>(1, std::min(chunks, max_chunks));
    const int64_t bpc = (idx->n_blocks + chunks - 1) / chunks;
    p->blocks_per_chunk = (int32_t)bpc;
    p->n_chunks = (int32_t)((idx->n_blocks + bpc - 1) / bpc);
}

// The matrix-core scan serves batches of 8-bit-table queries on a flat index of 4-bit codes.
static bool use_mfma_scan(const avq_index *idx, int nq, int lut_mode)
{
    return idx->tune_mfma == 0 && lut_mode == AVQ_LUT_U8 && idx->cfg.n_leaves == 0 && nq >= 16 &&
           scan_mfma_supported(idx->NB, idx->cfg.bits);
}

// Batches with fp32 tables on a flat index of 4-bit codes: the matrix-core scan over the 8-bit
// tables collects every point that the rounding of the tables could still place among the R
// best, and those are re-scored and ranked in fp32.
static bool use_prefilter(const avq_index *idx, int nq, int lut_mode, int R)
{
    return idx->tune_prefilter != 1 && idx->tune_mfma == 0 && lut_mode == AVQ_LUT_F32 && idx->cfg.n_leaves == 0 &&
           nq >= 16 && scan_mfma_supported(idx->NB, idx->cfg.bits) && idx->cfg.M <= 64 && idx->n > R;
}

// Whether the matrix-core scan of this batch would be given bounds guessed from a sample.
static bool mfma_scan_samples(const avq_index *idx, int nq, int R, int ns)
{
    if (idx->tune_sample == 1) return false;
    ScanParams p, sample;
    memset(&p, 0, sizeof(p));
    p.R = R;
    p.ns = ns;
    scan_mfma_plan(nq, idx->n_blocks, idx->tune_target_wgs, &p);
    return scan_mfma_sample_plan(p, &sample);
}

// u8: the 8-bit-table search itself through the same machinery (fixed bounds from a sample, kept
// keys ranked by their integer sums: no margin, no fp32 tables); only called when the scan samples.
static int search_through_candidates(avq_index *idx, const float *queries, int nq, int k, int reorder_k, int R, int ns,
                              bool u8, int32_t *ids_out, float *scores_out, hipStream_t st)
{
    const avq_config &c = idx->cfg;
    const int C = 64 * ns;
    // 1. matrix-core scan over the 8-bit tables in candidate mode
    ScanParams pm;
    fill_scan_params(idx, nq, R, ns, &pm);
    scan_mfma_plan(nq, idx->n_blocks, idx->tune_target_wgs, &pm);
    pm.cand_cap = idx->tune_prefilter_cap > 0 ? std::max(128, idx->tune_prefilter_cap) : std::max(2048, 16 * C);
    // 2. the plain fp32 scan for the queries whose candidates cannot be used (no margin, a buffer
    // that overflowed): its grid is cut on the device to the number of such queries
    ScanParams pf;
    fill_scan_params(idx, nq, R, ns, &pf);
    ScanShape shape;
    AVQ_TRY(scan_pick_shape(idx->NB, c.bits, u8, ns, nq, false, 8, idx->tune_waves, &shape));
    pf.n_tiles = (nq + shape.qt - 1) / shape.qt;
    pf.n_chunks = (int32_t)std::max<int64_t>(1, std::min<int64_t>(128, idx->n_blocks / shape.waves)); // at most
    pf.blocks_per_chunk = 0; // derived on the device

    const size_t partial_m = sizeof(u64) * (size_t)nq * pm.n_chunks * C;
    // the plain scan writes (live queries, rounded up to tiles) x chunks lists: at most max(kDynamicItems, tiles) tiles' worth
    const size_t partial_f = sizeof(u64) * (size_t)std::max(kDynamicItems, pf.n_tiles) * shape.qt * C;
    AVQ_TRY(idx->partial.reserve(std::max(partial_m, partial_f)));
    const size_t lists_f = shape.lists_global ? sizeof(u64) * (size_t)std::max(kDynamicItems, pf.n_tiles) * shape.waves * shape.qt * C : 0;
    AVQ_TRY(idx->lists.reserve(std::max(scan_mfma_lists_bytes(pm), lists_f)));
    const size_t thr_bytes = sizeof(uint32_t) * (size_t)nq * (1 + (size_t)pm.n_chunks);
    AVQ_TRY(idx->thr.reserve(thr_bytes));
    AVQ_TRY(idx->cand.reserve(sizeof(u64) * (size_t)nq * C));
    AVQ_TRY(idx->refined.reserve(sizeof(u64) * (size_t)nq * C));
    const size_t row_floats = u8 ? (size_t)c.M * idx->kc / 4 : (size_t)c.M * idx->kc; // a query's tables, in 4-byte units
    AVQ_TRY(idx->lut_fail.reserve(sizeof(float) * (size_t)pf.n_tiles * shape.qt * row_floats));
    // fail: [4] count | [nq] list | [nq] margins | [nq][chunks] candidate counts
    AVQ_TRY(idx->fail.reserve(sizeof(int32_t) * (4 + (size_t)nq * (2 + (size_t)pm.n_chunks))));
    AVQ_TRY(idx->cand_keys.reserve(sizeof(uint32_t) * (size_t)nq * pm.n_chunks * pm.cand_cap));
    uint32_t *fail_count = idx->fail.as<uint32_t>();
    int32_t *fail_list = idx->fail.as<int32_t>() + 4;
    int32_t *margin = fail_list + nq;

    pm.partial = idx->partial.as<u64>();
    pm.lists_ws = idx->lists.as<u64>();
    pm.thr_shared = idx->thr.as<uint32_t>();
    pm.kth_shared = pm.thr_shared + nq;
    pm.cand_keys = idx->cand_keys.as<uint32_t>();
    pm.cand_cnt = (uint32_t *)(margin + nq);
    pm.cand_margin = u8 ? nullptr : margin;
    {
        StageTimer t(idx, AVQ_STAGE_SAMPLE, st);
        AVQ_HIP(hipMemsetAsync(fail_count, 0, 16, st));
        AVQ_HIP(hipMemsetAsync(pm.thr_shared, 0, thr_bytes, st));
        if (!u8) AVQ_TRY(launch_prefilter_margin(idx->lut.as<float>(), idx->scale.as<float>(), c.M, idx->NB, nq, margin, st));
        // guess the bounds from a sample of the index and scan against them, where the index is large
        // enough for that; otherwise the scan keeps lists and raises its bounds itself
        ScanParams sample;
        if (idx->tune_sample != 1 && scan_mfma_sample_plan(pm, &sample)) {
            // The r-th best sum of the sample. With enough waves per query it comes without lists: every wave
            // records the best sum of each of its 32 disjoint point classes, and the r-th largest of a query's
            // class maxima is the r-th best of the sample unless two of those fell into one class (then it is a
            // little lower, which only keeps more points). Otherwise, or when asked, from sorted lists.
            const int classes = sample.n_chunks * 32;
            if (idx->tune_sample != 2 && classes >= 8 * sample.R && classes <= 8192) {
                sample.sample_max = (uint32_t *)idx->lists.p; // the lists' scratch: no launch here keeps lists
                AVQ_TRY(launch_scan_mfma(sample, st));
                AVQ_TRY(launch_sample_bound(sample.sample_max, classes, sample.R, nq, pm.thr_shared, st));
            } else {
                AVQ_TRY(launch_scan_mfma(sample, st));
                const u64 *best = sample.partial;
                if (sample.n_chunks > 1) {
                    AVQ_TRY(launch_merge_partials(sample.partial, nq, sample.n_chunks, sample.ns, idx->cand.as<u64>(), st));
                    best = idx->cand.as<u64>();
                }
                AVQ_TRY(launch_list_bound(best, sample.ns, sample.R, nq, pm.thr_shared, st));
            }
            pm.fixed_bound = 1;
        }
    }
    {
        StageTimer t(idx, AVQ_STAGE_SCAN, st); // the launch over all blocks, nothing else
        AVQ_TRY(launch_scan_mfma(pm, st));
    }
    const u64 *top = pm.fixed_bound ? nullptr : pm.partial;
    if (!pm.fixed_bound && pm.n_chunks > 1) {
        StageTimer t(idx, AVQ_STAGE_MERGE, st);
        AVQ_TRY(launch_merge_partials(pm.partial, nq, pm.n_chunks, ns, idx->cand.as<u64>(), st));
        top = idx->cand.as<u64>();
    }
    {
        StageTimer t(idx, AVQ_STAGE_RESCAN, st);
        RefineCandParams r;
        r.top = top;
        r.bound = pm.fixed_bound ? pm.thr_shared : nullptr;
        r.R = R; r.ns = ns; r.nq = nq; r.M = c.M; r.NB = idx->NB;
        r.n_chunks = pm.n_chunks;
        r.cand_cap = pm.cand_cap;
        r.chunk_points = (int64_t)pm.blocks_per_chunk * kBlockPoints;
        r.cand_keys = pm.cand_keys;
        r.cand_cnt = pm.cand_cnt;
        r.margin = u8 ? nullptr : margin;
        r.lut = u8 ? nullptr : idx->lut.as<float>();
        r.codes = idx->codes_logical.as<uint8_t>();
        r.out = idx->refined.as<u64>();
        r.fail_list = fail_list;
        r.fail_count = fail_count;
        r.force_fail_odd = idx->tune_prefilter == 2;
        AVQ_TRY(launch_refine_cand(r, st));
        // the other queries: their tables side by side, the plain scan over them, and their lists
        // merged into their own rows of the refined candidates
        AVQ_TRY(launch_gather_rows(u8 ? (const float *)idx->lut8.p : idx->lut.as<float>(), idx->lut_fail.as<float>(), fail_list,
                                   fail_count, nq, (int)row_floats, st));
        pf.lut = idx->lut_fail.as<float>();
        pf.lut8 = idx->lut_fail.as<uint8_t>();
        pf.partial = idx->partial.as<u64>(); // the matrix-core scan's lists are merged by now
        if (shape.lists_global) pf.lists_ws = idx->lists.as<u64>();
        pf.active_queries = fail_count;
        AVQ_TRY(launch_scan(pf, u8, SCAN_CHUNK, shape, st));
        AVQ_TRY(launch_merge_partials(pf.partial, nq, pf.n_chunks, ns, idx->refined.as<u64>(), st, fail_list, fail_count,
                                      shape.qt));
    }
    StageTimer t(idx, AVQ_STAGE_FINAL, st);
    return launch_finalize(idx->refined.as<u64>(), ns, nq, R, k, reorder_k != 0, u8 ? 1 : 0, idx->x, c.d, queries,
                           idx->scale.as<float>(), idx->bias.as<float>(), ids_out, scores_out, st);
}

// What a call on 8-bit codes takes (us): queries one by one, sixteen to a scan, or through the product of the queries with the
// decoded points. Fitted to 3,132 calls: 2,000 to 10,000,000 points of 8, 13, 25 and 32 code bytes (32 to 256 dimensions), 1 to 1,000
// queries, 1 to 500 results, tables of either kind; the forms chosen by these lines take 1.012 (up to 32 queries) and 1.008 times as
// long as the best ones in the mean. Measured, one by one / sixteen to a scan, 25 bytes, R = 100, fp32 tables: 200,000 points, 16
// queries 59 / 63, 32 82 / 75; 500,000, 8 54 / 56, 16 72 / 63, 32 109 / 78; 1,183,514, 4 55 / 60, 6 71 / 62, 16 110 / 71, 32 177 / 100;
// 5,000,000, 2 79 / 102, 4 110 / 110, 16 289 / 127, 64 1,016 / 341; 256 dimensions in 32 bytes, 2,000,000, 4 80 / 85, 8 112 / 88, 64
// 580 / 256; 250,000, 16 68 / 73. Sixteen to a scan / product: 2,000 points, 150 queries 66 / 113, 300 96 / 116, 1,000 170 / 126; 16,000,
// 48 100 / 95, 150 147 / 95; 600,000, 80 137 / 123; R = 500: 4,000, 300 133 / 198; 16,000, 80 132 / 178, 150 162 / 185.
static double listed_blocks(const avq_index *idx, int R) { return (double)std::min<int64_t>(R, 2 * idx->n_blocks); }
static double per_query_us(const avq_index *idx, int R) // blocks listed, scored and ranked
{
    const double listed = listed_blocks(idx, R);
    return 0.25 + 0.005 * std::min(100.0, listed) + 0.009 * std::max(0.0, listed - 100.0);
}
static double single_us(const avq_index *idx, int nq, int R)
{
    return 35.0 + nq * (0.1 + per_query_us(idx, R) + 3.3e-5 * idx->NB * (double)idx->n_blocks);
}
static double tile_us(const avq_index *idx, int nq, int R, bool u8)
{
    const double q = nq, d = idx->cfg.d, r = R, blocks = (double)idx->n_blocks, tiles = (nq + 15) / 16, codes = idx->NB * blocks;
    if (nq <= 32) { // the launches' latencies, for the most part
        const double rows = u8 || blocks <= 4000.0 ? 0.0 : 0.006 * std::max(0.0, listed_blocks(idx, R) - 100.0);
        return 45.0 + 0.03 * std::max(0.0, d - 100.0) + 1.28e-4 * codes * tiles + q * (per_query_us(idx, R) + (blocks < 4000.0 ? 0.1 : 0.0) + rows);
    }
    const double listed = std::min(r, blocks), all = r >= 0.9 * blocks ? listed : 0.0; // all: every block of the index is listed
    return 21.0 + 0.28 * d + 1.26e-4 * codes * tiles + 0.11 * listed + 0.57 * all + q * (0.126 + 0.0033 * listed + 0.0021 * all);
}
static double product8_us(const avq_index *idx, int nq, int R, bool u8)
{
    const double n = (double)idx->n, q = nq, d = idx->cfg.d, r = R;
    return 44.0 + 0.32 * d + 0.133 * r + 0.108 * std::max(0.0, r - 200.0) + 5.1e-7 * std::max(0.0, n - 3e5) * d + q * (0.038 + 0.0002 * r) +
           1.95e-9 * n * q * d + (u8 ? 17.0 + 0.11 * d : 0.0);
}

// Batches on a flat index through the product of the queries with the decoded points (product.hip), where it is expected to
// be faster than the path that the call takes otherwise, for which few_max is the number of queries answered one by one.
// What the other paths cost is estimated from below. Measured, other path / product, us a call (100 dimensions, R = 100):
//  4-bit codes, fp32 tables: 1,000,000 points 93 / 120 (16 queries), 144 / 121 (32), 505 / 297 (1,024), 1,697 / 932 (4,096);
//    200,000 points 66 / 69 (32), 170 / 87 (256), 581 / 376; 32,000 points 59 / 70 (64), 109 / 77 (256), 287 / 203; up to
//    16,384 points one launch answers 256 queries in about 20 us: 4,000 points 68 / 109 (1,024), 264 / 212 (4,096), and
//    R = 500 432 / 567.
//  4-bit codes, 8-bit tables, whose rounding lets through several times R: 1,000,000 points 168 / 150 (64), 1,560 / 1,089;
//    64,000 points 131 / 104 (256), 308 / 324 (4,096); R = 500: 200,000 points 790 / 1,078, 1,000,000 1,904 / 1,803.
//  code sizes without matrix-core kernels (192 dimensions, 96 subspaces): 1,000,000 points 360 / 264 (32), 12,877 / 1,788.
//  8-bit codes: product8_us and the lines above it.
//  and where the other batch path cannot guess its bounds (guessed false: 20,000 points, R = 100) 151 / 98 (256), 718 / 196.
static bool use_product(const avq_index *idx, int nq, int R, bool u8, int few_max, bool guessed)
{
    const avq_config &c = idx->cfg;
    if (idx->tune_product == 1 || c.n_leaves > 0 || !product_supported(c.d, c.M, idx->n, R)) return false;
    if (idx->tune_product == 2) return true;
    // any tuning of the other kernels' launches asks for those kernels
    if (idx->tune_target_wgs || idx->tune_waves || idx->tune_qt || idx->tune_mfma || idx->tune_prefilter == 1 || idx->tune_prefilter_cap ||
        idx->tune_sample || idx->tune_small_impl || idx->tune_bound_bits || idx->tune_small_batch >= 0) return false;
    if (nq < 16) return false;
    const double n = (double)idx->n, q = (double)nq, d = (double)c.d, r = (double)R;
    const double few = 20.0 + q * (0.1 + 0.000037 * idx->NB * (double)idx->n_blocks + (guessed ? 0.001 : 0.002) * r);
    if (c.bits == 8) {
        if (!block_bound_supported(idx->NB, c.bits)) return true; // plain scans: 400 us and more
        return product8_us(idx, nq, R, u8) < (nq > few_max ? tile_us(idx, nq, R, u8) : few);
    }
    const double decode = std::max(0.0, n - 3e5) * d * (d > 128 ? 6e-7 : 4.8e-7);
    double product = 30.0 + 0.35 * d + 0.14 * r + decode + q * (0.02 + 0.00018 * r) + 1.6e-9 * n * q * d;
    const bool own = scan_mfma_supported(idx->NB, c.bits);
    if (u8) product += 12.0;
    if (idx->n <= 16384) {
        if (u8) return own ? nq >= 2048 && R >= 50 && R <= 100 : nq > few_max && (c.d <= 128 || (nq >= 1024 && n >= 8192.0));
        return own ? nq >= 2048 && R <= 100 : nq > few_max;
    }
    if (u8 && own && guessed && (n < 2000.0 * r || n < 32768.0)) return false;
    return nq > few_max || product < (own && !guessed ? std::min(560.0, few) : few);
}

// The most scratch that a part of a batch through the product takes ("scratch_limit_kb" where that is less); parts cost: the
// points are decoded again for each. The flat batches' measured range ends at 16,384 queries a part.
constexpr size_t kProductScratch = (size_t)4 << 30;
static size_t product_scratch(const avq_index *idx) { return idx->product.limit ? std::min(idx->product.limit, kProductScratch) : kProductScratch; }

// the plain scan of queries that the product hands back
static int product_shape(const avq_index *idx, int nq, int ns, bool u8, bool leaves, ScanShape *shape)
{
    const int bits = idx->cfg.bits, qt = !leaves && bits == 4 ? 8 : 0, waves = leaves ? 16 : 0;
    if ((qt || waves) && scan_pick_shape(idx->NB, bits, u8, ns, nq, leaves, qt, waves, shape) == AVQ_OK) return AVQ_OK;
    return scan_pick_shape(idx->NB, bits, u8, ns, nq, leaves, 0, 0, shape);
}

// Queries of one part of a batch.
static int product_part(const avq_index *idx, int nq, int R, int ns, int L, bool u8, int *per)
{
    const avq_config &c = idx->cfg;
    ScanShape shape;
    AVQ_TRY(product_shape(idx, nq, ns, u8, L > 0, &shape));
    // bytes of a query beside the product's own: its tables twice (8-bit ones with the fp32 ones they are made from), the lists
    // and, on a partitioned index, the leaves of the plain scan
    const size_t entries = (size_t)c.M * idx->kc, list = sizeof(u64) * 64 * (size_t)ns;
    const size_t other = entries * (u8 ? 6 : 4) + list + (shape.lists_global ? list * shape.waves * shape.qt : 0) + (size_t)L * 8;
    if (L > 0) {
        *per = product_leaf_part(nq, L, c.n_leaves, idx->n, idx->n_blocks, idx->max_leaf_blocks, c.d, R, u8, other, product_scratch(idx));
        return AVQ_OK;
    }
    const ProductPlan pl = product_plan(std::min(nq, 16384), idx->n, c.d, R, u8);
    const size_t row = (size_t)pl.n_classes * 4 + (size_t)pl.kept_cap * 8 + (size_t)pl.steps * 32 + 256 + other;
    const int64_t most = std::max<int64_t>(64, std::min<int64_t>(16384, (int64_t)(product_scratch(idx) / row)));
    const int parts = (int)((nq + most - 1) / most); // of about the same size
    *per = (nq + parts - 1) / parts;
    return AVQ_OK;
}

// A batch in parts through go(first query, queries, whether it is the first part). AVQ_ENOMEM: no room for a part's scratch
// (nothing of that part was launched); what it had of it is given back, as the other paths, which take less, need it now.
template <class Go>
static int product_in_parts(avq_index *idx, int nq, int per, Go go)
{
    int rc = AVQ_OK;
    for (int q0 = 0; q0 < nq && rc == AVQ_OK; q0 += per) rc = go(q0, std::min(per, nq - q0), q0 == 0);
    if (rc == AVQ_ENOMEM) {
        idx->product.release();
        idx->lut_fail.release();
        idx->fail_rows.release();
    }
    return rc;
}

static int search_product(avq_index *idx, const float *queries, int nq, int k, int reorder_k, int R, int ns, bool u8, bool first,
                          int32_t *ids_out, float *scores_out, hipStream_t st)
{
    const avq_config &c = idx->cfg;
    const int C = 64 * ns;
    const ProductPlan pl = product_plan(nq, idx->n, c.d, R, u8);
    ProductParams p;
    memset(&p, 0, sizeof(p));
    p.codes = idx->codes_blocked.as<uint8_t>();
    p.n = idx->n;
    p.nq = nq; p.d = c.d; p.M = c.M; p.bits = c.bits; p.NB = idx->NB;
    p.n_tiles = pl.n_tiles;
    p.n_classes = pl.n_classes;
    p.run = pl.run;
    p.kept_cap = pl.kept_cap;
    p.cnt_stride = pl.cnt_stride;
    // scratch, 256-byte aligned pieces
    size_t off = 0;
    auto take = [&](size_t bytes) -> size_t { const size_t at = (off + 255) & ~(size_t)255; off = at + bytes; return at; };
    const size_t o_cb = take((size_t)c.M * idx->kc * idx->ds * 2), o_packed = take((size_t)pl.n_tiles * pl.steps * 1024),
                 o_meta = take(kProductInfoBytes), o_q = take(kProductInfoBytes * (size_t)nq),
                 o_thr = take(sizeof(float) * ((size_t)pl.n_tiles * 32 + 64)), o_margin = take(sizeof(float) * (size_t)nq * 2),
                 o_classes = take(sizeof(float) * (size_t)nq * pl.n_classes), o_kept = take(sizeof(u64) * (size_t)nq * pl.kept_cap),
                 o_cnt = take(sizeof(uint32_t) * (size_t)nq * pl.cnt_stride);
    AVQ_TRY(idx->product.reserve(off));
    unsigned char *base = (unsigned char *)idx->product.p;
    p.cb16 = base + o_cb;
    p.packed = base + o_packed;
    p.meta = (ProductMeta *)(base + o_meta);
    p.qinfo = (ProductQuery *)(base + o_q);
    p.thr = (float *)(base + o_thr);
    p.classes = (float *)(base + o_classes);
    p.kept = (u64 *)(base + o_kept);
    p.kept_cnt = (uint32_t *)(base + o_cnt);
    float *margin = (float *)(base + o_margin), *guess = margin + nq;
    // the plain scan for the queries whose candidates cannot be used: its grid is cut on the device to their number
    ScanParams pf;
    fill_scan_params(idx, nq, R, ns, &pf);
    ScanShape shape;
    AVQ_TRY(product_shape(idx, nq, ns, u8, false, &shape));
    pf.n_tiles = (nq + shape.qt - 1) / shape.qt;
    pf.n_chunks = (int32_t)std::max<int64_t>(1, std::min<int64_t>(128, idx->n_blocks / shape.waves)); // at most
    pf.blocks_per_chunk = 0; // derived on the device
    const size_t items = (size_t)std::max(kDynamicItems, pf.n_tiles); // (tiles of live queries) x chunks
    AVQ_TRY(idx->partial.reserve(sizeof(u64) * items * shape.qt * C));
    if (shape.lists_global) AVQ_TRY(idx->lists.reserve(sizeof(u64) * items * shape.waves * shape.qt * C));
    const size_t row_floats = u8 ? (size_t)c.M * idx->kc / 4 : (size_t)c.M * idx->kc; // a query's tables, in 4-byte units
    AVQ_TRY(idx->lut_fail.reserve(sizeof(float) * (size_t)pf.n_tiles * shape.qt * row_floats));
    AVQ_TRY(idx->fail.reserve(sizeof(int32_t) * (8 + (size_t)nq)));
    uint32_t *fail_total = idx->fail.as<uint32_t>(), *fail_count = fail_total + 4;
    int32_t *fail_list = idx->fail.as<int32_t>() + 8;
    {
        StageTimer t(idx, AVQ_STAGE_LUT, st);
        if (u8) AVQ_TRY(build_tables(idx, queries, nq, AVQ_LUT_U8, st));
        AVQ_TRY(launch_product_pack(p, queries, idx->codebooks.as<float>(), first ? fail_total : fail_count, first ? 8 : 4, false, st));
    }
    {
        StageTimer t(idx, AVQ_STAGE_SAMPLE, st);
        p.groups = pl.sample_groups;
        p.stages_per_chunk = pl.sample_stages_per_chunk;
        p.chunks = pl.sample_chunks;
        p.stride = pl.stride;
        AVQ_TRY(launch_product_scan(p, true, st));
        AVQ_TRY(launch_product_bound(p, pl.r, u8 ? idx->scale.as<float>() : nullptr, margin, guess, nullptr, nullptr, 0, st));
    }
    {
        StageTimer t(idx, AVQ_STAGE_SCAN, st); // the launch over all points, nothing else
        p.groups = pl.groups;
        p.stages_per_chunk = pl.stages_per_chunk;
        p.chunks = pl.chunks;
        p.stride = 1;
        AVQ_TRY(launch_product_scan(p, false, st));
    }
    StageTimer t(idx, AVQ_STAGE_RESCAN, st);
    ProductRefineParams r;
    memset(&r, 0, sizeof(r));
    r.kept = p.kept;
    r.kept_cnt = p.kept_cnt;
    r.margin = margin;
    r.guess = guess;
    r.queries = queries;
    r.codebooks = idx->codebooks.as<float>();
    r.x = idx->x;
    r.codes = idx->codes_logical.as<uint8_t>();
    r.lut8 = u8 ? idx->lut8.as<uint8_t>() : nullptr;
    r.scale = idx->scale.as<float>();
    r.bias = idx->bias.as<float>();
    r.ids_out = ids_out;
    r.scores_out = scores_out;
    r.fail_list = fail_list;
    r.fail_count = fail_count;
    r.fail_total = fail_total;
    r.fail_lut = idx->lut_fail.p;
    r.kept_cap = pl.kept_cap; r.cnt_stride = pl.cnt_stride;
    r.nq = nq; r.d = c.d; r.M = c.M; r.NB = idx->NB; r.R = R; r.k = k; r.reorder = reorder_k != 0;
    r.force_fail_odd = idx->tune_prefilter == 2;
    AVQ_TRY(launch_product_refine(r, u8, c.bits, st));
    // the other queries, whose tables lie side by side now: the plain scan over them
    pf.lut = idx->lut_fail.as<float>();
    pf.lut8 = idx->lut_fail.as<uint8_t>();
    pf.partial = idx->partial.as<u64>();
    if (shape.lists_global) pf.lists_ws = idx->lists.as<u64>();
    pf.active_queries = fail_count;
    AVQ_TRY(launch_scan(pf, u8, SCAN_CHUNK, shape, st));
    return launch_product_fallback(r, pf.partial, pf.n_chunks, shape.qt, ns, u8, st);
}

// Batches on a partitioned index of 4-bit codes: the (query, leaf) pairs are regrouped by leaf and
// every leaf is scanned once per 32 of its queries on the matrix cores, against a bound per query
// that the query's best few leaves supply; the kept points are scored and ranked per query.
static bool use_grouped_leaves(const avq_index *idx, int nq, int L, int R)
{
    // below about 1.3e5 pairs (1,300 queries x 100 leaves) one workgroup per query is faster: regrouping, bounds and
    // the hand-over of kept points cost a fixed 0.2 ms
    const int64_t min_pairs = idx->tune_group_min > 0 ? idx->tune_group_min : 100000;
    return idx->tune_prefilter != 1 && idx->tune_mfma == 0 && idx->cfg.n_leaves > 0 && nq >= 64 && nq <= (1 << 16) &&
           (int64_t)nq * L >= min_pairs &&
           scan_mfma_supported(idx->NB, idx->cfg.bits) && idx->cfg.M <= 64 && L >= 16 && L <= 512 &&
           idx->cfg.n_leaves <= (1 << 21) && idx->max_leaf_blocks <= 1024 && R <= 2048;
}

static int search_leaves_grouped(avq_index *idx, const float *queries, int nq, int k, int reorder_k, int R, int ns, int L,
                                 bool u8, int32_t *ids_out, float *scores_out, hipStream_t st)
{
    const avq_config &c = idx->cfg;
    const int C = 64 * ns;
    AVQ_TRY(idx->leaf_ids.reserve(sizeof(int32_t) * (size_t)nq * L));
    AVQ_TRY(idx->leaf_ip.reserve(sizeof(float) * (size_t)nq * L));
    AVQ_TRY(idx->groups.reserve(sizeof(uint32_t) * group_by_leaf_words(nq, L, c.n_leaves)));
    LeafGroups g;
    {
        StageTimer t(idx, AVQ_STAGE_LEAF, st);
        AVQ_TRY(group_by_leaf_prepare(nq, L, c.n_leaves, idx->groups.as<uint32_t>(), &g, st));
        AVQ_TRY(launch_leaf_select(idx->centers_t.as<float>(), c.n_leaves, c.d, queries, nq, L,
                                   idx->leaf_ids.as<int32_t>(), idx->leaf_ip.as<float>(), st, g.cnt_wide, g.pos, g.cnt_stride));
    }
    // scratch: [4] counts | [nq] unverified queries | [nq] margins | [nq] bounds | [nq] kept counts
    AVQ_TRY(idx->fail.reserve(sizeof(int32_t) * (4 + (size_t)4 * nq)));
    uint32_t *fail_count = idx->fail.as<uint32_t>();
    int32_t *fail_list = idx->fail.as<int32_t>() + 4;
    int32_t *margin = fail_list + nq;
    uint32_t *bound = (uint32_t *)(margin + nq);
    uint32_t *kept_cnt = bound + nq;
    const int kept_cap = idx->tune_prefilter_cap > 0 ? std::min(4096, std::max(128, idx->tune_prefilter_cap)) : 2048;
    AVQ_TRY(idx->kept.reserve(sizeof(u64) * (size_t)nq * kept_cap));
    AVQ_TRY(idx->cand.reserve(sizeof(u64) * (size_t)nq * C));
    AVQ_TRY(idx->refined.reserve(sizeof(u64) * (size_t)nq * C));

    // the plain scan over leaves, used twice: over the first leaves of every query for the bounds, and
    // over all leaves of the queries that are handed back
    ScanShape shape;
    const int waves_hint = idx->tune_waves > 0 ? idx->tune_waves : 0;
    AVQ_TRY(scan_pick_shape(idx->NB, c.bits, u8, ns, nq, true, idx->tune_qt, waves_hint, &shape));
    ScanParams pl;
    fill_scan_params(idx, nq, R, ns, &pl);
    pl.perm = idx->perm.as<int32_t>();
    pl.leaf_ids = idx->leaf_ids.as<int32_t>();
    pl.leaf_ip = idx->leaf_ip.as<float>();
    pl.leaf_blk = idx->leaf_blk.as<int32_t>();
    pl.n_tiles = nq;
    pl.n_chunks = 1;
    AVQ_TRY(idx->partial.reserve(sizeof(u64) * (size_t)nq * C));
    pl.partial = idx->partial.as<u64>();
    if (shape.lists_global) {
        AVQ_TRY(idx->lists.reserve(sizeof(u64) * (size_t)nq * shape.waves * shape.qt * C));
        pl.lists_ws = idx->lists.as<u64>();
    }
    const int bound_leaves = idx->tune_bound_leaves > 0 ? std::min(L, idx->tune_bound_leaves) : std::min(L, std::max(8, u8 ? (L + 11) / 12 : (2 * L + 24) / 25));
    ScanParams pi;
    {
        StageTimer t(idx, AVQ_STAGE_SAMPLE, st); // here: margins, bounds from the first leaves, regrouping
        AVQ_HIP(hipMemsetAsync(fail_count, 0, 16, st));
        AVQ_HIP(hipMemsetAsync(kept_cnt, 0, sizeof(uint32_t) * (size_t)nq, st));
        if (!u8) AVQ_TRY(launch_prefilter_margin(idx->lut.as<float>(), idx->scale.as<float>(), c.M, idx->NB, nq, margin, st));
        ScanParams pb = pl;
        pb.Lp = bound_leaves;
        pb.leaf_stride = L;
        if (idx->max_leaf_blocks <= kLeafBoundMaxBlocks) {
            AVQ_TRY(launch_leaf_bound(pb, u8, (int)idx->max_leaf_blocks, (int)((idx->n_blocks + c.n_leaves - 1) / c.n_leaves), bound, st));
        } else {
            AVQ_TRY(launch_scan(pb, u8, SCAN_LEAVES, shape, st));
            AVQ_TRY(launch_list_bound(pb.partial, ns, R, nq, bound, st));
        }
        AVQ_TRY(launch_group_by_leaf(idx->leaf_ids.as<int32_t>(), nq, L, c.n_leaves, g, st));
        fill_scan_params(idx, nq, R, ns, &pi);
        pi.n_valid = 0x7fffffff; // padding slots are told from points by perm, afterwards
        pi.leaf_blk = idx->leaf_blk.as<int32_t>();
        pi.leaf_ip = idx->leaf_ip.as<float>();
        pi.Lp = L;
        pi.leaf_stride = L;
        pi.item_list = g.item_list;
        pi.n_items = g.n_items;
        pi.qlist = g.qlist;
        pi.leaf_off = g.leaf_off;
        pi.leaf_cnt = g.leaf_cnt;
        pi.max_items = g.max_items;
        pi.item_bound = bound;
        pi.cand_margin = u8 ? nullptr : margin;
        pi.kept = idx->kept.as<u64>();
        pi.kept_cnt = kept_cnt;
        pi.kept_cap = kept_cap;
    }
    {
        StageTimer t(idx, AVQ_STAGE_SCAN, st); // the scan over all leaves, nothing else
        AVQ_TRY(launch_scan_mfma(pi, st));
    }
    {
        StageTimer t(idx, AVQ_STAGE_RESCAN, st);
        IvfRefineParams r;
        r.kept = idx->kept.as<u64>();
        r.kept_cnt = kept_cnt;
        r.kept_cap = kept_cap;
        r.R = R; r.ns = ns; r.nq = nq; r.M = c.M; r.NB = idx->NB; r.leaf_stride = L;
        r.lut = u8 ? nullptr : idx->lut.as<float>();
        r.scale = idx->scale.as<float>();
        r.bias = idx->bias.as<float>();
        r.leaf_ip = idx->leaf_ip.as<float>();
        r.margin = u8 ? nullptr : margin;
        r.leaf_blk = idx->leaf_blk.as<int32_t>();
        r.perm = idx->perm.as<int32_t>();
        r.codes = idx->codes_logical.as<uint8_t>();
        r.out = idx->refined.as<u64>();
        r.fail_list = fail_list;
        r.fail_count = fail_count;
        r.force_fail_odd = idx->tune_prefilter == 2;
        AVQ_TRY(launch_ivf_refine(r, st));
        // the queries handed back: their rows (tables, scale, bias, probed leaves) side by side, the plain
        // scan over all their leaves, and their lists into their own rows of the refined candidates
        const size_t lut_row = u8 ? (size_t)c.M * idx->kc / 4 : (size_t)c.M * idx->kc; // 4-byte units
        AVQ_TRY(idx->lut_fail.reserve(sizeof(float) * (size_t)nq * lut_row));
        AVQ_TRY(idx->fail_rows.reserve(sizeof(float) * (size_t)nq * (2 + (size_t)2 * L)));
        float *scale_c = idx->fail_rows.as<float>(), *bias_c = scale_c + nq;
        float *ip_c = bias_c + nq;
        int32_t *ids_c = (int32_t *)(ip_c + (size_t)nq * L);
        AVQ_TRY(launch_gather_rows(u8 ? (const float *)idx->lut8.p : idx->lut.as<float>(), idx->lut_fail.as<float>(), fail_list,
                                   fail_count, nq, (int)lut_row, st));
        AVQ_TRY(launch_gather_rows(idx->scale.as<float>(), scale_c, fail_list, fail_count, nq, 1, st));
        AVQ_TRY(launch_gather_rows(idx->bias.as<float>(), bias_c, fail_list, fail_count, nq, 1, st));
        AVQ_TRY(launch_gather_rows(idx->leaf_ip.as<float>(), ip_c, fail_list, fail_count, nq, L, st));
        AVQ_TRY(launch_gather_rows((const float *)idx->leaf_ids.p, (float *)ids_c, fail_list, fail_count, nq, L, st));
        // few queries, one workgroup each: as many waves per workgroup as the kernel takes
        ScanShape shape_f;
        AVQ_TRY(scan_pick_shape(idx->NB, c.bits, u8, ns, nq, true, idx->tune_qt, waves_hint ? waves_hint : 16, &shape_f));
        ScanParams pf = pl;
        pf.lut = idx->lut_fail.as<float>();
        pf.lut8 = idx->lut_fail.as<uint8_t>();
        pf.scale = scale_c;
        pf.bias = bias_c;
        pf.leaf_ip = ip_c;
        pf.leaf_ids = ids_c;
        pf.Lp = L;
        pf.active_queries = fail_count;
        AVQ_TRY(launch_scan(pf, u8, SCAN_LEAVES, shape_f, st));
        AVQ_TRY(launch_merge_partials(pf.partial, nq, 1, ns, idx->refined.as<u64>(), st, fail_list, fail_count, 0));
    }
    StageTimer t(idx, AVQ_STAGE_FINAL, st);
    return launch_finalize(idx->refined.as<u64>(), ns, nq, R, k, reorder_k != 0, 0, idx->x, c.d, queries,
                           idx->scale.as<float>(), idx->bias.as<float>(), ids_out, scores_out, st);
}

// Batches on a partitioned index through the product of the queries with the decoded points of the leaves they probe
// (product_leaf.hip). Both launches decode every block of every probed leaf whatever its queries, and those are rounded up to 32, so
// what counts beside the points scored (queries x probed leaves x points of a leaf) is the queries of a leaf. Measured, other path /
// product, us a call, R = 100 and fp32 tables unless said otherwise:
//  points scored: 100 dimensions, 4-bit codes: 1e7 137 / 124 (500 queries), 1.8e7 266 / 220, 6e7 536 / 313, 6e8 2,822 / 1,222; R = 500
//   2,434 / 565 at 1.2e8; 8-bit tables, R = 500: 1,216 / 1,344 at 6e7.
//  queries of a leaf, where the other path is one workgroup a query: 10,000,000 points: 3 (64 queries) 226 / 1,536, 16 665 / 1,747,
//   25 1,449 / 1,800; 5,000,000 x 105 points: 24 785 / 1,236, 30 1,050 / 910; 1,183,514 x 128: 25 330 / 451, 50 647 / 524; 8-bit codes of 256
//   dimensions 50 479 / 508; R = 500: 24 689 / 500.
//  where it is regrouped by leaf: leaves of 1,000 points 10 3,029 / 2,228, 75 6,085 / 3,012; of 3,300 to 5,000 points 75 2,034 / 2,041,
//   80 760 / 1,098, 90 1,499 / 1,248, 250 3,660 / 2,949; R = 500 50 10,194 / 5,023.
//  few of the leaves probed (many small classes of points): 1,183,514 points, 30 of 2,000 leaves, 45 queries a leaf 452 / 605, 10,000,000,
//   100 of 10,000, 100 a leaf, 8-bit codes 4,297 / 4,921; 1,183,514, 5 of 500 leaves, 100 a leaf 1,093 / 704: the two estimates below.
static bool use_product_leaves(const avq_index *idx, int nq, int L, int R, bool u8)
{
    const avq_config &c = idx->cfg;
    if (idx->tune_product == 1 || c.n_leaves <= 0 ||
        !product_leaf_supported(c.d, c.M, c.n_leaves, idx->n_blocks, idx->max_leaf_blocks, nq, L, R)) return false;
    if (idx->tune_product == 2) return true;
    // any tuning of the other kernels' launches asks for those kernels
    if (idx->tune_target_wgs || idx->tune_waves || idx->tune_qt || idx->tune_mfma || idx->tune_prefilter == 1 || idx->tune_prefilter_cap ||
        idx->tune_sample || idx->tune_small_impl || idx->tune_small_batch >= 0 || idx->tune_group_min || idx->tune_bound_leaves) return false;
    const double n = (double)idx->n, q = (double)nq, leaf = n / c.n_leaves, work = q * L * leaf, per_leaf = q * L / c.n_leaves;
    if (nq < 64 || work < (u8 && R > 256 ? 1e8 : 2.5e7)) return false;
    if (use_grouped_leaves(idx, nq, L, R)) return per_leaf >= (leaf <= 1500.0 ? 8.0 : R <= 256 ? 100.0 : 50.0);
    if (per_leaf < (c.bits == 8 && c.d > 128 ? 100.0 : R <= 256 ? 30.0 : 28.0)) return false;
    if (!product_leaf_narrow(L, c.n_leaves, R)) return true;
    const ProductLeafPlan pl = product_leaf_plan(nq, L, c.n_leaves, idx->n, idx->n_blocks, idx->max_leaf_blocks, c.d, R, u8);
    const double slots = 256.0 * (double)idx->n_blocks;
    const double product = 125.0 + slots * pl.steps * (2e-5 + 8e-8 * (per_leaf + 16.0)) + q * (0.0001 * L + (u8 ? 0.00055 : 0.00025) * R + 8e-6 * pl.n_classes);
    const double plain = 130.0 + work * (idx->NB * (c.bits == 8 ? 1.4e-7 : idx->NB <= 32 ? 1.5e-7 : 2.8e-7) + 0.0007 / q) + q * (0.0002 * L + (u8 ? 0.0 : 0.0003) * R);
    return product < 1.15 * plain;
}

static int search_leaves_product(avq_index *idx, const float *queries, int nq, int k, int reorder_k, int R, int ns, int L, bool u8,
                                 bool first, int32_t *ids_out, float *scores_out, hipStream_t st)
{
    const avq_config &c = idx->cfg;
    const int C = 64 * ns;
    const ProductLeafPlan pl = product_leaf_plan(nq, L, c.n_leaves, idx->n, idx->n_blocks, idx->max_leaf_blocks, c.d, R, u8);
    const int64_t pairs = (int64_t)nq * L;
    ProductLeafParams p;
    memset(&p, 0, sizeof(p));
    p.base.codes = idx->codes_blocked.as<uint8_t>();
    p.base.n = idx->n_blocks * kBlockPoints;
    p.base.nq = nq; p.base.d = c.d; p.base.M = c.M; p.base.bits = c.bits; p.base.NB = idx->NB;
    p.base.n_tiles = pl.n_tiles;
    p.base.n_classes = pl.n_classes;
    p.base.kept_cap = pl.kept_cap;
    p.base.cnt_stride = pl.cnt_stride;
    p.L = L;
    p.run = pl.run;
    p.pair_classes = pl.pair_classes;
    // scratch, 256-byte aligned pieces
    size_t off = 0;
    auto take = [&](size_t bytes) -> size_t { const size_t at = (off + 255) & ~(size_t)255; off = at + bytes; return at; };
    const size_t class_bytes = sizeof(uint32_t) * (size_t)nq * pl.n_classes;
    const size_t o_cb = take((size_t)c.M * idx->kc * idx->ds * 2), o_packed = take((size_t)pl.n_tiles * pl.steps * 1024),
                 o_meta = take(kProductInfoBytes), o_q = take(kProductInfoBytes * (size_t)nq), o_thr = take(sizeof(float) * (size_t)pl.n_tiles * 32),
                 o_margin = take(sizeof(float) * (size_t)nq * 2), o_classes = take(class_bytes), o_kept = take(sizeof(u64) * (size_t)nq * pl.kept_cap),
                 o_slot = take(sizeof(uint16_t) * (size_t)nq * pl.kept_cap), o_cnt = take(sizeof(uint32_t) * (size_t)nq * pl.cnt_stride),
                 o_ip = take(sizeof(float) * (size_t)pairs), o_line = take(sizeof(float) * (size_t)pairs),
                 o_items = take(sizeof(uint2) * (size_t)pl.most_items), o_ni = take(sizeof(uint32_t));
    AVQ_TRY(idx->product.reserve(off));
    AVQ_TRY(idx->leaf_ids.reserve(sizeof(int32_t) * (size_t)pairs));
    AVQ_TRY(idx->leaf_ip.reserve(sizeof(float) * (size_t)pairs));
    // cleared in pieces of 16 bytes, from a piece's start on: the counters lie last in groups
    AVQ_TRY(idx->groups.reserve(sizeof(uint32_t) * group_by_leaf_words(nq, L, c.n_leaves) + 32));
    LeafGroups g;
    AVQ_TRY(group_by_leaf_lay_out(nq, L, c.n_leaves, idx->groups.as<uint32_t>(), &g));
    g.cnt_wide = (uint32_t *)(((uintptr_t)g.cnt_wide + 15) & ~(uintptr_t)15);
    unsigned char *base = (unsigned char *)idx->product.p;
    p.base.cb16 = base + o_cb;
    p.base.packed = base + o_packed;
    p.base.meta = (ProductMeta *)(base + o_meta);
    p.base.qinfo = (ProductQuery *)(base + o_q);
    p.base.thr = (float *)(base + o_thr);
    p.base.classes = (float *)(base + o_classes);
    p.base.kept = (u64 *)(base + o_kept);
    p.base.kept_cnt = (uint32_t *)(base + o_cnt);
    p.kept_slot = (uint16_t *)(base + o_slot);
    p.classes = (uint32_t *)(base + o_classes);
    p.pair_ip = (float *)(base + o_ip);
    p.pair_line = (float *)(base + o_line);
    p.perm = idx->perm.as<int32_t>();
    p.leaf_blk = idx->leaf_blk.as<int32_t>();
    p.leaf_off = g.leaf_off;
    p.leaf_cnt = g.leaf_cnt;
    p.qlist = g.qlist;
    uint2 *items = (uint2 *)(base + o_items);
    uint32_t *n_items = (uint32_t *)(base + o_ni);
    p.items = items;
    p.n_items = n_items;
    float *margin = (float *)(base + o_margin), *guess = margin + nq;
    // the plain scan over the leaves of the queries that are handed back
    ScanShape shape;
    AVQ_TRY(product_shape(idx, nq, ns, u8, true, &shape));
    AVQ_TRY(idx->partial.reserve(sizeof(u64) * (size_t)nq * C));
    if (shape.lists_global) AVQ_TRY(idx->lists.reserve(sizeof(u64) * (size_t)nq * shape.waves * shape.qt * C));
    const size_t lut_row = u8 ? (size_t)c.M * idx->kc / 4 : (size_t)c.M * idx->kc; // 4-byte units
    AVQ_TRY(idx->lut_fail.reserve(sizeof(float) * (size_t)nq * lut_row));
    AVQ_TRY(idx->fail_rows.reserve(sizeof(float) * (size_t)nq * (2 + (size_t)2 * L)));
    AVQ_TRY(idx->fail.reserve(sizeof(int32_t) * (8 + (size_t)nq)));
    uint32_t *fail_total = idx->fail.as<uint32_t>(), *fail_count = fail_total + 4;
    int32_t *fail_list = idx->fail.as<int32_t>() + 8;
    if (u8) {
        StageTimer t(idx, AVQ_STAGE_LUT, st);
        AVQ_TRY(build_tables(idx, queries, nq, AVQ_LUT_U8, st));
    }
    {
        StageTimer t(idx, AVQ_STAGE_LEAF, st);
        AVQ_TRY(launch_product_clear(g.cnt_wide, (sizeof(uint32_t) * (size_t)c.n_leaves * g.cnt_stride + 15) / 16 * 16, p.classes, class_bytes, st));
        AVQ_TRY(launch_leaf_select(idx->centers_t.as<float>(), c.n_leaves, c.d, queries, nq, L, idx->leaf_ids.as<int32_t>(),
                                   idx->leaf_ip.as<float>(), st, g.cnt_wide, g.pos, g.cnt_stride));
    }
    {
        StageTimer t(idx, AVQ_STAGE_SAMPLE, st); // here: operands, regrouping, bounds
        AVQ_TRY(launch_product_pack(p.base, queries, idx->codebooks.as<float>(), first ? fail_total : fail_count, first ? 8 : 4, true, st));
        AVQ_TRY(launch_group_offsets(g, c.n_leaves, st));
        AVQ_TRY(launch_product_pairs(p, idx->leaf_ids.as<int32_t>(), idx->leaf_ip.as<float>(), g.pos, c.n_leaves, items, pl.most_items, n_items, st));
        AVQ_TRY(launch_product_leaf(p, true, pl.most_items, st));
        AVQ_TRY(launch_product_bound(p.base, R, u8 ? idx->scale.as<float>() : nullptr, margin, guess, idx->leaf_ids.as<int32_t>(),
                                     idx->leaf_ip.as<float>(), L, st));
        AVQ_TRY(launch_product_lines(p, c.n_leaves, st));
    }
    {
        StageTimer t(idx, AVQ_STAGE_SCAN, st); // the launch over all leaves, nothing else
        AVQ_TRY(launch_product_leaf(p, false, pl.most_items, st));
    }
    StageTimer t(idx, AVQ_STAGE_RESCAN, st);
    ProductLeafRefineParams r;
    memset(&r, 0, sizeof(r));
    r.base.kept = p.base.kept;
    r.base.kept_cnt = p.base.kept_cnt;
    r.base.margin = margin;
    r.base.guess = guess;
    r.base.queries = queries;
    r.base.codebooks = idx->codebooks.as<float>();
    r.base.x = idx->x;
    r.base.codes = idx->codes_logical.as<uint8_t>();
    r.base.lut8 = u8 ? idx->lut8.as<uint8_t>() : nullptr;
    r.base.scale = idx->scale.as<float>();
    r.base.bias = idx->bias.as<float>();
    r.base.ids_out = ids_out;
    r.base.scores_out = scores_out;
    r.base.fail_list = fail_list;
    r.base.fail_count = fail_count;
    r.base.fail_total = fail_total;
    r.base.fail_lut = idx->lut_fail.p;
    r.base.kept_cap = pl.kept_cap; r.base.cnt_stride = pl.cnt_stride;
    r.base.nq = nq; r.base.d = c.d; r.base.M = c.M; r.base.NB = idx->NB; r.base.R = R; r.base.k = k; r.base.reorder = reorder_k != 0;
    r.base.force_fail_odd = idx->tune_prefilter == 2;
    r.kept_slot = p.kept_slot;
    r.perm = p.perm;
    r.leaf_ids = idx->leaf_ids.as<int32_t>();
    r.leaf_ip = idx->leaf_ip.as<float>();
    r.fail_scale = idx->fail_rows.as<float>();
    r.fail_bias = r.fail_scale + nq;
    r.fail_ip = r.fail_bias + nq;
    r.fail_ids = (int32_t *)(r.fail_ip + pairs);
    r.L = L;
    AVQ_TRY(launch_product_leaf_refine(r, u8, c.bits, st));
    ScanParams pf;
    fill_scan_params(idx, nq, R, ns, &pf);
    pf.perm = p.perm;
    pf.leaf_ids = r.fail_ids;
    pf.leaf_ip = r.fail_ip;
    pf.leaf_blk = p.leaf_blk;
    pf.lut = idx->lut_fail.as<float>();
    pf.lut8 = idx->lut_fail.as<uint8_t>();
    pf.scale = r.fail_scale;
    pf.bias = r.fail_bias;
    pf.Lp = L;
    pf.n_tiles = nq;
    pf.n_chunks = 1;
    pf.partial = idx->partial.as<u64>();
    if (shape.lists_global) pf.lists_ws = idx->lists.as<u64>();
    pf.active_queries = fail_count;
    AVQ_TRY(launch_scan(pf, u8, SCAN_LEAVES, shape, st));
    return launch_product_fallback(r.base, pf.partial, 1, 1, ns, false, st);
}

static int check_query_args(const avq_index *idx, const float *queries, int32_t nq, int32_t lut_mode)
{
    if (idx->n <= 0) { set_error("no database yet (avq_encode or avq_set_database first)"); return AVQ_ESTATE; }
    if (!idx->have_codebooks) { set_error("no dictionaries yet"); return AVQ_ESTATE; }
    if (!queries || nq < 1) { set_error("queries NULL or nq < 1"); return AVQ_EINVAL; }
    if (lut_mode != AVQ_LUT_F32 && lut_mode != AVQ_LUT_U8) { set_error("bad lut_mode %d", lut_mode); return AVQ_EINVAL; }
    return AVQ_OK;
}

// ---- a handful of queries on a flat index ------------------------------------------------
// Full scan recording block maxima, selection of the R best blocks, scan of those, final
// selection with exact re-scoring. Its device scratch is described by SmallWs, so that the
// same launches can run from buffers the index owns (avq_search) or from the library's static
// scratch array (avq_search_noalloc).
struct SmallWs {
    float *lut;          // [nq][M][kc]      (unused when the scan computes its own tables)
    uint8_t *lut8;       // [nq][M][kc]      (8-bit tables only)
    float *scale, *bias; // [nq]             (8-bit tables only)
    u64 *block_max;      // [nq][n_blocks]
    u64 *cand;           // [nq][256 * R]
    int32_t *sel_blk;    // [nq][R], or [nq][n_blocks] on the block-bound path
    SmallMeta *meta;     // [nq]
    uint32_t *block_bound; // [nq][n_blocks]   (block-bound path)
    BoundMeta *bound_meta; // [nq]             (block-bound path)
    uint8_t *bound_tbl;    // [nq][NB][256]    (block-bound path)
    uint32_t *sel_hist;    // [nq][8192]       (block-bound path, selection over several workgroups per query)
    u64 *fin_out;          // [nq][R]          (exact re-scoring over several workgroups per query)
    uint32_t *fin_n;       // [nq][2]
};

// 0: the scan records block maxima of 8-bit sums (bounds of the scores) where the code size has its
// kernels; 2 (tuning "small_batch_impl"): always the exact block maxima.
static bool small_uses_bounds(const avq_index *idx)
{
    return idx->tune_small_impl == 0 && block_bound_supported(idx->NB, idx->cfg.bits);
}

// Blocks per workgroup when the selection of a query's blocks is spread over several workgroups; 0: one workgroup
// per query. Built in: a few queries on an index of 32,768 blocks or more, where one compute unit's two passes over
// the block maxima take longer than everything else after the scan. Tuning "select_split": 1 never, v >= 2: always,
// v blocks per workgroup.
static int small_select_split_per(const avq_index *idx, int nq)
{
    if (!small_uses_bounds(idx) || idx->tune_select_split == 1) return 0;
    if (idx->tune_select_split >= 2) return std::min(idx->tune_select_split, 8192);
    return nq <= 16 && idx->n_blocks >= 32768 ? 8192 : 0;
}

// Candidates per workgroup when the exact re-scoring of a query's candidates is spread over several workgroups; 0:
// the final kernel does it. Built in: up to 16 queries whose R rows of d values one workgroup would stage in more
// than one pass (its LDS holds `stage_rows` of them): 64 rows per workgroup. Tuning "rerank_split": 1 never,
// v >= 2: always, v rows per workgroup (as many as fit LDS at most).
static int small_rerank_rows(const avq_index *idx, int nq, int R, int stage_rows, bool reorder)
{
    if (!reorder || idx->tune_rerank_split == 1) return 0;
    const int fit = (int)std::min<size_t>(1024, ((size_t)128 * 1024) / ((size_t)(idx->cfg.d + 1) * 4));
    if (fit < 1) return 0;
    if (idx->tune_rerank_split >= 2) return std::min(idx->tune_rerank_split, fit);
    return nq <= 16 && R > stage_rows ? std::min(64, fit) : 0;
}

// Lays the scratch out from `base` (256-byte aligned pieces); returns the bytes needed.
// base == NULL: only the size.
static size_t small_ws_carve(const avq_index *idx, int nq, int R, unsigned char *base, SmallWs *w)
{
    const int nq_tiles = (nq + 15) / 16 * 16; // the batch form of the block-bound scan lays its tables out in tiles of 16
    size_t off = 0;
    auto take = [&](size_t bytes) -> void * {
        const size_t at = (off + 255) & ~(size_t)255;
        off = at + bytes;
        return base ? (void *)(base + at) : nullptr;
    };
    const size_t entries = (size_t)nq * idx->cfg.M * idx->kc;
    w->lut = (float *)take(entries * sizeof(float));
    w->lut8 = (uint8_t *)take(entries);
    w->scale = (float *)take(sizeof(float) * (size_t)nq);
    w->bias = (float *)take(sizeof(float) * (size_t)nq);
    w->block_max = (u64 *)take(sizeof(u64) * (size_t)nq * idx->n_blocks);
    w->cand = (u64 *)take(sizeof(u64) * (size_t)nq * 256 * R);
    const bool bounds = small_uses_bounds(idx);
    w->sel_blk = (int32_t *)take(sizeof(int32_t) * (size_t)nq * (bounds ? (size_t)idx->n_blocks : (size_t)R));
    w->meta = (SmallMeta *)take(sizeof(SmallMeta) * (size_t)nq);
    w->block_bound = (uint32_t *)take(bounds ? sizeof(uint32_t) * (size_t)nq * idx->n_blocks : 0);
    w->bound_meta = (BoundMeta *)take(bounds ? sizeof(BoundMeta) * (size_t)nq : 0);
    w->bound_tbl = (uint8_t *)take(bounds ? (size_t)nq_tiles * idx->NB * 256 : 0);
    const bool split = small_select_split_per(idx, nq) > 0;
    w->sel_hist = (uint32_t *)take(split ? sizeof(uint32_t) * (size_t)nq * 8192 : 0);
    w->fin_out = (u64 *)take(sizeof(u64) * (size_t)nq * R);
    w->fin_n = (uint32_t *)take(sizeof(uint32_t) * (size_t)nq * 2);
    return off;
}

static int small_ws_from_index(avq_index *idx, int nq, int R, SmallWs *w)
{
    const size_t bytes = small_ws_carve(idx, nq, R, nullptr, w);
    AVQ_TRY(idx->tmp.reserve(bytes));
    small_ws_carve(idx, nq, R, (unsigned char *)idx->tmp.p, w);
    return AVQ_OK;
}

// Small flat indexes of 4-bit codes with fp32 tables: one launch answers the query.
// Its one compute unit adds up every point, so it grows with the blocks and their code bytes (and tables: n_blocks x
// (NB + 18) fits the times); the several launches cost about 40 us, and 55 to 65 once R reaches the number of blocks, whose
// points they then all score exactly. One launch / several (us a call), one query: 10,000 points, 16 subspaces, R = 100:
// 35 / 56, R = 10: 32 / 38; 16,384 points, R = 10: 16 subspaces 35 / 38, 50 subspaces 45 / 41, 64 50 / 43, 96 68 / 47 and
// R = 100: 39 / 62, 50 / 66, 53 / 67, 72 / 72; 12,288 points, 50 subspaces (the line, 48 x 43 = 2,064): 41 / 41; code sizes
// without kernels of their own cross earlier (8,192 x 72 subspaces, 32 x 54 = 1,728: 44 / 45). From sixteen queries on the
// several launches rise sooner (32 queries, 14,000 x 50 subspaces, R = 50: 45 / 55), from 64 on they never won (300
// queries, 16,384 x 50 subspaces, R = 10: 76 / 86) but where hundreds of queries want one or two points of a few blocks,
// for which sixteen waves are too many (16 subspaces, R = 1: 300 points, 1,000 queries 65 / 56, 3,000 152 / 103; 1,000 points,
// 3,000 queries 129 / 107; R = 10, 300 points, 1,000 queries: 66 / 80). Codes of one byte have so many equal sums that
// every pass of the selection carries them along (16,384 points, one query, R = 10: 42 / 38).
// Rows of R x d <= 100,000 floats are also re-scored by that one (500 x 100 at 2,000 points, one query: 25 / 46; 500 x 192:
// 35 / 53); more are left to the split re-scoring.
static bool use_search_one(const avq_index *idx, int nq, int R, bool fuse_tables, bool tile)
{
    if (!fuse_tables || tile || !search_one_supported(idx->n_blocks, idx->NB)) return false;
    if (R <= 2 && nq >= 256 * idx->n_blocks) return false;
    if (idx->NB == 1 && R <= idx->n_blocks) return false;
    const int64_t work = idx->n_blocks * (idx->NB + 18);
    const bool own = idx->NB == 8 || idx->NB == 13 || idx->NB == 25 || idx->NB == 32;
    if (nq < 64 && R <= idx->n_blocks && work > (own ? 2064 : 1750) && !(nq >= 16 && 2 * R > idx->n_blocks && work <= 2800)) return false;
    // any tuning of the other kernels' launches asks for those kernels
    return idx->tune_small_impl == 0 && idx->tune_waves == 0 && idx->tune_target_wgs == 0 && idx->tune_select_split == 0 &&
           idx->tune_rerank_split == 0 && idx->tune_stream_loads == 0;
}

// Launches only: no allocation, no synchronisation. timers: per-stage event pairs while profiling is on.
// tile: the batch form (8-bit codes): the full scan takes the queries sixteen at a time, with byte tables of 8 or 7 bits (own_bits below).
static int search_small(avq_index *idx, const float *queries, int nq, int k, int reorder_k, bool u8, bool fuse_tables,
                        const SmallWs &w, bool timers, int32_t *ids_out, float *scores_out, hipStream_t st, bool tile = false)
{
    const avq_config &c = idx->cfg;
    const int R = reorder_k ? reorder_k : k;
    const int ns = (R + 63) / 64;
    const bool bounds = small_uses_bounds(idx);
    if (!fuse_tables) {
        StageTimer t(idx, AVQ_STAGE_LUT, st, timers);
        AVQ_TRY(launch_lut(queries, nq, idx->codebooks.as<float>(), c.d, c.M, idx->kc, w.lut, u8 ? w.lut8 : nullptr, w.scale,
                           w.bias, st));
    }
    ScanParams p;
    fill_scan_params(idx, nq, R, ns, &p);
    p.lut = w.lut;
    p.lut8 = w.lut8;
    p.scale = w.scale;
    p.bias = w.bias;
    if (fuse_tables) {
        p.fuse_queries = queries;
        p.fuse_codebooks = idx->codebooks.as<float>();
        p.fuse_d = c.d;
    }
    p.block_max = w.block_max;
    p.n_tiles = nq;
    p.n_chunks = 1;
    p.max_wgs = idx->tune_target_wgs;
    p.nt_loads = stream_loads_nontemporal(idx, nq) ? 1 : 0;
    p.block_bound = w.block_bound;
    p.bound_meta = w.bound_meta;
    p.lut_out = fuse_tables ? w.lut : nullptr;
    p.bound_tbl = w.bound_tbl;
    p.sel_split_per = small_select_split_per(idx, nq);
    if (p.sel_split_per > 0) p.sel_hist = w.sel_hist;
    if (tile) {
        p.bound_tile = 16;
        // Entries of 6, 7 or 8 bits (tuning "bound_bits"): each bit more halves the width of the bounds, so fewer
        // blocks are scored exactly, and halves how many entries the full scan adds as packed bytes before it must
        // spread them into 16-bit sums. Seven is the best of the three at 1.2 and at 50 million points for batches; eight
        // for up to 64 queries on less than 40 MB of codes (1,183,514 x 25 bytes, fp32 tables, 7 / 8: 16 queries 78 / 71 us, 64
        // 175 / 160; 2,500,000: 90 / 88 and 230 / 232; 2,000,000 x 32 bytes, 8-bit tables, 64 queries 239 / 251).
        const int own_bits = nq <= 64 && R <= 200 && idx->n_blocks * idx->NB <= 150000 ? 8 : 7;
        const int bits_e = idx->tune_bound_bits >= 6 && idx->tune_bound_bits <= 8 ? idx->tune_bound_bits : own_bits;
        p.bound_levels = (1 << bits_e) - 1;
        p.bound_shift = 8 - bits_e;
        p.blocks_per_chunk = block_bound_tile_chunk(idx->n_blocks, nq);
    }
    FinishParams f;
    memset(&f, 0, sizeof(f));
    f.x = idx->x;
    f.queries = queries;
    f.d = c.d;
    f.k = k;
    f.reorder = reorder_k != 0;
    f.stage_rows = small_finish_stage_rows(p, c.d, u8);
    f.cand_stride = (int64_t)256 * R;
    f.cand = w.cand;
    f.sel_blk = w.sel_blk;
    f.meta = w.meta;
    f.ids_out = ids_out;
    f.scores_out = scores_out;
    f.rerank_rows = small_rerank_rows(idx, nq, R, f.stage_rows, f.reorder != 0);
    f.fin_out = w.fin_out;
    f.fin_n = w.fin_n;
    if (use_search_one(idx, nq, R, fuse_tables, tile) && (f.rerank_rows == 0 || (int64_t)R * c.d <= 100000)) {
        f.rerank_rows = 0;
        StageTimer t(idx, AVQ_STAGE_SCAN, st, timers);
        return launch_search_one(p, f, st);
    }
    if (bounds) {
        StageTimer t(idx, AVQ_STAGE_LUT, st, timers);
        AVQ_TRY(launch_bound_tables(p, u8, st));
    }
    {
        StageTimer t(idx, AVQ_STAGE_SCAN, st, timers);
        if (bounds && tile) AVQ_TRY(launch_block_bound_tile(p, st));
        else if (bounds) AVQ_TRY(launch_block_bound(p, idx->tune_waves, st));
        else AVQ_TRY(launch_block_max(p, u8, idx->tune_waves > 0 ? idx->tune_waves : 4, st));
    }
    if (bounds) {
        f.block_max = w.block_max;
        f.n_blocks = idx->n_blocks;
        f.n_valid = (int32_t)idx->n;
        f.NB = idx->NB;
        f.M = c.M;
        f.bits = c.bits;
        f.u8 = u8 ? 1 : 0;
        f.codes_logical = idx->codes_logical.as<uint8_t>();
        f.lut = w.lut;
        f.lut8 = w.lut8;
    }
    {
        StageTimer t(idx, AVQ_STAGE_MERGE, st, timers);
        if (bounds) AVQ_TRY(launch_select_bound_blocks(p, f, u8, st));
        else AVQ_TRY(launch_small_select(p, f, st));
    }
    {
        StageTimer t(idx, AVQ_STAGE_RESCAN, st, timers);
        if (bounds) AVQ_TRY(launch_rescan_listed(p, f, u8, st));
        else AVQ_TRY(launch_small_rescan(p, f, u8, st));
    }
    StageTimer t(idx, AVQ_STAGE_FINAL, st, timers);
    return launch_small_final(p, f, u8, st);
}


static int check_search_args(const avq_index *idx, const float *queries, int32_t nq, int32_t k, int32_t reorder_k,
                             int32_t lut_mode, int32_t leaves_to_search, const int32_t *ids_out, const float *scores_out)
{
    AVQ_TRY(check_index(idx));
    AVQ_TRY(check_query_args(idx, queries, nq, lut_mode));
    const avq_config &c = idx->cfg;
    if (!ids_out || !scores_out) { set_error("avq_search: output pointer is NULL"); return AVQ_EINVAL; }
    if (k < 1 || k > AVQ_MAX_SELECT || k > idx->n || (reorder_k != 0 && (reorder_k < k || reorder_k > AVQ_MAX_SELECT))) {
        set_error("avq_search: need 1 <= k <= min(n, %d) and reorder_k == 0 or k <= reorder_k <= %d",
                  AVQ_MAX_SELECT, AVQ_MAX_SELECT);
        return AVQ_EINVAL;
    }
    if (reorder_k != 0 && !idx->x) { set_error("avq_search: re-scoring needs the datapoints"); return AVQ_ESTATE; }
    if (c.n_leaves > 0 && (leaves_to_search < 1 || leaves_to_search > c.n_leaves || leaves_to_search > AVQ_MAX_SELECT)) {
        set_error("avq_search: leaves_to_search must be in [1, min(n_leaves, %d)]", AVQ_MAX_SELECT);
        return AVQ_EINVAL;
    }
    return AVQ_OK;
}

// ---- a handful of queries on a partitioned index -------------------------------------------
// Leaf selection, exact block maxima over the blocks of the probed leaves, selection of the R best blocks, the
// points of those at or above the R-th best maximum, final selection with exact re-scoring: the first design of the
// flat small-batch path, run on the few hundred blocks a query probes. Up to this many queries (measured crossover
// with the one-query-per-workgroup scan over leaves, which keeps sorted lists per wave: between 64 and 96 queries at
// 100 of 2,000 leaves).
constexpr int kLeafSmallMaxQueries = 80;
// 8-bit codes and code sizes without kernels of their own take it too, but
//  - for a few results from a few blocks, where the four launches of the list scan are done before the six here;
//  - where all of a query's blocks, and of more than 64, are scored twice and all of their points are candidates, for many queries:
//    those go to a query's list one by one, while the list scan's time hardly grows with the queries;
//  - beyond 64 queries, where the list scan has four waves a workgroup rather than sixteen;
//  - large codes for many queries, whose tables each workgroup copies.
// List scan / this, us a call, fp32 tables, queries 1 / 24 / 60 / 80:
//  16 bytes of 4-bit codes, 25 of 500 leaves, 32 blocks: R = 100 63/40 66/51 67/55 63/57, R = 500 208/50 216/63 218/71 234/76;
//   60 of 300, 342 blocks: R = 30 67/40 78/58 78/74 94/84, 200 176/48 193/115 201/204 175/246, 350 280/136 310/450 312/785 250/964;
//   100 of 2,000, 245 blocks: R = 200 170/49 204/134 296/242 201/285, 350 258/101 317/229 457/317 286/467, 500 379/104 438/248 623/390
//   384/499; 10 of 100, 396 blocks: R = 350 451/83 511/282 530/526 421/608, 500 640/192 698/559 701/1,032 568/1,219.
//  48 bytes of 4-bit codes, 342 blocks: R = 200 216/64 248/168 248/313 267/408, 245 blocks 258/76 361/241 442/423 348/486.
//  8-bit codes, 342 blocks, R = 350: 25 bytes 301/136 326/314 340/584 273/670, 48 bytes 304/146 339/378 354/631 339/781; 48 bytes, 32
//   blocks, R = 30: 60/49 62/61 74/92 76/103; 48 bytes of 4-bit codes, 4 blocks, R = 100, 60 queries 47 / 51.
// Of 6,174 calls 23 take more than 5 % longer than by the list scan, 15 % at most (48 bytes of 8-bit codes, 342 blocks, 60 queries).
static bool use_leaf_small(const avq_index *idx, int nq, int L, int R)
{
    const int max_q = idx->tune_small_batch >= 0 ? std::min(idx->tune_small_batch, 4096) : kLeafSmallMaxQueries;
    if (idx->cfg.n_leaves == 0 || idx->tune_small_impl == 1 || nq > max_q || L > 512 || !leaf_small_supported(idx->NB, idx->cfg.bits) ||
        !leaf_select_few_supported(idx->cfg.d)) return false;
    if (idx->tune_small_batch >= 0) return true;
    const bool own = idx->cfg.bits == 4 && block_bound_supported(idx->NB, 4), wide = idx->cfg.bits == 8;
    const double listed = (double)L * (double)idx->n_blocks / idx->cfg.n_leaves; // blocks of a query's leaves
    if (own) return R <= 200 || nq <= 64 || nq * listed <= 20000.0;
    const bool all = R >= 0.9 * listed;
    if (R < 32 && (listed < 12.0 || (all && nq > 24))) return false;
    if (!wide && idx->NB > 32 && nq > 24 && R <= 100 && listed < 12.0) return false;
    if (wide && idx->NB > 32 && nq > 32 && R <= 100 && listed < 2.0 * L) return false;
    if (listed <= 64.0) return true;
    if (nq > 64 && R > 128 && !(L < 16 && R <= 200)) return false;
    if (all) return nq * listed <= R * (L >= 100 ? 44.0 : wide && idx->NB <= 32 ? 32.0 : 20.0);
    return wide || idx->NB <= 32 || L < 16 || nq * R <= 10000;
}

// AVQ_ENOMEM, with nothing launched, where there is no room for the scratch: 2 KB a result and query, for the points of the
// listed blocks (64 queries, 512 results: 67 MB), and 16 bytes a block and query.
static int search_leaves_small(avq_index *idx, const float *queries, int nq, int k, int reorder_k, int R, int L, bool u8,
                               int32_t *ids_out, float *scores_out, hipStream_t st)
{
    const avq_config &c = idx->cfg;
    const int ns = (R + 63) / 64;
    // a few queries: every workgroup computes the short fp32 tables itself (one launch less); more: the table kernel
    const bool fuse_tables = nq <= 4 && small_batch_can_fuse_tables(c.bits, c.M, c.d, u8);
    const int64_t stride = std::min<int64_t>(idx->n_blocks, (int64_t)L * std::max<int64_t>(1, idx->max_leaf_blocks));
    // scratch, 256-byte aligned pieces of idx->tmp
    size_t off = 0;
    auto take = [&](size_t bytes) -> size_t { const size_t at = (off + 255) & ~(size_t)255; off = at + bytes; return at; };
    const size_t entries = (size_t)nq * c.M * idx->kc;
    const size_t o_lut = take(entries * sizeof(float)), o_lut8 = take(entries), o_scale = take(sizeof(float) * (size_t)nq),
                 o_bias = take(sizeof(float) * (size_t)nq), o_best = take(sizeof(u64) * (size_t)nq * stride),
                 o_blk = take(sizeof(int32_t) * (size_t)nq * stride), o_ip = take(sizeof(float) * (size_t)nq * stride),
                 o_n = take(sizeof(uint32_t) * (size_t)nq), o_sel = take(sizeof(int32_t) * (size_t)nq * R),
                 o_meta = take(sizeof(SmallMeta) * (size_t)nq), o_cand = take(sizeof(u64) * (size_t)nq * 256 * R),
                 o_keys = take(sizeof(u64) * (size_t)nq * c.n_leaves);
    if (idx->product.limit != 0 && off > idx->product.limit) { set_error("%zu bytes of scratch exceed the limit", off); return AVQ_ENOMEM; }
    AVQ_TRY(idx->tmp.reserve(off));
    unsigned char *base = (unsigned char *)idx->tmp.p;
    AVQ_TRY(idx->leaf_ids.reserve(sizeof(int32_t) * (size_t)nq * L));
    AVQ_TRY(idx->leaf_ip.reserve(sizeof(float) * (size_t)nq * L));
    {
        StageTimer t(idx, AVQ_STAGE_LEAF, st);
        AVQ_TRY(launch_leaf_select_few(idx->centers_t.as<float>(), c.n_leaves, c.d, queries, nq, L, (u64 *)(base + o_keys),
                                       idx->leaf_ids.as<int32_t>(), idx->leaf_ip.as<float>(), st));
    }
    ScanParams p;
    fill_scan_params(idx, nq, R, ns, &p);
    p.lut = (float *)(base + o_lut);
    p.lut8 = base + o_lut8;
    p.scale = (float *)(base + o_scale);
    p.bias = (float *)(base + o_bias);
    if (fuse_tables) {
        p.fuse_queries = queries;
        p.fuse_codebooks = idx->codebooks.as<float>();
        p.fuse_d = c.d;
    } else {
        StageTimer t(idx, AVQ_STAGE_LUT, st);
        AVQ_TRY(launch_lut(queries, nq, idx->codebooks.as<float>(), c.d, c.M, idx->kc, (float *)(base + o_lut),
                           u8 ? base + o_lut8 : nullptr, (float *)(base + o_scale), (float *)(base + o_bias), st));
    }
    p.perm = idx->perm.as<int32_t>();
    p.leaf_ids = idx->leaf_ids.as<int32_t>();
    p.leaf_ip = idx->leaf_ip.as<float>();
    p.leaf_blk = idx->leaf_blk.as<int32_t>();
    p.Lp = L;
    LeafSmallBuffers b;
    b.best = (u64 *)(base + o_best);
    b.blk = (int32_t *)(base + o_blk);
    b.ip = (float *)(base + o_ip);
    b.n_listed = (uint32_t *)(base + o_n);
    b.stride = stride;
    FinishParams f;
    memset(&f, 0, sizeof(f));
    f.x = idx->x;
    f.queries = queries;
    f.d = c.d;
    f.k = k;
    f.reorder = reorder_k != 0;
    f.stage_rows = small_finish_stage_rows(p, c.d, u8);
    f.cand_stride = (int64_t)256 * R;
    f.cand = (u64 *)(base + o_cand);
    f.sel_blk = (int32_t *)(base + o_sel);
    f.meta = (SmallMeta *)(base + o_meta);
    f.ids_out = ids_out;
    f.scores_out = scores_out;
    {
        StageTimer t(idx, AVQ_STAGE_SCAN, st);
        AVQ_TRY(launch_leaf_block_max(p, u8, b, st));
    }
    {
        StageTimer t(idx, AVQ_STAGE_MERGE, st);
        AVQ_TRY(launch_select_listed_blocks(p, f, b, st));
    }
    {
        StageTimer t(idx, AVQ_STAGE_RESCAN, st);
        AVQ_TRY(launch_rescan_leaf_blocks(p, f, u8, b, st));
    }
    StageTimer t(idx, AVQ_STAGE_FINAL, st);
    return launch_small_final(p, f, false, st); // keys carry fp32 scores with either kind of table
}

extern "C" int avq_search(avq_index *idx, const float *queries, int32_t nq, int32_t k, int32_t reorder_k,
                          int32_t lut_mode, int32_t leaves_to_search, int32_t *ids_out, float *scores_out,
                          void *hip_stream)
{
    AVQ_TRY(check_search_args(idx, queries, nq, k, reorder_k, lut_mode, leaves_to_search, ids_out, scores_out));
    hipStream_t st = (hipStream_t)hip_stream;
    const avq_config &c = idx->cfg;
    const bool ivf = c.n_leaves > 0;
    const int R = reorder_k ? reorder_k : k;
    const int ns = (R + 63) / 64;
    const int C = 64 * ns;
    const bool u8 = lut_mode == AVQ_LUT_U8;

    // 4-bit codes: the block-maxima path costs about 4.5 us per query and million points, the batch scans a fixed
    // 0.2 ms per million points up to a few hundred queries: measured crossover near 36 queries
    // 8-bit codes: a query by itself costs a scan of its own, sixteen share one (byte tables side by side), which takes four
    // times as long (single_us, tile_us)
    // 4-bit codes: the per-query path costs about 40 us + (0.1 + 0.00093 x blocks) us per query, the batch path
    // 150 us + 0.017 us per block up to a few hundred queries -- or 600 us on an index so small that its bounds
    // cannot be guessed from the class maxima of a sample and sorted lists take nearly every point. Measured
    // crossovers: 36 to 44 queries at 1.2 million points, 20 at 10 million, about 200 at 100,000, thousands at
    // 10,000 points.
    int small_max = c.bits == 4 ? (idx->n_blocks < 12000 ? 35 : 20) : 8; // code sizes without kernels of their own: as measured at first
    bool guessed = false; // whether the matrix-core scan of this batch would guess its bounds from class maxima
    if (c.bits == 4 && small_uses_bounds(idx)) {
        const double nb = (double)idx->n_blocks;
        double batch_us = 150.0 + 0.017 * nb;
        ScanParams plan, sample;
        fill_scan_params(idx, nq, R, ns, &plan);
        scan_mfma_plan(nq, idx->n_blocks, idx->tune_target_wgs, &plan);
        guessed = scan_mfma_sample_plan(plan, &sample) && sample.n_chunks * 32 >= 8 * sample.R && sample.n_chunks * 32 <= 8192;
        if (!guessed) batch_us = 600.0;
        small_max = (int)std::min(4096.0, std::max(8.0, (batch_us - 40.0) / (0.1 + 0.00093 * nb)));
    }
    if (c.bits == 8 && block_bound_supported(idx->NB, c.bits) && idx->tune_small_impl == 0)
        // (more than 200 results: as measured at first, 24 queries at 1.2 million points, two in any case)
        small_max = R > 200 ? (int)std::min<int64_t>(32, std::max<int64_t>(2, 120000 / std::max<int64_t>(1, idx->n_blocks)))
                            : nq <= 2 || (nq <= 32 && single_us(idx, nq, R) <= tile_us(idx, nq, R, u8)) ? nq : 0;
    if (idx->tune_small_batch >= 0) small_max = idx->tune_small_batch;
    const bool product = use_product(idx, nq, R, u8, small_max, guessed);
    const bool small = !ivf && !product && nq <= small_max;
    // the single-query kernels compute short fp32 tables themselves (one launch less)
    const bool fuse_tables = small && idx->tune_small_impl != 1 && small_batch_can_fuse_tables(c.bits, c.M, c.d, u8);
    const bool prefilter = !small && use_prefilter(idx, nq, lut_mode, R);
    if (ivf && use_product_leaves(idx, nq, leaves_to_search, R, u8)) {
        int per = 0;
        AVQ_TRY(product_part(idx, nq, R, ns, leaves_to_search, u8, &per));
        const int rc = product_in_parts(idx, nq, per, [&](int q0, int m, bool first) {
            return search_leaves_product(idx, queries + (size_t)q0 * c.d, m, k, reorder_k, R, ns, leaves_to_search, u8, first,
                                         ids_out + (size_t)q0 * k, scores_out + (size_t)q0 * k, st);
        });
        if (rc != AVQ_ENOMEM) return rc;
    }
    const bool grouped = ivf && use_grouped_leaves(idx, nq, leaves_to_search, R);
    if (ivf && use_leaf_small(idx, nq, leaves_to_search, R)) {
        const int rc = search_leaves_small(idx, queries, nq, k, reorder_k, R, leaves_to_search, u8, ids_out, scores_out, st);
        if (rc != AVQ_ENOMEM) return rc; // the list scan needs less
    }
    if (small && idx->tune_small_impl != 1) {
        SmallWs w;
        AVQ_TRY(small_ws_from_index(idx, nq, R, &w));
        return search_small(idx, queries, nq, k, reorder_k, u8, fuse_tables, w, true, ids_out, scores_out, st);
    }
    if (product) {
        int per = 0;
        AVQ_TRY(product_part(idx, nq, R, ns, 0, u8, &per));
        const int rc = product_in_parts(idx, nq, per, [&](int q0, int m, bool first) {
            return search_product(idx, queries + (size_t)q0 * c.d, m, k, reorder_k, R, ns, u8, first, ids_out + (size_t)q0 * k,
                                  scores_out + (size_t)q0 * k, st);
        });
        if (rc != AVQ_ENOMEM) return rc;
    }
    // Batches of 8-bit codes on a flat index: the same search through block bounds, the full scan taking the queries
    // sixteen at a time (byte tables of eight or seven bits); "scan_prefilter" = 1 scores every point instead
    if (!ivf && !small && c.bits == 8 && idx->tune_prefilter != 1 && small_uses_bounds(idx)) {
        SmallWs w;
        AVQ_TRY(small_ws_from_index(idx, nq, R, &w));
        return search_small(idx, queries, nq, k, reorder_k, u8, false, w, true, ids_out, scores_out, st, true);
    }
    if (!fuse_tables) {
        StageTimer t(idx, AVQ_STAGE_LUT, st);
        AVQ_TRY(build_tables(idx, queries, nq, (prefilter || grouped) ? AVQ_LUT_U8 : lut_mode, st));
    }
    if (grouped) return search_leaves_grouped(idx, queries, nq, k, reorder_k, R, ns, leaves_to_search, u8, ids_out, scores_out, st);
    if (prefilter) return search_through_candidates(idx, queries, nq, k, reorder_k, R, ns, false, ids_out, scores_out, st);
    ScanParams p;
    fill_scan_params(idx, nq, R, ns, &p);
    const int key_kind = (u8 && !ivf) ? 1 : 0;
    if (small) {
        // three-kernel variant of the same algorithm (kept as a cross-check)
        AVQ_TRY(idx->block_max.reserve(sizeof(u64) * (size_t)nq * idx->n_blocks));
        AVQ_TRY(idx->cand.reserve(sizeof(u64) * (size_t)nq * C));
        AVQ_TRY(idx->partial.reserve(sizeof(u64) * (size_t)nq * C));
        p.block_max = idx->block_max.as<u64>();
        p.block_keys = idx->cand.as<u64>();
        p.partial = idx->partial.as<u64>();
        p.n_tiles = nq;
        p.n_chunks = 1;
        p.max_wgs = idx->tune_target_wgs;
        {
            StageTimer t(idx, AVQ_STAGE_SCAN, st);
            AVQ_TRY(launch_block_max(p, u8, idx->tune_waves > 0 ? idx->tune_waves : 4, st));
        }
        {
            StageTimer t(idx, AVQ_STAGE_MERGE, st);
            AVQ_TRY(launch_select_keys(p.block_max, nq, idx->n_blocks, ns, R, idx->cand.as<u64>(), st));
        }
        ScanShape shape;
        int rc = AVQ_EINVAL;
        for (int w16 = 16; w16 >= 1 && rc != AVQ_OK; w16 /= 2) rc = scan_pick_shape(idx->NB, idx->cfg.bits, u8, ns, nq, true, 1, w16, &shape);
        AVQ_TRY(rc);
        {
            StageTimer t(idx, AVQ_STAGE_RESCAN, st);
            AVQ_TRY(launch_scan(p, u8, SCAN_BLOCKLIST, shape, st));
        }
        StageTimer t(idx, AVQ_STAGE_FINAL, st);
        return launch_finalize(p.partial, ns, nq, R, k, reorder_k != 0, key_kind, idx->x, c.d, queries,
                               idx->scale.as<float>(), idx->bias.as<float>(), ids_out, scores_out, st);
    }
    if (use_mfma_scan(idx, nq, lut_mode) && idx->tune_prefilter != 1 && c.M <= 64 && idx->n > R && mfma_scan_samples(idx, nq, R, ns))
        return search_through_candidates(idx, queries, nq, k, reorder_k, R, ns, true, ids_out, scores_out, st);
    if (use_mfma_scan(idx, nq, lut_mode)) {
        // 4-bit codes, 8-bit tables, flat index: the table sums are a one-hot contraction on the matrix cores
        scan_mfma_plan(nq, idx->n_blocks, idx->tune_target_wgs, &p);
        AVQ_TRY(idx->partial.reserve(sizeof(u64) * (size_t)nq * p.n_chunks * C));
        AVQ_TRY(idx->lists.reserve(scan_mfma_lists_bytes(p)));
        const size_t thr_bytes = sizeof(uint32_t) * (size_t)nq * (1 + (size_t)p.n_chunks);
        AVQ_TRY(idx->thr.reserve(thr_bytes));
        p.partial = idx->partial.as<u64>();
        p.lists_ws = idx->lists.as<u64>();
        p.thr_shared = idx->thr.as<uint32_t>();
        p.kth_shared = p.thr_shared + nq;
        {
            StageTimer t(idx, AVQ_STAGE_SCAN, st);
            AVQ_HIP(hipMemsetAsync(p.thr_shared, 0, thr_bytes, st));
            AVQ_TRY(launch_scan_mfma(p, st));
        }
        const u64 *cand = p.partial;
        if (p.n_chunks > 1) {
            AVQ_TRY(idx->cand.reserve(sizeof(u64) * (size_t)nq * C));
            StageTimer t(idx, AVQ_STAGE_MERGE, st);
            AVQ_TRY(launch_merge_partials(p.partial, nq, p.n_chunks, ns, idx->cand.as<u64>(), st));
            cand = idx->cand.as<u64>();
        }
        StageTimer t(idx, AVQ_STAGE_FINAL, st);
        return launch_finalize(cand, ns, nq, R, k, reorder_k != 0, key_kind, idx->x, c.d, queries,
                               idx->scale.as<float>(), idx->bias.as<float>(), ids_out, scores_out, st);
    }
    ScanShape shape;
    // few queries on a partitioned index: sixteen waves per workgroup and several workgroups per query
    const int waves_hint = idx->tune_waves > 0 ? idx->tune_waves : (ivf && nq <= 64 ? 16 : 0);
    if (scan_pick_shape(idx->NB, idx->cfg.bits, u8, ns, nq, ivf, idx->tune_qt, waves_hint, &shape) != AVQ_OK)
        AVQ_TRY(scan_pick_shape(idx->NB, idx->cfg.bits, u8, ns, nq, ivf, idx->tune_qt, idx->tune_waves, &shape));
    if (ivf) {
        const int L = leaves_to_search;
        AVQ_TRY(idx->leaf_ids.reserve(sizeof(int32_t) * (size_t)nq * L));
        AVQ_TRY(idx->leaf_ip.reserve(sizeof(float) * (size_t)nq * L));
        {
            StageTimer t(idx, AVQ_STAGE_LEAF, st);
            AVQ_TRY(launch_leaf_select(idx->centers_t.as<float>(), c.n_leaves, c.d, queries, nq, L,
                                       idx->leaf_ids.as<int32_t>(), idx->leaf_ip.as<float>(), st));
        }
        p.perm = idx->perm.as<int32_t>();
        p.leaf_ids = idx->leaf_ids.as<int32_t>();
        p.leaf_ip = idx->leaf_ip.as<float>();
        p.leaf_blk = idx->leaf_blk.as<int32_t>();
        p.Lp = L;
        p.n_tiles = nq;
        // about one leaf per wave when the batch alone cannot fill the chip
        const int target = idx->tune_target_wgs > 0 ? idx->tune_target_wgs : 512;
        int chunks = target / nq;
        const int max_chunks = (L + shape.waves - 1) / shape.waves;
        p.n_chunks = std::max(1, std::min(chunks, max_chunks));
    } else {
        plan_flat(idx, shape, nq, &p);
    }
    AVQ_TRY(idx->partial.reserve(sizeof(u64) * (size_t)p.n_tiles * shape.qt * p.n_chunks * C));
    p.partial = idx->partial.as<u64>();
    if (shape.lists_global) {
        AVQ_TRY(idx->lists.reserve(sizeof(u64) * (size_t)p.n_tiles * p.n_chunks * shape.waves * shape.qt * C));
        p.lists_ws = idx->lists.as<u64>();
    }
    {
        StageTimer t(idx, AVQ_STAGE_SCAN, st);
        AVQ_TRY(launch_scan(p, u8, ivf ? SCAN_LEAVES : SCAN_CHUNK, shape, st));
    }
    const u64 *cand = p.partial;
    if (p.n_chunks > 1) {
        AVQ_TRY(idx->cand.reserve(sizeof(u64) * (size_t)nq * C));
        StageTimer t(idx, AVQ_STAGE_MERGE, st);
        AVQ_TRY(launch_merge_partials(p.partial, nq, p.n_chunks, ns, idx->cand.as<u64>(), st));
        cand = idx->cand.as<u64>();
    }
    StageTimer t(idx, AVQ_STAGE_FINAL, st);
    return launch_finalize(cand, ns, nq, R, k, reorder_k != 0, key_kind, idx->x, c.d, queries,
                           idx->scale.as<float>(), idx->bias.as<float>(), ids_out, scores_out, st);
}

// ---- the entry point that allocates nothing ---------------------------------------------
// Device scratch of avq_search_noalloc: one array per GPU, part of the library's code object,
// held from the moment the library is loaded on that GPU until the process ends. In host code
// the array's name only stands for the symbol; the address on the current device comes from
// hipGetSymbolAddress and is looked up once per device.
static __device__ __align__(256) unsigned char scratch[AVQ_NOALLOC_SCRATCH_BYTES];
constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mutex;
static unsigned char *g_scratch_ptr[kMaxDevices] = {};

static int noalloc_scratch(unsigned char **out)
{
    int dev = -1;
    AVQ_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) { set_error("avq_search_noalloc: device %d not supported", dev); return AVQ_EINVAL; }
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        unsigned char *ptr = nullptr;
        AVQ_HIP(hipGetSymbolAddress((void **)&ptr, HIP_SYMBOL(scratch)));
        if (!ptr) { set_error("avq_search_noalloc: no address for the scratch array"); return AVQ_EHIP; }
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return AVQ_OK;
}

extern "C" int avq_search_noalloc(avq_index *idx, const float *queries, int32_t nq, int32_t k, int32_t reorder_k,
                                  int32_t lut_mode, int32_t *ids_out, float *scores_out, void *hip_stream)
{
    AVQ_TRY(check_index(idx));
    const avq_config &c = idx->cfg;
    if (c.n_leaves > 0) { set_error("avq_search_noalloc: flat index only"); return AVQ_EINVAL; }
    AVQ_TRY(check_search_args(idx, queries, nq, k, reorder_k, lut_mode, 0, ids_out, scores_out));
    if (nq > AVQ_NOALLOC_MAX_QUERIES) {
        set_error("avq_search_noalloc: at most %d queries per call (got %d)", AVQ_NOALLOC_MAX_QUERIES, nq);
        return AVQ_EINVAL;
    }
    const int R = reorder_k ? reorder_k : k;
    const bool u8 = lut_mode == AVQ_LUT_U8;
    SmallWs w;
    const size_t need = small_ws_carve(idx, nq, R, nullptr, &w);
    if (need > (size_t)AVQ_NOALLOC_SCRATCH_BYTES) {
        set_error("avq_search_noalloc: %d queries x %lld points with reorder_k %d need %zu bytes of scratch, the library holds %zu",
                  nq, (long long)idx->n, reorder_k, need, (size_t)AVQ_NOALLOC_SCRATCH_BYTES);
        return AVQ_EINVAL;
    }
    if ((size_t)idx->NB * 256 * 4 > kMaxDynLds && !(c.bits == 4 && (size_t)c.M * 64 <= 60 * 1024)) {
        set_error("avq_search_noalloc: the tables of this index do not fit the single-query kernels");
        return AVQ_EINVAL;
    }
    unsigned char *base = nullptr;
    AVQ_TRY(noalloc_scratch(&base));
    small_ws_carve(idx, nq, R, base, &w);
    const bool fuse_tables = small_batch_can_fuse_tables(c.bits, c.M, c.d, u8);
    return search_small(idx, queries, nq, k, reorder_k, u8, fuse_tables, w, false, ids_out, scores_out, (hipStream_t)hip_stream);
}

extern "C" int avq_brute_force(avq_index *idx, const float *queries, int32_t nq, int32_t k,
                               int32_t *ids_out, float *scores_out, void *hip_stream)
{
    AVQ_TRY(check_index(idx));
    if (idx->n <= 0 || !idx->x) { set_error("avq_brute_force: no datapoints stored"); return AVQ_ESTATE; }
    if (!queries || nq < 1 || !ids_out || !scores_out || k < 1 || k > AVQ_MAX_SELECT || k > idx->n) {
        set_error("avq_brute_force: bad argument");
        return AVQ_EINVAL;
    }
    hipStream_t st = (hipStream_t)hip_stream;
    const int d = idx->cfg.d, ns = (k + 63) / 64;
    bool product = exact_supported(idx->n, d, nq, k);
    int per = nq;
    if (product) {
        const size_t most = exact_scratch(idx->n, d);
        per = exact_queries_per_launch(idx->n, d, nq, idx->exact_ws.limit ? std::min(most, idx->exact_ws.limit) : most);
        const int rc = idx->exact_ws.reserve(exact_ws_bytes(idx->n, d, per));
        if (rc == AVQ_ENOMEM) { product = false; per = nq; } // the plain kernel needs none of it
        else AVQ_TRY(rc);
    }
    const int chunks = brute_force_chunks(idx->n, per);
    AVQ_TRY(idx->partial.reserve(sizeof(u64) * (size_t)per * chunks * 64 * ns));
    AVQ_TRY(idx->cand.reserve(sizeof(u64) * (size_t)per * 64 * ns));
    for (int q0 = 0; q0 < nq; q0 += per) {
        const int m = std::min(per, nq - q0);
        const float *qs = queries + (size_t)q0 * d;
        int32_t *ids = ids_out + (size_t)q0 * k;
        float *scores = scores_out + (size_t)q0 * k;
        const uint32_t *need = nullptr; // without the product every query is answered by the plain kernel
        if (product) AVQ_TRY(launch_exact(idx->x, idx->n, d, qs, m, k, idx->exact_ws.p, ids, scores, &need, st));
        AVQ_TRY(launch_brute_force(idx->x, idx->n, d, qs, m, k, idx->partial.as<u64>(), chunks, idx->cand.as<u64>(), ids, scores, st, need));
    }
    return AVQ_OK;
}

// ---- stage-level inspection -------------------------------------------------------------

extern "C" int avq_debug_lut(avq_index *idx, const float *queries, int32_t nq, int32_t lut_mode,
                             void *lut_out, float *scale_out, float *bias_out, void *hip_stream)
{
    AVQ_TRY(check_index(idx));
    if (!idx->have_codebooks) { set_error("avq_debug_lut: no dictionaries yet"); return AVQ_ESTATE; }
    if (!queries || nq < 1 || !lut_out) { set_error("avq_debug_lut: bad argument"); return AVQ_EINVAL; }
    if (lut_mode != AVQ_LUT_F32 && lut_mode != AVQ_LUT_U8) { set_error("bad lut_mode"); return AVQ_EINVAL; }
    if (lut_mode == AVQ_LUT_U8 && (!scale_out || !bias_out)) { set_error("avq_debug_lut: scale/bias NULL"); return AVQ_EINVAL; }
    hipStream_t st = (hipStream_t)hip_stream;
    const avq_config &c = idx->cfg;
    if (lut_mode == AVQ_LUT_F32)
        return launch_lut(queries, nq, idx->codebooks.as<float>(), c.d, c.M, idx->kc, (float *)lut_out, nullptr,
                          nullptr, nullptr, st);
    return launch_lut(queries, nq, idx->codebooks.as<float>(), c.d, c.M, idx->kc, nullptr, (uint8_t *)lut_out,
                      scale_out, bias_out, st);
}

extern "C" int avq_debug_adc_scores(avq_index *idx, const float *queries, int32_t nq, int32_t lut_mode,
                                    void *scores_out, void *hip_stream)
{
    AVQ_TRY(check_index(idx));
    AVQ_TRY(check_query_args(idx, queries, nq, lut_mode));
    if (idx->cfg.n_leaves > 0) { set_error("avq_debug_adc_scores: flat index only"); return AVQ_ESTATE; }
    if (!scores_out) { set_error("avq_debug_adc_scores: NULL output"); return AVQ_EINVAL; }
    hipStream_t st = (hipStream_t)hip_stream;
    const bool u8 = lut_mode == AVQ_LUT_U8;
    AVQ_TRY(build_tables(idx, queries, nq, lut_mode, st));
    ScanParams p;
    fill_scan_params(idx, nq, 1, 2, &p);
    if (use_mfma_scan(idx, nq, lut_mode)) {
        scan_mfma_plan(nq, idx->n_blocks, idx->tune_target_wgs, &p);
        p.scores_out = scores_out;
        p.score_stride = idx->n;
        return launch_scan_mfma(p, st);
    }
    ScanShape shape;
    AVQ_TRY(scan_pick_shape(idx->NB, idx->cfg.bits, u8, 2, nq, false, idx->tune_qt, idx->tune_waves, &shape));
    plan_flat(idx, shape, nq, &p);
    p.scores_out = scores_out;
    p.score_stride = idx->n;
    AVQ_TRY(idx->partial.reserve(64));
    p.partial = idx->partial.as<u64>();
    if (shape.lists_global) {
        AVQ_TRY(idx->lists.reserve(sizeof(u64) * (size_t)p.n_tiles * p.n_chunks * shape.waves * shape.qt * 128));
        p.lists_ws = idx->lists.as<u64>();
    }
    return launch_scan(p, u8, SCAN_CHUNK, shape, st);
}

extern "C" int avq_debug_stream_codes(avq_index *idx, uint32_t *words_out, int64_t *n_blocks_out, void *hip_stream)
{
    AVQ_TRY(check_index(idx));
    if (idx->n <= 0) { set_error("avq_debug_stream_codes: no codes yet"); return AVQ_ESTATE; }
    if (n_blocks_out) *n_blocks_out = idx->n_blocks;
    if (!words_out) return AVQ_OK;
    return launch_stream_codes(idx->codes_blocked.as<uint8_t>(), idx->n_blocks, idx->NB, words_out, (hipStream_t)hip_stream,
                               stream_loads_nontemporal(idx, 1));
}

extern "C" int avq_debug_scan_parts(avq_index *idx, const float *queries, int32_t nq, int32_t lut_mode, int32_t part,
                                    int32_t reps, void *hip_stream)
{
    AVQ_TRY(check_index(idx));
    AVQ_TRY(check_query_args(idx, queries, nq, lut_mode));
    if (idx->cfg.n_leaves > 0) { set_error("avq_debug_scan_parts: flat index only"); return AVQ_ESTATE; }
    if (part < 0 || part > 2 || reps < 1 || nq > 64) { set_error("avq_debug_scan_parts: bad argument"); return AVQ_EINVAL; }
    hipStream_t st = (hipStream_t)hip_stream;
    const avq_config &c = idx->cfg;
    const bool u8 = lut_mode == AVQ_LUT_U8;
    const bool bounds = small_uses_bounds(idx);
    if (part == 2 && !bounds) { set_error("avq_debug_scan_parts: no lookup-only kernel for this code size"); return AVQ_EINVAL; }
    SmallWs w;
    AVQ_TRY(small_ws_from_index(idx, nq, 1, &w));
    const bool fuse_tables = small_batch_can_fuse_tables(c.bits, c.M, c.d, u8);
    if (!fuse_tables)
        AVQ_TRY(launch_lut(queries, nq, idx->codebooks.as<float>(), c.d, c.M, idx->kc, w.lut, u8 ? w.lut8 : nullptr, w.scale,
                           w.bias, st));
    ScanParams p;
    fill_scan_params(idx, nq, 1, 1, &p);
    p.lut = w.lut; p.lut8 = w.lut8; p.scale = w.scale; p.bias = w.bias;
    if (fuse_tables) { p.fuse_queries = queries; p.fuse_codebooks = idx->codebooks.as<float>(); p.fuse_d = c.d; }
    p.block_max = w.block_max;
    p.block_bound = w.block_bound;
    p.bound_meta = w.bound_meta;
    p.bound_tbl = w.bound_tbl;
    p.lut_out = fuse_tables ? w.lut : nullptr;
    p.n_tiles = nq;
    p.n_chunks = 1;
    p.max_wgs = idx->tune_target_wgs;
    p.nt_loads = stream_loads_nontemporal(idx, nq) ? 1 : 0;
    if (bounds) AVQ_TRY(launch_bound_tables(p, u8, st));
    for (int r = 0; r < reps; ++r) {
        if (part == 1) AVQ_TRY(launch_stream_codes(idx->codes_blocked.as<uint8_t>(), idx->n_blocks, idx->NB, (uint32_t *)w.block_max, st, stream_loads_nontemporal(idx, nq)));
        else if (bounds) AVQ_TRY(launch_block_bound(p, idx->tune_waves, st, part == 2));
        else AVQ_TRY(launch_block_max(p, u8, idx->tune_waves > 0 ? idx->tune_waves : 4, st));
    }
    return AVQ_OK;
}

extern "C" int avq_debug_unverified_queries(avq_index *idx, int32_t *counts_out)
{
    AVQ_TRY(check_index(idx));
    if (!counts_out) { set_error("avq_debug_unverified_queries: NULL"); return AVQ_EINVAL; }
    counts_out[0] = -1;
    counts_out[1] = counts_out[2] = counts_out[3] = 0;
    if (!idx->fail.p) return AVQ_OK;
    AVQ_HIP(hipDeviceSynchronize());
    uint32_t c[4] = {0, 0, 0, 0};
    AVQ_HIP(hipMemcpy(c, idx->fail.p, sizeof(c), hipMemcpyDeviceToHost));
    for (int i = 0; i < 4; ++i) counts_out[i] = (int32_t)c[i];
    return AVQ_OK;
}

extern "C" int avq_debug_leaf_select(avq_index *idx, const float *queries, int32_t nq, int32_t L,
                                     int32_t *leaf_ids_out, float *leaf_ip_out, void *hip_stream)
{
    AVQ_TRY(check_index(idx));
    const avq_config &c = idx->cfg;
    if (c.n_leaves <= 0 || !idx->have_centers) { set_error("avq_debug_leaf_select: no leaf centers"); return AVQ_ESTATE; }
    if (!queries || nq < 1 || !leaf_ids_out || !leaf_ip_out || L < 1 || L > c.n_leaves || L > AVQ_MAX_SELECT) {
        set_error("avq_debug_leaf_select: bad argument");
        return AVQ_EINVAL;
    }
    if (nq <= 32) { // the kernels the few-query search uses
        AVQ_TRY(idx->tmp.reserve(sizeof(u64) * (size_t)nq * c.n_leaves));
        return launch_leaf_select_few(idx->centers_t.as<float>(), c.n_leaves, c.d, queries, nq, L, (u64 *)idx->tmp.p,
                                      leaf_ids_out, leaf_ip_out, (hipStream_t)hip_stream);
    }
    return launch_leaf_select(idx->centers_t.as<float>(), c.n_leaves, c.d, queries, nq, L, leaf_ids_out,
                              leaf_ip_out, (hipStream_t)hip_stream);
}
