// Host side of the C ABI declared in include/sj.h: argument checking, memory ownership, weight
// upload / re-tiling, and the kernel sequence of one verification step.
#include "../../include/sj.h"
#include "sj_kernels.h"
#include "sj_plan.h"
#include "sj_attn.h"
#include "sj_attn_rows.h"
#include "sj_gemm_rows.h"
#include "sj_gemm_tile.h"
#include "sj_gemm_ring.h"

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <memory>
#include <mutex>
#include <string>
#include <type_traits>
#include <vector>

using namespace sj;

// ------------------------------------------------------------------------------------------------
// errors

static thread_local std::string g_err;

static int fail(int code, const char* fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_err = buf;
    return code;
}

#define HIPCHK(expr)                                                                              \
    do {                                                                                          \
        hipError_t e_ = (expr);                                                                   \
        if (e_ != hipSuccess) return fail(SJ_EHIP, "%s failed: %s", #expr, hipGetErrorString(e_)); \
    } while (0)

#define LAUNCHCHK(name)                                                                          \
    do {                                                                                         \
        hipError_t e_ = hipGetLastError();                                                       \
        if (e_ != hipSuccess) return fail(SJ_EHIP, "launch of %s failed: %s", name, hipGetErrorString(e_)); \
    } while (0)

// ------------------------------------------------------------------------------------------------
// objects

struct LayerW {
    void *attn_norm = nullptr, *wqkv = nullptr, *wo = nullptr, *ffn_norm = nullptr, *wgu = nullptr, *wd = nullptr;
};

struct TunedPlans;

struct sj_model {
    sj_config cfg{};
    ModelDims md{};
    size_t esz = 0;
    void *embed = nullptr, *final_norm = nullptr, *lm_head = nullptr, *judge_w = nullptr, *judge_b = nullptr;
    std::vector<LayerW> layers;
    std::vector<void*> allocs;
    int64_t weight_bytes = 0;
    int device = 0;
    unsigned temp_gen = 0;                     // bumped by sj_set_temperature: captured launch graphs carry the old value
    // launch shapes measured for this model, keyed by (rows, operand planes): a second cache object on the same
    // model reuses them, so two objects of one process run the same kernels (bit-identical results)
    mutable std::mutex tuned_mu;
    mutable std::map<std::pair<int, int>, std::shared_ptr<TunedPlans>> tuned;
};

struct TunedPlans { GemmPlan qkv, o, d, gu, lm; };

// Buffers of a forward over up to `rpad` rows: residual stream, operand planes, projection partials, rotary table.
struct Forward {
    int rpad = 0;
    size_t part_elems = 0;     // of `part`
    float *x = nullptr, *part = nullptr, *cs = nullptr, *ss = nullptr;
    void *xn = nullptr, *attn_out = nullptr, *act = nullptr;
    int32_t *row_tok = nullptr, *prefill_tok = nullptr;
};

enum class Product { qkv, o, down };          // the split-K projections
static Sums sums_of(Product p) { return p == Product::qkv ? Sums::attention : Sums::closing; }

struct sj_kv : Forward {       // the inherited buffers serve the blocks of up to max_gamma + 1 rows per sequence
    const sj_model* m = nullptr;
    int batch = 0, max_rows = 0, mpad = 0, cap_max = 64;
    Forward chunk;             // those of a prompt chunk of sj_prefill
    int pf_rows = 0;           // rows of one prompt chunk of sj_prefill (0: no buffers for them, chunks of max_gamma + 1 rows)
    std::vector<int32_t> cap, len_upper;
    std::vector<int64_t> seq_off;
    int64_t layer_stride = 0;
    void *K = nullptr, *V = nullptr;
    int64_t* seq_off_dev = nullptr;
    int32_t *cap_dev = nullptr, *len_dev = nullptr, *pending_dev = nullptr;
    // workspace
    StepParams* sp_dev = nullptr;
    float *hn32 = nullptr, *opart = nullptr, *logits = nullptr;
    float *scores = nullptr, *p_at_d = nullptr;
    int32_t* ranks = nullptr;        // [R] rank of every draft token in its target row (top-k mode)
    int topk = 2;
    unsigned* tickets = nullptr;
    unsigned* close_tickets = nullptr;            // of the split-K products that close a sub-layer: one per n-tile
    float4 *stats = nullptr, *rowstat = nullptr;
    int32_t *bits = nullptr, *nacc = nullptr, *draft_tok = nullptr;
    double *epart = nullptr, *wpart = nullptr, *eblk = nullptr, *wblk = nullptr;
    int chunk_keys = 64, nchunk_max = 1, nslab = 0, slab_len = 0;
    GemmPlan plan_qkv[2], plan_o[2], plan_d[2];   // [0]: few-row kernel (at most 32 rows), [1]: more
    const GemmPlan* plans(Product p) const { return p == Product::qkv ? plan_qkv : p == Product::o ? plan_o : plan_d; }
    GemmPlan plan_gu;                             // gate / up projection with few rows (no K-slices)
    GemmPlan plan_lm{8, 4, 1, 2};                 // LM head with few rows
    int few_rows = 1;                             // rows that the few-row shapes were made for
    int mode = SJ_MODE_TWO_STAGE;
    int ring_rows = RING_ROWS;            // the rules take the LDS-ring kernel up to this many rows
    int planes = 2;            // bf16 planes of the activation operand (fp32 storage: always 1)
    int32_t* pinned_state = nullptr;      // [2*batch] staging of sj_kv_rewind
    hipEvent_t rewind_done = nullptr;
    bool rewind_pending = false;
    // optional timing of one kernel class (eager launches only)
    // captured launch graphs of the full step, keyed by (gamma, planes)
    std::map<int, hipGraphExec_t> graphs;
    unsigned graph_gen = 0;               // temp_gen of the model the graphs were captured with
    hipStream_t cap_stream = nullptr;
    bool use_graph = true;
    int timing_class = 0;
    std::vector<hipEvent_t> tev;          // start/stop pairs
    size_t tev_used = 0;
    int last_gamma = 0, last_rows = 0;
    // judge scores, p(draft) and accept bits of the last call, max_rows words each, in host memory that the device writes: there from
    // the first sj_debug_fetch of one of them on
    mutable std::atomic<float*> mirror{nullptr};
    mutable std::mutex mirror_mu;
    bool mirrored = false;                // the last call wrote it
    bool captured = false;                // graphs of the caller hold verification calls: a replay writes results without the host knowing
    std::vector<void*> allocs;
};

static size_t esz_of(int dtype) { return dtype == SJ_DTYPE_FP32 ? 4 : 2; }

template <typename P> static int dev_alloc(std::vector<void*>& owner, P** p, size_t bytes, bool zero = true) {
    void* q = nullptr;
    if (bytes == 0) bytes = 256;
    hipError_t e = hipMalloc(&q, bytes);
    if (e != hipSuccess) return fail(e == hipErrorOutOfMemory ? SJ_ENOMEM : SJ_EHIP, "hipMalloc(%zu) failed: %s", bytes,
                                     hipGetErrorString(e));
    owner.push_back(q);
    if (zero) HIPCHK(hipMemset(q, 0, bytes));
    *p = reinterpret_cast<P*>(q);
    return SJ_OK;
}

static void free_all(std::vector<void*>& v) {
    for (void* p : v) (void)hipFree(p);
    v.clear();
}

// ------------------------------------------------------------------------------------------------
// model load

static int check_config(const sj_config* c) {
    if (!c) return fail(SJ_EINVAL, "config is null");
    if (c->dtype != SJ_DTYPE_FP32 && c->dtype != SJ_DTYPE_BF16) return fail(SJ_EINVAL, "dtype must be 0 (fp32) or 1 (bf16)");
    if (c->n_layers < 0 || c->d_model <= 0 || c->vocab <= 0) return fail(SJ_EINVAL, "non-positive model dimension");
    if (c->d_model % 64 || c->vocab % 128) return fail(SJ_EINVAL, "d_model must be a multiple of 64 and vocab of 128");
    if (c->d_model > 16384) return fail(SJ_EINVAL, "d_model above 16384 is not supported");
    if (c->max_gamma < 1 || c->max_gamma > 63) return fail(SJ_EINVAL, "max_gamma must be in 1..63");
    if (!(c->temperature >= 0.f)) return fail(SJ_EINVAL, "temperature must be >= 0");
    if (c->n_layers > 0) {
        if (c->n_q_heads <= 0 || c->n_kv_heads <= 0 || c->d_ffn <= 0) return fail(SJ_EINVAL, "non-positive model dimension");
        if (c->head_dim != 64 && c->head_dim != 128) return fail(SJ_EINVAL, "head_dim must be 64 or 128");
        if (c->n_q_heads % c->n_kv_heads) return fail(SJ_EINVAL, "n_q_heads must be a multiple of n_kv_heads");
        if (c->d_ffn % 64) return fail(SJ_EINVAL, "d_ffn must be a multiple of 64");
        if (!(c->rope_base > 1.f) || !(c->rms_eps >= 0.f)) return fail(SJ_EINVAL, "bad rope_base / rms_eps");
    }
    return SJ_OK;
}

namespace {
struct Loader {
    sj_model* m;
    sj_tensor_fn fn;
    void* user;
    void* host = nullptr;      // pinned staging
    void* dev = nullptr;       // device staging (source of the re-tile)
    size_t cap = 0;

    int fetch(int id, int layer, size_t off_bytes, size_t bytes) {
        if (off_bytes + bytes > cap) return fail(SJ_EINVAL, "internal: staging too small");
        if (fn(user, id, layer, (char*)host + off_bytes, bytes) != 0)
            return fail(SJ_ECALLBACK, "tensor provider failed for tensor %d layer %d", id, layer);
        return SJ_OK;
    }
    int plain(int id, int layer, size_t elems, void** out) {       // vectors, embedding: kept row-major
        const size_t bytes = elems * m->esz;
        int rc = fetch(id, layer, 0, bytes);
        if (rc) return rc;
        rc = dev_alloc(m->allocs, out, bytes, false);
        if (rc) return rc;
        HIPCHK(hipMemcpy(*out, host, bytes, hipMemcpyHostToDevice));
        return SJ_OK;
    }
    // one or more [n_i, K] matrices stacked along N, re-tiled into one device matrix
    int tiled(const int* ids, const int* ns, int count, int layer, int K, int interleave, void** out) {
        size_t off = 0;
        int N = 0;
        for (int i = 0; i < count; ++i) {
            const size_t bytes = (size_t)ns[i] * K * m->esz;
            int rc = fetch(ids[i], layer, off, bytes);
            if (rc) return rc;
            off += bytes;
            N += ns[i];
        }
        HIPCHK(hipMemcpy(dev, host, off, hipMemcpyHostToDevice));
        int rc = dev_alloc(m->allocs, out, off, false);
        if (rc) return rc;
        const int blocks = 4096;
        if (m->cfg.dtype == SJ_DTYPE_FP32)
            retile_kernel<float><<<blocks, 256>>>((const float*)dev, (float*)*out, N, K, interleave);
        else
            retile_kernel<bf16_t><<<blocks, 256>>>((const bf16_t*)dev, (bf16_t*)*out, N, K, interleave);
        LAUNCHCHK("retile");
        HIPCHK(hipDeviceSynchronize());
        m->weight_bytes += (int64_t)off;
        return SJ_OK;
    }
};
}  // namespace

extern "C" int sj_model_load(const sj_config* cfg, sj_tensor_fn provider, void* user, sj_model** out) {
    int rc = check_config(cfg);
    if (rc) return rc;
    if (!provider || !out) return fail(SJ_EINVAL, "provider / out is null");
    sj_model* m = new (std::nothrow) sj_model();
    if (!m) return fail(SJ_ENOMEM, "host allocation failed");
    m->cfg = *cfg;
    m->esz = esz_of(cfg->dtype);
    const int d = cfg->d_model, hd = cfg->head_dim, V = cfg->vocab, F = cfg->d_ffn;
    const int Nq = cfg->n_q_heads * hd, Nk = cfg->n_kv_heads * hd;
    ModelDims& md = m->md;
    md.d = d; md.Hq = cfg->n_q_heads; md.Hkv = cfg->n_kv_heads; md.hd = hd; md.F = F; md.V = V;
    md.G = cfg->n_layers > 0 ? cfg->n_q_heads / cfg->n_kv_heads : 1;
    md.eps = cfg->rms_eps;
    md.temperature = cfg->temperature;
    md.inv_temp = cfg->temperature > 0.f ? 1.0f / cfg->temperature : 0.f;
    md.scale = cfg->n_layers > 0 ? (float)(1.0 / std::sqrt((double)hd)) : 1.f;

    Loader ld{m, provider, user};
    size_t need = (size_t)V * d;
    if (cfg->n_layers > 0) need = std::max({need, (size_t)(Nq + 2 * Nk) * d, (size_t)2 * F * d});
    ld.cap = need * m->esz;
    auto cleanup = [&](int code) {
        if (ld.host) (void)hipHostFree(ld.host);
        if (ld.dev) (void)hipFree(ld.dev);
        if (code) { free_all(m->allocs); delete m; }
        return code;
    };
    if (hipGetDevice(&m->device) != hipSuccess) return cleanup(fail(SJ_EHIP, "no HIP device available"));
    {
        hipError_t e = hipHostMalloc(&ld.host, ld.cap, hipHostMallocDefault);
        if (e != hipSuccess) { ld.host = nullptr; return cleanup(fail(SJ_EHIP, "hipHostMalloc(%zu) failed: %s", ld.cap, hipGetErrorString(e))); }
        e = hipMalloc(&ld.dev, ld.cap);
        if (e != hipSuccess) { ld.dev = nullptr; return cleanup(fail(SJ_ENOMEM, "hipMalloc(%zu) failed: %s", ld.cap, hipGetErrorString(e))); }
    }
    m->layers.resize(cfg->n_layers);
    if (cfg->n_layers > 0) {
        if ((rc = ld.plain(SJ_T_EMBED, -1, (size_t)V * d, &m->embed))) return cleanup(rc);
        if ((rc = ld.plain(SJ_T_FINAL_NORM, -1, d, &m->final_norm))) return cleanup(rc);
    }
    for (int l = 0; l < cfg->n_layers; ++l) {
        LayerW& L = m->layers[l];
        if ((rc = ld.plain(SJ_T_ATTN_NORM, l, d, &L.attn_norm))) return cleanup(rc);
        if ((rc = ld.plain(SJ_T_FFN_NORM, l, d, &L.ffn_norm))) return cleanup(rc);
        const int qkv_ids[3] = {SJ_T_WQ, SJ_T_WK, SJ_T_WV}, qkv_ns[3] = {Nq, Nk, Nk};
        if ((rc = ld.tiled(qkv_ids, qkv_ns, 3, l, d, 0, &L.wqkv))) return cleanup(rc);
        const int o_id = SJ_T_WO, o_n = d;
        if ((rc = ld.tiled(&o_id, &o_n, 1, l, Nq, 0, &L.wo))) return cleanup(rc);
        const int gu_ids[2] = {SJ_T_W_GATE, SJ_T_W_UP}, gu_ns[2] = {F, F};
        if ((rc = ld.tiled(gu_ids, gu_ns, 2, l, d, 1, &L.wgu))) return cleanup(rc);
        const int d_id = SJ_T_W_DOWN, d_n = d;
        if ((rc = ld.tiled(&d_id, &d_n, 1, l, F, 0, &L.wd))) return cleanup(rc);
    }
    const int lm_id = SJ_T_LM_HEAD, lm_n = V;
    if ((rc = ld.tiled(&lm_id, &lm_n, 1, -1, d, 0, &m->lm_head))) return cleanup(rc);
    if ((rc = ld.plain(SJ_T_JUDGE_W, -1, d, &m->judge_w))) return cleanup(rc);
    if ((rc = ld.plain(SJ_T_JUDGE_B, -1, 1, &m->judge_b))) return cleanup(rc);
    cleanup(0);
    *out = m;
    return SJ_OK;
}

extern "C" int sj_model_free(sj_model* m) {
    if (!m) return fail(SJ_EINVAL, "model is null");
    free_all(m->allocs);
    delete m;
    return SJ_OK;
}

extern "C" int64_t sj_model_weight_bytes(const sj_model* m) { return m ? m->weight_bytes : 0; }

extern "C" int sj_set_temperature(sj_model* m, float temperature) {
    if (!m) return fail(SJ_EINVAL, "model is null");
    if (!(temperature >= 0.f)) return fail(SJ_EINVAL, "temperature must be >= 0");
    HIPCHK(hipDeviceSynchronize());                            // no step in flight still reads the old value
    m->cfg.temperature = temperature;
    m->md.temperature = temperature;
    m->md.inv_temp = temperature > 0.f ? 1.0f / temperature : 0.f;
    ++m->temp_gen;
    return SJ_OK;
}

// ------------------------------------------------------------------------------------------------
// kv / workspace

// Rows of one prompt chunk.  Every chunk streams all weights once, so a chunk should be so long that its work outweighs
// that: four row groups of the loader-wave kernel (the two-plane products of 576 rows take 5 x the time of the
// weight stream).
constexpr int PREFILL_ROWS = 4 * ROWS_MT * 16;

static int tune_plans(sj_kv* kv, int rows);

// The LM head's launch shape by the rule; planes of its operand: one for hidden states handed in by the caller of a head-only model.
static void rule_lm_head(sj_kv* kv, int planes) {
    const sj_config& c = kv->m->cfg;
    const bool bf16 = c.dtype == SJ_DTYPE_BF16;
    kv->few_rows = std::min(kv->max_rows, FEW_ROWS);
    kv->plan_lm = rule_logits(c.vocab / 16, c.d_model / (bf16 ? 32 : 16), kv->few_rows, planes, bf16, kv->ring_rows);
}

// the launch shapes the rule gives (before any measurement)
static void rule_plans(sj_kv* kv) {
    const sj_config& c = kv->m->cfg;
    const int d = c.d_model, hd = c.head_dim, Nq = c.n_q_heads * hd, Nk = c.n_kv_heads * hd, F = c.d_ffn;
    const bool bf16 = c.dtype == SJ_DTYPE_BF16;
    const int kstep = bf16 ? 32 : 16, planes = bf16 ? kv->planes : 1, rows = std::min(kv->max_rows, FEW_ROWS);
    // bf16 with one or two planes: the LDS-ring kernel where a shape of it fits (4 - 13 % faster than the register-ring kernel from 1 to 32 rows; the
    // start-up measurement may still prefer another shape).  SJ_RING_ROWS = 0..32 moves the row limit of this rule.
    if (const char* e = std::getenv("SJ_RING_ROWS")) kv->ring_rows = std::min(std::max(std::atoi(e), 0), RING_ROWS);
    auto partial = [&](GemmPlan (&plan)[2], int N, int K, Sums sums) {
        plan[0] = rule_partial(N / 16, K / kstep, rows, planes, bf16, kv->ring_rows, sums);
        plan[1] = plan_partial(N / 16, K / kstep, false);
    };
    partial(kv->plan_qkv, Nq + 2 * Nk, d, Sums::attention);
    partial(kv->plan_o, d, Nq, Sums::closing);
    partial(kv->plan_d, d, F, Sums::closing);
    kv->plan_gu = rule_gate_up(2 * F / 16, d / kstep, rows, planes, bf16, kv->ring_rows);
    rule_lm_head(kv, planes);
}

// fp32 elements of the projections' partials for blocks of up to `rows` rows; element offsets into them are 32-bit
constexpr size_t PART_LIMIT = (size_t)1 << 31;
static size_t forward_elems(const sj_kv* kv, int rows) {
    const sj_config& c = kv->m->cfg;
    const int d = c.d_model, Nq = c.n_q_heads * c.head_dim, Nk = c.n_kv_heads * c.head_dim, kstep = c.dtype == SJ_DTYPE_FP32 ? 16 : 32;
    return std::max({part_elems(kv->plan_qkv[1].split, Nq + 2 * Nk, d / kstep, rows), part_elems(kv->plan_o[1].split, d, Nq / kstep, rows),
                     part_elems(kv->plan_d[1].split, d, c.d_ffn / kstep, rows)});
}

// Buffers of a prompt chunk, as long as the longest sequence allows, up to PREFILL_ROWS: allocated with the cache object's first
// prompt of more than a block, so that objects which see none (draft and scoring caches filled by sj_kv_set) neither hold them (120 MB
// for the 8B shape) nor take the time (0.3 ms).  They are apart from those of the blocks (a block's planes then stay close together:
// with one set for both, the steps of small models took 3 % longer), in one allocation.  Where it does not fit, prompts go through in
// blocks of max_gamma + 1 rows.
static void get_chunk(sj_kv* kv) {
    const sj_model* m = kv->m;
    const sj_config& c = m->cfg;
    const int pf = std::min(PREFILL_ROWS, kv->cap_max), pad = (pf + 15) / 16 * 16;
    if (kv->pf_rows || pf <= c.max_gamma + 1) return;
    const size_t elems = forward_elems(kv, pf);
    if (elems >= PART_LIMIT) return;
    const int d = c.d_model, Nq = c.n_q_heads * c.head_dim;
    Forward& w = kv->chunk;
    char* base = nullptr;
    size_t used = 0;
    auto carve = [&](auto*& ptr, size_t bytes) {
        if (base) ptr = reinterpret_cast<std::remove_reference_t<decltype(ptr)>>(base + used);
        used = (used + bytes + 255) / 256 * 256;
    };
    for (int round = 0; round < 2; ++round) {                  // sizes first, then the pieces
        used = 0;
        carve(w.xn, (size_t)3 * pad * d * m->esz);
        carve(w.row_tok, (size_t)pf * 4);
        carve(w.x, (size_t)pf * d * 4);
        carve(w.part, elems * 4);
        carve(w.attn_out, (size_t)3 * pad * Nq * m->esz);
        // also holds the chunk's rotated query fragments (pad x Nq elements per plane) until the gate / up projection
        carve(w.act, (size_t)3 * pad * std::max(c.d_ffn, Nq) * m->esz);
        carve(w.cs, (size_t)pf * c.head_dim * 4);
        carve(w.ss, (size_t)std::min(pf, FEW_ROWS) * (d / 16) * 4);
        carve(w.prefill_tok, (size_t)pf * 4);
        if (round == 0 && hipMalloc((void**)&base, used) != hipSuccess) { (void)hipGetLastError(); return; }
    }
    kv->allocs.push_back(base);
    w.rpad = pad;
    w.part_elems = elems;
    kv->pf_rows = pf;
}

extern "C" int sj_kv_create(const sj_model* m, int32_t batch, const int32_t* capacity, sj_kv** out) {
    if (!m || !out) return fail(SJ_EINVAL, "model / out is null");
    if (batch < 1 || batch > 4096) return fail(SJ_EINVAL, "batch must be in 1..4096");
    const sj_config& c = m->cfg;
    if (c.n_layers > 0 && !capacity) return fail(SJ_EINVAL, "capacity is null");
    sj_kv* kv = new (std::nothrow) sj_kv();
    if (!kv) return fail(SJ_ENOMEM, "host allocation failed");
    kv->m = m;
    kv->batch = batch;
    if (const char* e = std::getenv("SJ_NO_GRAPH")) kv->use_graph = !(e[0] == '1');
    kv->cap.assign(batch, 64);
    kv->len_upper.assign(batch, 0);
    kv->seq_off.assign(batch, 0);
    int64_t off = 0;
    int cap_max = 64;
    for (int b = 0; b < batch; ++b) {
        int cp = 64;
        if (c.n_layers > 0) {
            if (capacity[b] < 1 || capacity[b] > (1 << 24)) { delete kv; return fail(SJ_EINVAL, "capacity[%d] out of range", b); }
            cp = (capacity[b] + 63) / 64 * 64;
        }
        kv->cap[b] = cp;
        kv->seq_off[b] = off;
        off += (int64_t)cp * c.n_kv_heads * c.head_dim;
        cap_max = std::max(cap_max, cp);
    }
    kv->cap_max = cap_max;
    kv->layer_stride = off;
    const int R = batch * (c.max_gamma + 1);
    kv->max_rows = R;
    kv->rpad = (R + 15) / 16 * 16;
    const int d = c.d_model, V = c.vocab;
    auto& A = kv->allocs;
    int rc = SJ_OK;
    auto bail = [&](int code) { free_all(kv->allocs); delete kv; return code; };
#define ALLOC(ptr, bytes) if ((rc = dev_alloc(A, &(ptr), (bytes)))) return bail(rc)
    ALLOC(kv->seq_off_dev, sizeof(int64_t) * batch);
    ALLOC(kv->cap_dev, sizeof(int32_t) * batch);
    ALLOC(kv->len_dev, sizeof(int32_t) * 2 * batch);           // lengths, then pending tokens: one copy rewinds both
    kv->pending_dev = kv->len_dev + batch;
    ALLOC(kv->sp_dev, sizeof(StepParams));
    ALLOC(kv->hn32, (size_t)R * d * 4);
    ALLOC(kv->logits, (size_t)R * V * 4);
    ALLOC(kv->stats, (size_t)R * (V / 16) * sizeof(float4));
    ALLOC(kv->rowstat, (size_t)R * sizeof(float4));
    ALLOC(kv->scores, (size_t)R * 4);
    ALLOC(kv->ranks, (size_t)R * 4);
    ALLOC(kv->p_at_d, (size_t)R * 4);
    ALLOC(kv->bits, (size_t)R * 4);
    ALLOC(kv->nacc, (size_t)batch * 4);
    ALLOC(kv->draft_tok, (size_t)batch * 4);
    // resampling slabs: about 16 vocabulary entries per thread
    {
        int blocks = std::max(1, (V / 16 + 255) / 256);
        kv->nslab = blocks * 256;
        kv->slab_len = (V + kv->nslab - 1) / kv->nslab;
    }
    const size_t slabs = (size_t)batch * kv->nslab;            // a multiple of 256
    ALLOC(kv->epart, (2 * slabs + slabs / 128) * 8);           // slab sums of both passes, then their workgroup sums (an allocation takes 20 us)
    kv->wpart = kv->epart + slabs;
    kv->eblk = kv->wpart + slabs;
    kv->wblk = kv->eblk + slabs / 256;
    if (c.n_layers == 0) {
        ALLOC(kv->xn, (size_t)3 * kv->rpad * d * m->esz);      // up to three operand planes
        rule_lm_head(kv, 1);
    }
    if (c.n_layers > 0) {
        const int hd = c.head_dim, Nq = c.n_q_heads * hd, F = c.d_ffn;
        const int G = c.n_q_heads / c.n_kv_heads;
        rule_plans(kv);
        kv->mpad = (G * (c.max_gamma + 1) + 63) / 64 * 64;   // whole groups of 4 MFMA tiles
        // key ranges of attention: one wave takes chunk_keys keys (at least one 32-key step, more when the
        // total context would otherwise need more than 1024 waves: every range costs a partial
        // result and a share of the final merge), a workgroup 4 waves' worth
        {
            const int64_t total_keys = off / ((int64_t)c.n_kv_heads * hd);
            int ck = 32;
            while (ck < 1024 && total_keys * c.n_kv_heads / ck > 1024) ck *= 2;
            if (const char* e = std::getenv("SJ_ATTN_CK")) { const int v = std::atoi(e); if (v >= 32 && v <= 4096 && (v & (v - 1)) == 0) ck = v; }
            kv->chunk_keys = ck;
            kv->nchunk_max = (cap_max + 4 * ck - 1) / (4 * ck);
        }
        ALLOC(kv->K, (size_t)kv->layer_stride * c.n_layers * m->esz);
        ALLOC(kv->V, (size_t)kv->layer_stride * c.n_layers * m->esz);
        // per (sequence, kv head, key range): mpad rows of hd accumulators + (max, sum) in lane order
        ALLOC(kv->opart, (size_t)batch * c.n_kv_heads * kv->nchunk_max * kv->mpad * (hd + 8) * 4);
        const size_t attn_tickets = (size_t)batch * c.n_kv_heads * (kv->mpad / 16);
        ALLOC(kv->tickets, (attn_tickets + d / 16) * 4);
        kv->close_tickets = kv->tickets + attn_tickets;
        kv->part_elems = forward_elems(kv, R);
        if (kv->part_elems >= PART_LIMIT) return bail(fail(SJ_EINVAL, "batch * (max_gamma + 1) rows need a projection workspace beyond 2^31 elements"));
        ALLOC(kv->xn, (size_t)3 * kv->rpad * d * m->esz);      // up to three operand planes
        ALLOC(kv->row_tok, (size_t)R * 4);
        ALLOC(kv->x, (size_t)R * d * 4);
        ALLOC(kv->part, kv->part_elems * 4);
        ALLOC(kv->attn_out, (size_t)3 * kv->rpad * Nq * m->esz);
        // also holds the rotated query fragments of many-row attention until the gate / up projection (whole tiles of 16 columns)
        const size_t qcols = (size_t)(G * (c.max_gamma + 1) + 15) / 16 * 16;
        ALLOC(kv->act, (size_t)3 * std::max((size_t)kv->rpad * F, R > FEW_ROWS ? batch * c.n_kv_heads * qcols * hd : 0) * m->esz);
        ALLOC(kv->cs, ((size_t)R * hd + (size_t)std::min(R, FEW_ROWS) * (d / 16)) * 4);
        kv->ss = kv->cs + (size_t)R * hd;                      // 16-byte pieces: hd and d are multiples of 64
        ALLOC(kv->prefill_tok, (size_t)R * 4);
    }
#undef ALLOC
    if (hipMemcpy(kv->seq_off_dev, kv->seq_off.data(), sizeof(int64_t) * batch, hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(kv->cap_dev, kv->cap.data(), sizeof(int32_t) * batch, hipMemcpyHostToDevice) != hipSuccess)
        return bail(fail(SJ_EHIP, "hipMemcpy of cache geometry failed"));
    if (c.n_layers > 0) {
        const char* e = std::getenv("SJ_TUNE");
        if (!(e && e[0] == '0') && (rc = tune_plans(kv, std::min(R, FEW_ROWS)))) return bail(rc);
    }
    *out = kv;
    return SJ_OK;
}

// Host memory for the mirrors of cache objects.  Taking and returning pinned memory costs a program that makes a cache object per batch
// 80 us, so up to eight blocks of one size (1365 rows) wait for the next object; larger ones go back at once.
constexpr size_t MIRROR_BYTES = 16384, MIRROR_POOL = 8;
static std::mutex mirror_pool_mu;
static float* mirror_pool[MIRROR_POOL];       // plain storage: giving a block back cannot throw, and nothing is destroyed before a late caller
static size_t mirror_pooled = 0;
static float* mirror_take(int rows) {
    const size_t bytes = (size_t)3 * rows * 4;
    if (bytes <= MIRROR_BYTES) {
        std::lock_guard<std::mutex> lock(mirror_pool_mu);
        if (mirror_pooled) return mirror_pool[--mirror_pooled];
    }
    void* h = nullptr;
    if (hipHostMalloc(&h, std::max(bytes, MIRROR_BYTES), hipHostMallocPortable) == hipSuccess) return (float*)h;
    (void)hipGetLastError();
    return nullptr;
}
// (no kernel writes to it any more)
static void mirror_give(float* h, int rows) {
    if (!h) return;
    if ((size_t)3 * rows * 4 <= MIRROR_BYTES) {
        std::lock_guard<std::mutex> lock(mirror_pool_mu);
        if (mirror_pooled < MIRROR_POOL) { mirror_pool[mirror_pooled++] = h; return; }
    }
    (void)hipHostFree(h);
}

extern "C" int sj_kv_free(sj_kv* kv) {
    if (!kv) return fail(SJ_EINVAL, "kv is null");
    (void)hipDeviceSynchronize();
    if (kv->pinned_state) (void)hipHostFree(kv->pinned_state);
    if (kv->rewind_done) (void)hipEventDestroy(kv->rewind_done);
    for (hipEvent_t e : kv->tev) (void)hipEventDestroy(e);
    for (auto& g : kv->graphs) (void)hipGraphExecDestroy(g.second);
    if (kv->cap_stream) (void)hipStreamDestroy(kv->cap_stream);
    free_all(kv->allocs);                                     // waits for the device that holds them
    mirror_give(kv->mirror, kv->max_rows);
    delete kv;
    return SJ_OK;
}

extern "C" int sj_set_mode(sj_kv* kv, int32_t mode) {
    if (!kv) return fail(SJ_EINVAL, "kv is null");
    if (mode < 0 || mode > 3) return fail(SJ_EINVAL, "mode must be 0, 1, 2 or 3");
    kv->mode = mode;
    return SJ_OK;
}

extern "C" int sj_set_topk(sj_kv* kv, int32_t k) {
    if (!kv) return fail(SJ_EINVAL, "kv is null");
    if (k < 1) return fail(SJ_EINVAL, "k must be at least 1");
    kv->topk = k;
    return SJ_OK;
}

extern "C" int sj_kv_rewind(sj_kv* kv, const int32_t* len_host, const int32_t* pending_host, void* stream) {
    if (!kv || !len_host || !pending_host) return fail(SJ_EINVAL, "null argument");
    for (int b = 0; b < kv->batch; ++b) {
        if (len_host[b] < 0 || len_host[b] > kv->cap[b]) return fail(SJ_ECAPACITY, "len[%d] = %d outside capacity %d", b, len_host[b], kv->cap[b]);
        if (pending_host[b] < 0 || pending_host[b] >= kv->m->cfg.vocab) return fail(SJ_EINVAL, "pending[%d] out of range", b);
    }
    hipStream_t st = (hipStream_t)stream;
    if (kv->batch <= REWIND_SEQS) {                            // the values travel as kernel arguments: no staging, no copy
        RewindArgs a{};
        for (int b = 0; b < kv->batch; ++b) { a.len[b] = len_host[b]; a.pending[b] = pending_host[b]; }
        rewind_kernel<<<1, REWIND_SEQS, 0, st>>>(a, kv->batch, kv->len_dev, kv->pending_dev);
        LAUNCHCHK("rewind");
        for (int b = 0; b < kv->batch; ++b) kv->len_upper[b] = len_host[b];
        return SJ_OK;
    }
    if (!kv->pinned_state) {
        HIPCHK(hipHostMalloc((void**)&kv->pinned_state, sizeof(int32_t) * 2 * kv->batch, hipHostMallocDefault));
        HIPCHK(hipEventCreateWithFlags(&kv->rewind_done, hipEventDisableTiming));
    }
    if (kv->rewind_pending) HIPCHK(hipEventSynchronize(kv->rewind_done));   // staging still being read
    std::memcpy(kv->pinned_state, len_host, sizeof(int32_t) * kv->batch);
    std::memcpy(kv->pinned_state + kv->batch, pending_host, sizeof(int32_t) * kv->batch);
    HIPCHK(hipMemcpyAsync(kv->len_dev, kv->pinned_state, sizeof(int32_t) * 2 * kv->batch, hipMemcpyHostToDevice, st));
    HIPCHK(hipEventRecord(kv->rewind_done, st));
    kv->rewind_pending = true;
    for (int b = 0; b < kv->batch; ++b) kv->len_upper[b] = len_host[b];
    return SJ_OK;
}

extern "C" int sj_set_kernel_timing(sj_kv* kv, int32_t kernel_class) {
    if (!kv) return fail(SJ_EINVAL, "kv is null");
    if (kernel_class < 0 || kernel_class > 4) return fail(SJ_EINVAL, "kernel_class must be 0..4");
    kv->timing_class = kernel_class;
    kv->tev_used = 0;
    return SJ_OK;
}

extern "C" int sj_kernel_class_shape(const sj_kv* kv, int32_t kernel_class, int32_t rows, char* buf, int32_t buf_len) {
    if (!kv || !buf || buf_len < 1) return fail(SJ_EINVAL, "kv / buf is null");
    if (kernel_class < 1 || kernel_class > 5) return fail(SJ_EINVAL, "kernel_class must be in 1..5");
    if (rows < 1) return fail(SJ_EINVAL, "rows must be positive");
    if (rows > FEW_ROWS) {
        const sj_config& c = kv->m->cfg;
        const int Nq = c.n_q_heads * c.head_dim, kstep = c.dtype == SJ_DTYPE_FP32 ? 16 : 32;
        const int planes = c.dtype == SJ_DTYPE_FP32 ? 0 : kv->planes;
        const GemmPlan* p = kernel_class == 1 ? &kv->plan_qkv[1] : kernel_class == 2 ? &kv->plan_o[1] : kernel_class == 4 ? &kv->plan_d[1] : nullptr;
        const int N = kernel_class == 1 ? Nq + 2 * c.n_kv_heads * c.head_dim : c.d_model;
        const int K = kernel_class == 1 ? c.d_model : kernel_class == 2 ? Nq : c.d_ffn;
        const int lm_planes = !planes || c.n_layers ? planes : 1;      // a head alone: its input is in the storage type
        const int trt = kernel_class == 3 && planes == 2 ? tile_rows(rows, 2 * c.d_ffn / 16) : kernel_class == 5 ? tile_logits(rows, c.vocab / 16, lm_planes) : 0;
        if (trt) snprintf(buf, (size_t)buf_len, "gemm_tile: row groups of %d in one launch, %d n-tiles per workgroup", trt * 16, TILE_NT);
        else snprintf(buf, (size_t)buf_len, "gemm_rows8: row groups of %d in one launch, 8 or 7 n-tiles per workgroup, %d K-slice(s)",
                 row_tiles(planes, rows) * 16, p ? rows_split(p->split, N / 16, K / kstep, rows, planes) : 1);
        return SJ_OK;
    }
    // what Runner launches
    const sj_config& c = kv->m->cfg;
    const bool bf16 = c.dtype == SJ_DTYPE_BF16;
    const int kstep = bf16 ? 32 : 16, planes = bf16 ? kv->planes : 1, d = c.d_model, Nq = c.n_q_heads * c.head_dim;
    auto partial = [&](const GemmPlan& q, int N, int K, Sums sums) { return few_partial_plan(q, kv->few_rows, N / 16, K / kstep, rows, planes, bf16, kv->ring_rows, sums); };
    GemmPlan p;
    switch (kernel_class) {
        case 1: p = partial(kv->plan_qkv[0], Nq + 2 * c.n_kv_heads * c.head_dim, d, Sums::attention); break;
        case 3: p = few_gate_up_plan(kv->plan_gu, kv->few_rows, 2 * c.d_ffn / 16, d / kstep, rows, planes, bf16, kv->ring_rows); break;
        case 5: p = few_logits_plan(kv->plan_lm, kv->few_rows, c.vocab / 16, d / kstep, rows, c.n_layers ? planes : 1, bf16, kv->ring_rows); break;
        default: {
            const int K = kernel_class == 2 ? Nq : c.d_ffn;
            p = resid_plan(d, K, kstep, rows, planes, bf16, kv->ring_rows);
            if (!p.nt) p = partial(kernel_class == 2 ? kv->plan_o[0] : kv->plan_d[0], d, K, Sums::closing);
        }
    }
    if (p.waves == RING_WAVES)
        snprintf(buf, (size_t)buf_len, "gemm_ring: %d n-tiles per workgroup, 8 waves, %d K-slice(s), LDS ring of %d KB a wave",
                 p.nt, p.split, p.depth);
    else
        snprintf(buf, (size_t)buf_len, "gemm_skinny: %d n-tiles x %d waves per workgroup, %d K-slice(s), register ring of %d", p.nt, p.waves,
                 p.split, p.depth);
    return SJ_OK;
}

extern "C" int sj_get_kernel_timing(sj_kv* kv, double* total_ms, int64_t* launches) {
    if (!kv || !total_ms || !launches) return fail(SJ_EINVAL, "null argument");
    HIPCHK(hipDeviceSynchronize());
    double tot = 0.0;
    for (size_t i = 0; i + 1 < kv->tev_used; i += 2) {
        float ms = 0.f;
        HIPCHK(hipEventElapsedTime(&ms, kv->tev[i], kv->tev[i + 1]));
        tot += ms;
    }
    *total_ms = tot;
    *launches = (int64_t)(kv->tev_used / 2);
    kv->tev_used = 0;
    return SJ_OK;
}

// records an event on the stream if kernel class `cls` is being timed; pairs are (start, stop)
static int time_mark(sj_kv* kv, int cls, hipStream_t st) {
    if (kv->timing_class != cls) return SJ_OK;
    if (kv->tev_used == kv->tev.size()) {
        if (kv->tev.size() >= (1u << 16)) return SJ_OK;         // enough samples; stop recording
        hipEvent_t e;
        HIPCHK(hipEventCreate(&e));
        kv->tev.push_back(e);
    }
    HIPCHK(hipEventRecord(kv->tev[kv->tev_used++], st));
    return SJ_OK;
}

extern "C" int sj_set_operand_planes(sj_kv* kv, int32_t planes) {
    if (!kv) return fail(SJ_EINVAL, "kv is null");
    if (planes < 1 || planes > 3) return fail(SJ_EINVAL, "planes must be 1, 2 or 3");
    if (planes == kv->planes) return SJ_OK;
    kv->planes = planes;
    // the launch shapes were chosen for the previous plane count (some exist for one or two planes only): back to
    // the rule's shapes, then the measured ones for this count (taken from the model's record when there is one)
    if (kv->m->cfg.n_layers > 0 && kv->m->cfg.dtype == SJ_DTYPE_BF16) {
        HIPCHK(hipDeviceSynchronize());
        rule_plans(kv);
        const char* e = std::getenv("SJ_TUNE");
        if (!(e && e[0] == '0')) {
            const int rc = tune_plans(kv, std::min(kv->max_rows, FEW_ROWS));
            if (rc) return rc;
        }
    }
    return SJ_OK;
}

static int check_seq_layer(const sj_kv* kv, int seq, int layer) {
    if (!kv) return fail(SJ_EINVAL, "kv is null");
    if (kv->m->cfg.n_layers == 0) return fail(SJ_EINVAL, "head-only model has no cache");
    if (seq < 0 || seq >= kv->batch) return fail(SJ_EINVAL, "seq %d out of range", seq);
    if (layer < 0 || layer >= kv->m->cfg.n_layers) return fail(SJ_EINVAL, "layer %d out of range", layer);
    return SJ_OK;
}

extern "C" int sj_kv_set_layer(sj_kv* kv, int32_t seq, int32_t layer, const void* k_host, const void* v_host, int32_t len) {
    int rc = check_seq_layer(kv, seq, layer);
    if (rc) return rc;
    if (!k_host || !v_host) return fail(SJ_EINVAL, "k_host / v_host is null");
    if (len < 0 || len > kv->cap[seq]) return fail(SJ_ECAPACITY, "len %d exceeds capacity %d", len, kv->cap[seq]);
    if (len == 0) return SJ_OK;
    const sj_config& c = kv->m->cfg;
    const size_t esz = kv->m->esz, bytes = (size_t)c.n_kv_heads * len * c.head_dim * esz;
    void *ks = nullptr, *vs = nullptr;
    HIPCHK(hipMalloc(&ks, bytes));
    if (hipMalloc(&vs, bytes) != hipSuccess) { (void)hipFree(ks); return fail(SJ_ENOMEM, "hipMalloc failed"); }
    hipError_t e1 = hipMemcpy(ks, k_host, bytes, hipMemcpyHostToDevice);
    hipError_t e2 = hipMemcpy(vs, v_host, bytes, hipMemcpyHostToDevice);
    if (e1 == hipSuccess && e2 == hipSuccess) {
        const size_t off = (size_t)layer * kv->layer_stride + kv->seq_off[seq];
        if (c.dtype == SJ_DTYPE_FP32)
            kv_scatter_kernel<float><<<1024, 256>>>((const float*)ks, (const float*)vs, (float*)kv->K + off,
                                                     (float*)kv->V + off, c.n_kv_heads, len, kv->cap[seq], c.head_dim);
        else
            kv_scatter_kernel<bf16_t><<<1024, 256>>>((const bf16_t*)ks, (const bf16_t*)vs, (bf16_t*)kv->K + off,
                                                      (bf16_t*)kv->V + off, c.n_kv_heads, len, kv->cap[seq], c.head_dim);
        e1 = hipGetLastError();
        e2 = hipDeviceSynchronize();
    }
    (void)hipFree(ks);
    (void)hipFree(vs);
    if (e1 != hipSuccess || e2 != hipSuccess)
        return fail(SJ_EHIP, "cache upload failed: %s", hipGetErrorString(e1 != hipSuccess ? e1 : e2));
    return SJ_OK;
}

extern "C" int sj_kv_set_state(sj_kv* kv, int32_t seq, int32_t len, int32_t pending_token) {
    if (!kv) return fail(SJ_EINVAL, "kv is null");
    if (seq < 0 || seq >= kv->batch) return fail(SJ_EINVAL, "seq %d out of range", seq);
    if (len < 0 || len > kv->cap[seq]) return fail(SJ_ECAPACITY, "len %d exceeds capacity %d", len, kv->cap[seq]);
    if (pending_token < 0 || pending_token >= kv->m->cfg.vocab) return fail(SJ_EINVAL, "pending token out of range");
    HIPCHK(hipDeviceSynchronize());
    set_state_kernel<<<1, 1>>>(kv->len_dev, kv->pending_dev, seq, len, pending_token);
    LAUNCHCHK("set_state");
    HIPCHK(hipDeviceSynchronize());
    kv->len_upper[seq] = len;
    return SJ_OK;
}

extern "C" int sj_kv_set(sj_kv* kv, int32_t seq, const void* k_host, const void* v_host, int32_t len, int32_t pending_token) {
    int rc = check_seq_layer(kv, seq, 0);
    if (rc) return rc;
    if (len < 0 || len > kv->cap[seq]) return fail(SJ_ECAPACITY, "len %d exceeds capacity %d", len, kv->cap[seq]);
    if (pending_token < 0 || pending_token >= kv->m->cfg.vocab) return fail(SJ_EINVAL, "pending token out of range");
    if (len > 0 && (!k_host || !v_host)) return fail(SJ_EINVAL, "k_host / v_host is null");
    const sj_config& c = kv->m->cfg;
    const size_t per_layer = (size_t)c.n_kv_heads * len * c.head_dim * kv->m->esz;
    for (int l = 0; l < c.n_layers && len > 0; ++l)
        if ((rc = sj_kv_set_layer(kv, seq, l, (const char*)k_host + l * per_layer, (const char*)v_host + l * per_layer, len)))
            return rc;
    return sj_kv_set_state(kv, seq, len, pending_token);
}

extern "C" int sj_kv_read(const sj_kv* kv, int32_t seq, int32_t layer, int32_t pos0, int32_t n, void* k_host, void* v_host) {
    int rc = check_seq_layer(kv, seq, layer);
    if (rc) return rc;
    if (!k_host || !v_host) return fail(SJ_EINVAL, "k_host / v_host is null");
    if (pos0 < 0 || n < 1 || pos0 + n > kv->cap[seq]) return fail(SJ_EINVAL, "rows %d..%d outside capacity %d", pos0, pos0 + n, kv->cap[seq]);
    const sj_config& c = kv->m->cfg;
    const size_t esz = kv->m->esz, bytes = (size_t)c.n_kv_heads * n * c.head_dim * esz;
    void *ks = nullptr, *vs = nullptr;
    HIPCHK(hipDeviceSynchronize());
    HIPCHK(hipMalloc(&ks, bytes));
    if (hipMalloc(&vs, bytes) != hipSuccess) { (void)hipFree(ks); return fail(SJ_ENOMEM, "hipMalloc failed"); }
    const size_t off = (size_t)layer * kv->layer_stride + kv->seq_off[seq];
    if (c.dtype == SJ_DTYPE_FP32)
        kv_gather_kernel<float><<<256, 256>>>((float*)ks, (float*)vs, (const float*)kv->K + off, (const float*)kv->V + off,
                                               c.n_kv_heads, pos0, n, kv->cap[seq], c.head_dim);
    else
        kv_gather_kernel<bf16_t><<<256, 256>>>((bf16_t*)ks, (bf16_t*)vs, (const bf16_t*)kv->K + off, (const bf16_t*)kv->V + off,
                                                c.n_kv_heads, pos0, n, kv->cap[seq], c.head_dim);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) e = hipMemcpy(k_host, ks, bytes, hipMemcpyDeviceToHost);
    if (e == hipSuccess) e = hipMemcpy(v_host, vs, bytes, hipMemcpyDeviceToHost);
    (void)hipFree(ks);
    (void)hipFree(vs);
    if (e != hipSuccess) return fail(SJ_EHIP, "cache read failed: %s", hipGetErrorString(e));
    return SJ_OK;
}

static int refresh_lengths(sj_kv* kv) {
    HIPCHK(hipDeviceSynchronize());
    HIPCHK(hipMemcpy(kv->len_upper.data(), kv->len_dev, sizeof(int32_t) * kv->batch, hipMemcpyDeviceToHost));
    return SJ_OK;
}

// May sequences lo .. hi - 1 take `rows` more positions, by the lengths on the device once all of its work is done?  Draft blocks, scoring
// and prompts wait here for the whole device: callers rely on it for inputs and outputs still in use on other streams, and for an object
// handed from one thread or stream to another (a stream's handle does not tell: hipStreamPerThread is one handle for many streams, a
// destroyed stream's handle is given out again).
static int check_room(sj_kv* kv, int lo, int hi, int rows) {
    const int rc = refresh_lengths(kv);
    if (rc) return rc;
    for (int b = lo; b < hi; ++b)
        if (kv->len_upper[b] + rows > kv->cap[b])
            return fail(SJ_ECAPACITY, "sequence %d: len %d + %d rows exceeds capacity %d", b, kv->len_upper[b], rows, kv->cap[b]);
    return SJ_OK;
}

// The host's bound counts a call's rows before its first launch: a call that fails part of the way has moved the lengths on the device, and
// one counted too many only costs the next step a look at them.
static void raise_bound(sj_kv* kv, int lo, int hi, int rows) {
    for (int b = lo; b < hi; ++b) kv->len_upper[b] += rows;
}

extern "C" int sj_kv_state(const sj_kv* kv, int32_t* len_host, int32_t* pending_host) {
    if (!kv) return fail(SJ_EINVAL, "kv is null");
    HIPCHK(hipDeviceSynchronize());
    if (len_host) HIPCHK(hipMemcpy(len_host, kv->len_dev, sizeof(int32_t) * kv->batch, hipMemcpyDeviceToHost));
    if (pending_host) HIPCHK(hipMemcpy(pending_host, kv->pending_dev, sizeof(int32_t) * kv->batch, hipMemcpyDeviceToHost));
    return SJ_OK;
}

// ------------------------------------------------------------------------------------------------
// kernel sequence


// Few rows (at most 32 = two MFMA row tiles): Y = X W^T with the few-row kernel.  X has SPL planes `xplane`
// elements apart; act (EPI_SWIGLU) planes are `actplane` apart.  NT n-tiles per workgroup (N/16 must be a
// multiple of NT), WAVES waves split the K-slice, D = depth of the register ring.
// What a few-row product knows of its surroundings: whether its operand and result planes are packed (gemm_ring_kernel), and of
// the norms around it `ss_in` when its operand lacks the 1/rms factor, the others for EPI_RESID (GemmArgs).
constexpr int RM_ROWS = 2;             // packed planes of up to this many rows keep a row's lane groups side by side
template <typename T> constexpr size_t packed_plane(int rm) { return rm ? 8 * Traits<T>::KSTEP : 8 * Traits<T>::KF; }
struct FewArgs {
    bool packed = false;
    int rm = 0;                        // inner order of packed planes (opnd_off)
    const float* ss_in = nullptr;
    float eps = 0.f;
    float* x = nullptr;
    const void* gain = nullptr;
    float* ss_out = nullptr;
    unsigned* tickets = nullptr;       // split-K product that closes its sub-layer: the next operand goes to xg
    void* xg = nullptr;
    size_t xgplane = 0;
    template <typename T> void put(GemmArgs& a) const {
        if (tickets) { a.tickets = tickets; a.act = xg; a.actplane = xgplane; }
        if (packed) a.xplane = a.actplane = packed_plane<T>(rm);
        a.rm = rm;
        a.ss_in = ss_in; a.eps = eps; a.x = x; a.gain = gain; a.ss_out = ss_out;
    }
};
// blocks whose operand planes are packed: both planes of at most 8 rows in one fragment
template <typename T, int SPL> constexpr bool packed_rows(int rows) { return std::is_same<T, bf16_t>::value && SPL == 2 && rows <= RING_PACK_ROWS; }

// The kernels apply 1/rms in the products that follow a residual epilogue, the register-ring kernel up to `most` = 8 rows, the LDS-ring kernel
// up to 32; elsewhere an operand that lacks it would go through unscaled.
template <int EPI> static int check_scaled(const FewArgs& fa, int rows, int most) {
    if (!fa.ss_in || ((EPI == EPI_PARTIAL || EPI == EPI_SWIGLU) && rows <= most)) return SJ_OK;
    return fail(SJ_EINVAL, "internal: product %d of %d rows with an operand that lacks its norm", EPI, rows);
}

template <typename T, int NT, int EPI, int SPL, int WAVES, int D = 2>
static int gemm(hipStream_t st, const void* Wt, const void* X, size_t xplane, int K, int N, int rows, int split,
                float* out, void* act, size_t actplane, float4* stats, float inv_temp, const FewArgs& fa = FewArgs{}) {
    if (rows > FEW_ROWS) return fail(SJ_EINVAL, "internal: few-row kernel called with %d rows", rows);
    if (const int rc = check_scaled<EPI>(fa, rows, RING_PACK_ROWS)) return rc;
    if (fa.tickets) return fail(SJ_EINVAL, "internal: the register-ring kernel closes no split-K product");
    const int ngroups = N / 16 / NT;
    GemmArgs a{};
    a.Wt = Wt; a.X = X; a.xplane = xplane; a.actplane = actplane;
    a.K = K; a.N = N; a.R = rows; a.slice_rows = rows;
    a.inv_temp = inv_temp;
    a.out = out; a.stats = stats; a.act = act;
    fa.put<T>(a);
    if (rows <= 16) gemm_skinny_kernel<T, NT, 1, EPI, SPL, WAVES, D><<<dim3(ngroups, split), WAVES * 64, 0, st>>>(a);
    else gemm_skinny_kernel<T, NT, 2, EPI, SPL, WAVES, D><<<dim3(ngroups, split), WAVES * 64, 0, st>>>(a);
    LAUNCHCHK("gemm_skinny");
    return SJ_OK;
}

// The same product on the LDS-ring kernel (bf16, at most two planes; ring_fits has been checked).
template <typename T, int NT, int EPI, int SPL, int DEPTH>
static int gemm_ring(hipStream_t st, const void* Wt, const void* X, size_t xplane, int K, int N, int rows, int split,
                     float* out, void* act, size_t actplane, float4* stats, float inv_temp, const FewArgs& fa = FewArgs{}) {
    if (const int rc = check_scaled<EPI>(fa, rows, RING_ROWS)) return rc;
    GemmArgs a{};
    a.Wt = Wt; a.X = X; a.xplane = xplane; a.actplane = actplane;
    a.K = K; a.N = N; a.R = rows; a.slice_rows = rows;
    a.inv_temp = inv_temp;
    a.out = out; a.stats = stats; a.act = act;
    fa.put<T>(a);
    const dim3 grid(N / 16 / NT, split);
    if (EPI == EPI_RESID && rows > RING_PACK_ROWS) return fail(SJ_EINVAL, "internal: residual epilogue over %d rows", rows);
    constexpr bool FEWER = EPI == EPI_RESID;                       // no more than 8 rows: two planes are packed, one row tile
    if (SPL == 2 && (FEWER || rows <= RING_PACK_ROWS)) gemm_ring_kernel<T, NT, 1, EPI, 2, true, DEPTH><<<grid, RING_CW * 64, 0, st>>>(a);
    else if constexpr (!FEWER || SPL == 1) {
        if (FEWER || rows <= 16) gemm_ring_kernel<T, NT, 1, EPI, SPL, false, DEPTH><<<grid, RING_CW * 64, 0, st>>>(a);
        else if constexpr (!FEWER) gemm_ring_kernel<T, NT, 2, EPI, SPL, false, DEPTH><<<grid, RING_CW * 64, 0, st>>>(a);
    }
    LAUNCHCHK("gemm_ring");
    return SJ_OK;
}

// The few-row split-K projection in exactly the launch shape of a plan (partial_fits has been checked): the consumer of the partials
// goes by the plan's K-slices.
template <typename T, int SPL>
static int few_partial(const GemmPlan& p, hipStream_t st, const void* W, const void* X, size_t xplane, int K, int N,
                       int rows, float* out, const FewArgs& fa = FewArgs{}) {
    constexpr bool BF16 = std::is_same<T, bf16_t>::value;
    if (partial_fits(p, N / 16, K / Traits<T>::KSTEP, rows, SPL, BF16)) {
        if constexpr (BF16 && SPL <= 2) {
#define SJ_RING(NT, DEPTH)                                                                                            \
    if (p.waves == RING_WAVES && p.nt == NT && p.depth == DEPTH)                                                      \
        return gemm_ring<T, NT, EPI_PARTIAL, SPL, DEPTH>(st, W, X, xplane, K, N, rows, p.split, out, nullptr, 0, nullptr, 0.f, fa);
            SJ_RING_PARTIAL_SHAPES(SJ_RING)
#undef SJ_RING
        }
#define SJ_SHAPE(NT, WV, D)                                                                                         \
    if (p.nt == NT && p.waves == WV && p.depth == D)                                                                \
        return gemm<T, NT, EPI_PARTIAL, SPL, WV, D>(st, W, X, xplane, K, N, rows, p.split, out, nullptr, 0, nullptr, 0.f, fa);
        SJ_FEW_PARTIAL_SHAPES(SJ_SHAPE)
        if constexpr (SPL <= 2) { SJ_FEW_PARTIAL_SHAPES_2(SJ_SHAPE) }
#undef SJ_SHAPE
    }
    return fail(SJ_EINVAL, "internal: no few-row kernel for %d tiles x %d waves, %d K-slice(s), ring %d", p.nt, p.waves, p.split, p.depth);
}

// The few-row gate / up projection (SwiGLU epilogue, no K-slices) in exactly the launch shape of a plan (resolve_gate_up).
template <typename T, int SPL>
static int few_swiglu(const GemmPlan& p, hipStream_t st, const void* W, const void* X, size_t xplane, int K, int N2, int rows,
                      void* act, size_t actplane, const FewArgs& fa = FewArgs{}) {
    constexpr bool BF16 = std::is_same<T, bf16_t>::value;
    if (gate_up_fits(p, N2 / 16, K / Traits<T>::KSTEP, rows, SPL, BF16)) {
        if constexpr (BF16 && SPL <= 2) {
#define SJ_RING(NT, DEPTH)                                                                                            \
    if (p.waves == RING_WAVES && p.nt == NT && p.depth == DEPTH)                                                      \
        return gemm_ring<T, NT, EPI_SWIGLU, SPL, DEPTH>(st, W, X, xplane, K, N2, rows, 1, nullptr, act, actplane, nullptr, 0.f, fa);
            SJ_RING_GATE_UP_SHAPES(SJ_RING)
#undef SJ_RING
        }
#define SJ_SHAPE(NT, WV, D)                                                                                         \
    if (p.nt == NT && p.waves == WV && p.depth == D)                                                                \
        return gemm<T, NT, EPI_SWIGLU, SPL, WV, D>(st, W, X, xplane, K, N2, rows, 1, nullptr, act, actplane, nullptr, 0.f, fa);
        SJ_FEW_GATE_UP_SHAPES(SJ_SHAPE)
        if constexpr (SPL <= 2) { SJ_FEW_GATE_UP_SHAPES_2(SJ_SHAPE) }
#undef SJ_SHAPE
    }
    return fail(SJ_EINVAL, "internal: no few-row gate/up kernel for %d tiles x %d waves, ring %d", p.nt, p.waves, p.depth);
}

template <typename T, int SPL>
static int few_resid(const GemmPlan& p, hipStream_t st, const void* W, const void* X, size_t xplane, int K, int N, int rows, void* xg,
                     size_t xgplane, const FewArgs& fa) {
    if constexpr (SPL <= 2) {
        if constexpr (std::is_same<T, bf16_t>::value) {
#define SJ_RING(NT, DEPTH)                                                                                            \
    if (p.waves == RING_WAVES && p.nt == NT && p.depth == DEPTH)                                                      \
        return gemm_ring<T, NT, EPI_RESID, SPL, DEPTH>(st, W, X, xplane, K, N, rows, 1, nullptr, xg, xgplane, nullptr, 0.f, fa);
            SJ_RING_RESID_SHAPES(SJ_RING)
#undef SJ_RING
        }
#define SJ_SHAPE(NT)                                                                                                \
    if (p.waves == 8 && p.nt == NT)                                                                                 \
        return gemm<T, NT, EPI_RESID, SPL, 8, 2>(st, W, X, xplane, K, N, rows, 1, nullptr, xg, xgplane, nullptr, 0.f, fa);
        SJ_SHAPE(1) SJ_SHAPE(2) SJ_SHAPE(4)
#undef SJ_SHAPE
    }
    return fail(SJ_EINVAL, "internal: no residual kernel for %d tiles x %d waves", p.nt, p.waves);
}

// The few-row LM head (logits + per-workgroup softmax statistics: V / 16 / nt entries per row) in exactly the launch shape of a plan.
template <typename T, int SPL>
static int few_logits(const GemmPlan& p, hipStream_t st, const void* W, const void* X, size_t xplane, int K, int V, int rows,
                      float* logits, float4* stats, float inv_temp, const FewArgs& fa = FewArgs{}) {
    constexpr bool BF16 = std::is_same<T, bf16_t>::value;
    if (logits_fits(p, V / 16, K / Traits<T>::KSTEP, rows, SPL, BF16)) {
        if constexpr (BF16 && SPL <= 2) {
#define SJ_RING(NT, DEPTH)                                                                                            \
    if (p.waves == RING_WAVES && p.nt == NT && p.depth == DEPTH)                                                      \
        return gemm_ring<T, NT, EPI_LOGITS, SPL, DEPTH>(st, W, X, xplane, K, V, rows, 1, logits, nullptr, 0, stats, inv_temp, fa);
            SJ_RING_LOGITS_SHAPES(SJ_RING)
#undef SJ_RING
        }
#define SJ_SHAPE(NT, WV, D)                                                                                         \
    if (p.nt == NT && p.waves == WV && p.depth == D)                                                                \
        return gemm<T, NT, EPI_LOGITS, SPL, WV, D>(st, W, X, xplane, K, V, rows, 1, logits, nullptr, 0, stats, inv_temp, fa);
        SJ_FEW_LOGITS_SHAPES(SJ_SHAPE)
        if constexpr (SPL <= 2) { SJ_FEW_LOGITS_SHAPES_2(SJ_SHAPE) }
#undef SJ_SHAPE
    }
    return fail(SJ_EINVAL, "internal: no few-row LM-head kernel for %d tiles x %d waves, ring %d", p.nt, p.waves, p.depth);
}

// Picks between the rule's plan and measured candidates.  time_plan(plan, us) times one plan.  The first timings of
// a process run on a GPU that is still raising its clocks, so the rule's plan is timed (and discarded) first; the
// fastest candidate then has to beat the rule's plan by 5 % in two alternating confirmation rounds before it
// replaces it - a choice made on one noisy sample would differ from run to run, and the measurement does not see
// what more K-slices cost the kernel that sums them.
template <typename TimeFn>
static int pick_plan(GemmPlan& plan, const std::vector<GemmPlan>& candidates, TimeFn time_plan) {
    int rc;
    double us = 0.0, best_us = 1e30;
    if ((rc = time_plan(plan, us)) || (rc = time_plan(plan, us))) return rc;       // warm-up
    GemmPlan best = plan;
    bool found = false;
    for (const GemmPlan& p : candidates) {
        if (p.nt == plan.nt && p.waves == plan.waves && p.split == plan.split && p.depth == plan.depth) continue;
        if ((rc = time_plan(p, us))) return rc;
        if (us < best_us) { best_us = us; best = p; found = true; }
    }
    if (!found) return SJ_OK;
    double base_sum = 0.0, cand_sum = 0.0;
    for (int round = 0; round < 2; ++round) {
        if ((rc = time_plan(plan, us))) return rc;
        base_sum += us;
        if ((rc = time_plan(best, us))) return rc;
        cand_sum += us;
    }
    if (cand_sum < 0.95 * base_sum) plan = best;
    return SJ_OK;
}

// Launch shapes of the three split-K projections for few rows, chosen by measurement when the cache object is created: which of
// (n-tiles, waves, K-slices, ring depth) streams a given weight matrix fastest depends on its shape and on the number of row tiles in ways the workgroup-count rule of plan_partial does not capture (70B-shaped
// QKV with two row tiles: 50 us with the rule's shape, 35 us with the best one).  Every candidate runs over up to 16
// layers' weights back to back (distinct layers, so nothing is served from cache); the rule's plan stays unless a
// candidate is at least 5 % faster (pick_plan).  `closes` (tune_plans): O and down are timed as they run, with the tickets of their K-slices and
// the end of the sub-layer, into buffers that hold nothing between calls.  SJ_TUNE=0 keeps the rule's plans (launch shapes then never differ between runs).
template <typename T, int SPL>
static int tune_one(sj_kv* kv, GemmPlan& plan, void* LayerW::*which, const void* X, int K, int N, int rows, Sums sums, bool closes,
                    hipEvent_t e0, hipEvent_t e1) {
    const sj_model* m = kv->m;
    const int ksteps = K / Traits<T>::KSTEP, ntiles = N / 16;
    const int nl = std::min(m->cfg.n_layers, 16);
    const size_t xplane = (size_t)kv->rpad * K;
    FewArgs fa;
    fa.packed = packed_rows<T, SPL>(rows);
    fa.rm = fa.packed && rows <= RM_ROWS;
    if (closes && sums == Sums::closing) {
        fa.x = kv->x; fa.gain = m->layers[0].ffn_norm; fa.ss_out = kv->ss;
        fa.tickets = kv->close_tickets; fa.xg = kv->xn; fa.xgplane = (size_t)kv->rpad * N;
    }
    auto time_plan = [&](const GemmPlan& p, double& us) -> int {
        float ms = 0.f;
        for (int rep = 0; rep < 2; ++rep) {                 // the first repetition warms up
            HIPCHK(hipEventRecord(e0, nullptr));
            for (int l = 0; l < nl; ++l) {
                const int rc = few_partial<T, SPL>(p, nullptr, m->layers[l].*which, X, xplane, K, N, rows, kv->part, fa);
                if (rc) return rc;
            }
            HIPCHK(hipEventRecord(e1, nullptr));
            HIPCHK(hipEventSynchronize(e1));
            HIPCHK(hipEventElapsedTime(&ms, e0, e1));
        }
        us = (double)ms * 1e3 / nl;
        return SJ_OK;
    };
    return pick_plan(plan, measured_partials(plan, ntiles, ksteps, rows, SPL, std::is_same<T, bf16_t>::value, sums, closes), time_plan);
}

template <typename T, int SPL>
static int tune_gate_up(sj_kv* kv, int rows, bool closes, hipEvent_t e0, hipEvent_t e1) {
    const sj_model* m = kv->m;
    const int d = m->cfg.d_model, F = m->cfg.d_ffn, ntiles = 2 * F / 16;
    const int nl = std::min(m->cfg.n_layers, 16);
    FewArgs fa;
    fa.packed = packed_rows<T, SPL>(rows);
    fa.rm = fa.packed && rows <= RM_ROWS;
    auto time_plan = [&](const GemmPlan& p, double& us) -> int {
        float ms = 0.f;
        for (int rep = 0; rep < 2; ++rep) {                 // the first repetition warms up
            HIPCHK(hipEventRecord(e0, nullptr));
            for (int l = 0; l < nl; ++l) {
                const int rc = few_swiglu<T, SPL>(p, nullptr, m->layers[l].wgu, kv->xn, (size_t)kv->rpad * d, d, 2 * F, rows, kv->act,
                                                  (size_t)kv->rpad * F, fa);
                if (rc) return rc;
            }
            HIPCHK(hipEventRecord(e1, nullptr));
            HIPCHK(hipEventSynchronize(e1));
            HIPCHK(hipEventElapsedTime(&ms, e0, e1));
        }
        us = (double)ms * 1e3 / nl;
        return SJ_OK;
    };
    const int ksteps = d / Traits<T>::KSTEP;
    const bool one = rule_gate_up(ntiles, SPL).nt == 1;          // small matrices: the rule's shape, where it starts from a ring
    std::vector<GemmPlan> cands;
    auto offer = [&](int nt, int waves, int depth) {
        const GemmPlan p{nt, waves, 1, depth};
        if (!gate_up_fits(p, ntiles, ksteps, rows, SPL, std::is_same<T, bf16_t>::value) || (closes && waves != RING_WAVES)) return;
        const bool wide = ntiles / nt >= 128 && (waves == RING_WAVES || ksteps / waves >= 4);
        if (one && waves != RING_WAVES ? nt == 1 : wide) cands.push_back(p);
    };
#define SJ_OFFER(NT, WV, D) offer(NT, WV, D);
    SJ_FEW_GATE_UP_SHAPES(SJ_OFFER)
    SJ_FEW_GATE_UP_SHAPES_2(SJ_OFFER)
#undef SJ_OFFER
#define SJ_OFFER(NT, D) offer(NT, RING_WAVES, D);
    SJ_RING_GATE_UP_SHAPES(SJ_OFFER)
#undef SJ_OFFER
    return pick_plan(kv->plan_gu, cands, time_plan);
}

template <typename T, int SPL>
static int tune_lm_head(sj_kv* kv, int rows, hipEvent_t e0, hipEvent_t e1) {
    const sj_model* m = kv->m;
    const int d = m->cfg.d_model, V = m->cfg.vocab;
    FewArgs fa;
    fa.packed = packed_rows<T, SPL>(rows);
    fa.rm = fa.packed && rows <= RM_ROWS;
    auto time_plan = [&](const GemmPlan& p, double& us) -> int {
        float ms = 0.f;
        for (int rep = 0; rep < 2; ++rep) {                 // the first repetition warms up
            HIPCHK(hipEventRecord(e0, nullptr));
            for (int l = 0; l < 3; ++l) {
                const int rc = few_logits<T, SPL>(p, nullptr, m->lm_head, kv->xn, (size_t)kv->rpad * d, d, V, rows, kv->logits, kv->stats,
                                                  m->md.inv_temp, fa);
                if (rc) return rc;
            }
            HIPCHK(hipEventRecord(e1, nullptr));
            HIPCHK(hipEventSynchronize(e1));
            HIPCHK(hipEventElapsedTime(&ms, e0, e1));
        }
        us = (double)ms * 1e3 / 3;
        return SJ_OK;
    };
    const int ntiles = V / 16, ksteps = d / Traits<T>::KSTEP;
    const GemmPlan rule = rule_logits(ntiles);
    std::vector<GemmPlan> cands{rule};
    auto offer = [&](int nt, int waves, int depth) {
        const GemmPlan p{nt, waves, 1, depth};
        if (!logits_fits(p, ntiles, ksteps, rows, SPL, std::is_same<T, bf16_t>::value)) return;
        // (a small matrix: the rule's shape, where it starts from a ring; a large one: none of the small ones')
        if (waves == RING_WAVES || (rule.nt != 2 && nt != 2 && ksteps / waves >= 4)) cands.push_back(p);
    };
#define SJ_OFFER(NT, WV, D) offer(NT, WV, D);
    SJ_FEW_LOGITS_SHAPES(SJ_OFFER)
    if (SPL <= 2) { SJ_FEW_LOGITS_SHAPES_2(SJ_OFFER) }
#undef SJ_OFFER
#define SJ_OFFER(NT, D) offer(NT, RING_WAVES, D);
    SJ_RING_LOGITS_SHAPES(SJ_OFFER)
#undef SJ_OFFER
    return pick_plan(kv->plan_lm, cands, time_plan);
}

static int tune_plans(sj_kv* kv, int rows) {
    const sj_model* m = kv->m;
    const sj_config& c = m->cfg;
    const int d = c.d_model, Nq = c.n_q_heads * c.head_dim, Nk = c.n_kv_heads * c.head_dim, F = c.d_ffn;
    const std::pair<int, int> key(rows, c.dtype == SJ_DTYPE_FP32 ? 1 : kv->planes);
    {
        std::lock_guard<std::mutex> lock(m->tuned_mu);
        auto it = m->tuned.find(key);
        if (it != m->tuned.end()) {                          // measured before on this model: same shapes again
            const TunedPlans& t = *it->second;
            kv->plan_qkv[0] = t.qkv; kv->plan_o[0] = t.o; kv->plan_d[0] = t.d; kv->plan_gu = t.gu; kv->plan_lm = t.lm;
            return SJ_OK;
        }
    }
    hipEvent_t e0 = nullptr, e1 = nullptr;
    HIPCHK(hipEventCreate(&e0));
    if (hipEventCreate(&e1) != hipSuccess) { (void)hipEventDestroy(e0); return fail(SJ_EHIP, "hipEventCreate failed"); }
    int rc = SJ_OK;
    // From 9 rows on O and down close their sub-layers where they and their consumers run on the LDS-ring kernel: where the rule has it so, the
    // measurement stays with that kernel (another, 5 % faster by itself, would bring back a norm launch of 4.7 us).
    const bool closes = rows > RING_PACK_ROWS && std::min({kv->plan_qkv[0].waves, kv->plan_o[0].waves, kv->plan_d[0].waves, kv->plan_gu.waves}) == RING_WAVES;
#define SJ_TUNE3(T, SPL)                                                                                          \
    do {                                                                                                          \
        if (!rc) rc = tune_one<T, SPL>(kv, kv->plan_qkv[0], &LayerW::wqkv, kv->xn, d, Nq + 2 * Nk, rows, Sums::attention, closes, e0, e1);  \
        if (!rc) rc = tune_one<T, SPL>(kv, kv->plan_o[0], &LayerW::wo, kv->attn_out, Nq, d, rows, Sums::closing, closes, e0, e1);  \
        if (!rc) rc = tune_one<T, SPL>(kv, kv->plan_d[0], &LayerW::wd, kv->act, F, d, rows, Sums::closing, closes, e0, e1);  \
        if (!rc) rc = tune_gate_up<T, SPL>(kv, rows, closes, e0, e1);                                                  \
        if (!rc) rc = tune_lm_head<T, SPL>(kv, rows, e0, e1);                                                     \
    } while (0)
    if (c.dtype == SJ_DTYPE_FP32) SJ_TUNE3(float, 1);
    else if (kv->planes == 1) SJ_TUNE3(bf16_t, 1);
    else if (kv->planes == 3) SJ_TUNE3(bf16_t, 3);
    else SJ_TUNE3(bf16_t, 2);
#undef SJ_TUNE3
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (!rc) {
        auto t = std::make_shared<TunedPlans>();
        t->qkv = kv->plan_qkv[0]; t->o = kv->plan_o[0]; t->d = kv->plan_d[0]; t->gu = kv->plan_gu; t->lm = kv->plan_lm;
        std::lock_guard<std::mutex> lock(m->tuned_mu);
        m->tuned.emplace(key, t);
    }
    if (const char* e = std::getenv("SJ_TUNE_LOG")) {
        if (e[0] == '1') {
            auto show = [](const char* name, const GemmPlan& p) {
                fprintf(stderr, "[sj] %-8s %d n-tiles x %d waves, %d K-slice(s), ring %d\n", name, p.nt, p.waves, p.split, p.depth);
            };
            fprintf(stderr, "[sj] launch shapes for %d rows, d_model %d:\n", rows, d);
            show("QKV", kv->plan_qkv[0]); show("O", kv->plan_o[0]); show("gate/up", kv->plan_gu); show("down", kv->plan_d[0]);
            show("LM head", kv->plan_lm);
        }
    }
    return rc;
}

// The gate / up projection, or the LM head, of many rows on large tiles; rt = row tiles of a row group (tile_rows, tile_logits).
template <typename T, int EPI, int SPL>
static int gemm_tile(hipStream_t st, const void* Wt, const void* X, size_t xplane, int K, int N, int rows, int rt, float* out, void* act, size_t actplane,
                     float4* stats, float inv_temp) {
    GemmArgs a{};
    a.Wt = Wt; a.X = X; a.xplane = xplane; a.actplane = actplane;
    a.K = K; a.N = N; a.R = rows;
    a.act = act; a.out = out; a.stats = stats; a.inv_temp = inv_temp;
    a.rgroups = (rows + rt * 16 - 1) / (rt * 16);
    const int ngroups = (N / 16 + TILE_NT - 1) / TILE_NT;
    const int grid = std::min(TILE_WGS, (ngroups + 7) / 8 * 8 * a.rgroups);        // whole rounds of the 8 XCDs
    bool done = false;
    auto launch = [&](auto rt_tag) {
        constexpr int RT = decltype(rt_tag)::value, NS = std::min(5, 160 / (RT * SPL + TILE_NT));      // as many stages as 160 KB hold, up to five
        if (rt != RT) return;
        gemm_tile_kernel<T, EPI, SPL, RT, NS><<<grid, TILE_WAVES * 64, 0, st>>>(a);
        done = true;
    };
    if constexpr (EPI == EPI_LOGITS) {                 // tile_rows has no group below ten row tiles
        launch(std::integral_constant<int, 6>{});
        launch(std::integral_constant<int, 8>{});
        if constexpr (SPL == 2) {
            launch(std::integral_constant<int, 9>{});
            launch(std::integral_constant<int, 11>{});
            launch(std::integral_constant<int, 13>{});
            launch(std::integral_constant<int, 15>{});
        } else launch(std::integral_constant<int, 18>{});
    }
    launch(std::integral_constant<int, 10>{});
    launch(std::integral_constant<int, 12>{});
    launch(std::integral_constant<int, 14>{});
    launch(std::integral_constant<int, 16>{});
    if (!done) return fail(SJ_EINVAL, "internal: no large-tile kernel for %d row tiles", rt);
    LAUNCHCHK("gemm_tile");
    return SJ_OK;
}

// More rows: all row groups in one launch of the loader-wave kernel, the workgroups of an n-tile group side by side on one XCD, so that the
// weights are fetched from HBM once for all rows.  The statistics of EPI_LOGITS are per workgroup (of 8 n-tiles).
template <typename T, int SPL> constexpr int rows_planes = std::is_same<T, float>::value ? 0 : SPL;   // as row_tiles and rows_split count them
template <typename T, int EPI, int SPL>
static int gemm_rows(hipStream_t st, const void* Wt, const void* X, size_t xplane, int K, int N, int rows, int split,
                     float* out, void* act, size_t actplane, float4* stats, float inv_temp) {
    if constexpr (EPI == EPI_SWIGLU && SPL == 2 && std::is_same<T, bf16_t>::value) {
        if (const int trt = tile_rows(rows, N / 16)) return gemm_tile<T, EPI, SPL>(st, Wt, X, xplane, K, N, rows, trt, nullptr, act, actplane, nullptr, 0.f);
    }
    if constexpr (EPI == EPI_LOGITS && SPL <= 2 && std::is_same<T, bf16_t>::value) {
        if (const int trt = tile_logits(rows, N / 16, SPL)) return gemm_tile<T, EPI, SPL>(st, Wt, X, xplane, K, N, rows, trt, out, nullptr, 0, stats, inv_temp);
    }
    const int ntiles = N / 16, rt = row_tiles(rows_planes<T, SPL>, rows), rgroups = (rows + rt * 16 - 1) / (rt * 16);
    const int mt = (std::min(rows, rt * 16) + 15) / 16;
    GemmArgs a{};
    a.Wt = Wt; a.X = X; a.xplane = xplane; a.actplane = actplane;
    a.K = K; a.N = N; a.R = rows; a.slice_rows = rows;
    a.inv_temp = inv_temp;
    a.out = out; a.stats = stats; a.act = act;
    a.rgroups = rgroups;
    // 7 n-tiles per workgroup where that fills whole rounds of the chip and 8 do not (gate/up of the 8B shape: 256 workgroups instead of
    // 224), from 8 row tiles on (below that the lighter weight stream per CU loses)
    const bool seven = EPI == EPI_SWIGLU && mt >= 8 && rt >= 8 && ntiles % 7 == 0 && (ntiles / 7) % 256 == 0 && ((ntiles + 7) / 8) % 256 != 0;
    const int per = seven ? 7 : ROWS_NT, ngroups = (ntiles + per - 1) / per;
    const dim3 grid(rgroups > 1 ? (ngroups + 7) / 8 * 8 * rgroups : ngroups, EPI == EPI_PARTIAL ? split : 1);
    auto launch = [&](auto rt_tag) {
        constexpr int RT = decltype(rt_tag)::value;
        if (rt != RT) return;
        if constexpr (EPI == EPI_SWIGLU && RT >= 8) {
            if (seven) gemm_rows8_kernel<T, EPI, SPL, 7, RT><<<grid, (R8_CW + R4_LW) * 64, 0, st>>>(a, mt);
        }
        if (!seven) gemm_rows8_kernel<T, EPI, SPL, ROWS_NT, RT><<<grid, (R8_CW + R4_LW) * 64, 0, st>>>(a, mt);
    };
    launch(std::integral_constant<int, 4>{});              // the sizes of row_tiles
    if constexpr (SPL == 3) { launch(std::integral_constant<int, 5>{}); launch(std::integral_constant<int, 6>{}); }
    else launch(std::integral_constant<int, 9>{});
    if constexpr (SPL == 2) { launch(std::integral_constant<int, 6>{}); launch(std::integral_constant<int, 8>{}); }
    if constexpr (SPL == 1 && std::is_same<T, bf16_t>::value) { launch(std::integral_constant<int, 16>{}); launch(std::integral_constant<int, 18>{}); }
    LAUNCHCHK("gemm_rows");
    return SJ_OK;
}

// Blocks whose attention runs in two launches: more rows than the few-row kernels take, at least one full query tile per kv head
// and sequence, and contexts of at most 2048 keys.  The single launch sums and rotates the query rows again for every key range
// (score block of 6 x 21 rows, up to 721 keys: 83 us a layer against 26); with long contexts that work is small beside the keys, and
// its split of a sequence's keys over workgroups balances a ragged batch better (16 x 9 rows, up to 4096 keys: 69 against 81).
constexpr int ROWS_ATTN_KEYS = 2048;
static bool many_rows_attention(const ModelDims& md, int rows, int rps, int cap_max) {
    return rows > FEW_ROWS && rps * md.G >= 16 && cap_max <= ROWS_ATTN_KEYS;
}

template <typename T, int SPL>
struct Runner {
    const sj_model* m;
    sj_kv* kv;
    hipStream_t st;
    int nseq, rps, R;
    const Forward* w = kv;     // the buffers it works in
    int seq_base = 0;          // first sequence (a prompt's: its index)

    KvView<T> view() const {
        KvView<T> v;
        v.K = (T*)kv->K; v.V = (T*)kv->V; v.seq_off = kv->seq_off_dev; v.cap = kv->cap_dev;
        v.len = kv->len_dev; v.pending = kv->pending_dev; v.layer_stride = kv->layer_stride;
        return v;
    }
    bool packed() const { return packed_rows<T, SPL>(R); }
    int rm() const { return packed() && R <= RM_ROWS; }
    size_t plane(int ld) const { return packed() ? packed_plane<T>(rm()) : (size_t)w->rpad * ld; }
    // launch shape of a split-K projection for this row count
    GemmPlan plan_of(Product product, int K, int N) const {
        const int ksteps = K / Traits<T>::KSTEP;
        const GemmPlan* pl = kv->plans(product);
        if (R <= FEW_ROWS) return few_partial_plan(pl[0], kv->few_rows, N / 16, ksteps, R, SPL, std::is_same<T, bf16_t>::value, kv->ring_rows, sums_of(product));
        GemmPlan p = pl[1];
        p.split = rows_split(p.split, N / 16, ksteps, R, rows_planes<T, SPL>);
        return p;
    }
    // `parts`: the K-slices it leaves in w->part
    int partial_gemm(const void* W, const void* X, int K, int N, Product product, int* parts = nullptr, bool unscaled = false) {
        const GemmPlan p = plan_of(product, K, N);
        if (parts) *parts = p.split;
        if ((size_t)p.split * R * N > w->part_elems) return fail(SJ_EINVAL, "internal: %d K-slices of %d rows exceed the partials' buffer", p.split, R);
        if (R > FEW_ROWS) return gemm_rows<T, EPI_PARTIAL, SPL>(st, W, X, plane(K), K, N, R, p.split, w->part, nullptr, 0, nullptr, 0.f);
        return few_partial<T, SPL>(p, st, W, X, plane(K), K, N, R, w->part, few_args(unscaled));
    }
    // does the product that reads what O or down leaves run on the LDS-ring kernel?
    bool ring_consumer(Product product) const {
        const ModelDims& md = m->md;
        const GemmPlan p = product == Product::o ? few_gate_up_plan(kv->plan_gu, kv->few_rows, 2 * md.F / 16, md.d / Traits<T>::KSTEP, R, SPL, std::is_same<T, bf16_t>::value, kv->ring_rows)
                                                 : plan_of(Product::qkv, md.d, (md.Hq + 2 * md.Hkv) * md.hd);
        return p.waves == RING_WAVES;
    }
    // the operand in w->xn lacks its 1/rms factors (it came from a residual epilogue)
    FewArgs few_args(bool unscaled) const {
        FewArgs n;
        n.packed = packed();
        n.rm = rm();
        if (unscaled) { n.ss_in = w->ss; n.eps = m->md.eps; }
        return n;
    }
    // O or down projection with its sub-layer's residual add, either in its epilogue (`unscaled`: the next operand, with the norm
    // gain, is in w->xn without its 1/rms factors) or left in `parts` K-slices for norm()
    // (or, from 9 rows on, in the epilogue of the last of its K-slices, where both this product and the next run on the LDS-ring kernel)
    int closing_gemm(const void* W, const void* X, int K, Product product, const void* gain, int& parts, bool& unscaled) {
        const int d = m->md.d;
        const GemmPlan p = resid_plan(d, K, Traits<T>::KSTEP, R, SPL, std::is_same<T, bf16_t>::value, kv->ring_rows);
        unscaled = p.nt > 0;
        if (!unscaled) {
            const GemmPlan q = plan_of(product, K, d);
            if (R > FEW_ROWS || R <= RING_PACK_ROWS || q.waves != RING_WAVES || !ring_consumer(product)) return partial_gemm(W, X, K, d, product, &parts);
            if ((size_t)q.split * R * d > w->part_elems) return fail(SJ_EINVAL, "internal: %d K-slices of %d rows exceed the partials' buffer", q.split, R);
            unscaled = true;
            FewArgs n = few_args(false);
            n.x = w->x; n.gain = gain; n.ss_out = w->ss;
            n.tickets = kv->close_tickets; n.xg = w->xn; n.xgplane = plane(d);
            return few_partial<T, SPL>(q, st, W, X, plane(K), K, d, R, w->part, n);
        }
        FewArgs n = few_args(false);
        n.x = w->x; n.gain = gain; n.ss_out = w->ss;
        return few_resid<T, SPL>(p, st, W, X, plane(K), K, d, R, w->xn, plane(d), n);
    }
    // the same up to and including the next norm
    int close(const void* W, const void* X, int K, Product product, const void* gain, int cls, bool& unscaled) {
        int rc, parts = 0;
        if ((rc = time_mark(kv, cls, st))) return rc;
        if ((rc = closing_gemm(W, X, K, product, gain, parts, unscaled))) return rc;
        if ((rc = time_mark(kv, cls, st))) return rc;
        if (!unscaled) {
            norm(parts, gain, nullptr);
            LAUNCHCHK("add_rmsnorm");
        }
        return SJ_OK;
    }
    // gate / up projection with the SwiGLU epilogue; few rows: the plan's launch shape, or the rule's where that does not take them
    int gate_up(const void* W, bool unscaled = false) {
        const ModelDims& md = m->md;
        if (R > FEW_ROWS) return gemm_rows<T, EPI_SWIGLU, SPL>(st, W, w->xn, plane(md.d), md.d, 2 * md.F, R, 1, nullptr, w->act, plane(md.F), nullptr, 0.f);
        const GemmPlan p = few_gate_up_plan(kv->plan_gu, kv->few_rows, 2 * md.F / 16, md.d / Traits<T>::KSTEP, R, SPL, std::is_same<T, bf16_t>::value, kv->ring_rows);
        return few_swiglu<T, SPL>(p, st, W, w->xn, plane(md.d), md.d, 2 * md.F, R, w->act, plane(md.F), few_args(unscaled));
    }

    // rotary + cache append + attention of one layer from the QKV partials in w->part
    int attention(int layer, int parts) {
        const ModelDims& md = m->md;
        if (rps > m->cfg.max_gamma + 1 || many_rows_attention(md, R, rps, kv->cap_max)) return rows_attention(layer, parts);
        const int M = md.G * rps;
        const int mtiles = (M + 15) / 16;
        // one query tile per workgroup while the launch stays small (shortest dependent chain per wave;
        // K / V are then read once per tile), up to 4 tiles per workgroup for large batches
        const bool small = (long long)nseq * md.Hkv * kv->nchunk_max * mtiles <= 512;
        const int mq = small ? 1 : std::min(mtiles, 4);
        const int qgroups = (mtiles + mq - 1) / mq;
        dim3 grid(kv->nchunk_max, md.Hkv * qgroups, nseq);
        // A batch of loads asks for that many of a value's QKV partials at once (surplus loads repeat the last one): two where there are no
        // more; six for five or six of them in the launches of three and four query tiles, one trip instead of two (8B shape, 16 x 9 rows, five: 67.5 -> 66.2 us
        // a layer); else four (1B shape, eight: 39.3 us, in sixes 40.8; 70B shape, three and four: the same either way).
        const int pb = parts <= 2 ? 2 : mq >= 3 && (parts == 5 || parts == 6) ? 6 : 4;
#define ATTN_PB(HD, MQ, PB)                                                                                            \
    attn_fused_kernel<T, HD, MQ, SPL, PB><<<grid, 256, 0, st>>>(seq_base, rps, md, w->part, parts, R, w->cs, view(), \
                                                                layer, kv->chunk_keys, kv->nchunk_max, kv->opart, kv->tickets,  \
                                                                (T*)w->attn_out, plane(md.Hq * md.hd), rm())
#define ATTN(HD, MQ)                                                                                                   \
    do { if (pb == 2) ATTN_PB(HD, MQ, 2); else if (pb == 4) ATTN_PB(HD, MQ, 4); else ATTN_PB(HD, MQ, (MQ >= 3 ? 6 : 4)); } while (0)
        if (md.hd == 128) {
            switch (mq) { case 1: ATTN(128, 1); break; case 2: ATTN(128, 2); break; case 3: ATTN(128, 3); break; default: ATTN(128, 4); }
        } else {
            switch (mq) { case 1: ATTN(64, 1); break; case 2: ATTN(64, 2); break; case 3: ATTN(64, 3); break; default: ATTN(64, 4); }
        }
#undef ATTN
#undef ATTN_PB
        LAUNCHCHK("attn_fused");
        return SJ_OK;
    }

    // the same in two launches, for many rows (sj_attn_rows.h); `tail`: only its rows, the last ones of every sequence, want the
    // attention's output (it goes to the tail's operand planes), perhaps none
    int rows_attention(int layer, int parts, const Runner* tail = nullptr) {
        const ModelDims& md = m->md;
        const int q0 = tail ? rps - tail->rps : 0;
        const int blocks = (rps + ROT_POS - 1) / ROT_POS, ntiles = (rps * md.G + 15) / 16, used = ntiles - q0 * md.G / 16;
        u32x4* qbuf = (u32x4*)w->act;
        // waves per tile: as many as leave a workgroup for every CU
        const long long tiles = (long long)used * md.Hkv * nseq;
        const int kw = tiles >= 1024 ? 2 : tiles >= 512 ? 4 : 8;
        const int grid = (used * kw + ROWS_WAVES - 1) / ROWS_WAVES * ((nseq * md.Hkv + 7) / 8 * 8);
        const Runner& to = tail ? *tail : *this;
#define ROWS_ATTN_KW(HD, KW)                                                                                           \
    rows_attn_kernel<T, HD, KW, SPL><<<grid, ROWS_WAVES * 64, 0, st>>>(kv->sp_dev, md, view(), layer, qbuf, ntiles, q0, \
                                                                       (T*)w->attn_out, to.plane(md.Hq * md.hd), to.rm())
#define ROWS_ATTN(HD)                                                                                                  \
    do {                                                                                                               \
        const dim3 rgrid(blocks, 3 * md.Hkv, nseq);                                                                    \
        if (parts <= 2) rows_rotary_kernel<T, HD, SPL, 2><<<rgrid, 256, 0, st>>>(kv->sp_dev, md, w->part, parts, R, w->cs, view(), layer, qbuf, ntiles, q0); \
        else rows_rotary_kernel<T, HD, SPL, 6><<<rgrid, 256, 0, st>>>(kv->sp_dev, md, w->part, parts, R, w->cs, view(), layer, qbuf, ntiles, q0); \
        LAUNCHCHK("rows_rotary");                                                                                      \
        if (q0 == rps) break;                                                                                          \
        if (kw == 2) ROWS_ATTN_KW(HD, 2); else if (kw == 4) ROWS_ATTN_KW(HD, 4); else ROWS_ATTN_KW(HD, 8);             \
        LAUNCHCHK("rows_attn");                                                                                        \
    } while (0)
        if (md.hd == 128) ROWS_ATTN(128); else ROWS_ATTN(64);
#undef ROWS_ATTN
#undef ROWS_ATTN_KW
        return SJ_OK;
    }

    // residual add of `parts` pending split-K partials + RMSNorm into the operand planes (batches of loads as wide as
    // the partials there are: an eight-wide clamped batch for two partials repeats six loads)
    void norm(int parts, const void* gain, float* xn32) { norm_rows(parts, gain, xn32, 0, R, 0, plane(m->md.d), rm()); }
    // rows r0 .. r0 + n - 1 of the block into rows 0 .. of the operand planes and rows o0 .. of xn32
    void norm_rows(int parts, const void* gain, float* xn32, int r0, int n, int o0, size_t oplane, int orm) {
        const int d = m->md.d;
        float *x = w->x + (size_t)r0 * d, *part = w->part + (size_t)r0 * d, *h = xn32 ? xn32 + (size_t)o0 * d : nullptr;
        T* xn = (T*)w->xn;
        if (parts <= 2) add_rmsnorm_kernel<T, 2, SPL><<<n, 1024, 0, st>>>(R, d, m->md.eps, x, part, parts, (const T*)gain, xn, oplane, h, orm);
        else if (parts <= 4) add_rmsnorm_kernel<T, 4, SPL><<<n, 1024, 0, st>>>(R, d, m->md.eps, x, part, parts, (const T*)gain, xn, oplane, h, orm);
        else add_rmsnorm_kernel<T, 8, SPL><<<n, 1024, 0, st>>>(R, d, m->md.eps, x, part, parts, (const T*)gain, xn, oplane, h, orm);
    }

    // a layer behind its attention: O, gate / up, down; after the last one the down projection's K-slices stay pending in w->part
    int feed_forward(int l, int& parts, bool& unscaled) {
        const ModelDims& md = m->md;
        const LayerW& L = m->layers[l];
        int rc;
        if ((rc = close(L.wo, w->attn_out, md.Hq * md.hd, Product::o, L.ffn_norm, 2, unscaled))) return rc;
        if ((rc = time_mark(kv, 3, st))) return rc;
        if ((rc = gate_up(L.wgu, unscaled))) return rc;
        if ((rc = time_mark(kv, 3, st))) return rc;
        if (l + 1 < m->cfg.n_layers) return close(L.wd, w->act, md.F, Product::down, m->layers[l + 1].attn_norm, 4, unscaled);
        if ((rc = time_mark(kv, 4, st))) return rc;
        if ((rc = partial_gemm(L.wd, w->act, md.F, md.d, Product::down, &parts))) return rc;
        return time_mark(kv, 4, st);
    }

    // decoder layers (Eq. 2 / Eq. 4): leaves the last down-projection's K-slices pending in w->part (their number in `parts`).
    // `tail` (a prompt chunk): the runner of the chunk's last rows, the only ones whose final states are wanted, perhaps none.  Nobody reads
    // what the last layer makes of the other rows beyond their keys and values, so behind its QKV projection that layer is the tail's:
    // 509 rows of the 8B shape cut to 4 layers, blocks of 6: 367 us of products and attention over all rows give way to 95.
    int decoder(int& parts, Runner* tail = nullptr) {
        const ModelDims& md = m->md;
        const sj_config& c = m->cfg;
        const int d = md.d, Nq = md.Hq * md.hd, Nk = md.Hkv * md.hd, Nqkv = Nq + 2 * Nk;
        step_begin_kernel<T, SPL><<<R, 1024, 0, st>>>(kv->sp_dev, md, (const T*)m->embed, kv->len_dev, kv->pending_dev, w->x, w->cs, w->row_tok,
                                                  std::log((double)c.rope_base), (const T*)m->layers[0].attn_norm, (T*)w->xn, plane(d), rm());
        LAUNCHCHK("step_begin");
        parts = 0;
        bool unscaled = false;
        int rc;
        for (int l = 0; l < c.n_layers; ++l) {
            const LayerW& L = m->layers[l];
            if ((rc = time_mark(kv, 1, st))) return rc;
            if ((rc = partial_gemm(L.wqkv, w->xn, d, Nqkv, Product::qkv, &parts, unscaled))) return rc;
            if ((rc = time_mark(kv, 1, st))) return rc;
            if (tail && l + 1 == c.n_layers) {
                if ((rc = rows_attention(l, parts, tail))) return rc;
                unscaled = false;
                return tail->R > 0 ? tail->feed_forward(l, parts, unscaled) : SJ_OK;
            }
            if ((rc = attention(l, parts))) return rc;
            if ((rc = feed_forward(l, parts, unscaled))) return rc;
        }
        return SJ_OK;
    }
    int layers() {
        int parts = 0;
        const int rc = decoder(parts);
        if (rc) return rc;
        norm(parts, m->final_norm, kv->hn32);
        LAUNCHCHK("add_rmsnorm");
        return SJ_OK;
    }

    // LM head -> logits + softmax statistics of every row (Eq. 2's p, kept as (max, Z, arg-max)).
    // Hidden states handed in by the caller are already in the storage dtype: one plane suffices then.
    int lm_gemm(bool exact_operand, int& nblk) {
        const ModelDims& md = m->md;
        int rc;
        if (R > FEW_ROWS) {
            rc = exact_operand
                ? gemm_rows<T, EPI_LOGITS, 1>(st, m->lm_head, w->xn, plane(md.d), md.d, md.V, R, 1, kv->logits, nullptr, 0, kv->stats, md.inv_temp)
                : gemm_rows<T, EPI_LOGITS, SPL>(st, m->lm_head, w->xn, plane(md.d), md.d, md.V, R, 1, kv->logits, nullptr, 0, kv->stats, md.inv_temp);
            const int planes = std::is_same<T, float>::value ? 0 : exact_operand ? 1 : SPL;
            nblk = md.V / 16 / (tile_logits(R, md.V / 16, planes) ? TILE_STAT : ROWS_NT);
        } else {
            const GemmPlan p = few_logits_plan(kv->plan_lm, kv->few_rows, md.V / 16, md.d / Traits<T>::KSTEP, R, exact_operand ? 1 : SPL, std::is_same<T, bf16_t>::value, kv->ring_rows);
            rc = exact_operand
                ? few_logits<T, 1>(p, st, m->lm_head, w->xn, plane(md.d), md.d, md.V, R, kv->logits, kv->stats, md.inv_temp)
                : few_logits<T, SPL>(p, st, m->lm_head, w->xn, plane(md.d), md.d, md.V, R, kv->logits, kv->stats, md.inv_temp, few_args(false));
            nblk = md.V / 16 / p.nt;
        }
        return rc;
    }
    // judge_gamma > 0: the judge scores of the gamma draft tokens per sequence (Eq. 5) are computed by the same launch
    // that merges the softmax statistics (tail() is then told that they exist)
    int lm_head(bool exact_operand, int judge_gamma = 0) {
        int nblk = 0;
        const int rc = lm_gemm(exact_operand, nblk);
        if (rc) return rc;
        const ModelDims& md = m->md;
        if (judge_gamma > 0) {
            merge_judge_kernel<T><<<R + nseq * judge_gamma, 256, 0, st>>>(R, kv->stats, nblk, md.inv_temp, kv->rowstat, kv->sp_dev, md.d, kv->hn32,
                                                                          (const T*)m->judge_w, (const T*)m->judge_b, kv->scores, md.V,
                                                                          kv->logits, kv->ranks);
            LAUNCHCHK("merge_judge");
        } else {
            softmax_merge_kernel<<<R, 256, 0, st>>>(kv->stats, nblk, md.inv_temp, kv->rowstat);
            LAUNCHCHK("softmax_merge");
        }
        return SJ_OK;
    }

    // Eq. 3, Eq. 5, scan, extra token, state commit
    int tail(int gamma, bool judged) {
        const ModelDims& md = m->md;
        if (gamma > 0 && !judged) {                        // gamma = 0: a plain decode step (draft proposal)
            judge_kernel<T><<<nseq * gamma, 256, 0, st>>>(kv->sp_dev, md.d, kv->hn32, nullptr, (const T*)m->judge_w, (const T*)m->judge_b, kv->scores,
                                                             md.V, kv->logits, kv->ranks);
            LAUNCHCHK("judge");
        }
        ResampleArgs ra{};
        ra.V = md.V; ra.nslab = kv->nslab; ra.slab_len = kv->slab_len; ra.inv_temp = md.inv_temp;
        ra.logits = kv->logits; ra.rowstat = kv->rowstat; ra.nacc = kv->nacc; ra.epart = kv->epart; ra.wpart = kv->wpart;
        ra.eblk = kv->eblk; ra.wblk = kv->wblk;
        if (md.inv_temp > 0.f && kv->nslab == 256) {       // one workgroup holds the vocabulary
            scan_draw_kernel<<<dim3(1, nseq), 256, 0, st>>>(kv->sp_dev, ra, kv->scores, kv->p_at_d, kv->bits, kv->nacc, kv->ranks, kv->len_dev,
                                                            kv->pending_dev);
            LAUNCHCHK("scan_draw");
            return SJ_OK;
        }
        if (md.inv_temp > 0.f) {
            dim3 g(kv->nslab / 256, nseq);
            scan_resample_e_kernel<<<g, 256, 0, st>>>(kv->sp_dev, ra, kv->scores, kv->p_at_d, kv->bits, kv->nacc, kv->ranks);
            LAUNCHCHK("scan_resample_e");
            if (gamma > 0) {                               // gamma = 0: always the bonus draw from the row itself, no residual
                resample_w_kernel<<<g, 256, 0, st>>>(kv->sp_dev, ra);
                LAUNCHCHK("resample_w");
            }
        } else {
            accept_scan_kernel<<<nseq, 64, 0, st>>>(kv->sp_dev, md.V, md.inv_temp, kv->logits, kv->rowstat, kv->scores, kv->p_at_d,
                                                     kv->bits, kv->nacc, kv->ranks);
            LAUNCHCHK("accept_scan");
        }
        if (gamma == 0 && !(md.inv_temp > 0.f)) {          // a draft block's decode step: its law (T > 0: written by pass 1)
            draft_onehot_kernel<<<dim3(std::min(64, (md.V + 255) / 256), nseq), 256, 0, st>>>(kv->sp_dev, md.V, kv->rowstat);
            LAUNCHCHK("draft_onehot");
        }
        resample_pick_kernel<<<nseq, 256, 0, st>>>(kv->sp_dev, ra, kv->len_dev, kv->pending_dev, kv->scores, kv->p_at_d, kv->bits);
        LAUNCHCHK("resample_pick");
        return SJ_OK;
    }
};

static int set_params(sj_kv* kv, hipStream_t st, const StepParams& p) {
    set_params_kernel<<<1, 1, 0, st>>>(p, kv->sp_dev);
    LAUNCHCHK("set_params");
    return SJ_OK;
}

template <typename T, int SPL>
static int enqueue_step(sj_model* m, sj_kv* kv, int gamma, hipStream_t st, bool head_only, const void* hidden) {
    int rc;
    Runner<T, SPL> run{m, kv, st, kv->batch, gamma + 1, kv->batch * (gamma + 1)};
    if (head_only) {
        hidden_in_kernel<T><<<1024, 256, 0, st>>>((const T*)hidden, (T*)kv->xn, kv->hn32, run.R, m->md.d);
        LAUNCHCHK("hidden_in");
    } else {
        if ((rc = run.layers())) return rc;
    }
    if ((rc = run.lm_head(head_only, gamma))) return rc;
    return run.tail(gamma, gamma > 0);
}

// Launches what `enqueue` puts on a stream, from a launch graph captured once per key: a forward is ~200 dependent launches of a few
// microseconds each.  Only the per-call parameter block, written by a tiny kernel in front of the replay, changes between calls.
template <typename Enqueue>
static int replay(const sj_model* m, sj_kv* kv, int key, hipStream_t st, Enqueue enqueue) {
    if (!kv->use_graph || kv->timing_class != 0) return enqueue(st);
    if (kv->graph_gen != m->temp_gen) {                        // the temperature changed: the graphs hold the old one
        for (auto& g : kv->graphs) (void)hipGraphExecDestroy(g.second);
        kv->graphs.clear();
        kv->graph_gen = m->temp_gen;
    }
    auto it = kv->graphs.find(key);
    if (it == kv->graphs.end()) {
        if (!kv->cap_stream) HIPCHK(hipStreamCreateWithFlags(&kv->cap_stream, hipStreamNonBlocking));
        HIPCHK(hipStreamBeginCapture(kv->cap_stream, hipStreamCaptureModeRelaxed));
        const int rc = enqueue(kv->cap_stream);
        hipGraph_t g = nullptr;
        hipError_t e = hipStreamEndCapture(kv->cap_stream, &g);
        if (rc) { if (g) (void)hipGraphDestroy(g); return rc; }
        if (e != hipSuccess) return fail(SJ_EHIP, "hipStreamEndCapture failed: %s", hipGetErrorString(e));
        hipGraphExec_t ex = nullptr;
        e = hipGraphInstantiate(&ex, g, nullptr, nullptr, 0);
        (void)hipGraphDestroy(g);
        if (e != hipSuccess) return fail(SJ_EHIP, "hipGraphInstantiate failed: %s", hipGetErrorString(e));
        it = kv->graphs.emplace(key, ex).first;
    }
    HIPCHK(hipGraphLaunch(it->second, st));
    return SJ_OK;
}
constexpr int FEED_KEY = 64 * 4;                               // keys below: gamma * 4 + planes, gamma <= 63

template <typename T, int SPL>
static int verify_step_impl(sj_model* m, sj_kv* kv, int gamma, const StepParams& p, hipStream_t st, bool head_only,
                            const void* hidden) {
    const int rc = set_params(kv, st, p);
    if (rc) return rc;
    if (head_only) return enqueue_step<T, SPL>(m, kv, gamma, st, true, hidden);
    return replay(m, kv, gamma * 4 + SPL, st, [&](hipStream_t s) { return enqueue_step<T, SPL>(m, kv, gamma, s, false, nullptr); });
}

static int dispatch_step(sj_model* m, sj_kv* kv, int gamma, const StepParams& p, hipStream_t st, bool head_only,
                         const void* hidden) {
    if (m->cfg.dtype == SJ_DTYPE_FP32) return verify_step_impl<float, 1>(m, kv, gamma, p, st, head_only, hidden);
    switch (kv->planes) {
        case 1: return verify_step_impl<bf16_t, 1>(m, kv, gamma, p, st, head_only, hidden);
        case 3: return verify_step_impl<bf16_t, 3>(m, kv, gamma, p, st, head_only, hidden);
        default: return verify_step_impl<bf16_t, 2>(m, kv, gamma, p, st, head_only, hidden);
    }
}

template <typename T, int SPL>
static int time_kernel_impl(sj_model* m, sj_kv* kv, int cls, int launches, int gamma, hipStream_t st, double* total_ms) {
    Runner<T, SPL> run{m, kv, st, kv->batch, gamma + 1, kv->batch * (gamma + 1)};
    const ModelDims& md = m->md;
    const int d = md.d, Nq = md.Hq * md.hd, Nk = md.Hkv * md.hd;
    hipEvent_t e0, e1;
    HIPCHK(hipEventCreate(&e0));
    HIPCHK(hipEventCreate(&e1));
    int rc = SJ_OK, parts = 0;
    bool unscaled = false;
    HIPCHK(hipEventRecord(e0, st));
    for (int i = 0; i < launches && !rc; ++i) {
        if (cls == 5) {                                          // LM head (1 GB at the paper's vocabulary: no reuse either)
            int nblk = 0;
            rc = run.lm_gemm(m->cfg.n_layers == 0, nblk);
            continue;
        }
        const LayerW& L = m->layers[i % m->cfg.n_layers];        // a different layer each time: no cache reuse
        switch (cls) {
            case 1: rc = run.partial_gemm(L.wqkv, kv->xn, d, Nq + 2 * Nk, Product::qkv); break;
            case 2: rc = run.closing_gemm(L.wo, kv->attn_out, Nq, Product::o, L.ffn_norm, parts, unscaled); break;
            case 3: rc = run.gate_up(L.wgu); break;
            default: rc = run.closing_gemm(L.wd, kv->act, md.F, Product::down, L.ffn_norm, parts, unscaled); break;
        }
    }
    hipError_t e = hipEventRecord(e1, st);
    if (e == hipSuccess) e = hipEventSynchronize(e1);
    float ms = 0.f;
    if (e == hipSuccess) e = hipEventElapsedTime(&ms, e0, e1);
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (rc) return rc;
    if (e != hipSuccess) return fail(SJ_EHIP, "kernel timing failed: %s", hipGetErrorString(e));
    *total_ms = ms;
    return SJ_OK;
}

extern "C" int sj_time_kernel_class(sj_model* m, sj_kv* kv, int32_t kernel_class, int32_t launches, void* stream, double* total_ms) {
    if (!m || !kv || !total_ms) return fail(SJ_EINVAL, "null argument");
    if (kv->m != m) return fail(SJ_EINVAL, "kv was created for a different model");
    if (kernel_class < 1 || kernel_class > 5 || launches < 1) return fail(SJ_EINVAL, "kernel_class must be 1..5, launches >= 1");
    if (kernel_class != 5 && m->cfg.n_layers == 0) return fail(SJ_EINVAL, "a head-only model has only the LM head (class 5)");
    if (kv->last_gamma < 1) return fail(SJ_EINVAL, "run a verification step first (the operands of the last step are reused)");
    hipStream_t st = (hipStream_t)stream;
    if (m->cfg.dtype == SJ_DTYPE_FP32) return time_kernel_impl<float, 1>(m, kv, kernel_class, launches, kv->last_gamma, st, total_ms);
    if (kv->planes == 1) return time_kernel_impl<bf16_t, 1>(m, kv, kernel_class, launches, kv->last_gamma, st, total_ms);
    if (kv->planes == 3) return time_kernel_impl<bf16_t, 3>(m, kv, kernel_class, launches, kv->last_gamma, st, total_ms);
    return time_kernel_impl<bf16_t, 2>(m, kv, kernel_class, launches, kv->last_gamma, st, total_ms);
}

static int check_step_args(sj_model* m, sj_kv* kv, int gamma, const void* a, const void* b, const void* c, const void* d,
                           const void* e) {
    if (!m || !kv) return fail(SJ_EINVAL, "model / kv is null");
    if (kv->m != m) return fail(SJ_EINVAL, "kv was created for a different model");
    if (gamma < 1 || gamma > m->cfg.max_gamma) return fail(SJ_EINVAL, "gamma %d outside 1..%d", gamma, m->cfg.max_gamma);
    if (!a || !b || !c || !d || !e) return fail(SJ_EINVAL, "null device pointer argument");
    return SJ_OK;
}

// A verification call is about to go to `st`: its draw's last kernel also leaves the small per-draft results in host memory where
// they have been asked for.  A call that the caller captures does not, and ends it for the object: which of its calls ran last is then known
// to the caller alone.  (The default stream cannot be captured, and must not be asked while another is.)
static void set_mirror(sj_kv* kv, hipStream_t st, StepParams& p) {
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    if (st && hipStreamIsCapturing(st, &status) != hipSuccess) (void)hipGetLastError();
    if (status != hipStreamCaptureStatusNone) kv->captured = true;
    p.mirror = kv->captured ? nullptr : kv->mirror.load();
    p.mirror_stride = kv->max_rows;
}

extern "C" int sj_verify_step(sj_model* m, sj_kv* kv, int32_t gamma, const int32_t* draft_tokens, const float* draft_probs,
                              const float* uniforms, float judge_threshold, int32_t* accepted_len, int32_t* next_token,
                              void* stream) {
    int rc = check_step_args(m, kv, gamma, draft_tokens, draft_probs, uniforms, accepted_len, next_token);
    if (rc) return rc;
    if (m->cfg.n_layers == 0) return fail(SJ_EINVAL, "head-only model: use sj_verify_head");
    if (!(judge_threshold == judge_threshold)) return fail(SJ_EINVAL, "judge_threshold is NaN");
    // capacity: the host keeps an upper bound of every length; refresh it only when the bound trips
    bool tight = true;
    for (int b = 0; b < kv->batch; ++b) tight = tight && (kv->len_upper[b] + gamma + 1 <= kv->cap[b]);
    if (!tight) {
        if ((rc = refresh_lengths(kv))) return rc;
        for (int b = 0; b < kv->batch; ++b)
            if (kv->len_upper[b] + gamma + 1 > kv->cap[b])
                return fail(SJ_ECAPACITY, "sequence %d: len %d + gamma + 1 exceeds capacity %d", b, kv->len_upper[b], kv->cap[b]);
    }
    StepParams p{};
    p.nseq = kv->batch; p.seq_base = 0; p.rps = gamma + 1; p.gamma = gamma; p.tok_mode = 0; p.mode = kv->mode; p.topk = kv->topk;
    p.theta = judge_threshold;
    p.draft_tokens = draft_tokens; p.draft_probs = draft_probs; p.uniforms = uniforms;
    p.accepted_len = accepted_len; p.next_token = next_token;
    hipStream_t st = (hipStream_t)stream;
    set_mirror(kv, st, p);
    raise_bound(kv, 0, kv->batch, gamma + 1);
    rc = dispatch_step(m, kv, gamma, p, st, false, nullptr);
    if (rc) return rc;
    kv->mirrored = p.mirror != nullptr;
    kv->last_gamma = gamma;
    kv->last_rows = kv->batch * (gamma + 1);
    return SJ_OK;
}

// gamma decode steps - each a verification step without draft tokens: the "all accepted" token is drawn from the row's distribution
// with the step's uniform and becomes the pending token, length += 1 - and, with feed_last, the layers alone (no LM head, no
// decisions) over the last token, whose rows are kept.  The parameters are written once: the steps count themselves, and write
// their column of the block's outputs (a launch between two replays cost a gap of 8 us before and after it, and the layers of the
// last token, launched one by one, 0.4 ms of a 5 ms block).
template <typename T, int SPL>
static int draft_block_impl(sj_model* m, sj_kv* kv, int gamma, bool feed_last, const StepParams& p, hipStream_t st) {
    int rc = set_params(kv, st, p);
    for (int j = 0; j < gamma && !rc; ++j)
        rc = replay(m, kv, SPL, st, [&](hipStream_t s) { return enqueue_step<T, SPL>(m, kv, 0, s, false, nullptr); });
    if (rc || !feed_last) return rc;
    return replay(m, kv, FEED_KEY + SPL, st, [&](hipStream_t s) -> int {
        Runner<T, SPL> run{m, kv, s, kv->batch, 1, kv->batch};
        const int rc2 = run.layers();
        if (rc2) return rc2;
        advance_len_kernel<<<(kv->batch + 63) / 64, 64, 0, s>>>(kv->sp_dev, kv->len_dev);
        LAUNCHCHK("advance_len");
        return SJ_OK;
    });
}

extern "C" int sj_draft_block(sj_model* m, sj_kv* kv, int32_t gamma, const float* uniforms, int32_t feed_last,
                              int32_t* draft_tokens, float* draft_probs, void* stream) {
    if (!m || !kv) return fail(SJ_EINVAL, "model / kv is null");
    if (kv->m != m) return fail(SJ_EINVAL, "kv was created for a different model");
    if (gamma < 1 || gamma > 63) return fail(SJ_EINVAL, "gamma %d outside 1..63", gamma);
    if (!uniforms || !draft_tokens || !draft_probs) return fail(SJ_EINVAL, "null device pointer argument");
    if (m->cfg.n_layers == 0) return fail(SJ_EINVAL, "head-only model has no decode loop");
    const int need = gamma + (feed_last ? 1 : 0);
    hipStream_t st = (hipStream_t)stream;
    int rc = check_room(kv, 0, kv->batch, need);
    if (rc) return rc;
    raise_bound(kv, 0, kv->batch, need);
    StepParams p{};
    p.nseq = kv->batch; p.seq_base = 0; p.rps = 1; p.gamma = 0; p.tok_mode = 0; p.mode = kv->mode; p.topk = kv->topk;
    p.theta = 0.5f;
    p.draft_tokens = nullptr; p.draft_probs = nullptr; p.uniforms = uniforms;
    p.accepted_len = kv->nacc; p.next_token = kv->draft_tok;       // scratch: the tokens go to emit_tokens and the state
    p.emit_gamma = gamma; p.emit_tokens = draft_tokens; p.emit_probs = draft_probs;
    if (m->cfg.dtype == SJ_DTYPE_FP32) rc = draft_block_impl<float, 1>(m, kv, gamma, feed_last != 0, p, st);
    else if (kv->planes == 1) rc = draft_block_impl<bf16_t, 1>(m, kv, gamma, feed_last != 0, p, st);
    else if (kv->planes == 3) rc = draft_block_impl<bf16_t, 3>(m, kv, gamma, feed_last != 0, p, st);
    else rc = draft_block_impl<bf16_t, 2>(m, kv, gamma, feed_last != 0, p, st);
    if (rc) return rc;
    kv->last_gamma = 0;
    kv->last_rows = kv->batch;
    return SJ_OK;
}

// forward + LM head over given tokens, then the gather of the targets' log-probabilities
template <typename T, int SPL>
static int score_impl(sj_model* m, sj_kv* kv, int n, const int32_t* targets, float* logprob, int hrow, float* hidden_out,
                      hipStream_t st) {
    Runner<T, SPL> run{m, kv, st, kv->batch, n, kv->batch * n};
    int rc;
    if ((rc = run.layers())) return rc;
    if ((rc = run.lm_head(false))) return rc;
    const int R = kv->batch * n, work = std::max(R, hidden_out ? kv->batch * m->md.d : 0);
    score_gather_kernel<<<std::min(256, (work + 255) / 256), 256, 0, st>>>(kv->batch, n, m->md.V, m->md.d, m->md.inv_temp, kv->logits,
                                                                       kv->rowstat, targets, logprob, kv->hn32, hrow, hidden_out);
    LAUNCHCHK("score_gather");
    return SJ_OK;
}

extern "C" int sj_score_block(sj_model* m, sj_kv* kv, int32_t n, const int32_t* input_tokens, const int32_t* target_tokens,
                              float* logprob, int32_t hidden_row, float* hidden_out, void* stream) {
    if (!m || !kv) return fail(SJ_EINVAL, "model / kv is null");
    if (kv->m != m) return fail(SJ_EINVAL, "kv was created for a different model");
    if (m->cfg.n_layers == 0) return fail(SJ_EINVAL, "head-only model has no forward");
    if (n < 1 || n > m->cfg.max_gamma + 1) return fail(SJ_EINVAL, "n %d outside 1..max_gamma + 1 = %d", n, m->cfg.max_gamma + 1);
    if (!input_tokens || !target_tokens || !logprob) return fail(SJ_EINVAL, "null device pointer argument");
    if (hidden_out && (hidden_row < 0 || hidden_row >= n)) return fail(SJ_EINVAL, "hidden_row %d outside the block", hidden_row);
    hipStream_t st = (hipStream_t)stream;
    int rc = check_room(kv, 0, kv->batch, n);
    if (rc) return rc;
    StepParams p{};
    p.nseq = kv->batch; p.seq_base = 0; p.rps = n; p.gamma = n - 1; p.tok_mode = 2; p.mode = kv->mode; p.topk = kv->topk;
    p.draft_tokens = input_tokens;
    if ((rc = set_params(kv, st, p))) return rc;
    if (m->cfg.dtype == SJ_DTYPE_FP32) rc = score_impl<float, 1>(m, kv, n, target_tokens, logprob, hidden_row, hidden_out, st);
    else if (kv->planes == 1) rc = score_impl<bf16_t, 1>(m, kv, n, target_tokens, logprob, hidden_row, hidden_out, st);
    else if (kv->planes == 3) rc = score_impl<bf16_t, 3>(m, kv, n, target_tokens, logprob, hidden_row, hidden_out, st);
    else rc = score_impl<bf16_t, 2>(m, kv, n, target_tokens, logprob, hidden_row, hidden_out, st);
    if (rc) return rc;
    kv->last_gamma = 0;
    kv->last_rows = kv->batch * n;
    return SJ_OK;
}

extern "C" int sj_verify_head(sj_model* m, sj_kv* kv, int32_t gamma, const void* hidden, const int32_t* draft_tokens,
                              const float* draft_probs, const float* uniforms, float judge_threshold, int32_t* accepted_len,
                              int32_t* next_token, void* stream) {
    int rc = check_step_args(m, kv, gamma, draft_tokens, draft_probs, uniforms, accepted_len, next_token);
    if (rc) return rc;
    if (!hidden) return fail(SJ_EINVAL, "hidden is null");
    if (!(judge_threshold == judge_threshold)) return fail(SJ_EINVAL, "judge_threshold is NaN");
    StepParams p{};
    p.nseq = kv->batch; p.seq_base = 0; p.rps = gamma + 1; p.gamma = gamma; p.tok_mode = 0; p.mode = kv->mode; p.topk = kv->topk;
    p.theta = judge_threshold;
    p.draft_tokens = draft_tokens; p.draft_probs = draft_probs; p.uniforms = uniforms;
    p.accepted_len = accepted_len; p.next_token = next_token;
    p.step = 0;
    hipStream_t st = (hipStream_t)stream;
    set_mirror(kv, st, p);
    rc = dispatch_step(m, kv, gamma, p, st, true, hidden);
    if (rc) return rc;
    kv->mirrored = p.mirror != nullptr;
    kv->last_gamma = gamma;
    kv->last_rows = kv->batch * (gamma + 1);
    return SJ_OK;
}

// ------------------------------------------------------------------------------------------------
// sj_verify_head for callers that cannot allocate: the workspace lives in a static device array.

constexpr size_t SJ_STATIC_BYTES = SJ_STATIC_WORKSPACE_BYTES;  // per GPU, held until the process ends
static __device__ __align__(256) unsigned char scratch[SJ_STATIC_BYTES];

// The array's device address: looked up once per device with that device current (every GPU holds its own copy).
static int static_scratch_base(unsigned char** out) {
    constexpr int MAXDEV = 64;
    static unsigned char* base[MAXDEV] = {};
    static std::mutex mu;
    int dev = 0;
    HIPCHK(hipGetDevice(&dev));
    if (dev < 0 || dev >= MAXDEV) return fail(SJ_EINVAL, "device index %d not supported by the static workspace", dev);
    std::lock_guard<std::mutex> lock(mu);
    if (!base[dev]) {
        void* p = nullptr;
        HIPCHK(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p) return fail(SJ_EHIP, "hipGetSymbolAddress returned a null address");
        base[dev] = (unsigned char*)p;
    }
    *out = base[dev];
    return SJ_OK;
}

__global__ void fill_i32_kernel(int32_t* p, int n, int32_t v) {
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) p[i] = v;
}

extern "C" int sj_verify_head_static(sj_model* m, int32_t batch, int32_t gamma, const void* hidden, const int32_t* draft_tokens,
                                     const float* draft_probs, const float* uniforms, float judge_threshold,
                                     int32_t* accepted_len, int32_t* next_token, void* stream) {
    if (!m) return fail(SJ_EINVAL, "model is null");
    if (batch < 1) return fail(SJ_EINVAL, "batch must be positive");
    if (gamma < 1 || gamma > m->cfg.max_gamma) return fail(SJ_EINVAL, "gamma %d outside 1..%d", gamma, m->cfg.max_gamma);
    if (!hidden || !draft_tokens || !draft_probs || !uniforms || !accepted_len || !next_token)
        return fail(SJ_EINVAL, "null device pointer argument");
    if (!(judge_threshold == judge_threshold)) return fail(SJ_EINVAL, "judge_threshold is NaN");
    const int64_t R = (int64_t)batch * (gamma + 1);
    const int d = m->cfg.d_model, V = m->cfg.vocab;
    if (R > SJ_STATIC_MAX_ROWS) return fail(SJ_EINVAL, "batch * (gamma + 1) = %lld rows exceed the static workspace's %d", (long long)R, SJ_STATIC_MAX_ROWS);
    unsigned char* base = nullptr;
    int rc = static_scratch_base(&base);
    if (rc) return rc;
    // carve the workspace (256-byte aligned pieces); a shape that does not fit is refused
    sj_kv kv;
    kv.m = m;
    kv.batch = batch;
    kv.max_rows = kv.few_rows = (int)R;
    kv.rpad = ((int)R + 15) / 16 * 16;
    kv.use_graph = false;
    // eight n-tiles a statistic, as the workspace below has it, on either few-row kernel
    if (const GemmPlan ring{8, RING_WAVES, 1, RING_TWO}; logits_fits(ring, V / 16, d * (int)m->esz / 64, (int)R, 1, m->cfg.dtype == SJ_DTYPE_BF16)) kv.plan_lm = ring;
    kv.nslab = std::max(1, (V / 16 + 255) / 256) * 256;
    kv.slab_len = (V + kv.nslab - 1) / kv.nslab;
    size_t off = 0;
    bool fits = true;
    auto take = [&](size_t bytes) -> void* {
        const size_t at = off;
        off = (off + bytes + 255) / 256 * 256;
        if (off > SJ_STATIC_BYTES) { fits = false; return (void*)base; }
        return (void*)(base + at);
    };
    kv.sp_dev = (StepParams*)take(sizeof(StepParams));
    kv.len_dev = (int32_t*)take(sizeof(int32_t) * 2 * batch);
    kv.pending_dev = kv.len_dev + batch;
    kv.xn = take((size_t)kv.rpad * d * m->esz);                // hidden states are in the storage type: one plane
    kv.hn32 = (float*)take((size_t)R * d * 4);
    kv.logits = (float*)take((size_t)R * V * 4);
    kv.stats = (float4*)take((size_t)R * (V / 16) * sizeof(float4));
    kv.rowstat = (float4*)take((size_t)R * sizeof(float4));
    kv.scores = (float*)take((size_t)R * 4);
    kv.ranks = (int32_t*)take((size_t)R * 4);
    kv.p_at_d = (float*)take((size_t)R * 4);
    kv.bits = (int32_t*)take((size_t)R * 4);
    kv.nacc = (int32_t*)take((size_t)batch * 4);
    kv.epart = (double*)take((size_t)batch * kv.nslab * 8);
    kv.wpart = (double*)take((size_t)batch * kv.nslab * 8);
    // the few-row LM head leaves one statistic per 8 n-tiles: the workgroup sums of the draw take the rest of `stats`
    kv.eblk = (double*)(kv.stats + (size_t)R * (V / 128));
    kv.wblk = kv.eblk + (size_t)batch * (kv.nslab / 256);
    if (!fits)
        return fail(SJ_EINVAL, "%lld rows of vocabulary %d, width %d need more than the %zu bytes of the static workspace", (long long)R, V, d,
                    SJ_STATIC_BYTES);
    hipStream_t st = (hipStream_t)stream;
    // the resampling step adds to a length word: it starts at zero on every call (the array keeps the last call's contents)
    fill_i32_kernel<<<1, 256, 0, st>>>(kv.len_dev, 2 * batch, 0);
    LAUNCHCHK("fill_i32");
    StepParams p{};
    p.nseq = batch; p.seq_base = 0; p.rps = gamma + 1; p.gamma = gamma; p.tok_mode = 0; p.mode = SJ_MODE_TWO_STAGE; p.topk = 2;
    p.theta = judge_threshold;
    p.draft_tokens = draft_tokens; p.draft_probs = draft_probs; p.uniforms = uniforms;
    p.accepted_len = accepted_len; p.next_token = next_token;
    p.step = 0;
    return dispatch_step(m, &kv, gamma, p, st, true, hidden);
}

// A prompt of at most max_gamma + 1 tokens is one block of the decode kernels.  A longer one goes through in chunks of up to
// pf_rows rows of nearly equal length: every chunk streams all weights, so their number is what a prompt costs (509 tokens of a
// 4-layer 8B shape: 85 chunks of 6 rows took 36.9 ms).  The LM head, and the final norm, run over the
// rows that a chain of max_gamma + 1 - row blocks would have in its last block; sj_debug_fetch finds them where that chain leaves
// them (rows after those of the last block: the ones just before it).
template <typename T, int SPL>
static int prefill_impl(sj_model* m, sj_kv* kv, int seq, const int32_t* tokens, int n, hipStream_t st) {
    const int block = std::min(kv->max_rows, m->cfg.max_gamma + 1);
    if (n > block) get_chunk(kv);
    const int rows_max = n > block && kv->pf_rows > block ? kv->pf_rows : block;
    const bool long_chunks = rows_max > block;
    const int nchunks = (n + rows_max - 1) / rows_max;
    for (int i = 0; i < nchunks; ++i) {
        const int t0 = long_chunks ? (int)((long long)n * i / nchunks) : i * rows_max;
        const int t1 = long_chunks ? (int)((long long)n * (i + 1) / nchunks) : std::min(n, t0 + rows_max);
        const int cn = t1 - t0;
        const bool last = (t1 == n);
        const Forward* fw = long_chunks ? &kv->chunk : kv;
        HIPCHK(hipMemcpyAsync(fw->prefill_tok, tokens + t0, sizeof(int32_t) * cn, hipMemcpyHostToDevice, st));
        StepParams p{};
        p.nseq = 1; p.seq_base = seq; p.rps = cn; p.gamma = cn - 1; p.tok_mode = 1; p.prefill_tokens = fw->prefill_tok;
        int rc = set_params(kv, st, p);
        if (rc) return rc;
        Runner<T, SPL> run{m, kv, st, 1, cn, cn, fw, seq};
        int head_rows = cn;
        if (!long_chunks) {
            if ((rc = run.layers())) return rc;
        } else {
            int parts = 0;
            const int keep = last ? std::min(block, cn) : 0;   // chunks are longer than a block: cn > block
            Forward tail_fw = *fw;                             // the same buffers, the residual stream from the first kept row on
            tail_fw.x += (size_t)(cn - keep) * m->md.d;
            Runner<T, SPL> tail{m, kv, st, 1, keep, keep, &tail_fw, seq};
            if ((rc = run.decoder(parts, &tail))) return rc;
            if (last) {
                head_rows = n - (n - 1) / block * block;
                Runner<T, SPL> head{m, kv, st, 1, head_rows, head_rows, fw};
                if (keep > head_rows) tail.norm_rows(parts, m->final_norm, kv->hn32, 0, keep - head_rows, head_rows, tail.plane(m->md.d), tail.rm());   // (its operand rows give way to the next ones)
                tail.norm_rows(parts, m->final_norm, kv->hn32, keep - head_rows, head_rows, 0, head.plane(m->md.d), head.rm());
                LAUNCHCHK("add_rmsnorm");
            }
        }
        if (last) {
            Runner<T, SPL> head{m, kv, st, 1, head_rows, head_rows, fw};
            if ((rc = head.lm_head(false))) return rc;
        }
        prefill_commit_kernel<<<1, 1, 0, st>>>(kv->sp_dev, kv->rowstat, kv->len_dev, kv->pending_dev, last ? 1 : 0, head_rows);
        LAUNCHCHK("prefill_commit");
        HIPCHK(hipStreamSynchronize(st));     // the pageable token copy of the next chunk must not race
    }
    return SJ_OK;
}

extern "C" int sj_prefill(sj_model* m, sj_kv* kv, int32_t seq, const int32_t* tokens_host, int32_t n, void* stream) {
    if (!m || !kv || !tokens_host) return fail(SJ_EINVAL, "null argument");
    if (kv->m != m) return fail(SJ_EINVAL, "kv was created for a different model");
    if (m->cfg.n_layers == 0) return fail(SJ_EINVAL, "head-only model has no cache");
    if (seq < 0 || seq >= kv->batch) return fail(SJ_EINVAL, "seq %d out of range", seq);
    if (n < 1) return fail(SJ_EINVAL, "n must be positive");
    for (int i = 0; i < n; ++i)
        if (tokens_host[i] < 0 || tokens_host[i] >= m->cfg.vocab) return fail(SJ_EINVAL, "token %d out of range", i);
    hipStream_t st = (hipStream_t)stream;
    int rc = check_room(kv, seq, seq + 1, n);
    if (rc) return rc;
    raise_bound(kv, seq, seq + 1, n);
    if (m->cfg.dtype == SJ_DTYPE_FP32) rc = prefill_impl<float, 1>(m, kv, seq, tokens_host, n, st);
    else if (kv->planes == 1) rc = prefill_impl<bf16_t, 1>(m, kv, seq, tokens_host, n, st);
    else if (kv->planes == 3) rc = prefill_impl<bf16_t, 3>(m, kv, seq, tokens_host, n, st);
    else rc = prefill_impl<bf16_t, 2>(m, kv, seq, tokens_host, n, st);
    if (rc) return rc;
    kv->last_gamma = 0;
    kv->last_rows = std::min(n, std::min(kv->max_rows, m->cfg.max_gamma + 1));
    return SJ_OK;
}

extern "C" int sj_debug_fetch(const sj_kv* kv, int32_t what, void* dst_host, size_t nbytes) {
    if (!kv || !dst_host) return fail(SJ_EINVAL, "null argument");
    const int R = kv->last_rows, gamma = kv->last_gamma;
    if (R <= 0) return fail(SJ_EINVAL, "no step has run yet");
    const void* src = nullptr;
    size_t want = 0;
    switch (what) {
        case SJ_DBG_LOGITS: src = kv->logits; want = (size_t)R * kv->m->cfg.vocab * 4; break;
        case SJ_DBG_HIDDEN: src = kv->hn32; want = (size_t)R * kv->m->cfg.d_model * 4; break;
        case SJ_DBG_JUDGE_SCORES: src = kv->scores; want = (size_t)kv->batch * gamma * 4; break;
        case SJ_DBG_P_AT_DRAFT: src = kv->p_at_d; want = (size_t)kv->batch * gamma * 4; break;
        case SJ_DBG_ACCEPT_BITS: src = kv->bits; want = (size_t)kv->batch * gamma * 4; break;
        default: return fail(SJ_EINVAL, "unknown debug item %d", what);
    }
    if (want == 0) return fail(SJ_EINVAL, "item not produced by the last call");
    if (nbytes != want) return fail(SJ_EINVAL, "nbytes %zu != expected %zu", nbytes, want);
    // Everything on the device first, on whatever stream: results may come from a graph of the caller's.
    HIPCHK(hipDeviceSynchronize());
    // Per-draft results (a few words a sequence) are then in host memory, from the call after the first fetch on (three small
    // launches and the wait: 21 us, with a copy of 40 bytes behind it 33, of 96 KB 32).
    const int slot = what == SJ_DBG_JUDGE_SCORES ? 0 : what == SJ_DBG_P_AT_DRAFT ? 1 : what == SJ_DBG_ACCEPT_BITS ? 2 : -1;
    if (slot >= 0 && !kv->captured) {
        if (kv->mirrored) {
            std::memcpy(dst_host, kv->mirror + (size_t)slot * kv->max_rows, want);
            return SJ_OK;
        }
        std::lock_guard<std::mutex> lock(kv->mirror_mu);
        if (!kv->mirror) kv->mirror = mirror_take(kv->max_rows);       // null: fetched by copies
    }
    HIPCHK(hipMemcpy(dst_host, src, want, hipMemcpyDeviceToHost));
    return SJ_OK;
}

// the library's other translation units report their errors through this
__attribute__((visibility("hidden"))) int sj_set_error(int code, const char* msg) {
    g_err = msg;
    return code;
}

extern "C" const char* sj_last_error(void) { return g_err.c_str(); }
extern "C" const char* sj_version(void) { return "sj-verify 0.1 (gfx950)"; }
