// libsrm: C ABI and step scheduler for SRM generation on gfx950.
// The exported calls are declared and documented in include/srm.h.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <algorithm>
#include <cstring>
#include <mutex>
#include <new>
#include <string>
#include <vector>

#include "srm.h"
#include "gemm.hpp"
#include "gemm_f32.hpp"
#include "gemm_persist.hpp"
#include "gemm_slices.hpp"
#include "mega.hpp"
#include "mixer.hpp"
#include "norm.hpp"
#include "probe.hpp"
#include "sample.hpp"
#include "tokmix.hpp"

// ------------------------------------------------------------------ errors
static thread_local std::string g_err;

static int fail(int code, const char *fmt, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_err = buf;
    return code;
}

#define HIP_TRY(expr)                                                                       \
    do {                                                                                    \
        hipError_t e_ = (expr);                                                             \
        if (e_ != hipSuccess)                                                               \
            return fail(SRM_EHIP, "%s failed: %s (%s:%d)", #expr, hipGetErrorString(e_),    \
                        __FILE__, __LINE__);                                                \
    } while (0)

#define SRM_TRY(expr)                 \
    do {                              \
        int rc_ = (expr);             \
        if (rc_ != SRM_OK) return rc_; \
    } while (0)

static inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }
static inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// ------------------------------------------------------------------ model
struct LayerDev {
    const float *ln1_g, *ln1_b, *b_in, *alpha, *beta, *lam, *b_out, *ln2_g, *ln2_b, *b_up, *b_down;
    const void *w_in, *w_out, *w_up, *w_down;
};

struct FewLayer;              // (few.hpp)
typedef unsigned long long few_word;
constexpr int kFewDevices = 64;                      // devices that few_launch keeps events for
constexpr int kFewShare = 64, kFewShares = 8;        // CUs of one of its shares of a device; shares at most
constexpr int kFewMaxLayers = 64;                    // their pointers are kept in LDS

struct srm_model {
    srm_config cfg;
    int device;
    int d, ff, V, L, H;
    // The mixer's own geometry: row width dm, Hs heads of which the first hrow are row-repeat.
    // Mixed, row-only and column-only layouts: dm = d, Hs = H.  Combined heads (one row-repeat
    // and one column-repeat matrix per head, outputs added) run as a mixer of width 2d with 2H
    // heads, the H row-repeat ones first: the in-projection's rows and the out-projection's
    // columns are stored twice, so that both halves see the same input and the out-projection
    // adds their outputs.  A mixer with k filters along the hidden dimension (Eq. 11) runs the
    // same way with k copies, all column-repeat, copy i of the in-projection shifted by i rows.
    int dm, Hs, hrow;
    bool noproj;           // non-projected mixer layers
    bool shalf;            // recurrent state (and lambda) in binary16
    size_t ssize;          // bytes per state element
    size_t wsize;          // bytes per matrix element
    void *slab;
    MegaLayer *mega_layers;   // device copy of the layers' pointers for the one-kernel small-batch path, or null
    FewLayer *few_layers;     // ... and for the steps of few.hpp, or null,
    void *few_slab;           // which read matrices packed for them
    unsigned char *few_words; // and, in groups of fp32 rows, exchange words here (see few_group_rows)
    const void *few_head;
    const void *embed, *head;
    const float *lnf_g, *lnf_b;
    std::vector<LayerDev> layers;
    // cached graph of one decode step for srm_generate (see there)
    hipGraphExec_t gexec;
    struct { int64_t B; const void *tok, *state, *store, *ws; float temp; uint32_t seed; float top_p; const void *logits; size_t ws_bytes; const void *pos; int eos_plus1; } gkey;
};

static uint16_t host_f32_to_bf16(float f)
{
    uint32_t u;
    memcpy(&u, &f, 4);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40);   // NaN stays NaN
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

namespace {
struct SlabBuilder {
    std::vector<unsigned char> host;
    size_t add(const float *src, size_t n, bool as_bf16)
    {
        size_t off = align_up(host.size(), 256);
        size_t bytes = n * (as_bf16 ? 2 : 4);
        host.resize(off + bytes);
        if (as_bf16) {
            uint16_t *dst = reinterpret_cast<uint16_t *>(host.data() + off);
            for (size_t i = 0; i < n; ++i) dst[i] = host_f32_to_bf16(src[i]);
        } else {
            memcpy(host.data() + off, src, bytes);
        }
        return off;
    }
};
}  // namespace

extern "C" const char *srm_last_error(void) { return g_err.c_str(); }

// Checks a configuration and fills the sizes derived from it (no device work): what srm_init_weights
// starts with, and all that the host-side planning queries need of a model.
static int model_geometry(const char *who, const srm_config *cfg, srm_model *m)
{
    if (cfg->vocab <= 0 || cfg->d_model <= 0 || cfg->n_layers <= 0 || cfg->n_heads <= 0 ||
        cfg->mlp_expansion <= 0 || cfg->n_ctx <= 0)
        return fail(SRM_EINVAL, "%s: sizes must be positive", who);
    const int layout = cfg->head_layout;
    if (layout < SRM_HEADS_MIXED || layout > SRM_HEADS_COMBINED)
        return fail(SRM_EINVAL, "%s: unknown head_layout %d", who, layout);
    const int kmix = cfg->mixer_kernel > 1 ? cfg->mixer_kernel : 1;
    if (cfg->mixer_kernel < 0 || kmix > cfg->d_model)
        return fail(SRM_EINVAL, "%s: mixer_kernel %d outside [0, d_model]", who, cfg->mixer_kernel);
    if (kmix > 1 && (layout != SRM_HEADS_COLUMN || cfg->no_projections))
        return fail(SRM_EINVAL, "%s: mixer_kernel > 1 needs column-repeat heads and the head projections", who);
    const int slots = cfg->n_heads * (kmix > 1 ? kmix : layout == SRM_HEADS_COMBINED ? 2 : 1);
    if ((layout == SRM_HEADS_MIXED && cfg->n_heads % 2) || slots > kMaxHeads)
        return fail(SRM_EINVAL, "%s: n_heads must be even for mixed heads, and at most %d "
                                "coefficient rows per layer", who, kMaxHeads);
    if (layout == SRM_HEADS_COMBINED && cfg->no_projections)
        return fail(SRM_EINVAL, "%s: combined heads need the head projections", who);
    if (cfg->d_model % (4 * cfg->n_heads))
        return fail(SRM_EINVAL, "%s: d_model must be a multiple of 4*n_heads", who);
    if (cfg->d_model > 4096) return fail(SRM_EINVAL, "%s: d_model > 4096 unsupported", who);
    if (cfg->weight_dtype != SRM_FP32 && cfg->weight_dtype != SRM_BF16)
        return fail(SRM_EINVAL, "%s: unknown weight_dtype %d", who, cfg->weight_dtype);
    if (cfg->weight_dtype == SRM_BF16 && cfg->d_model % 64)
        return fail(SRM_EINVAL, "%s: bf16 needs d_model %% 64 == 0", who);
    if (!(cfg->ln_eps > 0.0f)) return fail(SRM_EINVAL, "%s: ln_eps must be > 0", who);
    if (cfg->state_dtype != SRM_FP32 && cfg->state_dtype != SRM_FP16)
        return fail(SRM_EINVAL, "%s: unknown state_dtype %d", who, cfg->state_dtype);
    m->cfg = *cfg;
    m->device = -1;
    m->d = cfg->d_model; m->ff = cfg->mlp_expansion * cfg->d_model; m->V = cfg->vocab; m->L = cfg->n_layers;
    m->H = cfg->n_heads;
    const int copies = kmix > 1 ? kmix : layout == SRM_HEADS_COMBINED ? 2 : 1;   // times the mixer row repeats the head input
    m->dm = copies * m->d;
    m->Hs = slots;
    m->hrow = layout == SRM_HEADS_MIXED ? m->H / 2 : layout == SRM_HEADS_COLUMN ? 0 : m->H;
    m->noproj = cfg->no_projections != 0;
    m->shalf = cfg->state_dtype == SRM_FP16;
    m->ssize = m->shalf ? 2 : 4;
    m->wsize = cfg->weight_dtype == SRM_BF16 ? 2 : 4;
    m->slab = nullptr;
    m->mega_layers = nullptr;
    m->few_layers = nullptr;
    m->few_slab = nullptr;
    m->few_words = nullptr;
    m->few_head = nullptr;
    m->gexec = nullptr;
    m->gkey = {0, nullptr, nullptr, nullptr, nullptr, 0.0f, 0, 1.0f, nullptr, 0, nullptr, 0};
    return SRM_OK;
}

// Models whose steps of a few rows can be one kernel (few.hpp), the rows that are, and the columns (and computing wavefronts)
// of a work-group.  Measured per step (us, step kernels | one kernel): d = 1024, 16 layers, 32000 tokens: 1 row 349 | 196, 2:
// 355 | 234, 4: 360 | 288; without projections 299 | 148, 302 | 170, 305 | 202; d = 512, 8 layers: 1 row 136 | 73, 2: 137 | 82, 4:
// 138 | 98, without projections 124 | 54, 4: 131 | 69; fp32, d = 256, 4 layers, 4096 tokens, steps of one launch: 1 row 80 | 32, 8:
// 84 | 52 (few_group_rows has shorter ones).  (Eight rows of d = 512 with projections: 141 | 143.)  Eight columns instead of four: d = 1024, 1 row 231 | 213, 4 rows
// 333 | 323; fp32, 1 row 31 | 29, 8 rows 52 | 55.
// The bounds are where the measuring ended, not where the step kernels win (but for those eight rows): the widths are those of
// the benchmark's models, of which the kernel's code exists; it could be made for other multiples of 512 (bf16) and 256 (fp32) up to
// 2048 and 1024, for eight bf16 rows without projections and for 16 fp32 rows.
static int few_max_rows(const srm_model *m)
{
    if (m->dm != m->d || m->ff != 4 * m->d || m->L > kFewMaxLayers || m->V < 4) return 0;
    if (m->wsize == 2) return m->d == 512 || m->d == 1024 ? 4 : 0;
    return m->d == 256 && !m->noproj ? 8 : 0;
}
static int few_columns(const srm_model *m) { return m->wsize == 2 ? 8 : 4; }
static int few_bucket(int64_t B) { return B <= 1 ? 1 : B <= 2 ? 2 : B <= 4 ? 4 : 8; }         // rows the kernel is unrolled for
// Its memory in the workspace, in the place of the row arrays: the nucleus pass's list (Workspace::slow) of B rows, then the words
// of the rows that the kernel is unrolled for.
static size_t few_list_bytes(int64_t B) { return align_up(256 + (size_t)B * 4, 256); }
static size_t few_words_bytes(const srm_model *m, int64_t B)
{
    const size_t gw = m->wsize == 2 ? m->ff / 2 : m->ff;
    return (size_t)few_bucket(B) * ((size_t)2 * m->d + gw + 2 * (m->d / few_columns(m))) * sizeof(few_word) + 256;
}
static size_t few_bytes(const srm_model *m, int64_t B) { return few_list_bytes(B) + few_words_bytes(m, B); }

static bool few_packable(const srm_model *m);
static int few_pack(srm_model *m);

extern "C" int srm_init_weights(const srm_config *cfg, const srm_host_weights *w, srm_model **out)
{
    if (!cfg || !w || !out) return fail(SRM_EINVAL, "srm_init_weights: null argument");
    *out = nullptr;
    srm_model *m = new (std::nothrow) srm_model();
    if (!m) return fail(SRM_ENOMEM, "srm_init_weights: host allocation failed");
    const int grc = model_geometry("srm_init_weights", cfg, m);
    if (grc != SRM_OK) { delete m; return grc; }
    if (!w->embed || !w->head || !w->lnf_g || !w->lnf_b || !w->layers) {
        delete m;
        return fail(SRM_EINVAL, "srm_init_weights: null weight pointer");
    }
    const int d = m->d, L = m->L, H = m->H, V = m->V;
    const int layout = cfg->head_layout;
    const int kmix = cfg->mixer_kernel > 1 ? cfg->mixer_kernel : 1;
    const int slots = m->Hs, copies = m->dm / d;
    const bool comb = layout == SRM_HEADS_COMBINED;
    (void)comb;
    const bool bf = cfg->weight_dtype == SRM_BF16;
    const size_t ff = (size_t)m->ff, nc = cfg->n_ctx;
    for (int l = 0; l < L; ++l) {
        const srm_host_layer &y = w->layers[l];
        const float *ptrs[] = {y.ln1_g, y.ln1_b, y.alpha, y.beta, y.lambda, y.ln2_g, y.ln2_b, y.w_up, y.b_up,
                               y.w_down, y.b_down};
        for (const float *p : ptrs)
            if (!p) { delete m; return fail(SRM_EINVAL, "srm_init_weights: null weight pointer in layer %d", l); }
        if (!cfg->no_projections && (!y.w_in || !y.b_in || !y.w_out || !y.b_out)) {
            delete m;
            return fail(SRM_EINVAL, "srm_init_weights: null projection weights in layer %d", l);
        }
        for (int h = 0; h < slots; ++h)
            if (!(y.lambda[h] > 0.0f && y.lambda[h] <= 1.0f)) {
                delete m;
                return fail(SRM_EINVAL, "srm_init_weights: lambda[%d][%d] = %g outside (0, 1]", l, h,
                            (double)y.lambda[h]);
            }
    }

    struct Offs { size_t v[15]; };
    std::vector<Offs> lo(L);
    size_t o_embed, o_head, o_lnfg, o_lnfb;
    SlabBuilder sb;
    try {
        o_embed = sb.add(w->embed, (size_t)V * d, bf);
        o_head = sb.add(w->head, (size_t)V * d, bf);
        o_lnfg = sb.add(w->lnf_g, d, false);
        o_lnfb = sb.add(w->lnf_b, d, false);
        for (int l = 0; l < L; ++l) {
            const srm_host_layer &y = w->layers[l];
            size_t *o = lo[l].v;
            o[0] = sb.add(y.ln1_g, d, false);          o[1] = sb.add(y.ln1_b, d, false);
            const bool pj = !m->noproj;
            if (copies > 1) {
                // W_in [d][d] -> [copies*d][d], W_out [d][d] -> [d][copies*d] (columns repeated).  Copy i of
                // W_in / b_in holds rows i .. d-1 followed by i zero rows (combined heads: no shift), so that
                // mixer channel i*d + c receives head input c + i, or zero past the last channel (Eq. 11).
                std::vector<float> t((size_t)copies * d * d, 0.0f), tb((size_t)copies * d, 0.0f);
                for (int i = 0; i < copies; ++i) {
                    const int sh = kmix > 1 ? i : 0;
                    memcpy(t.data() + (size_t)i * d * d, y.w_in + (size_t)sh * d, (size_t)(d - sh) * d * 4);
                    memcpy(tb.data() + (size_t)i * d, y.b_in + sh, (size_t)(d - sh) * 4);
                }
                o[2] = sb.add(t.data(), t.size(), bf);
                o[3] = sb.add(tb.data(), tb.size(), false);
            } else {
                o[2] = pj ? sb.add(y.w_in, (size_t)d * d, bf) : 0;   o[3] = pj ? sb.add(y.b_in, d, false) : 0;
            }
            o[4] = sb.add(y.alpha, slots * nc, false);
            if (kmix > 1) {                              // beta [H][n_ctx] is added once: rows of filter 0, zeros after
                std::vector<float> t((size_t)slots * nc, 0.0f);
                memcpy(t.data(), y.beta, (size_t)H * nc * 4);
                o[5] = sb.add(t.data(), t.size(), false);
            } else {
                o[5] = sb.add(y.beta, slots * nc, false);
            }
            if (m->shalf) {                              // decay constants as binary16 values
                float lh[kMaxHeads];
                for (int h = 0; h < slots; ++h) lh[h] = (float)(_Float16)y.lambda[h];
                o[6] = sb.add(lh, slots, false);
            } else {
                o[6] = sb.add(y.lambda, slots, false);
            }
            if (copies > 1) {
                std::vector<float> t((size_t)copies * d * d);
                for (int i = 0; i < d; ++i)
                    for (int c = 0; c < copies; ++c)
                        memcpy(t.data() + ((size_t)i * copies + c) * d, y.w_out + (size_t)i * d, (size_t)d * 4);
                o[7] = sb.add(t.data(), t.size(), bf);
                o[8] = sb.add(y.b_out, d, false);
            } else {
                o[7] = pj ? sb.add(y.w_out, (size_t)d * d, bf) : 0;  o[8] = pj ? sb.add(y.b_out, d, false) : 0;
            }
            o[9] = sb.add(y.ln2_g, d, false);           o[10] = sb.add(y.ln2_b, d, false);
            o[11] = sb.add(y.w_up, ff * d, bf);         o[12] = sb.add(y.b_up, ff, false);
            o[13] = sb.add(y.w_down, (size_t)d * ff, bf); o[14] = sb.add(y.b_down, d, false);
        }
    } catch (const std::bad_alloc &) {
        delete m;
        return fail(SRM_ENOMEM, "srm_init_weights: host staging allocation failed");
    }
    hipError_t e = hipGetDevice(&m->device);
    if (e == hipSuccess) e = hipMalloc(&m->slab, align_up(sb.host.size(), 256));
    if (e != hipSuccess) {
        delete m;
        return fail(e == hipErrorOutOfMemory ? SRM_ENOMEM : SRM_EHIP, "srm_init_weights: hipMalloc(%zu): %s",
                    sb.host.size(), hipGetErrorString(e));
    }
    e = hipMemcpy(m->slab, sb.host.data(), sb.host.size(), hipMemcpyHostToDevice);
    if (e != hipSuccess) {
        (void)hipFree(m->slab);
        delete m;
        return fail(SRM_EHIP, "srm_init_weights: hipMemcpy: %s", hipGetErrorString(e));
    }
    const unsigned char *base = static_cast<const unsigned char *>(m->slab);
    auto F = [&](size_t off) { return reinterpret_cast<const float *>(base + off); };
    m->embed = base + o_embed; m->head = base + o_head;
    m->lnf_g = F(o_lnfg); m->lnf_b = F(o_lnfb);
    m->layers.resize(L);
    for (int l = 0; l < L; ++l) {
        const size_t *o = lo[l].v;
        LayerDev &y = m->layers[l];
        y.ln1_g = F(o[0]); y.ln1_b = F(o[1]); y.w_in = base + o[2]; y.b_in = F(o[3]);
        y.alpha = F(o[4]); y.beta = F(o[5]); y.lam = F(o[6]); y.w_out = base + o[7];
        y.b_out = F(o[8]); y.ln2_g = F(o[9]); y.ln2_b = F(o[10]); y.w_up = base + o[11];
        y.b_up = F(o[12]); y.w_down = base + o[13]; y.b_down = F(o[14]);
    }
    if (!bf && !m->noproj) {
        std::vector<MegaLayer> ml(L);
        for (int l = 0; l < L; ++l) {
            const LayerDev &y = m->layers[l];
            ml[l] = MegaLayer{y.ln1_g, y.ln1_b, static_cast<const float *>(y.w_in), y.b_in, y.alpha, y.beta, y.lam,
                              static_cast<const float *>(y.w_out), y.b_out, y.ln2_g, y.ln2_b,
                              static_cast<const float *>(y.w_up), y.b_up, static_cast<const float *>(y.w_down), y.b_down};
        }
        e = hipMalloc(reinterpret_cast<void **>(&m->mega_layers), sizeof(MegaLayer) * L);
        if (e == hipSuccess) e = hipMemcpy(m->mega_layers, ml.data(), sizeof(MegaLayer) * L, hipMemcpyHostToDevice);
        if (e != hipSuccess) {
            if (m->mega_layers) (void)hipFree(m->mega_layers);
            (void)hipFree(m->slab);
            delete m;
            return fail(SRM_EHIP, "srm_init_weights: layer table: %s", hipGetErrorString(e));
        }
    }
    if (few_packable(m)) {
        const int rc = few_pack(m);
        if (rc != SRM_OK) { srm_free(m); return rc; }
    }
    *out = m;
    return SRM_OK;
}

extern "C" void srm_free(srm_model *m)
{
    if (!m) return;
    if (m->gexec) (void)hipGraphExecDestroy(m->gexec);
    if (m->mega_layers) (void)hipFree(m->mega_layers);
    if (m->few_slab) (void)hipFree(m->few_slab);
    if (m->slab) (void)hipFree(m->slab);
    delete m;
}

extern "C" size_t srm_state_bytes(const srm_model *m, int64_t batch)
{
    if (!m || batch <= 0) return 0;
    return (size_t)m->L * (size_t)batch * (size_t)m->dm * m->ssize;
}

// Layer l's [B][dm] slab of a state array.
static void *layer_state(const srm_model *m, void *state, int l, int64_t B)
{
    return static_cast<unsigned char *>(state) + (size_t)l * (size_t)B * (size_t)m->dm * m->ssize;
}

// ------------------------------------------------------------------ workspace
// Column-tile width that bounds the number of argmax partials per row.
static int head_min_bn(const srm_model *m) { return m->cfg.weight_dtype == SRM_BF16 ? 128 : 64; }

struct Workspace {
    float *x;          // [rows][d]  residual stream
    void *a;           // [rows][d]  activation type
    void *u, *mx;      // [rows][dm] activation type: mixer input and output
    void *g;           // [rows][ff] activation type
    float *pv;         // [rows][nparts]
    int32_t *pi;       // [rows][nparts]
    int *ctr;          // [2] position and step counters of srm_generate
    int *slow;         // [64 + rows] nucleus pass: count, then (from slow + 64) the rows that need the search
    unsigned char *mega;  // [kMegaScratch] one-kernel small-batch path: partial winners and the barrier words
    float *part;       // [d / 128][rows][d] slabs of the one-kernel token mixing where it can run (rows <= kSplitMaxRows), else null
    size_t bytes;
};

// Slabs of the out-projection that the one-kernel token mixing leaves and the following LayerNorm kernel adds to the
// residual stream, in slab order (deterministic): d / 128 of them, for calls of at most kSplitMaxRows rows of a model
// whose token mixing can be one kernel.
constexpr int64_t kSplitMaxRows = 2048;
static bool token_mix_shape_ok(const srm_model *m)
{
    return m->wsize == 2 && !m->noproj && m->dm == m->d && (m->d == 256 || m->d == 512);
}
// fp32 calls of at most kGemvRows rows: the LM head runs as a GEMV, the other GEMMs with finer sums (see gemm_f32.hpp).
constexpr int64_t kGemvRows = 32;

// Scratch of the one-kernel path: [kMegaMaxBlocks][kMegaMaxB] floats, the same of ints, then the barrier's
// 64-byte slots (one per work-group) and its give-up flag.
constexpr size_t kMegaScratch = (size_t)kMegaMaxBlocks * kMegaMaxB * 8 + (size_t)kMegaMaxBlocks * 64 + 256;

static Workspace carve(const srm_model *m, void *base, int64_t rows)
{
    Workspace w;
    unsigned char *p = static_cast<unsigned char *>(base);
    size_t off = 0;
    auto take = [&](size_t bytes) {
        unsigned char *r = p ? p + off : nullptr;
        off += align_up(bytes, 256);
        return r;
    };
    const size_t r = (size_t)rows, d = m->d, dm = m->dm, s = m->wsize;
    const size_t nparts = cdiv(m->V, head_min_bn(m));
    w.x = reinterpret_cast<float *>(take(r * d * 4));
    w.a = take(r * d * s);
    w.u = m->noproj ? w.a : take(r * dm * s);     // without projections the mixer reads the LayerNorm output
    w.mx = take(r * dm * s);
    w.g = take(r * (size_t)m->ff * s);
    w.pv = reinterpret_cast<float *>(take(r * nparts * 4));
    w.pi = reinterpret_cast<int32_t *>(take(r * nparts * 4));
    w.slow = reinterpret_cast<int *>(take(256 + r * 4));
    // sized so that the workspace grows monotonically with the row count
    const size_t slabs = token_mix_shape_ok(m) ? d / kTokMixCols : 0;
    float *part = reinterpret_cast<float *>(take(slabs * std::min<int64_t>(rows, kSplitMaxRows) * d * 4));
    w.part = slabs && rows <= kSplitMaxRows ? part : nullptr;
    w.mega = take(kMegaScratch);
    w.ctr = reinterpret_cast<int *>(take(256));
    w.bytes = off;
    return w;
}

// The arrays of `rows` rows: what every call needs of its workspace, whatever its kernels.
static size_t row_bytes(const srm_model *m, int64_t rows) { return rows > 0 ? carve(m, nullptr, rows).bytes : 0; }

// What srm_workspace_bytes promises to be enough: also for the words of few.hpp, which are more than the arrays of a few rows.  A
// workspace without room for them takes the step kernels.
extern "C" size_t srm_workspace_bytes(const srm_model *m, int64_t rows)
{
    if (!m || rows <= 0) return 0;
    const int few = few_max_rows(m);
    return std::max(row_bytes(m, rows), few ? few_bytes(m, std::min<int64_t>(rows, few)) : 0);
}

// ------------------------------------------------------------------ launchers
template <int BM, int BN, int WM, int WN, int EPI, typename TAct, int NS = 2>
static int launch_bf16_tile(const bf16 *A, const bf16 *W, int M, int N, int K, const GemmEpi &ep, hipStream_t st)
{
    constexpr size_t smem = (size_t)NS * (BM + BN) * 64 * sizeof(bf16);
    auto kern = gemm_bf16_kernel<BM, BN, WM, WN, EPI, TAct, NS>;
    static bool attr_set = false;
    if (!attr_set) {
        HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem));
        attr_set = true;
    }
    const int64_t nb = cdiv(M, BM) * cdiv(N, BN);
    hipLaunchKernelGGL(kern, dim3((unsigned)nb), dim3(WM * WN * 64), smem, st, A, W, M, N, K, ep);
    HIP_TRY(hipGetLastError());
    return SRM_OK;
}

// The 256x256 tile as a persistent kernel (gemm_persist.hpp), one work-group per CU.  It needs two k tiles or more and
// whole quads of columns.
static bool persist_ok(int64_t M, int N, int K)
{
    return K % 64 == 0 && K >= 128 && (N & 3) == 0 && cdiv(M, 256) * cdiv(N, 256) < (1 << 30);
}
static int device_cus()
{
    static thread_local int dev_of = -1, cus_of = 0;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (dev != dev_of) {
        int cus = 0;
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
        dev_of = dev;
        cus_of = cus;
    }
    return cus_of;
}
template <int EPI, typename TAct>
static int launch_bf16_persist(const bf16 *A, const bf16 *W, int M, int N, int K, const GemmEpi &ep, hipStream_t st)
{
    auto kern = gemm_bf16_persist_kernel<EPI, TAct>;
    static bool attr_set = false;
    if (!attr_set) {
        HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, kPersistLds));
        attr_set = true;
    }
    const int cus = device_cus();
    if (cus <= 0) return fail(SRM_EHIP, "cannot read the number of compute units");
    const int64_t nb = cdiv(M, 256) * cdiv(N, 256);
    hipLaunchKernelGGL(kern, dim3((unsigned)std::min<int64_t>(nb, cus)), dim3(512), kPersistLds, st, A, W, M, N, K, ep);
    HIP_TRY(hipGetLastError());
    return SRM_OK;
}

// Few rows: the streaming GEMV (gemv_rows_kernel), 16 * CPG columns per block.
constexpr int kGemvMB = 8;                 // rows per pass over W
constexpr size_t kGemvMaxLds = 128 * 1024;
template <typename TW, typename TAct, int EPI, int CPG, bool LNA = false>
static int launch_gemv_rows(const TAct *A, const TW *W, int M, int N, int K, GemmEpi ep, hipStream_t st,
                            int *nparts_out)
{
    const size_t lds = (size_t)kGemvMB * K * sizeof(float);
    auto kern = gemv_rows_kernel<TW, TAct, EPI, kGemvMB, CPG, LNA>;
    static bool attr_set = false;
    if (!attr_set) {
        HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                    (int)kGemvMaxLds));
        attr_set = true;
    }
    ep.nparts = (int)cdiv(N, 16 * CPG);
    if (nparts_out) *nparts_out = ep.nparts;
    hipLaunchKernelGGL(kern, dim3((unsigned)ep.nparts), dim3(256), lds, st, A, W, M, N, K, ep);
    HIP_TRY(hipGetLastError());
    return SRM_OK;
}
// whether the streaming GEMV applies: few rows, whole 16-byte weight vectors, the rows' stage within LDS
template <typename TW>
static bool gemv_rows_ok(int64_t M, int K)
{
    const int vw = 16 / (int)sizeof(TW);
    return M <= kGemvRows && K % vw == 0 && (size_t)kGemvMB * K * sizeof(float) <= kGemvMaxLds;
}

// The slice form (gemm_slices.hpp) with a tile of 16 RT x 16 CT and a ring of NS line steps per wavefront.
template <int EPI, int RT, int CT, int NS, bool LNA = false>
static int launch_slices_tile(const bf16 *A, const bf16 *W, int M, int N, int K, const GemmEpi &ep, hipStream_t st)
{
    constexpr int rings = kSliceWaves * slices_wave_lds<RT, CT, NS, LNA>();
    const int smem = rings + (LNA ? K / 64 * 2048 : 0);
    auto kern = gemm_bf16_slices_kernel<EPI, RT, CT, NS, LNA>;
    static bool attr_set = false;
    if (!attr_set) {
        HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                    rings + (LNA ? 1024 / 64 * 2048 : 0)));
        attr_set = true;
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)(cdiv(M, 16 * RT) * cdiv(N, 16 * CT))), dim3(kSliceWaves * 64), smem, st, A, W,
                       M, N, K, ep);
    HIP_TRY(hipGetLastError());
    return SRM_OK;
}
// Whether a GEMM takes the slice form: while its 64x64 tiles number at most one per CU.  Measured (us, 64x64 or
// 128x128 tile | slices): 256 x 4096 x 1024, 256 tiles: 8.4 | 6.9; 1024 x 1024 x 1024, 256: 8.5 | 7.0; 1024 x 1024 x
// 4096, 256: 19.1 | 15.8; 1900 x 512 x 2048, 240: 12.2 | 9.7; 300 x 4096 x 1024, 320 tiles: 9.4 | 11.4; 3000 x 512 x
// 512, 376: 7.5 | 9.7 (rows x columns x K).  M is the row count of the whole call: its sums run in another order than
// those of the other tiles, and a prefill or sequence-form call that the workspace cuts into passes does not change with
// the cut (nor does an fp32 step; a bf16 step does, see decode_rows).
// With fewer than five k tiles half of the wavefronts have no slice; there the form ends with its 64x32 tile (2500 x 256 x
// 64: 3.5 | 4.3, x 256: 4.2 | 4.7, 1024 x 1024 x 128: 3.9 | 4.6; with five k tiles it is the faster one again).
static bool slices_ok(int64_t M, int N, int K)
{
    return N % 4 == 0 && K % 64 == 0 && cdiv(M, 64) * cdiv(N, K > 32 * kSliceWaves ? 64 : 32) <= device_cus();
}
// ... and with which tile: the smallest whose tiles still fit the chip in one round, since the time of a work-group
// is proportional to the cache lines it loads (us with tiles of 16x16 | 32x16 | 32x32 | 64x32 | 64x64: 64 x 1024 x
// 4096: 5.2 | 6.5 | 7.6 | 10.5 | 14; 128 x 1024 x 4096 (512 tiles of 16x16): 8.6 | 6.6 | 7.5 | 10 | 14; 300 x 1024 x
// 1024: 7.5 | 7.6 | 6.6 | 5.0 | 6.5; 1024 x 1024 x 1024: 18 | 18 | 12 | 8.7 | 7.0).  Every tile gives the same bits.
template <int EPI>
static int launch_slices(const bf16 *A, const bf16 *W, int M, int N, int K, const GemmEpi &ep, hipStream_t st)
{
    const int cus = device_cus();
    auto fits = [&](int rt, int ct) { return cdiv(M, 16 * rt) * cdiv(N, 16 * ct) <= cus; };
    if (fits(1, 1)) return launch_slices_tile<EPI, 1, 1, 4>(A, W, M, N, K, ep, st);
    if (fits(2, 1)) return launch_slices_tile<EPI, 2, 1, 2>(A, W, M, N, K, ep, st);
    if (fits(2, 2)) return launch_slices_tile<EPI, 2, 2, 2>(A, W, M, N, K, ep, st);
    if (fits(4, 2)) return launch_slices_tile<EPI, 4, 2, 1>(A, W, M, N, K, ep, st);
    return launch_slices_tile<EPI, 4, 4, 1>(A, W, M, N, K, ep, st);
}
// whether the work-groups of a GEMM can make the LayerNorm of their rows themselves (whole k tiles of 128 bytes)
template <typename T>
static bool lna_ok(int64_t M, int N, int K) { return M <= kLnaRows && K <= 1024 && K % (128 / (int)sizeof(T)) == 0 && N % 4 == 0; }
// ... or, bf16, those of several row tiles of 16 that are one round of the chip with the columns
static bool lna_tiles_ok(int64_t M, int N, int K)
{
    return lna_ok<bf16>(1, N, K) && cdiv(M, kLnaRows) * cdiv(N, 16) <= device_cus();
}

// The 64x64 tile with few blocks on the chip: its k loop is bound by the latency of the tile loads, so
// the LDS ring is deepened as far as the blocks per CU allow (8 stages = 128 KB: one block per CU;
// 4 stages = 64 KB: two).
template <int EPI, typename TAct>
static int launch_bf16_small(const bf16 *A, const bf16 *W, int M, int N, int K, const GemmEpi &ep, hipStream_t st)
{
    const int64_t blocks = cdiv(M, 64) * cdiv(N, 64);
    const int kt = K / 64;
    if (blocks <= 256 && kt > 4) return launch_bf16_tile<64, 64, 2, 2, EPI, TAct, 8>(A, W, M, N, K, ep, st);
    if (blocks <= 512 && kt > 2) return launch_bf16_tile<64, 64, 2, 2, EPI, TAct, 4>(A, W, M, N, K, ep, st);
    return launch_bf16_tile<64, 64, 2, 2, EPI, TAct>(A, W, M, N, K, ep, st);
}

// Tile codes of the bf16 GEMM: 0 = 256x256 (8 waves), 1 = 128x128 (4 waves),
// 2 = 64x64 (4 waves), 3 = 128x128 (8 waves), 4 = 256x128 (8 waves); 5 .. 8 pin the
// ring depth of a tile for sweeps, 9 / 10 pin the persistent / one-tile-per-work-group form of 256x256, 11 .. 15 the
// slice form with tiles of 16x16, 32x16, 32x32, 64x32 and 64x64; 16 = 192x256 (8 waves), 17 = 96x128, 18 = 128x64 (4
// waves, ring of four).  min_bn > 64 rules out the 64-wide tile (the LM
// head's partial buffers are sized for column tiles >= 128).  The big tile wins once it fills most of the chip in
// whole rounds (one block per CU; us, 128x128 | 256x256, rows x columns x K: 12544 x 1024 x 1024, 196 tiles: 31.9 | 28.1, 5120
// x 4096 x 1024, 320: 43.6 | 46.1, 6144, 384: 48.2 | 47.2, 6700, 432: 58.3 | 48.4, 13000, 816: 104.3 | 94.2); 128x128 wins
// over 64x64 from about 144 blocks on (700 x 4096 x 1024, 192: 10.2 | 11.4; 2048 x 1024 x 1024, 128: 9.9 | 8.7).
constexpr int kNumTiles = 19;
static int choose_tile(int64_t M, int N, int K, int min_bn)
{
    const int64_t t256 = cdiv(M, 256) * cdiv(N, 256), t128 = cdiv(M, 128) * cdiv(N, 128);
    int tile;
    // (a long k loop makes up for CUs left idle: with K >= 2048 the big tile wins from 160 tiles on)
    const int64_t t256_min = K >= 2048 ? 160 : 200;
    if (t256 >= t256_min && (t256 >= 1024 || t256 < 256 || (double)t256 / (double)(cdiv(t256, 256) * 256) >= 0.8)) tile = 0;
    else if (t128 >= 144) tile = 1;
    else tile = 2;
    if (tile == 2 && min_bn > 64) tile = 1;
    return tile;
}
// Launches whose 256x256 tiles do not fill the chip and whose 128x128 tiles leave the last round part empty: the tile
// that makes one round of it (-1: none does, choose_tile decides).  Measured (us, choose_tile's tile | this; rows x
// columns x K): 128x64 up to 256 tiles: 1300 x 1024 x 4096: 24.6 | 20.3, 2048 x 1024 x 1024: 8.7 | 8.1, 700 x 2048 x
// 1024: 8.4 | 8.0 (384 tiles: 10.2 | 12.9).  96x128 up to 256: 2500 x 1024 x 4096: 27.6 | 25.1, 3000 x 1024 x 1024:
// 10.6 | 9.5, 700 x 4096 x 1024: 10.2 | 9.2 (296: 10.6 | 16.4).  192x256 from 188 to 256: 2500 x 4096 x 1024: 27.9 |
// 22.3 (the 256x256 tile 24.7), 9000 x 1024 x 4096: 91.9 | 65.4 (77.7), 10240 x 1024 x 4096: 82.5 | 69.3 (176 tiles: 27.3 |
// 21.2, 304: 27.7 | 41.2; not while the 128x128 tiles fit two per CU, where its rows are padding: 1000 x 8192 x 2048: 30.8 |
// 34.4, 200 x 32000 x 1024: 23.7 | 27.7), and two or three rounds of it that are full where the 256x256 tile's are not:
// 9000 x 4096 x 1024, 752 of 768: 73.2 | 67.6 (256x256: 70.8), GELU 80.4 | 76.5, residual 6000 x 4096 x 1024: 63.8 | 64.6
// (with K = 512 not with vectors of fp32 to store: residual 9000 x 4096: 64.3 | 68.9, fp32 rows of odd width 81.3 | 85.8;
// GELU 51.3 | 52.5).  Every tile gives the same bits.
// At most one 64x64 tile per CU (one pass of a larger call; calls that small take the slice form): that tile on its deep
// ring (us, 64x64 | 128x64: 200 x 1024 x 1024: 8.2 | 8.1, 1000 x 512 x 2048: 9.1 | 11.6, 512 x 1024 x 4096: 15.4 | 18.9).
// Rows of odd width (N % 4) are stored by element, which the small tiles spread over more wavefronts: where choose_tile
// takes the 64x64 tile, that stays up to about one tile per CU (300 x 1022 x 1024: 8.5 | 8.9, with the residual epilogue
// 10.4 | 15.0; 1800 x 514 x 4096, 261 tiles: 20.7 | 22.5; 297: 25.3 | 21.6), and, unless the epilogue is a plain store, for
// short k loops beyond (us, 64x64 | 96x128, residual: 2100 x 1022 x 512: 13.8 | 19.1, x 1024: 18.0 | 22.2, x 4096: 40.7 |
// 38.5; store, x 512: 10.0 | 9.2).
// slow_update: a state update in the epilogue with a short k loop in front of it or a state in 16 bits, whose rows the
// 64x64 tile takes with twice the wavefronts: 2300 x 512 x 512: 9.6 | 11.0, state in 16 bits 10.6 | 13.4, 2049 x 1024 x
// 1024 so: 15.3 | 19.3; with K = 1024 and a state in 32 bits: 15.6 | 15.0.  (Larger launches than one round of 128x64 take
// the 96x128 tile all the same: 2300 x 1024 x 1024, 16 bits: 23.0 | 20.2.  These with 32x32x16 products.)
static int choose_one_round_tile(int64_t M, int N, int K, bool plain_store, bool slow_update, bool fp32_store)
{
    if (K < 512) return -1;                          // (rings of four k tiles)
    const int64_t t64 = cdiv(M, 64) * cdiv(N, 64);
    if (choose_tile(M, N, K, 64) == 2 && (t64 <= 256 || (N % 4 && (t64 <= 288 || (!plain_store && K < 4096))))) return -1;
    if (cdiv(M, 128) * cdiv(N, 64) <= 256) return slow_update ? -1 : 18;
    if (cdiv(M, 96) * cdiv(N, 128) <= 256) return 17;
    const int64_t t192 = cdiv(M, 192) * cdiv(N, 256), t256 = cdiv(M, 256) * cdiv(N, 256);
    if (t192 >= 188 && t192 <= 256 && cdiv(M, 128) * cdiv(N, 128) > 512) return 16;
    const int64_t r192 = cdiv(t192, 256) * 256, r256 = cdiv(t256, 256) * 256;
    if ((K >= 1024 || !fp32_store) && t192 > 256 && t192 <= 768 && t192 * 20 >= r192 * 19 && t256 * 5 < r256 * 4) return 16;
    return -1;
}
static int tile_bn(int tile) { return tile == 0 || tile >= 9 ? 256 : (tile == 2 || tile >= 6) ? 64 : 128; }

static thread_local int g_force_tile = -1;   // test/bench hook of srm_linear only
static thread_local unsigned long long *g_clock_probe = nullptr;   // measuring hook of srm_linear only
static thread_local int64_t g_clock_blocks = 0;

template <int EPI, typename TAct>
static int launch_bf16(const bf16 *A, const bf16 *W, int64_t M, int N, int K, GemmEpi ep, hipStream_t st,
                       int min_bn, int *nparts_out, int64_t call_rows)
{
    if (K % 64) return fail(SRM_EINVAL, "bf16 GEMM needs K %% 64 == 0 (K = %d)", K);
    if (M <= 0 || M >= (1 << 30) || N <= 0) return fail(SRM_EINVAL, "GEMM shape out of range");
    if ((int64_t)K * 256 * 2 >= (1LL << 31)) return fail(SRM_EINVAL, "bf16 GEMM: K = %d too large", K);
    const int m = (int)M;
    if constexpr (EPI != EPI_ARGMAX)                 // (whose partial winners are counted per 128 columns or more)
        if (g_force_tile < 0 && slices_ok(std::max(M, call_rows), N, K)) return launch_slices<EPI>(A, W, m, N, K, ep, st);
    int tile = g_force_tile;
    if constexpr (EPI != EPI_ARGMAX)
        if (tile < 0) tile = choose_one_round_tile(M, N, K, EPI == EPI_STORE || EPI == EPI_F32,
                                                   EPI == EPI_MIX && (K < 1024 || ep.state_half),
                                                   EPI == EPI_F32 || (EPI == EPI_RESID && N % 4 == 0));
    if (tile < 0) tile = choose_tile(M, N, K, min_bn);
    ep.nparts = (int)cdiv(N, tile_bn(tile));
    if (nparts_out) *nparts_out = ep.nparts;
    switch (tile) {
    case 0:
        if (persist_ok(M, N, K)) return launch_bf16_persist<EPI, TAct>(A, W, m, N, K, ep, st);
        return launch_bf16_tile<256, 256, 2, 4, EPI, TAct>(A, W, m, N, K, ep, st);
    case 1:
        // at most one block per CU: the k loop is bound by the latency of its tile loads (a 128x128x64 tile is
        // 0.27 us of MFMAs, a load about 1 us), so the LDS ring is deepened to keep three tiles in flight
        if (cdiv(M, 128) * cdiv(N, 128) <= 256 && K / 64 > 4)
            return launch_bf16_tile<128, 128, 2, 2, EPI, TAct, 4>(A, W, m, N, K, ep, st);
        return launch_bf16_tile<128, 128, 2, 2, EPI, TAct>(A, W, m, N, K, ep, st);
    case 2: return launch_bf16_small<EPI, TAct>(A, W, m, N, K, ep, st);
    case 3: return launch_bf16_tile<128, 128, 2, 4, EPI, TAct>(A, W, m, N, K, ep, st);
    case 4: return launch_bf16_tile<256, 128, 4, 2, EPI, TAct>(A, W, m, N, K, ep, st);
    // sweeps only: a fixed ring depth
    case 5: return launch_bf16_tile<128, 128, 2, 2, EPI, TAct, 4>(A, W, m, N, K, ep, st);
    case 6: return launch_bf16_tile<64, 64, 2, 2, EPI, TAct, 2>(A, W, m, N, K, ep, st);
    case 7: return launch_bf16_tile<64, 64, 2, 2, EPI, TAct, 4>(A, W, m, N, K, ep, st);
    case 8: return launch_bf16_tile<64, 64, 2, 2, EPI, TAct, 8>(A, W, m, N, K, ep, st);
    case 9:
        // (the pin keeps to an even number >= 4 of k tiles)
        if (!persist_ok(M, N, K) || K % 128 || K < 256) return fail(SRM_EINVAL, "the persistent GEMM does not take this shape");
        return launch_bf16_persist<EPI, TAct>(A, W, m, N, K, ep, st);
    case 10: return launch_bf16_tile<256, 256, 2, 4, EPI, TAct>(A, W, m, N, K, ep, st);
    default: break;
    }
    if constexpr (EPI != EPI_ARGMAX) {
        if (tile == 16) return launch_bf16_tile<192, 256, 2, 4, EPI, TAct>(A, W, m, N, K, ep, st);
        if (tile == 17) return launch_bf16_tile<96, 128, 1, 4, EPI, TAct, 4>(A, W, m, N, K, ep, st);
        if (tile == 18) return launch_bf16_tile<128, 64, 2, 2, EPI, TAct, 4>(A, W, m, N, K, ep, st);
        if (N % 4) return fail(SRM_EINVAL, "the slice form needs N %% 4 == 0 (N = %d)", N);
        switch (tile) {
        case 11: return launch_slices_tile<EPI, 1, 1, 4>(A, W, m, N, K, ep, st);
        case 12: return launch_slices_tile<EPI, 2, 1, 2>(A, W, m, N, K, ep, st);
        case 13: return launch_slices_tile<EPI, 2, 2, 2>(A, W, m, N, K, ep, st);
        case 14: return launch_slices_tile<EPI, 4, 2, 1>(A, W, m, N, K, ep, st);
        case 15: return launch_slices_tile<EPI, 4, 4, 1>(A, W, m, N, K, ep, st);
        default: break;
        }
    }
    return fail(SRM_EINVAL, "GEMM tile code %d does not exist for this epilogue", tile);
}

template <int EPI, int T, int NS, int NA, bool LNA = false>
static int launch_f32_slices(const float *A, const float *W, int M, int N, int K, const GemmEpi &ep, hipStream_t st)
{
    constexpr int rings = f32gemm::kSlices * NS * (LNA ? 1 : 2) * T * f32gemm::BK * (int)sizeof(float);
    const int smem = rings + (LNA ? K * T * (int)sizeof(float) : 0);
    auto kern = gemm_f32_slices_kernel<EPI, T, NS, NA, LNA>;
    static bool attr_set = false;
    if (!attr_set) {
        HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                    rings + (LNA ? 1024 * T * (int)sizeof(float) : 0)));
        attr_set = true;
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)(cdiv(M, T) * cdiv(N, T))), dim3(f32gemm::kSlices * 64), smem, st, A, W, M, N,
                       K, ep);
    HIP_TRY(hipGetLastError());
    return SRM_OK;
}
// The fp32 matrix-core kernels: which tile.  A launch of few tiles takes as long as one tile's trip through K, so
// the tile shrinks until the launch covers the chip; the 64x64 tile needs about a tile per CU.  Measured (graph of
// launches back to back; M x N x K: gemm_f32_kernel | 16 | 32 | 64, microseconds): 128 x 256 x 256: 28 | 3.1 | 4.5 |
// 9.3; 128 x 256 x 1024: 98 | 4.4 | 8.1 | 25; 512 x 256 x 1024 (512 tiles of 16): 98 | 5.9 | 8.2 | 25; 1024 x 256 x
// 1024 (1024 tiles of 16): 98 | 11 | 8.9 | 25; 1024 x 1024 x 256 (256 tiles of 64): 30 | 19 | 10.5 | 10.1;
// 2048 x 256 x 1024 (128 tiles of 64): 124 | 20 | 14.9 | 25; 4096 x 4096 x 256: 134 | 293 | 134 | 99 (87 TFLOP/s of
// the 157 the matrix cores peak at in fp32).  With eight sums per slice, i.e. at most 32 rows, the 32-wide tile also where
// the 64-wide one would be taken, half of whose rows or more do not exist (64 with one sum | 32 with eight: 16 x 16384 x
// 256: 9.3 | 6.7, 16 x 32000 x 256: 14.8 | 11.8, 32 x 32000 x 1024: 42.2 | 30.3).  All tiles give the same bits for one NA
// (see gemm_f32.hpp), which follows the rows of the call.
// LM head: always 64 columns per tile, which its partial winners are counted in.
template <int EPI, int NA>
static int launch_f32_tiles(const float *A, const float *W, int M, int N, int K, const GemmEpi &ep, hipStream_t st)
{
    static_assert(NA == 1 || EPI != EPI_ARGMAX, "the LM head of so few rows is a GEMV");
    const int64_t t64 = cdiv(M, 64) * cdiv(N, 64), t32 = cdiv(M, 32) * cdiv(N, 32), t16 = cdiv(M, 16) * cdiv(N, 16);
    if constexpr (EPI != EPI_ARGMAX) {
        // one work-group per CU: a deeper ring; else two fit a CU
        if (t16 <= 640) return launch_f32_slices<EPI, 16, 4, NA>(A, W, M, N, K, ep, st);
        if (NA > 1 || t64 < 200) {
            if (t32 <= 256) return launch_f32_slices<EPI, 32, 4, NA>(A, W, M, N, K, ep, st);
            return launch_f32_slices<EPI, 32, 2, NA>(A, W, M, N, K, ep, st);
        }
    }
    if constexpr (NA == 1) {
        hipLaunchKernelGGL(gemm_f32_tile_kernel<EPI>, dim3((unsigned)t64), dim3(256), 0, st, A, W, M, N, K, ep);
        HIP_TRY(hipGetLastError());
    }
    return SRM_OK;
}
// Whole 16-byte vectors along K, and of the outputs' rows where the tiles store them as vectors (N % 4 == 0; elements
// otherwise, so that a pass of a call with odd rows takes the kernel of its other passes wherever its output starts);
// byte offsets within a descriptor.
static bool f32_tiles_ok(const float *A, const float *W, int N, int K, const GemmEpi &ep)
{
    const uintptr_t outputs = N % 4 ? 0 : (uintptr_t)ep.out | (uintptr_t)ep.state;
    return K % 4 == 0 && K <= (1 << 20) && (((uintptr_t)A | (uintptr_t)W | outputs) & 15) == 0;
}

template <int EPI>
static int launch_f32(const float *A, const float *W, int64_t M, int N, int K, GemmEpi ep, hipStream_t st,
                      int *nparts_out, int64_t call_rows)
{
    if (M <= 0 || M >= (1 << 30) || N <= 0 || K <= 0) return fail(SRM_EINVAL, "GEMM shape out of range");
    ep.nparts = (int)cdiv(N, 64);
    if (nparts_out) *nparts_out = ep.nparts;
    // The streaming GEMV: the LM head of few rows, operands the tiles do not take, and at most one of its passes
    // (kGemvMB rows) over the widest matrices, where both are bound by reading W and it has less to do beside (us, 32-wide
    // slices | GEMV: 4 x 50000 x 256: 17.2 | 16.6, 4 x 32000 x 256: 11.6 | 10.7, x 64: 6.6 | 6.1; 4 x 24000 x 256: 9.6 |
    // 9.7; 4 x 16384 x 256: 6.6 | 7.7, 4 x 13000 x 1024: 15.4 | 22.1; rows x columns x K).  By the rows of the call: the
    // GEMV sums in an order of its own, see slices_ok.
    const int64_t call = std::max(M, call_rows);
    const bool wide = call <= kGemvMB && N >= 24000;
    if (gemv_rows_ok<float>(call, K) && (EPI == EPI_ARGMAX || wide || !f32_tiles_ok(A, W, N, K, ep))) {
        // (64 columns per block where the partial winners of the LM head are counted per 64 columns, or where 16 would
        // make too many blocks)
        if (EPI == EPI_ARGMAX || N >= 16384) return launch_gemv_rows<float, float, EPI, 4>(A, W, (int)M, N, K, ep, st, nparts_out);
        return launch_gemv_rows<float, float, EPI, 1>(A, W, (int)M, N, K, ep, st, nparts_out);
    } else if (f32_tiles_ok(A, W, N, K, ep)) {
        if constexpr (EPI != EPI_ARGMAX)
            if (call <= kGemvRows) return launch_f32_tiles<EPI, f32gemm::kFine>(A, W, (int)M, N, K, ep, st);
        return launch_f32_tiles<EPI, 1>(A, W, (int)M, N, K, ep, st);
    } else {
        const int64_t nb = cdiv(M, 64) * cdiv(N, 64);
        hipLaunchKernelGGL(gemm_f32_kernel<EPI>, dim3((unsigned)nb), dim3(256), 0, st, A, W, (int)M, N, K, ep);
    }
    HIP_TRY(hipGetLastError());
    return SRM_OK;
}

struct Sampling {          // temp == 0: greedy
    float temp = 0.0f;
    uint32_t seed = 0;
    int pos = 0;
    const int *pos_dev = nullptr;
    const int *pos_rows = nullptr;
    float top_p = 1.0f;    // < 1 (with temp > 0): nucleus truncation, needs the logits in memory
    uint32_t row_base = 0; // sample index of the first row
    int eos_plus1 = 0;     // ragged decode with advance: end-of-sequence token + 1 (0: none)
};

// Nucleus pass over the logits the LM head has just written; tok holds the
// unrestricted Gumbel-max winners and *slow (the row-list counter) is zero.
static int nucleus(const float *logits, int64_t rows, int V, const Sampling &sm, int32_t *tok, int32_t *store,
                   const int *step_dev, int64_t store_stride, int32_t *pos_advance, int *slow, hipStream_t st)
{
    constexpr int NT = 1024, EPT = 32;
    if (V > NT * EPT) {
        // vocabulary too large for the register-resident search: one kernel, searching from memory
        hipLaunchKernelGGL((nucleus_kernel<256, false, false>), dim3((unsigned)rows), dim3(256), 0, st, logits,
                           (int64_t)V, V, sm.temp, sm.top_p, sm.seed, sm.pos, sm.pos_dev, sm.pos_rows, tok, store,
                           step_dev, store_stride, pos_advance, nullptr, nullptr, sm.row_base, sm.eos_plus1);
        HIP_TRY(hipGetLastError());
        return SRM_OK;
    }
    hipLaunchKernelGGL((nucleus_kernel<256, false, true>), dim3((unsigned)rows), dim3(256), 0, st, logits, (int64_t)V,
                       V, sm.temp, sm.top_p, sm.seed, sm.pos, sm.pos_dev, sm.pos_rows, tok, store, step_dev,
                       store_stride, pos_advance, slow, slow + 64, sm.row_base, sm.eos_plus1);
    HIP_TRY(hipGetLastError());
    const unsigned nb = (unsigned)std::min<int64_t>(rows, 256);
    hipLaunchKernelGGL((nucleus_slow_kernel<NT, EPT>), dim3(nb), dim3(NT), 0, st, logits, (int64_t)V, V, sm.temp,
                       sm.top_p, sm.seed, sm.pos, sm.pos_dev, sm.pos_rows, tok, store, step_dev, store_stride,
                       pos_advance, slow, slow + 64, sm.row_base, sm.eos_plus1);
    HIP_TRY(hipGetLastError());
    return SRM_OK;
}

struct MixArgs {           // EPI_MIX: state slab of the layer and its coefficient tables
    void *state = nullptr;
    const float *alpha = nullptr, *beta = nullptr, *lam = nullptr;
    int n_ctx = 0, hrow = 0, dh = 0, state_half = 0;
};

struct LnArgs {            // A = LayerNorm(x) made by the GEMM itself (see lna_ok, lna_tiles_ok)
    const float *x = nullptr, *g = nullptr, *b = nullptr;
    float eps = 0.0f;
};

// out = epilogue(A W^T + bias) with operands of type T (float or bf16).  call_rows: the rows of the whole call where
// M is one of its passes (see slices_ok).
template <int EPI, typename T>
static int linear(const void *A, const void *W, const float *bias, int64_t M, int N, int K, void *out,
                  hipStream_t st, float *pv = nullptr, int32_t *pi = nullptr, int min_bn = 64,
                  int *nparts_out = nullptr, Sampling sm = Sampling(), MixArgs mx = MixArgs(),
                  int64_t call_rows = 0, LnArgs ln = LnArgs())
{
    GemmEpi ep{bias, out, (int64_t)N, pv, pi, 0, sm.temp, sm.seed, sm.pos, sm.pos_dev, sm.pos_rows, sm.row_base,
               mx.state, mx.alpha, mx.beta, mx.lam, mx.n_ctx, mx.hrow, mx.dh, mx.state_half};
    ep.clk = g_clock_probe; ep.clk_blocks = g_clock_blocks;
    if (ln.x) {
        if constexpr (EPI == EPI_STORE || EPI == EPI_GELU || EPI == EPI_MIX) {
            if (M <= 0 || N <= 0 || !(lna_ok<T>(M, N, K) || (sizeof(T) == 2 && lna_tiles_ok(M, N, K))))
                return fail(SRM_EINVAL, "linear: LayerNorm-on-load does not take %lld x %d x %d", (long long)M, N, K);
            ep.ln_x = ln.x; ep.ln_g = ln.g; ep.ln_b = ln.b; ep.ln_eps = ln.eps;
            const T *w = static_cast<const T *>(W);  // (in A's place: not read)
            if constexpr (sizeof(T) == 2) return launch_slices_tile<EPI, 1, 1, 4, true>(w, w, (int)M, N, K, ep, st);
            else return launch_f32_slices<EPI, 16, 4, f32gemm::kFine, true>(w, w, (int)M, N, K, ep, st);
        } else if constexpr (EPI == EPI_ARGMAX && sizeof(T) == 4) {
            if (M <= 0 || N <= 0 || M > kLnaRows || K > 1024 || !gemv_rows_ok<T>(M, K))
                return fail(SRM_EINVAL, "linear: LayerNorm-on-load needs at most %d rows, K <= 1024", kLnaRows);
            ep.ln_x = ln.x; ep.ln_g = ln.g; ep.ln_b = ln.b; ep.ln_eps = ln.eps;
            const T *w = static_cast<const T *>(W);  // (in A's place: not read)
            return launch_gemv_rows<T, T, EPI, 4, true>(w, w, (int)M, N, K, ep, st, nparts_out);
        } else {
            return fail(SRM_EINVAL, "linear: this epilogue has no LayerNorm-on-load");
        }
    }
    if constexpr (sizeof(T) == 2)
        return launch_bf16<EPI, bf16>(static_cast<const bf16 *>(A), static_cast<const bf16 *>(W), M, N, K, ep,
                                      st, min_bn, nparts_out, call_rows);
    else
        return launch_f32<EPI>(static_cast<const float *>(A), static_cast<const float *>(W), M, N, K, ep, st,
                               nparts_out, call_rows);
}

struct TokenStore {        // optional second destination of the greedy tokens (srm_generate)
    int32_t *store = nullptr;
    const int *step_dev = nullptr;
    int64_t stride = 0;
};

static int argmax_finalize(const float *pv, const int32_t *pi, int64_t rows, int nparts, int32_t *out,
                           int64_t row0, int rep, int vocab, hipStream_t st, TokenStore ts = TokenStore(),
                           FinalizeRagged rg = FinalizeRagged{})
{
    hipLaunchKernelGGL(argmax_finalize_kernel, dim3((unsigned)cdiv(rows, kFinalRows)), dim3(256), 0, st, pv, pi, rows,
                       nparts, out, row0, rep, vocab, ts.store, ts.step_dev, ts.stride, rg);
    HIP_TRY(hipGetLastError());
    return SRM_OK;
}

// What a launch's extra work-groups read (see Prefetch), in the order of use: the MLP of layer `mlp`, the projections of layer
// `mix` (-1: none), up to the first matrix above kPrefetchMatrix.  Their sum may exceed the 32 MB of the L2s: what the L2s give
// up the last-level cache still holds.  Decode steps of eight layers of 1536 and 1280 channels (MLP matrices of 18.9 and 13.1
// MB; us, none | the first one | both): 1536 channels, 40 rows 359 | 333 | 347, 300: 556 | 523 | 519, 3001: 2105 | 2028 | 1998,
// without projections 1 row 245 | 252 | 242, 300: 439 | 438 | 411; 1280 channels, 40 rows 300 | 279 | 283, 300: 471 | 450 | 443,
// 3001: 1388 | 1341 | 1288.
constexpr size_t kPrefetchMatrix = (size_t)20 << 20;
static Prefetch prefetch_of(const srm_model *m, int mlp, int mix)
{
    Prefetch pf{};
    int n = 0;
    bool more = true;
    auto add = [&](const void *mat, size_t elems) {
        const size_t bytes = elems * m->wsize;
        more = more && bytes <= kPrefetchMatrix;
        if (!more) return;
        pf.mat[n] = mat;
        pf.bytes[n++] = (uint32_t)bytes;
    };
    if (mlp >= 0) {
        add(m->layers[mlp].w_up, (size_t)m->d * m->ff);
        add(m->layers[mlp].w_down, (size_t)m->d * m->ff);
    }
    if (mix >= 0 && mix < m->L && !m->noproj) {
        add(m->layers[mix].w_in, (size_t)m->d * m->dm);
        add(m->layers[mix].w_out, (size_t)m->d * m->dm);
    }
    return pf;
}
// Extra work-groups of a LayerNorm launch (256 threads each).  For bf16 models whose matrices exceed the 256 MB of the
// last-level cache, so that a step finds them in HBM (the mid model's 74 MB: no gain, up to 2 % slower), and up to 12 288
// rows.  Measured per decode step of the large model (us, without | with): base 24 rows 445 | 436, 200: 605 | 574, 1000:
// 1081 | 1025, 3001: 1957 | 1890, 4000: 2208 | 2206, 8192: 4065 | 3804, 12000: 5582 | 5324, 14000: 6437 | 6441, 16384:
// 6846 | 6985; 17 rows 425 | 432; non-projected layers, whose token mixing is one such launch, 1 row: 322 | 314, 8: 325 |
// 306, 200: 466 | 430, 6000: 2646 | 2490, 16384: 5430 | 5540.  96 work-groups are too few for the time of the launch (30
// rows: 511, 192: 445, 384: 437), 768 no better.  The extra work-groups as part of the GEMM launches cost as much as they
// gave (1 row: 357 | 355).
static int prefetch_blocks(const srm_model *m, int64_t rows, int64_t least, const Prefetch &pf)
{
    const size_t elems = (size_t)m->L * ((m->noproj ? 0 : (size_t)2 * m->d * m->dm) + (size_t)2 * m->d * m->ff) + (size_t)m->V * m->d;
    if (!pf.mat[0] || m->wsize != 2 || elems * m->wsize <= (size_t)256 << 20) return 0;
    const char *e = getenv("SRM_READ_AHEAD");
    if (e && e[0] == '0') return 0;
    return rows >= least && rows <= 12288 ? 256 : 0;
}

template <typename T, bool GATHER>
static int layernorm(const srm_model *m, const float *x_in, int64_t in_stride, const int32_t *tok,
                     float *x_out, const float *g, const float *b, void *out, int64_t rows, hipStream_t st,
                     const int32_t *seq_end = nullptr, int64_t base = 0, int64_t src_rows = 0,
                     const float *part = nullptr, int nsplit = 0, const void *add_act = nullptr,
                     int *advance_ctr = nullptr, Prefetch pf = Prefetch{})
{
    const int d = m->d;
    T *o = static_cast<T *>(out);
    if (!GATHER && !seq_end && !part && !add_act && in_stride == d && rows >= 4096 && d <= 1024 && d % 256 == 0) {
        // plain, many rows: several rows per wavefront
        constexpr int RPW = 2;
        const unsigned nb2 = (unsigned)cdiv(rows, 4 * RPW);
        pf.blocks = prefetch_blocks(m, rows, 24, pf);
        const dim3 grid(nb2 + pf.blocks);
        if (d == 256) hipLaunchKernelGGL((ln_rows_kernel<T, 1, RPW>), grid, dim3(256), 0, st, x_in, g, b, o, rows, d, m->cfg.ln_eps, pf);
        else if (d == 512) hipLaunchKernelGGL((ln_rows_kernel<T, 2, RPW>), grid, dim3(256), 0, st, x_in, g, b, o, rows, d, m->cfg.ln_eps, pf);
        else if (d == 768) hipLaunchKernelGGL((ln_rows_kernel<T, 3, RPW>), grid, dim3(256), 0, st, x_in, g, b, o, rows, d, m->cfg.ln_eps, pf);
        else hipLaunchKernelGGL((ln_rows_kernel<T, 4, RPW>), grid, dim3(256), 0, st, x_in, g, b, o, rows, d, m->cfg.ln_eps, pf);
        HIP_TRY(hipGetLastError());
        return SRM_OK;
    }
    const unsigned nb = (unsigned)cdiv(rows, 4);
    pf.blocks = prefetch_blocks(m, rows, 24, pf);
    const T *emb = static_cast<const T *>(m->embed);
#define LN_CASE(VPL)                                                                                     \
    hipLaunchKernelGGL((ln_kernel<T, T, VPL, GATHER>), dim3(nb + pf.blocks), dim3(256), 0, st, x_in, in_stride, tok, \
                       emb, m->V, x_out, g, b, o, rows, d, m->cfg.ln_eps, seq_end, base, src_rows, part, nsplit,       \
                       (int64_t)rows * d, static_cast<const T *>(add_act), advance_ctr, pf)
    if (d <= 256) LN_CASE(1);
    else if (d <= 512) LN_CASE(2);
    else if (d <= 1024) LN_CASE(4);
    else if (d <= 2048) LN_CASE(8);
    else LN_CASE(16);
#undef LN_CASE
    HIP_TRY(hipGetLastError());
    return SRM_OK;
}

template <typename T>
static int state_update(const srm_model *m, int layer, int pos, int64_t B, const void *u, void *S, void *mx,
                        hipStream_t st, const int *pos_dev = nullptr)
{
    // Two 16-byte state vectors per thread and one pass over the slab (measured
    // best on MI355X: 6.15 TB/s at B = 16384, against 5.55 TB/s with four vectors
    // per thread and a capped grid).  The block count is rounded up so that
    // gridDim * 256 is a multiple of d/4: the kernel relies on a thread keeping
    // one channel group.
    constexpr int UNROLL = 2;
    const LayerDev &y = m->layers[layer];
    const int dv = m->dm / 4;
    const int64_t nvec = B * dv;
    int a = dv, b = 256;
    while (b) { int t = a % b; a = b; b = t; }
    const int step = dv / a;
    const int64_t nb = cdiv(cdiv(nvec, 256 * UNROLL), step) * step;
    if (m->shalf)
        hipLaunchKernelGGL((state_update_kernel<T, UNROLL, f16>), dim3((unsigned)nb), dim3(256), 0, st,
                           static_cast<const T *>(u), static_cast<f16 *>(S), static_cast<T *>(mx), y.alpha, y.beta,
                           y.lam, pos, pos_dev, m->cfg.n_ctx, m->Hs, m->hrow, m->dm, nvec);
    else
        hipLaunchKernelGGL((state_update_kernel<T, UNROLL>), dim3((unsigned)nb), dim3(256), 0, st,
                           static_cast<const T *>(u), static_cast<float *>(S), static_cast<T *>(mx), y.alpha, y.beta,
                           y.lam, pos, pos_dev, m->cfg.n_ctx, m->Hs, m->hrow, m->dm, nvec);
    HIP_TRY(hipGetLastError());
    return SRM_OK;
}

static hipStream_t as_stream(void *s) { return static_cast<hipStream_t>(s); }

static int check_device(const srm_model *m)
{
    int dev = -1;
    HIP_TRY(hipGetDevice(&dev));
    if (dev != m->device)
        return fail(SRM_EINVAL, "model lives on device %d but device %d is current", m->device, dev);
    return SRM_OK;
}

// Whether the state update rides in the in-projection's epilogue (EPI_MIX) instead of running as a
// kernel of its own.  bf16 models: always (few rows: one dependent kernel less per layer; many rows: the
// head input u is never written to memory and read back, 66 MB per layer at 16384 x 1024, measured
// 7.35 -> 7.15 ms per step there).  fp32 models: below 2^20 state elements per layer, where the step is
// bound by its number of kernels; the fp32 tile kernel has not been measured beyond.
// SRM_FUSE_MIXER=0 in the environment keeps the two kernels apart (tests, measurements).
static bool fuse_mixer(const srm_model *m, int64_t rows)
{
    if (m->noproj) return false;
    const char *e = getenv("SRM_FUSE_MIXER");
    if (e && e[0] == '0') return false;
    return m->wsize == 2 || rows * m->dm <= (1 << 20);
}

// A handful of samples: every LayerNorm between two GEMMs of the step is made by the GEMM that consumes it (the
// LNA form of the slice kernels) instead of a launch of its own.  Where the token mixing of a
// layer can be one kernel, that is the shorter step from kTokMixMinRows rows on.  SRM_LN_ON_LOAD=0 in the environment
// keeps the separate kernels.
constexpr int64_t kTokMixMinRows = 9;
static bool ln_on_load(const srm_model *m, int64_t rows)
{
    if (m->noproj || !(m->wsize == 2 ? lna_ok<bf16>(rows, m->dm, m->d) : lna_ok<float>(rows, m->dm, m->d))) return false;
    if (token_mix_shape_ok(m) && rows >= kTokMixMinRows) return false;
    const char *e = getenv("SRM_LN_ON_LOAD");
    return !(e && e[0] == '0');
}

// A dozen to about a thousand rows of a bf16 model with head projections: LayerNorm1, in-projection, state
// update and out-projection of a layer are one kernel (tokmix.hpp), which leaves the out-projection as d / 128
// slabs; the LayerNorm2 kernel adds them to x.  Taken while its work-groups (16 rows x 128 columns each) fit the chip in one
// round: measured on C3's model (d 512, L 8) per step 0.280 -> 0.248 ms at 16 rows, 0.298 -> 0.260 at 64,
// 0.318 -> 0.285 at 256, 0.353 -> 0.310 at 512, 0.378 -> 0.361 at 1024, and 0.473 -> 0.512 at 2048 (two rounds).
// SRM_TOKEN_MIX=0 in the environment keeps the separate kernels, =1 takes the one kernel wherever it can run.
static bool token_mix_one_kernel(const srm_model *m, int64_t rows)
{
    if (!token_mix_shape_ok(m) || ln_on_load(m, rows) || rows > kSplitMaxRows) return false;   // (w.part: see carve)
    if (!fuse_mixer(m, rows)) return false;          // (SRM_FUSE_MIXER=0 asks for the state update as a kernel of its own)
    const char *e = getenv("SRM_TOKEN_MIX");
    if (e && e[0] == '0') return false;
    if (e && e[0] == '1') return true;
    return rows >= kTokMixMinRows && cdiv(rows, 16) * (m->d / kTokMixCols) <= device_cus();
}
// Some dozens of rows of a bf16 model above that: the in-projection still normalises its rows, while tiles of 16 x 16 are one
// round of the chip (the up-projection has more of them and leaves that to a LayerNorm launch).  Decode steps of the large
// model (us, without | with): 17 rows 422 | 407, 24 with combined heads 443 | 440, 37: 445 | 443, 50: 446 | 443, 64 with a
// state in 16 bits 452 | 446.  Of eight layers at other widths: d = 64, 17 rows 135 | 132, 1000: 154 | 147; 128, 17: 140 | 133,
// 500: 152 | 146; 320, 40: 166 | 160; 768, 17: 184 | 179, 80: 203 | 198; 1024, 64: 212 | 205.
static bool in_projection_normalises(const srm_model *m, int64_t rows)
{
    if (m->noproj || m->wsize != 2 || !lna_tiles_ok(rows, m->dm, m->d)) return false;
    const char *e = getenv("SRM_LN_ON_LOAD");
    return !(e && e[0] == '0');
}
struct TokMixCall {
    const float *x;
    void *state;
    Sampling where;
    float *slabs;          // [d / 128][rows][d]
};
static int token_mix(const srm_model *m, int l, const TokMixCall &c, int64_t rows, hipStream_t st)
{
    const LayerDev &y = m->layers[l];
    TokMixArgs a{};
    a.x = c.x;
    a.ln1_g = y.ln1_g; a.ln1_b = y.ln1_b;
    a.eps = m->cfg.ln_eps;
    a.w_in = static_cast<const bf16 *>(y.w_in); a.w_out = static_cast<const bf16 *>(y.w_out);
    a.b_in = y.b_in; a.b_out = y.b_out;
    a.state = c.state;
    a.alpha = y.alpha; a.beta = y.beta; a.lam = y.lam;
    a.n_ctx = m->cfg.n_ctx; a.hrow = m->hrow; a.dh = m->dm / m->Hs;
    a.pos = c.where.pos; a.pos_dev = c.where.pos_dev; a.pos_rows = c.where.pos_rows;
    a.slabs = c.slabs;
    a.rows = rows;
    a.clk = g_clock_probe;
    a.clk_blocks = g_clock_blocks;
    const unsigned nb = (unsigned)(cdiv(rows, 16) * (m->d / kTokMixCols));
#define TOKMIX_LAUNCH(D, TS)                                                                                   \
    do {                                                                                                       \
        auto kern = token_mix_kernel<D, TS>;                                                                   \
        static bool attr_set = false;                                                                          \
        if (!attr_set) {                                                                                       \
            HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void *>(kern),                                  \
                                        hipFuncAttributeMaxDynamicSharedMemorySize, tokmix_lds_bytes<D>()));   \
            attr_set = true;                                                                                   \
        }                                                                                                      \
        hipLaunchKernelGGL(kern, dim3(nb), dim3(256), tokmix_lds_bytes<D>(), st, a);                           \
    } while (0)
    if (m->d == 256) { if (m->shalf) TOKMIX_LAUNCH(256, f16); else TOKMIX_LAUNCH(256, float); }
    else if (m->d == 512) { if (m->shalf) TOKMIX_LAUNCH(512, f16); else TOKMIX_LAUNCH(512, float); }
    else return fail(SRM_EINVAL, "token_mix: d = %d has no one-kernel form", m->d);
#undef TOKMIX_LAUNCH
    HIP_TRY(hipGetLastError());
    return SRM_OK;
}

// The rows of a prefill pass that matter behind the last layer's mixer, each sequence's last one: the state is written, and
// the head reads nothing else.  n rows of the pass, n_call of the call; row b ends at seq_end[b + 1] - base (packed
// sequences) or (b + 1) len.  n = 0: all rows.
struct LastRows {
    int64_t n = 0, n_call = 0, len = 0;
    const int32_t *seq_end = nullptr;
    int64_t base = 0;
};
// Whether a call of N sequences, `rows` rows, the shortest of `shortest`, continues on them.  The gathered rows lie in front of
// the last MLP's activations in w.g, where N sequences of that length leave room.  Behind the gather the last layer's
// out-projection, LayerNorm2 and MLP (3 / 4 of its products or more) run on N rows instead of all; what that saves grows with
// the rows times the width, what it costs is the gather's launch, 3 to 5 us (us per call, all rows | last rows; N x positions:
// d = 1024, 24 layers 1 x 64: 527 | 530, 64 x 3: 619 | 617, 8 x 32: 658 | 655, 256 x 16: 2026 | 1958, 256 x 128: 11833 | 11250; d = 512, 8
// layers 1 x 64: 205 | 208, 8 x 32: 241 | 236, 64 x 64: 503 | 476; fp32, d = 256, 4 layers 32 x 16: 165 | 169, 256 x 3: 176 | 174,
// 1024 x 8: 610 | 523).  A property of the whole call, so that results do not depend on its passes.
static bool last_rows_ok(const srm_model *m, int64_t N, int64_t rows, int64_t shortest)
{
    return (rows - N) * m->d >= (1 << 17) &&
           (size_t)(m->ff + m->dm) * m->wsize + (size_t)m->d * 4 + 512 <= (size_t)shortest * m->ff * m->wsize;
}
template <typename T>
static int gather_last_rows(const srm_model *m, Workspace &w, const LastRows &lr, int64_t rows, hipStream_t st);

// Streams whose kernels may use every CU: on one that keeps off some, work-groups that wait for others may find no room for those,
// whatever they wait for (0.5 us to ask).
// (where a question is refused the kernels without waits do the work, and its error must not be taken for one of theirs)
static bool refused(hipError_t e) { return e != hipSuccess && ((void)hipGetLastError(), true); }
// The default stream by its null name: hipExtStreamGetCUMask reads through the other one, hipStreamLegacy, as through a pointer.
static hipStream_t few_stream(hipStream_t st) { return st == hipStreamLegacy ? nullptr : st; }
static bool whole_device_stream(hipStream_t st)
{
    uint32_t mask[32] = {};
    if (refused(hipExtStreamGetCUMask(few_stream(st), 32, mask))) return false;
    int cus = 0;
    for (const uint32_t bits : mask) cus += __builtin_popcount(bits);
    return cus >= device_cus();
}

// Many rows of a bf16 model: the projections that add to the residual stream also make the LayerNorm behind them
// (EPI_RESID_LN), where both take the 256x256 persistent tile and a row is whole tiles of it, at most kLnTiles.  us, LayerNorm
// launches | this: decode step of the large model 13001 rows 5946 | 5763, 16384: 6727 | 6462, prefill 256 x 128 10946 | 10534, d = 512, state in
// 16 bits, 30001 rows 2976 | 2825; a projection of 16384 x 1024 and its LayerNorm 80.5 + 18.2 | 92.9.  (Smaller launches, in tiles of
// one round, stay as they are: up to 12 288 rows the LayerNorm launches read the next matrices ahead, worth 3 % at 3001 rows.)
// Not where the tiles of a row would lie in two rounds of the chip, and the first of them wait for what is not begun until they have
// left (27000 rows of 1024, us per step, LayerNorm launches | this: 11670 | 17236, with all that is left to the last ones 13960; 53000 of
// 512: 5128 | 5840).  Tiles are dealt in groups of eight row tiles, in line or, where that divides them evenly, an eighth to each XCD.
// (Models without projections have the same down-projection in prefill and sequence form; theirs has not been made.)
// SRM_LN_ON_LOAD=0 in the environment keeps the LayerNorm launches, and so does a stream whose CU mask leaves out some CUs: the tiles of a
// row are not worked on at the same time there, and each waits in vain (16384 rows, us per step of 192 | 128 | 64 CUs: 14485 |
// 13906 | 26490, with LayerNorm launches 10239 | 10561 | 19267).
static bool resid_ln_rounds_ok(int64_t rows, int d)
{
    const int64_t nbn = d / 256, n = cdiv(rows, 256) * nbn, group = 8 * nbn, cus = device_cus();
    if (nbn == 1 || n <= cus) return true;
    return n % 8 ? cus % group == 0 : (cus / 8) % group == 0 && n / 8 % group == 0;
}
static bool resid_ln_ok(const srm_model *m, int64_t rows, int64_t call_rows, hipStream_t st)
{
    if (m->wsize != 2 || m->noproj || m->d % 256 || m->d / 256 > kLnTiles || rows <= 0 || rows >= (1 << 30)) return false;
    if ((int64_t)2 * m->L * cdiv(rows, 256) > 64 + rows) return false;           // (the words lie in w.slow)
    if (!resid_ln_rounds_ok(rows, m->d)) return false;
    for (const int K : {m->dm, m->ff})
        if (slices_ok(std::max(rows, call_rows), m->d, K) || choose_one_round_tile(rows, m->d, K, false, false, true) >= 0 ||
            choose_tile(rows, m->d, K, 64) != 0 || !persist_ok(rows, m->d, K) || K % 64)
            return false;
    const char *e = getenv("SRM_LN_ON_LOAD");
    return !(e && e[0] == '0') && whole_device_stream(st);
}
// SRM_ONE_KERNEL_POLLS in the environment, for tests: a bound of waits, in all launches or ("n:g") in step g of a generate call alone
static unsigned poll_bound(unsigned otherwise, int step = 0)
{
    const char *e = getenv("SRM_ONE_KERNEL_POLLS"), *at = e ? strchr(e, ':') : nullptr;
    return e && (!at || atoi(at + 1) == step) ? (unsigned)std::max(0, atoi(e)) : otherwise;
}
// x += A W^T + bias, out = LayerNorm(x); launch: its number among the `launches` of so many rows in the pass, of which the first clears
// the words of all.  (The last rows of a prefill, which the last layer goes on with, count anew: the words lie by the row tiles.)
constexpr unsigned kLnPolls = 1u << 9;               // some 200 us: the tiles of a row that have been begun come within a few
static int resid_ln(const srm_model *m, Workspace &w, const void *A, const void *W, const float *bias, int64_t rows, int K, const float *g,
                    const float *b, int launch, int launches, hipStream_t st)
{
    const int nbm = (int)cdiv(rows, 256);
    if (launch == 0) {
        const int n = launches * nbm;
        hipLaunchKernelGGL(words_clear_kernel, dim3((unsigned)cdiv(n, 256)), dim3(256), 0, st, w.slow, n);
        HIP_TRY(hipGetLastError());
    }
    GemmEpi ep{bias, w.x, (int64_t)m->d};
    ep.ln_g = g; ep.ln_b = b; ep.ln_eps = m->cfg.ln_eps;
    ep.ln_out = w.a;
    ep.ln_stats = static_cast<float2 *>(w.u);        // (nobody reads u behind the mixer)
    ep.ln_words = reinterpret_cast<unsigned *>(w.slow) + (size_t)launch * nbm;
    ep.ln_polls = poll_bound(kLnPolls);
    ep.clk = g_clock_probe; ep.clk_blocks = g_clock_blocks;
    return launch_bf16_persist<EPI_RESID_LN, bf16>(static_cast<const bf16 *>(A), static_cast<const bf16 *>(W), (int)rows, m->d, K, ep, st);
}

// One block (token mixing + channel mixing) on `rows` token rows.  On entry
// w.a holds LayerNorm1(x) of this layer; mix(l) turns w.u into w.mx.  With
// norm_next, w.a leaves holding the next layer's LayerNorm1(x), or the final
// LayerNorm after the last layer.
// With lnf (decode of a handful of rows, see ln_on_load): no LayerNorm kernels between the GEMMs.  From layer 1 on w.a
// is not used: the in- and up-projection (and the fp32 LM head) normalise the rows of w.x themselves.  Layer 0 enters with w.a from the
// embedding kernel as usual.  With ln1f (see in_projection_normalises) that holds for the in-projection alone.  With one_mix (see token_mix_one_kernel) w.a on entry is not used either.
// call_rows: the rows of the whole call (rows are one of its passes; see slices_ok).  With last rows, what follows the mixer
// is done on those alone, and w.x leaves as them.
template <typename T, typename MIX>
static int block(const srm_model *m, int l, Workspace &w, int64_t rows, int64_t call_rows, hipStream_t st, MIX &&mix,
                 bool norm_next, void *fuse_state = nullptr, Sampling fuse_pos = Sampling(),
                 void *np_state = nullptr, bool lnf = false, bool one_mix = false, bool ln1f = false,
                 const LastRows &last = LastRows())
{
    auto keep_last = [&] {
        if (!last.n) return (int)SRM_OK;
        SRM_TRY((gather_last_rows<T>(m, w, last, rows, st)));
        rows = last.n;
        call_rows = last.n_call;
        return (int)SRM_OK;
    };
    const LayerDev &y = m->layers[l];
    const int d = m->d, dm = m->dm, ff = m->ff;
    const LnArgs ln1 = (lnf || ln1f) && l > 0 ? LnArgs{w.x, y.ln1_g, y.ln1_b, m->cfg.ln_eps} : LnArgs();
    const LnArgs ln2 = lnf ? LnArgs{w.x, y.ln2_g, y.ln2_b, m->cfg.ln_eps} : LnArgs();
    // read ahead: this layer's MLP (and the next layer's projections, if no launch stands in front of them), those projections
    Prefetch pf_mlp = prefetch_of(m, l, ln1f || one_mix ? l + 1 : -1), pf_next = prefetch_of(m, -1, l + 1);
    if constexpr (sizeof(T) == 2) {
        if (one_mix) {
            // token mixing in one kernel, which normalises w.x itself; LayerNorm2 adds its slabs to w.x
            SRM_TRY(token_mix(m, l, TokMixCall{w.x, np_state, fuse_pos, w.part}, rows, st));
            SRM_TRY((layernorm<T, false>(m, w.x, d, nullptr, w.x, y.ln2_g, y.ln2_b, w.a, rows, st, nullptr, 0, 0, w.part,
                                         d / kTokMixCols, nullptr, nullptr, pf_mlp)));
            SRM_TRY((linear<EPI_GELU, T>(w.a, y.w_up, y.b_up, rows, ff, d, w.g, st, nullptr, nullptr, 64, nullptr, Sampling(),
                                         MixArgs(), call_rows)));
            SRM_TRY((linear<EPI_RESID, T>(w.g, y.w_down, y.b_down, rows, d, ff, w.x, st, nullptr, nullptr, 64, nullptr,
                                          Sampling(), MixArgs(), call_rows)));
            if (l + 1 < m->L) return SRM_OK;
            return layernorm<T, false>(m, w.x, d, nullptr, nullptr, m->lnf_g, m->lnf_b, w.a, rows, st);
        }
    }
    if (m->noproj && np_state) {
        // non-projected layer, decode: LayerNorm1, state update, residual add and LayerNorm2 in one kernel
        const unsigned nb = (unsigned)cdiv(rows, 4);
        pf_mlp.blocks = prefetch_blocks(m, rows, 1, pf_mlp);
#define NP_LAUNCH(VPL, TS)                                                                                    \
    hipLaunchKernelGGL((np_token_mix_kernel<T, VPL, TS>), dim3(nb + pf_mlp.blocks), dim3(256), 0, st, w.x,                     \
                       static_cast<TS *>(np_state), static_cast<T *>(w.a), y.ln1_g, y.ln1_b, y.ln2_g, y.ln2_b, \
                       y.alpha, y.beta, y.lam, fuse_pos.pos, fuse_pos.pos_dev, fuse_pos.pos_rows, m->cfg.n_ctx, \
                       m->Hs, m->hrow, d, rows, m->cfg.ln_eps, pf_mlp)
#define NP_CASE(VPL)                                                                                          \
    do {                                                                                                      \
        if (m->shalf) NP_LAUNCH(VPL, f16);                                                                    \
        else NP_LAUNCH(VPL, float);                                                                           \
    } while (0)
        if (d <= 256) NP_CASE(1);
        else if (d <= 512) NP_CASE(2);
        else if (d <= 1024) NP_CASE(4);
        else if (d <= 2048) NP_CASE(8);
        else NP_CASE(16);
#undef NP_CASE
#undef NP_LAUNCH
        HIP_TRY(hipGetLastError());
    } else if (m->noproj) {
        // non-projected layer: mixer on the LayerNorm output, its result added to x by the LayerNorm kernel
        SRM_TRY(mix(l));
        SRM_TRY(keep_last());
        SRM_TRY((layernorm<T, false>(m, w.x, d, nullptr, w.x, y.ln2_g, y.ln2_b, w.a, rows, st, nullptr, 0, 0, nullptr,
                                     0, w.mx, nullptr, pf_mlp)));
    } else if (fuse_state) {
        // few rows: the state update rides in the in-projection's epilogue (one kernel less per layer)
        const MixArgs mx{fuse_state, y.alpha, y.beta, y.lam, m->cfg.n_ctx, m->hrow, dm / m->Hs, m->shalf ? 1 : 0};
        SRM_TRY((linear<EPI_MIX, T>(w.a, y.w_in, y.b_in, rows, dm, d, w.mx, st, nullptr, nullptr, 64, nullptr, fuse_pos,
                                    mx, call_rows, ln1)));
    } else {
        SRM_TRY((linear<EPI_STORE, T>(w.a, y.w_in, y.b_in, rows, dm, d, w.u, st, nullptr, nullptr, 64, nullptr, Sampling(),
                                      MixArgs(), call_rows, ln1)));
        SRM_TRY(mix(l));
        SRM_TRY(keep_last());
    }
    const bool fused_ln = resid_ln_ok(m, rows, call_rows, st);
    const int fused_at = last.n ? 0 : 2 * l, fused_n = last.n ? 2 : 2 * m->L;
    if (fused_ln) {
        SRM_TRY(resid_ln(m, w, w.mx, y.w_out, y.b_out, rows, dm, y.ln2_g, y.ln2_b, fused_at, fused_n, st));
    } else if (!m->noproj) {
        SRM_TRY((linear<EPI_RESID, T>(w.mx, y.w_out, y.b_out, rows, d, dm, w.x, st, nullptr, nullptr, 64, nullptr, Sampling(),
                                      MixArgs(), call_rows)));
        if (!lnf) SRM_TRY((layernorm<T, false>(m, w.x, d, nullptr, nullptr, y.ln2_g, y.ln2_b, w.a, rows, st, nullptr, 0, 0,
                                               nullptr, 0, nullptr, nullptr, pf_mlp)));
    }
    SRM_TRY((linear<EPI_GELU, T>(w.a, y.w_up, y.b_up, rows, ff, d, w.g, st, nullptr, nullptr, 64, nullptr, Sampling(),
                                 MixArgs(), call_rows, ln2)));
    if (fused_ln && norm_next)
        return resid_ln(m, w, w.g, y.w_down, y.b_down, rows, ff, l + 1 < m->L ? m->layers[l + 1].ln1_g : m->lnf_g,
                        l + 1 < m->L ? m->layers[l + 1].ln1_b : m->lnf_b, fused_at + 1, fused_n, st);
    SRM_TRY((linear<EPI_RESID, T>(w.g, y.w_down, y.b_down, rows, d, ff, w.x, st, nullptr, nullptr, 64, nullptr, Sampling(),
                                  MixArgs(), call_rows)));
    if ((lnf || ln1f) && l + 1 < m->L) return SRM_OK;              // the next layer's in-projection normalises
    if (norm_next && !(m->noproj && np_state && l + 1 < m->L)) {   // the fused kernel does its own LayerNorm1
        const float *g = l + 1 < m->L ? m->layers[l + 1].ln1_g : m->lnf_g;
        const float *b = l + 1 < m->L ? m->layers[l + 1].ln1_b : m->lnf_b;
        SRM_TRY((layernorm<T, false>(m, w.x, d, nullptr, nullptr, g, b, w.a, rows, st, nullptr, 0, 0, nullptr, 0, nullptr,
                                     nullptr, pf_next)));
    }
    return SRM_OK;
}

// LM head on M normalised rows `a` (of call_rows in the whole call): optional fp32 logits, greedy token written
// `rep` times at d_tok[(row0 + row) * rep + r].
template <typename T>
static int head_argmax(const srm_model *m, const Workspace &w, const void *a, int64_t M, int64_t call_rows, float *logits,
                       int32_t *d_tok, int64_t row0, int rep, hipStream_t st, TokenStore ts = TokenStore(),
                       Sampling sm = Sampling(), FinalizeRagged rg = FinalizeRagged{}, LnArgs ln = LnArgs())
{
    int nparts = 0;
    SRM_TRY((linear<EPI_ARGMAX, T>(a, m->head, nullptr, M, m->V, m->d, logits, st, w.pv, w.pi, head_min_bn(m),
                                   &nparts, sm, MixArgs(), call_rows, ln)));
    return argmax_finalize(w.pv, w.pi, M, nparts, d_tok, row0, rep, m->V, st, ts, rg);
}

// ------------------------------------------------------------------ decode
// One decode step for the rows b0 .. b0+nb-1 of a batch of B samples; uniform position
// (pos / pos_dev) or one position per sample (pos_rows, base pointer of the batch).
struct DecodeArgs {
    int64_t B;
    int pos;
    const int *pos_dev;
    int32_t *pos_rows;
    int advance;
    const int32_t *tok_in;
    void *state;
    int32_t *tok_out;
    float *logits, *hidden;
    TokenStore ts;
    float temperature;
    uint32_t seed;
    float top_p;
    int eos_plus1 = 0;
    int *advance_ctr = nullptr;     // step counters of srm_generate, advanced by the first kernel of the step
    size_t ws_bytes = 0;
    int step = 0;                   // of a generate call
    unsigned *gave_up = nullptr;    // ... whose steps may be kernels of all layers: not zero behind a wait that has given up
};
static bool stack_ok(const srm_model *m, int64_t rows, size_t ws_bytes, hipStream_t st);
static int stack_layers(srm_model *m, const DecodeArgs &a, const Workspace &w, int64_t b0, int64_t nb, hipStream_t st, const unsigned **dead);

template <typename T>
static int decode_rows(srm_model *m, const DecodeArgs &a, int64_t b0, int64_t nb, void *ws, hipStream_t st)
{
    Workspace w = carve(m, ws, nb);
    const int d = m->d, dm = m->dm;
    int32_t *pos_rows = a.pos_rows ? a.pos_rows + b0 : nullptr;
    auto slab = [&](int l) {       // rows b0.. of layer l's state
        return static_cast<void *>(static_cast<unsigned char *>(layer_state(m, a.state, l, a.B)) +
                                   (size_t)b0 * dm * m->ssize);
    };
    const bool stacked = sizeof(T) == 2 && stack_ok(m, nb, a.ws_bytes, st);
    const unsigned *dead = a.gave_up;
    if (stacked) SRM_TRY(stack_layers(m, a, w, b0, nb, st, &dead));
    else SRM_TRY((layernorm<T, true>(m, nullptr, 0, a.tok_in + b0, w.x, m->layers[0].ln1_g, m->layers[0].ln1_b, w.a, nb,
                                     st, nullptr, 0, 0, nullptr, 0, nullptr, b0 == 0 ? a.advance_ctr : nullptr,
                                     prefetch_of(m, -1, 0))));
    auto mix = [&](int l) {
        if (!pos_rows) return state_update<T>(m, l, a.pos, nb, w.u, slab(l), w.mx, st, a.pos_dev);
        const LayerDev &y = m->layers[l];
        const int64_t nvec = nb * (dm / 4);
        if (m->shalf)
            hipLaunchKernelGGL((state_update_ragged_kernel<T, f16>), dim3((unsigned)cdiv(nvec, 256)), dim3(256), 0, st,
                               static_cast<const T *>(w.u), static_cast<f16 *>(slab(l)), static_cast<T *>(w.mx),
                               y.alpha, y.beta, y.lam, pos_rows, m->cfg.n_ctx, m->Hs, m->hrow, dm, nvec);
        else
            hipLaunchKernelGGL((state_update_ragged_kernel<T>), dim3((unsigned)cdiv(nvec, 256)), dim3(256), 0, st,
                               static_cast<const T *>(w.u), static_cast<float *>(slab(l)), static_cast<T *>(w.mx),
                               y.alpha, y.beta, y.lam, pos_rows, m->cfg.n_ctx, m->Hs, m->hrow, dm, nvec);
        HIP_TRY(hipGetLastError());
        return (int)SRM_OK;
    };
    const bool fuse = fuse_mixer(m, nb);          // (same bits either way)
    const Sampling where{0.0f, 0, a.pos, a.pos_dev, pos_rows, 1.0f, 0};
    // A slice of a bf16 step takes the kernels of its own rows; fp32 results do not depend on the slicing, so whatever sums
    // in an order of its own follows the call there.  (4096 rows through a 512-row workspace, d = 1024: 6272 us by the
    // slice's rows, 9478 with the slice form of the GEMMs by the call's.)
    const int64_t call_rows = sizeof(T) == 4 ? a.B : nb;
    const bool lnf = ln_on_load(m, call_rows);
    const bool tm = token_mix_one_kernel(m, call_rows);
    const bool ln1f = !lnf && !tm && in_projection_normalises(m, call_rows);
    // ... and the LM head the last one, where it is the fp32 GEMV (bf16: one launch of many, for 64 rows of a tile)
    const bool head_norm = lnf && sizeof(T) == 4;
    for (int l = 0; l < m->L && !stacked; ++l)
        SRM_TRY((block<T>(m, l, w, nb, call_rows, st, mix, !head_norm, fuse ? slab(l) : nullptr, where, slab(l), lnf, tm,
                          ln1f)));
    if (a.hidden && !stacked)
        HIP_TRY(hipMemcpyAsync(a.hidden + (size_t)b0 * d, w.x, (size_t)nb * d * 4, hipMemcpyDeviceToDevice, st));
    const Sampling sm{a.temperature, a.seed, a.pos, a.pos_dev, pos_rows, a.top_p, (uint32_t)b0, a.eos_plus1};
    const bool topp = a.temperature > 0.0f && a.top_p < 1.0f;
    FinalizeRagged rg{};
    if (a.pos_rows) {
        rg.pos_rows = a.pos_rows;             // indexed with row0 + row
        rg.advance = a.advance && !topp;      // with a nucleus pass the positions move after it
        rg.n_ctx = m->cfg.n_ctx;
        rg.eos_plus1 = a.eos_plus1;
    }
    if (topp) rg.zero_counter = w.slow;
    rg.dead = dead;
    float *lg = a.logits ? a.logits + (size_t)b0 * m->V : nullptr;
    SRM_TRY((head_argmax<T>(m, w, w.a, nb, call_rows, lg, a.tok_out, b0, 1, st, a.ts, sm, rg,
                            head_norm ? LnArgs{w.x, m->lnf_g, m->lnf_b, m->cfg.ln_eps} : LnArgs())));
    if (topp)
        SRM_TRY(nucleus(lg, nb, m->V, sm, a.tok_out + b0, a.ts.store ? a.ts.store + b0 : nullptr, a.ts.step_dev,
                        a.ts.stride, (pos_rows && a.advance) ? pos_rows : nullptr, w.slow, st));
    return SRM_OK;
}

// Rows per pass of a decode call: the whole batch if the workspace holds it, else as many
// rows as it holds (the samples are independent, so a step can be taken in slices; this lets
// a caller keep far more sequences resident than one workspace covers).  0: too small.
// row_bytes(rows) = the row arrays + 256 bytes that srm_generate uses for its step
// counters at the very end of the caller's buffer, so the row arrays get workspace_bytes - 256.
static int64_t decode_rows_per_pass(const srm_model *m, int64_t B, size_t workspace_bytes)
{
    if (row_bytes(m, B) <= workspace_bytes) return B;
    int64_t lo = 0, hi = B;
    while (lo < hi) {
        const int64_t mid = (lo + hi + 1) / 2;
        if (row_bytes(m, mid) <= workspace_bytes) lo = mid; else hi = mid - 1;
    }
    if (lo >= 256) lo = lo / 256 * 256;       // whole GEMM tiles per pass
    return lo < std::min<int64_t>(B, 256) ? 0 : lo;
}

static int decode_batch(srm_model *m, DecodeArgs a, void *ws, size_t workspace_bytes, hipStream_t st)
{
    a.ws_bytes = workspace_bytes;
    const int64_t rpp = decode_rows_per_pass(m, a.B, workspace_bytes);
    if (rpp <= 0) return fail(SRM_ENOMEM, "workspace %zu bytes holds fewer than %lld rows", workspace_bytes,
                              (long long)std::min<int64_t>(a.B, 256));
    for (int64_t b0 = 0; b0 < a.B; b0 += rpp) {
        const int64_t nb = std::min<int64_t>(rpp, a.B - b0);
        SRM_TRY(m->wsize == 2 ? decode_rows<bf16>(m, a, b0, nb, ws, st) : decode_rows<float>(m, a, b0, nb, ws, st));
    }
    return SRM_OK;
}

static bool few_ok(const srm_model *m, int64_t B, int64_t G, size_t workspace_bytes, hipStream_t st);
static int few_run(srm_model *m, int64_t B, int pos0, int G, const int32_t *tok_in, int32_t *tok_out, int32_t *store,
                   void *state, float temperature, uint32_t seed, float *logits, float *hidden, void *ws, hipStream_t st);
static int few_group_rows(const srm_model *m, int64_t B, int64_t G);

static int decode_step_common(const char *who, srm_model *m, int64_t B, int32_t pos, const int32_t *d_tok_in,
                              void *d_state, int32_t *d_tok_out, float *d_logits, float *d_hidden,
                              void *d_workspace, size_t workspace_bytes, void *hip_stream, float temperature,
                              uint32_t seed, float top_p = 1.0f)
{
    if (!m || !d_tok_in || !d_state || !d_tok_out || !d_workspace) return fail(SRM_EINVAL, "%s: null argument", who);
    if (B <= 0 || B >= (1 << 30)) return fail(SRM_EINVAL, "%s: batch %lld out of range", who, (long long)B);
    if (pos < 0 || pos >= m->cfg.n_ctx) return fail(SRM_EINVAL, "%s: pos %d outside [0, %d)", who, pos, m->cfg.n_ctx);
    if (!(temperature >= 0.0f)) return fail(SRM_EINVAL, "%s: temperature must be >= 0", who);
    if (!(top_p > 0.0f)) return fail(SRM_EINVAL, "%s: top_p must be > 0", who);
    if (temperature > 0.0f && top_p < 1.0f && !d_logits)
        return fail(SRM_EINVAL, "%s: top_p < 1 needs a logits buffer", who);
    SRM_TRY(check_device(m));
    hipStream_t st = as_stream(hip_stream);
    if (few_ok(m, B, 1, workspace_bytes, st)) {
        SRM_TRY(few_run(m, B, pos, 1, d_tok_in, d_tok_out, nullptr, d_state, temperature, seed, d_logits, d_hidden,
                        d_workspace, st));
        if (!(temperature > 0.0f && top_p < 1.0f)) return SRM_OK;
        return nucleus(d_logits, B, m->V, Sampling{temperature, seed, pos, nullptr, nullptr, top_p}, d_tok_out, nullptr, nullptr,
                       0, nullptr, static_cast<int *>(d_workspace), st);
    }
    const DecodeArgs a{B, pos, nullptr, nullptr, 0, d_tok_in, d_state, d_tok_out, d_logits, d_hidden, TokenStore(),
                       temperature, seed, top_p};
    return decode_batch(m, a, d_workspace, workspace_bytes, st);
}

extern "C" int srm_decode_step(srm_model *m, int64_t B, int32_t pos, const int32_t *d_tok_in, void *d_state,
                               int32_t *d_tok_out, float *d_logits, float *d_hidden, void *d_workspace,
                               size_t workspace_bytes, void *hip_stream)
{
    return decode_step_common("srm_decode_step", m, B, pos, d_tok_in, d_state, d_tok_out, d_logits, d_hidden,
                              d_workspace, workspace_bytes, hip_stream, 0.0f, 0);
}

extern "C" int srm_decode_step_sampled(srm_model *m, int64_t B, int32_t pos, const int32_t *d_tok_in, void *d_state,
                                       int32_t *d_tok_out, float temperature, uint32_t seed, float *d_logits,
                                       float *d_hidden, void *d_workspace, size_t workspace_bytes, void *hip_stream)
{
    return decode_step_common("srm_decode_step_sampled", m, B, pos, d_tok_in, d_state, d_tok_out, d_logits, d_hidden,
                              d_workspace, workspace_bytes, hip_stream, temperature, seed);
}

extern "C" int srm_decode_step_topp(srm_model *m, int64_t B, int32_t pos, const int32_t *d_tok_in, void *d_state,
                                    int32_t *d_tok_out, float temperature, float top_p, uint32_t seed,
                                    float *d_logits, float *d_hidden, void *d_workspace, size_t workspace_bytes,
                                    void *hip_stream)
{
    return decode_step_common("srm_decode_step_topp", m, B, pos, d_tok_in, d_state, d_tok_out, d_logits, d_hidden,
                              d_workspace, workspace_bytes, hip_stream, temperature, seed, top_p);
}

// ------------------------------------------------------------------ decode, one position per sample
extern "C" int srm_decode_step_ragged(srm_model *m, int64_t B, int32_t *d_pos, int32_t advance,
                                      const int32_t *d_tok_in, void *d_state, int32_t *d_tok_out,
                                      float temperature, float top_p, uint32_t seed, float *d_logits,
                                      void *d_workspace, size_t workspace_bytes, void *hip_stream)
{
    const char *who = "srm_decode_step_ragged";
    if (!m || !d_pos || !d_tok_in || !d_state || !d_tok_out || !d_workspace)
        return fail(SRM_EINVAL, "%s: null argument", who);
    if (B <= 0 || B >= (1 << 30)) return fail(SRM_EINVAL, "%s: batch %lld out of range", who, (long long)B);
    if (!(temperature >= 0.0f)) return fail(SRM_EINVAL, "%s: temperature must be >= 0", who);
    if (!(top_p > 0.0f)) return fail(SRM_EINVAL, "%s: top_p must be > 0", who);
    if (temperature > 0.0f && top_p < 1.0f && !d_logits)
        return fail(SRM_EINVAL, "%s: top_p < 1 needs a logits buffer", who);
    SRM_TRY(check_device(m));
    const DecodeArgs a{B, 0, nullptr, d_pos, advance != 0, d_tok_in, d_state, d_tok_out, d_logits, nullptr, TokenStore(),
                       temperature, seed, top_p};
    return decode_batch(m, a, d_workspace, workspace_bytes, as_stream(hip_stream));
}

// ------------------------------------------------------------------ few samples: steps as one kernel (few.hpp)
// Whether G steps of B samples run as one kernel: the shapes of few_max_rows, a stream that is not being captured and may use
// every CU, and at least six layers or layers times steps.  That is faster at every size (us, step kernels | one kernel, d = 1024 with
// projections, 4 rows | 1 row: 6 layers 137 | 118, 134 | 79; 8: 168 | 146, 163 | 98; 24: 521 | 417, 507 | 281; d = 512: 6 layers
// 117 | 77, 114 | 59; fp32, d = 256: 8 rows 84 | 52, 1 row 80 | 32), and would be so at every depth (1 layer | 3 layers, 1 row: d = 1024
// 41 | 33, 76 | 51, d = 512 34 | 26, 63 | 39, fp32 30 | 20, 61 | 34; 4 rows of d = 1024 42 | 41, 77 | 71, 8 fp32 rows 30 | 28, 60 | 52).  The
// bound on the layers is there for the results, not for speed: steps of shallower models keep, bit for bit, the sums of the ragged
// step and of larger batches, which their users may compare.
// SRM_ONE_KERNEL_STEP=0 in the environment keeps the step kernels.
// Beside other work of the process it holds its gain (a stream of single steps next to one of other calls, large model, us per step and
// calls per second of the other stream, step kernels | one kernel: prefills of 256 x 128 11060 and 91 | 350 and 60; decode steps of
// 16384 samples 3340 and 148 | 320 and 93; of 3001 with top-p 1230 and 466 | 270 and 278).
static bool few_off()
{
    const char *e = getenv("SRM_ONE_KERNEL_STEP");
    return e && e[0] == '0';
}
static bool one_kernel_stream(hipStream_t st)
{
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    if (refused(hipStreamIsCapturing(st, &cs)) || cs != hipStreamCaptureStatusNone) return false;
    return whole_device_stream(st);
}
static bool few_ok(const srm_model *m, int64_t B, int64_t G, size_t workspace_bytes, hipStream_t st)
{
    if (!m->few_layers || (G > 1 && m->noproj) || G * m->L < 6 || few_off()) return false;
    if (B > few_max_rows(m) ? !few_group_rows(m, B, G) || row_bytes(m, B) > workspace_bytes : srm_workspace_bytes(m, B) > workspace_bytes)
        return false;
    return one_kernel_stream(few_stream(st));
}

// ------------------------------------------------------------------ generate, few samples: one persistent kernel
// Number of work-groups for the one-kernel path (see mega.hpp), or 0 if the call does not
// qualify: fp32 weights and state, head projections, at most kMegaMaxB samples, d <= 1024,
// the widest activation row of all samples within 128 KB of LDS, cooperative launches
// supported, and a model small enough for the small grid to win (see below).  SRM_MEGAKERNEL=0
// in the environment switches the path off, =2 takes it whatever the model's size,
// SRM_MEGA_BLOCKS=n sets the grid (default 16: a grid barrier costs about 1.4 us + 65 ns per
// work-group).
static int mega_rows(int64_t B) { return B <= 1 ? 1 : B <= 2 ? 2 : B <= 4 ? 4 : kMegaMaxB; }   // rows the kernel is unrolled for

static int mega_blocks(const srm_model *m, int64_t B)
{
    if (!m->mega_layers || m->shalf || B > kMegaMaxB || m->L > kMegaMaxLayers) return 0;
    const int widest = std::max(std::max(m->d, m->dm), m->ff);
    if (m->d > 1024 || m->d % 4 || m->dm % 4 || m->ff % 4 || (size_t)mega_rows(B) * widest * 4 > 128 * 1024) return 0;
    // The small grid has a fraction of the chip's arithmetic and cache bandwidth, so the path is for few rows of small
    // models: rows x matrix elements up to 16 M.  That limit was measured against step kernels of 132 us per step of C1's
    // model.  Against the present ones (us per step, one kernel | step kernels): C1's model 91 | 83 at B = 1, 100 | 83 at
    // 2, 112 | 84 at 4, 131 | 85 at 8; 128 wide, 2 layers, 1024 tokens 44 | 46, 47 | 47, 52 | 47, 58 | 48; 64 wide, 2
    // layers, 256 tokens 42 | 43, 44 | 43, 47 | 44, 53 | 44.
    const char *sw = getenv("SRM_MEGAKERNEL");
    if (sw && sw[0] == '0') return 0;
    const double elems = (double)m->L * ((double)2 * m->d * m->dm + (double)2 * m->d * m->ff) + (double)m->V * m->d;
    if (elems * mega_rows(B) > 16e6 && !(sw && sw[0] == '2')) return 0;      // SRM_MEGAKERNEL=2: whatever the size
    int coop = 0;
    if (hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, m->device) != hipSuccess || !coop) return 0;
    int nblk = 16;
    if (const char *nb = getenv("SRM_MEGA_BLOCKS")) nblk = atoi(nb);
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, m->device) != hipSuccess) return 0;
    return std::max(1, std::min(std::min(nblk, kMegaMaxBlocks), cus));
}

extern "C" int32_t srm_generate_one_kernel_blocks(const srm_model *m, int64_t B)
{
    return m && B > 0 ? mega_blocks(m, B) : 0;
}

static int mega_generate(srm_model *m, int B, int pos0, int G, int32_t *tok, void *state, int32_t *store,
                         float temperature, uint32_t seed, void *ws, int nblk, hipStream_t st)
{
    const Workspace w = carve(m, ws, B);
    MegaArgs a;
    a.layers = m->mega_layers;
    a.embed = static_cast<const float *>(m->embed);
    a.head = static_cast<const float *>(m->head);
    a.lnf_g = m->lnf_g; a.lnf_b = m->lnf_b;
    a.V = m->V; a.d = m->d; a.dm = m->dm; a.ff = m->ff; a.L = m->L; a.Hs = m->Hs; a.hrow = m->hrow;
    a.n_ctx = m->cfg.n_ctx; a.eps = m->cfg.ln_eps;
    a.B = B; a.pos0 = pos0; a.G = G;
    a.tok = tok; a.state = static_cast<float *>(state); a.store = store;
    a.temp = temperature; a.seed = seed;
    a.x = w.x; a.mbuf = static_cast<float *>(w.mx); a.gbuf = static_cast<float *>(w.g);
    a.pv = reinterpret_cast<float *>(w.mega);
    a.pi = reinterpret_cast<int32_t *>(w.mega + (size_t)kMegaMaxBlocks * kMegaMaxB * 4);
    a.bar = reinterpret_cast<unsigned *>(w.mega + (size_t)kMegaMaxBlocks * kMegaMaxB * 8);
    const int mb = mega_rows(B);
    const size_t lds = (size_t)mb * std::max(std::max(m->d, m->dm), m->ff) * 4;
    const void *kern = mb == 1 ? reinterpret_cast<const void *>(mega_generate_kernel<1>)
                       : mb == 2 ? reinterpret_cast<const void *>(mega_generate_kernel<2>)
                       : mb == 4 ? reinterpret_cast<const void *>(mega_generate_kernel<4>)
                                 : reinterpret_cast<const void *>(mega_generate_kernel<kMegaMaxB>);
    static bool attr_set[4] = {false, false, false, false};
    const int slot = mb == 1 ? 0 : mb == 2 ? 1 : mb == 4 ? 2 : 3;
    if (!attr_set[slot]) {
        HIP_TRY(hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, 128 * 1024));
        attr_set[slot] = true;
    }
    hipLaunchKernelGGL(mega_reset_kernel, dim3(1), dim3(256), 0, st, a.bar, store, G * B);
    HIP_TRY(hipGetLastError());
    void *args[] = {&a};
    HIP_TRY(hipLaunchCooperativeKernel(kern, dim3((unsigned)nblk), dim3(kMegaThreads), args, (unsigned)lds, st));
    return SRM_OK;
}

// ------------------------------------------------------------------ generate (G steps in one call)
static int generate_step(srm_model *m, int64_t B, int32_t *tok, void *state, void *ws, size_t ws_bytes, int *ctr,
                         TokenStore ts, hipStream_t st, float temperature, uint32_t seed, float top_p, float *logits,
                         int32_t *pos_rows, int eos_plus1, int step, bool stacked)
{
    // uniform position: read from the device counter; ragged: one position per sample, advanced on the device.
    // Every step but the first of a call advances the counters in its first kernel.
    DecodeArgs a{B, 0, pos_rows ? nullptr : ctr, pos_rows, pos_rows ? 1 : 0, tok, state, tok, logits, nullptr, ts,
                 temperature, seed, top_p, eos_plus1, step ? ctr : nullptr};
    a.step = step;
    if (stacked) a.gave_up = reinterpret_cast<unsigned *>(ctr + 2);
    return decode_batch(m, a, ws, ws_bytes, st);
}

static int generate_common(srm_model *m, int64_t B, int32_t pos0, int32_t G, int32_t *d_tok, void *d_state,
                           int32_t *d_tokens_out, float temperature, uint32_t seed, float top_p, float *d_logits,
                           void *d_workspace, size_t workspace_bytes, void *hip_stream, int32_t *d_pos = nullptr,
                           int eos_plus1 = 0)
{
    if (!m || !d_tok || !d_state || !d_tokens_out || !d_workspace) return fail(SRM_EINVAL, "srm_generate: null argument");
    if (!(top_p > 0.0f)) return fail(SRM_EINVAL, "srm_generate: top_p must be > 0");
    const bool topp = temperature > 0.0f && top_p < 1.0f;
    if (topp && !d_logits) return fail(SRM_EINVAL, "srm_generate: top_p < 1 needs a logits buffer");
    if (!topp) { d_logits = nullptr; top_p = 1.0f; }
    if (B <= 0 || B >= (1 << 30)) return fail(SRM_EINVAL, "srm_generate: batch %lld out of range", (long long)B);
    if (G <= 0) return fail(SRM_EINVAL, "srm_generate: G must be positive");
    if (!(temperature >= 0.0f)) return fail(SRM_EINVAL, "srm_generate: temperature must be >= 0");
    if (!d_pos && (pos0 < 0 || (int64_t)pos0 + G > m->cfg.n_ctx))
        return fail(SRM_EINVAL, "srm_generate: positions %d..%lld outside [0, %d)", pos0, (long long)pos0 + G - 1,
                    m->cfg.n_ctx);
    // the step counters live in the last 256 bytes of the workspace, whatever rows the rest is cut into
    if (workspace_bytes < 512) return fail(SRM_ENOMEM, "srm_generate: workspace too small");
    const size_t ws_bytes = workspace_bytes / 256 * 256;          // counters in its last 256 bytes
    if (decode_rows_per_pass(m, B, ws_bytes) <= 0)
        return fail(SRM_ENOMEM, "srm_generate: workspace %zu bytes holds fewer than %lld rows", workspace_bytes,
                    (long long)std::min<int64_t>(B, 256));
    SRM_TRY(check_device(m));
    hipStream_t st = as_stream(hip_stream);
    if (!topp && !d_pos && !eos_plus1 && !getenv("SRM_MEGAKERNEL") && few_ok(m, B, G, ws_bytes, st))
        return few_run(m, B, pos0, G, d_tok, d_tok, d_tokens_out, d_state, temperature, seed, nullptr, nullptr, d_workspace, st);
    if (!topp && !d_pos && !eos_plus1 && row_bytes(m, B) <= ws_bytes) {
        const int nblk = mega_blocks(m, B);
        if (nblk > 0)
            return mega_generate(m, (int)B, pos0, G, d_tok, d_state, d_tokens_out, temperature, seed, d_workspace, nblk, st);
    }
    int *ctr = reinterpret_cast<int *>(static_cast<unsigned char *>(d_workspace) + ws_bytes - 256);
    const TokenStore ts{d_tokens_out, ctr + 1, B};
    hipLaunchKernelGGL(counters_set_kernel, dim3(1), dim3(1), 0, st, ctr, pos0, 0);
    HIP_TRY(hipGetLastError());
    // Where the layers of a step, or of some slice of it, run as one kernel, all steps are launched one by one: a captured step would
    // take the step kernels, with their sums.
    const int64_t rpp = decode_rows_per_pass(m, B, ws_bytes);
    const bool stacked = stack_ok(m, rpp, ws_bytes, st) || (B % rpp && stack_ok(m, B % rpp, ws_bytes, st));
    // first step eagerly (it also performs every one-time kernel attribute set-up)
    SRM_TRY(generate_step(m, B, d_tok, d_state, d_workspace, ws_bytes, ctr, ts, st, temperature, seed, top_p, d_logits,
                          d_pos, eos_plus1, 0, stacked));
    if (G == 1) return SRM_OK;
    if (st == nullptr || stacked) {                  // (the legacy default stream cannot be captured either)
        for (int g = 1; g < G; ++g)
            SRM_TRY(generate_step(m, B, d_tok, d_state, d_workspace, ws_bytes, ctr, ts, st, temperature, seed, top_p,
                                  d_logits, d_pos, eos_plus1, g, stacked));
        return SRM_OK;
    }
    const bool hit = m->gexec && m->gkey.B == B && m->gkey.tok == d_tok && m->gkey.state == d_state &&
                     m->gkey.store == d_tokens_out && m->gkey.ws == d_workspace && m->gkey.temp == temperature &&
                     m->gkey.seed == seed && m->gkey.top_p == top_p && m->gkey.logits == d_logits &&
                     m->gkey.ws_bytes == workspace_bytes && m->gkey.pos == d_pos && m->gkey.eos_plus1 == eos_plus1;
    if (!hit) {
        if (m->gexec) { (void)hipGraphExecDestroy(m->gexec); m->gexec = nullptr; }
        hipGraph_t graph = nullptr;
        HIP_TRY(hipStreamBeginCapture(st, hipStreamCaptureModeThreadLocal));
        const int rc = generate_step(m, B, d_tok, d_state, d_workspace, ws_bytes, ctr, ts, st, temperature, seed, top_p,
                                     d_logits, d_pos, eos_plus1, 1, false);
        const hipError_t e = hipStreamEndCapture(st, &graph);
        if (rc != SRM_OK) { if (graph) (void)hipGraphDestroy(graph); return rc; }
        if (e != hipSuccess) return fail(SRM_EHIP, "srm_generate: stream capture failed: %s", hipGetErrorString(e));
        const hipError_t e2 = hipGraphInstantiate(&m->gexec, graph, nullptr, nullptr, 0);
        (void)hipGraphDestroy(graph);
        if (e2 != hipSuccess) { m->gexec = nullptr; return fail(SRM_EHIP, "srm_generate: hipGraphInstantiate: %s", hipGetErrorString(e2)); }
        m->gkey = {B, d_tok, d_state, d_tokens_out, d_workspace, temperature, seed, top_p, d_logits, workspace_bytes,
                   d_pos, eos_plus1};
        // the captured step was recorded, not run: replay it G - 1 times below
    }
    for (int g = 1; g < G; ++g) HIP_TRY(hipGraphLaunch(m->gexec, st));
    return SRM_OK;
}

extern "C" int srm_generate(srm_model *m, int64_t B, int32_t pos0, int32_t G, int32_t *d_tok, void *d_state,
                            int32_t *d_tokens_out, float temperature, uint32_t seed, void *d_workspace,
                            size_t workspace_bytes, void *hip_stream)
{
    return generate_common(m, B, pos0, G, d_tok, d_state, d_tokens_out, temperature, seed, 1.0f, nullptr, d_workspace,
                           workspace_bytes, hip_stream);
}

extern "C" int srm_generate_topp(srm_model *m, int64_t B, int32_t pos0, int32_t G, int32_t *d_tok, void *d_state,
                                 int32_t *d_tokens_out, float temperature, float top_p, uint32_t seed,
                                 float *d_logits, void *d_workspace, size_t workspace_bytes, void *hip_stream)
{
    return generate_common(m, B, pos0, G, d_tok, d_state, d_tokens_out, temperature, seed, top_p, d_logits,
                           d_workspace, workspace_bytes, hip_stream);
}

extern "C" int srm_generate_ragged(srm_model *m, int64_t B, int32_t G, int32_t *d_pos, int32_t *d_tok, void *d_state,
                                   int32_t *d_tokens_out, int32_t eos_id, float temperature, float top_p,
                                   uint32_t seed, float *d_logits, void *d_workspace, size_t workspace_bytes,
                                   void *hip_stream)
{
    if (!d_pos) return fail(SRM_EINVAL, "srm_generate_ragged: null argument");
    if (m && eos_id >= m->V) return fail(SRM_EINVAL, "srm_generate_ragged: eos_id %d outside the vocabulary", eos_id);
    return generate_common(m, B, 0, G, d_tok, d_state, d_tokens_out, temperature, seed, top_p, d_logits, d_workspace,
                           workspace_bytes, hip_stream, d_pos, eos_id >= 0 ? eos_id + 1 : 0);
}

// ------------------------------------------------------------------ prefill
// Whole sequences per pass that fit the workspace (0 if not even one does).
static int64_t seqs_per_pass(const srm_model *m, size_t workspace_bytes, int T, int64_t nseq)
{
    if (row_bytes(m, T) > workspace_bytes) return 0;
    int64_t lo = 1, hi = nseq;       // largest n with bytes(n*T) <= workspace_bytes
    while (lo < hi) {
        const int64_t mid = (lo + hi + 1) / 2;
        if (row_bytes(m, mid * T) <= workspace_bytes) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// Chunk length of the chunked scan for a call with nseq sequences of up to P
// positions, or 0 for the sequential kernel.  Chunks are used only while the
// sequential kernel (one thread per sequence and 4 channels) would leave the
// chip mostly idle; the choice depends on the whole call, not on how the
// workspace cuts it into passes, so results do not depend on the workspace size.
static int scan_chunk_len(const srm_model *m, int64_t nseq, int P)
{
    const int64_t dv = m->dm / 4;
    if (P < 64 || nseq * dv >= 65536 || m->shalf) return 0;   // a half-precision cache is rounded at every step
    for (int c : {16, 32, 64, 128}) {
        const int64_t nch = cdiv(P, c);
        if (nch < 2) break;
        if (nseq * dv * nch <= 262144) return c;
    }
    return 0;
}

// Where the chunked scan would run, mixer_parallel_kernel (one launch, every block reads the positions in front of it
// itself) is faster until those reads count: their bytes grow with sequences x channels x P^2.  Measured (chunked - block
// form, us per layer; in brackets the product in units of 2^30), d = 1024: 1 x 509 positions (0.25) +4.4, 8 x 320 (0.8)
// +4.8, 64 x 128 (1) +4.3, 32 x 200 (1.2) +0.9, 8 x 509 (2) +0.7, 64 x 200 (2.4) -3.5, 32 x 509 (8) -18; d = 512: 32 x 320
// (1.6) +5.3, 64 x 200 (1.2) +0.8, 120 x 200 (2.3) -4.  The limit keeps to the side where every call measured gains
// clearly; the calls between it and the crossover at about 2 take the chunked scan.  A property of the whole call, like
// the chunk length.
static bool scan_in_blocks(const srm_model *m, int chunk, int64_t nseq, int P)
{
    return chunk > 0 && P < 8192 && nseq * m->dm * (int64_t)P * P <= (1 << 30);
}

// The chunked scan keeps its per-chunk partial states F [nc][nchunks][dm] fp32 in the pass's MLP buffer
// w.g ([rows][ff] activation elements, free until the layer's MLP): whether they fit there.
static bool scan_scratch_fits(const srm_model *m, int64_t nc, int nchunks, int64_t rows)
{
    return (size_t)nc * (size_t)nchunks * (size_t)m->dm * sizeof(float) <= (size_t)rows * (size_t)m->ff * m->wsize;
}

// How srm_prefill_ragged cuts packed prompts into passes of whole prompts that fit max_rows workspace rows,
// and which mixer scan the call takes: the chunked one only if its partial states fit the MLP buffer in
// EVERY pass (many short prompts next to a long one do not: the chunk count follows the longest prompt of
// the call, the buffer the rows of the pass), so that one call uses one kind of scan whatever the workspace.
struct RaggedPlan {
    std::vector<int> first;        // first prompt of each pass, then N
    int chunk = 0, nchunks = 1;    // the scan taken (chunk 0: sequential)
    int chunk_by_shape = 0;        // what (N, longest prompt) alone would choose
    size_t need = 0, room = 0;     // tightest pass under chunk_by_shape: bytes of F, bytes of w.g
};
static RaggedPlan plan_ragged(const srm_model *m, const int32_t *h_off, int N, int64_t max_rows, int pmax_call)
{
    RaggedPlan pl;
    pl.chunk_by_shape = scan_chunk_len(m, N, pmax_call);
    const int nch = pl.chunk_by_shape ? (int)cdiv(pmax_call, pl.chunk_by_shape) : 1;
    bool fits = true;
    int n0 = 0;
    while (n0 < N) {
        int n1 = n0;
        while (n1 < N && (int64_t)h_off[n1 + 1] - h_off[n0] <= max_rows) ++n1;
        if (n1 == n0) break;                          // a prompt longer than the workspace: rejected by the caller
        pl.first.push_back(n0);
        if (pl.chunk_by_shape) {
            const int64_t nc = n1 - n0, rows = (int64_t)h_off[n1] - h_off[n0];
            const size_t need = (size_t)nc * nch * m->dm * sizeof(float), room = (size_t)rows * m->ff * m->wsize;
            if (!scan_scratch_fits(m, nc, nch, rows)) fits = false;
            if (pl.room == 0 || (double)need * (double)pl.room > (double)pl.need * (double)room) { pl.need = need; pl.room = room; }
        }
        n0 = n1;
    }
    pl.first.push_back(N);
    if (pl.chunk_by_shape && fits) { pl.chunk = pl.chunk_by_shape; pl.nchunks = nch; }
    return pl;
}

// mixer_parallel_kernel on nseq sequences of up to P positions, w.u -> w.mx.
template <typename T, bool PREFILL>
static int mixer_parallel(const srm_model *m, const LayerDev &y, const Workspace &w, int P, int64_t nseq, const PrefillSeqs &ps,
                          hipStream_t st)
{
    const unsigned tiles = (unsigned)cdiv(P, kParSquare), heads = (unsigned)(m->Hs * cdiv(m->dm / m->Hs, 64));
    const size_t lds = (size_t)parallel_table_floats(P) * sizeof(float);
#define PARALLEL_LAUNCH(FEW, WIDE, ...)                                                                         \
    hipLaunchKernelGGL((mixer_parallel_kernel<T, PREFILL, FEW, WIDE>), dim3(__VA_ARGS__), dim3(256), lds, st,     \
                       static_cast<const T *>(w.u), static_cast<T *>(w.mx), y.alpha, y.beta, y.lam, m->cfg.n_ctx, m->Hs, \
                       m->hrow, m->dm, P, ps)
    const bool few = (int64_t)tiles * heads * nseq <= device_cus();
    constexpr bool wide = sizeof(T) == 2;            // (fp32 rows are twice as wide, and never asked for by more than 16)
    if (few && P > 256 + kParSquare) PARALLEL_LAUNCH(true, wide, tiles, heads, (unsigned)nseq);
    else if (few) PARALLEL_LAUNCH(true, false, tiles, heads, (unsigned)nseq);
    else PARALLEL_LAUNCH(false, false, heads, (unsigned)nseq, tiles);
#undef PARALLEL_LAUNCH
    HIP_TRY(hipGetLastError());
    return SRM_OK;
}

// The mixer of one prefill pass: nc sequences in rows of w.u -> w.mx, final states to S_layer.
template <typename T>
static int prefill_mixer(const srm_model *m, int l, const Workspace &w, void *S_layer, int nc, int P, int chunk,
                         int nchunks, bool in_blocks, const int32_t *offsets, int64_t base, int64_t rows, int64_t seq0, int rep,
                         const int32_t *slot, int64_t nslots, hipStream_t st)
{
    const LayerDev &y = m->layers[l];
    const int d = m->dm;           // the mixer's row width
    if (in_blocks) {
        return mixer_parallel<T, true>(m, y, w, P, nc, PrefillSeqs{static_cast<float *>(S_layer), offsets, base, rows, seq0, rep, slot, nslots}, st);
    }
    if (chunk > 0) {
        float *F = static_cast<float *>(w.g);       // free until the MLP of this layer
        const unsigned nb = (unsigned)cdiv((int64_t)nc * nchunks * (d / 4), 256);
        hipLaunchKernelGGL((scan_chunk_partials_kernel<T>), dim3(nb), dim3(256), 0, st, static_cast<const T *>(w.u), F,
                           y.alpha, y.lam, m->cfg.n_ctx, m->Hs, m->hrow, d, nc, P, chunk, nchunks, offsets, base, rows, seq0);
        HIP_TRY(hipGetLastError());
        hipLaunchKernelGGL((scan_chunk_apply_kernel<T>), dim3(nb), dim3(256), 0, st, static_cast<const T *>(w.u),
                           static_cast<T *>(w.mx), static_cast<float *>(S_layer), F, y.alpha, y.beta, y.lam,
                           m->cfg.n_ctx, m->Hs, m->hrow, d, nc, P, chunk, nchunks, offsets, base, rows, seq0, rep, slot, nslots);
        HIP_TRY(hipGetLastError());
        return SRM_OK;
    }
    const unsigned nb = (unsigned)cdiv((int64_t)nc * (d / 4), 256);
    const size_t scan_lds = (size_t)2 * m->Hs * P * sizeof(float);
#define SCAN_LAUNCH(TS)                                                                                        \
    do {                                                                                                       \
        if (offsets)                                                                                           \
            hipLaunchKernelGGL((mixer_scan_ragged_kernel<T, TS>), dim3(nb), dim3(256), scan_lds, st,           \
                               static_cast<const T *>(w.u), static_cast<T *>(w.mx), static_cast<TS *>(S_layer), \
                               y.alpha, y.beta, y.lam, m->cfg.n_ctx, m->Hs, m->hrow, d, nc, P, offsets, base, rows, seq0, \
                               rep, slot, nslots);                                                             \
        else                                                                                                   \
            hipLaunchKernelGGL((mixer_scan_kernel<T, TS>), dim3(nb), dim3(256), scan_lds, st,                  \
                               static_cast<const T *>(w.u), static_cast<T *>(w.mx), static_cast<TS *>(S_layer), \
                               y.alpha, y.beta, y.lam, m->cfg.n_ctx, m->Hs, m->hrow, d, nc, P, seq0, rep);     \
    } while (0)
    if (m->shalf) SCAN_LAUNCH(f16);
    else SCAN_LAUNCH(float);
#undef SCAN_LAUNCH
    HIP_TRY(hipGetLastError());
    return SRM_OK;
}

template <typename T>
static int prefill_impl(srm_model *m, const int32_t *prompts, int N, int P, int k, void *state,
                        int32_t *next_tok, float *logits, void *ws, int64_t per_pass, int chunk, hipStream_t st)
{
    const int d = m->d;
    const int64_t Btot = (int64_t)N * k;
    const int nchunks = chunk ? (int)cdiv(P, chunk) : 1;
    const bool in_blocks = scan_in_blocks(m, chunk, N, P);
    for (int64_t n0 = 0; n0 < N; n0 += per_pass) {
        const int64_t nc = std::min<int64_t>(per_pass, N - n0);
        const int64_t rows = nc * P;
        Workspace w = carve(m, ws, rows);
        LastRows last;
        if (last_rows_ok(m, N, (int64_t)N * P, P)) last = {nc, N, P, nullptr, 0};
        SRM_TRY((layernorm<T, true>(m, nullptr, 0, prompts + n0 * P, w.x, m->layers[0].ln1_g,
                                    m->layers[0].ln1_b, w.a, rows, st)));
        auto mix = [&](int l) {
            return prefill_mixer<T>(m, l, w, layer_state(m, state, l, Btot), (int)nc, P, chunk, nchunks, in_blocks, nullptr, 0, rows,
                                    n0, k, nullptr, 0, st);
        };
        for (int l = 0; l < m->L; ++l)
            SRM_TRY((block<T>(m, l, w, rows, (int64_t)N * P, st, mix, l + 1 < m->L, nullptr, Sampling(), nullptr, false, false, false,
                              l + 1 < m->L ? LastRows() : last)));
        // final LayerNorm of each prompt's last position only, packed [nc][d] into w.a
        if (last.n)
            SRM_TRY((layernorm<T, false>(m, w.x, d, nullptr, nullptr, m->lnf_g, m->lnf_b, w.a, nc, st)));
        else
            SRM_TRY((layernorm<T, false>(m, w.x + (size_t)(P - 1) * d, (int64_t)P * d, nullptr, nullptr, m->lnf_g,
                                         m->lnf_b, w.a, nc, st)));
        SRM_TRY((head_argmax<T>(m, w, w.a, nc, N, logits ? logits + (size_t)n0 * m->V : nullptr, next_tok, n0, k, st)));
    }
    return SRM_OK;
}

extern "C" int srm_prefill(srm_model *m, const int32_t *d_prompts, int32_t N, int32_t P, int32_t fanout_k,
                           void *d_state, int32_t *d_next_tok, float *d_logits, void *d_workspace,
                           size_t workspace_bytes, void *hip_stream)
{
    if (!m || !d_prompts || !d_state || !d_next_tok || !d_workspace)
        return fail(SRM_EINVAL, "srm_prefill: null argument");
    if (N <= 0 || P <= 0 || fanout_k <= 0) return fail(SRM_EINVAL, "srm_prefill: N, P and fanout_k must be positive");
    if (P > m->cfg.n_ctx) return fail(SRM_EINVAL, "srm_prefill: P = %d exceeds n_ctx = %d", P, m->cfg.n_ctx);
    if ((int64_t)N * fanout_k >= (1 << 30)) return fail(SRM_EINVAL, "srm_prefill: N * fanout_k too large");
    // the chunked scan where the call's shape asks for it and its partial states fit the MLP buffer of a pass
    // (rows = prompts x P there, so the test does not depend on how many prompts a pass holds)
    int chunk = scan_chunk_len(m, N, P);
    if (chunk && !scan_scratch_fits(m, 1, (int)cdiv(P, chunk), P)) chunk = 0;
    if (!chunk && (size_t)2 * m->Hs * P * sizeof(float) > 64 * 1024)   // the sequential scan stages its coefficients in LDS
        return fail(SRM_EINVAL, "srm_prefill: n_heads * P too large for the coefficient stage");
    const int64_t max_seqs = std::max<int64_t>(1, ((1 << 30) - 1) / P);
    int64_t per_pass = seqs_per_pass(m, workspace_bytes, P, std::min<int64_t>(N, max_seqs));
    if (per_pass < 1)
        return fail(SRM_ENOMEM, "srm_prefill: workspace %zu < %zu bytes (one prompt)", workspace_bytes,
                    row_bytes(m, P));
    SRM_TRY(check_device(m));
    hipStream_t st = as_stream(hip_stream);
    return m->wsize == 2 ? prefill_impl<bf16>(m, d_prompts, N, P, fanout_k, d_state, d_next_tok, d_logits,
                                              d_workspace, per_pass, chunk, st)
                         : prefill_impl<float>(m, d_prompts, N, P, fanout_k, d_state, d_next_tok, d_logits,
                                               d_workspace, per_pass, chunk, st);
}

// ------------------------------------------------------------------ prefill of packed ragged prompts
template <typename T>
static int prefill_ragged_impl(srm_model *m, const int32_t *tokens, const int32_t *h_off, const int32_t *d_off, int N,
                               int k, const int32_t *slot, int64_t state_batch, void *state, int32_t *next_tok,
                               int32_t *pos_out, float *logits, void *ws, const RaggedPlan &plan, int pmax_call,
                               hipStream_t st)
{
    const int d = m->d;
    const int chunk = plan.chunk, nchunks = plan.nchunks;
    const bool in_blocks = scan_in_blocks(m, chunk, N, pmax_call);
    int shortest = pmax_call;
    for (int n = 0; n < N; ++n) shortest = std::min(shortest, h_off[n + 1] - h_off[n]);
    for (size_t pass = 0; pass + 1 < plan.first.size(); ++pass) {
        // as many whole prompts as the workspace holds
        const int n0 = plan.first[pass], n1 = plan.first[pass + 1];
        int pmax = 0;
        for (int n = n0; n < n1; ++n) pmax = std::max(pmax, h_off[n + 1] - h_off[n]);
        const int nc = n1 - n0;
        const int64_t base = h_off[n0], rows = (int64_t)h_off[n1] - base;
        Workspace w = carve(m, ws, rows);
        LastRows last;
        if (last_rows_ok(m, N, h_off[N] - h_off[0], shortest)) last = {nc, N, 0, d_off + n0, base};
        SRM_TRY((layernorm<T, true>(m, nullptr, 0, tokens + base, w.x, m->layers[0].ln1_g, m->layers[0].ln1_b, w.a,
                                    rows, st)));
        auto mix = [&](int l) {
            return prefill_mixer<T>(m, l, w, layer_state(m, state, l, state_batch), nc, chunk ? pmax_call : pmax, chunk,
                                    nchunks, in_blocks, d_off, base, rows, (int64_t)n0, k, slot, state_batch, st);
        };
        for (int l = 0; l < m->L; ++l)
            SRM_TRY((block<T>(m, l, w, rows, h_off[N] - h_off[0], st, mix, l + 1 < m->L, nullptr, Sampling(), nullptr, false, false,
                              false, l + 1 < m->L ? LastRows() : last)));
        // final LayerNorm of each prompt's last row, packed [nc][d] into w.a
        if (last.n)
            SRM_TRY((layernorm<T, false>(m, w.x, d, nullptr, nullptr, m->lnf_g, m->lnf_b, w.a, nc, st)));
        else
            SRM_TRY((layernorm<T, false>(m, w.x, d, nullptr, nullptr, m->lnf_g, m->lnf_b, w.a, nc, st, d_off + n0, base,
                                         rows)));
        FinalizeRagged rg{};
        rg.slot = slot;
        rg.nslots = state_batch;
        rg.offsets = d_off;
        rg.pos_set = pos_out;
        SRM_TRY((head_argmax<T>(m, w, w.a, nc, N, logits ? logits + (size_t)n0 * m->V : nullptr, next_tok, n0, k, st,
                                TokenStore(), Sampling(), rg)));
    }
    return SRM_OK;
}

// Host-side checks of a packed prompt list against a model and a workspace size: every length within
// [1, n_ctx] and within the rows the workspace holds; returns those rows and the longest prompt.
static int ragged_lengths(const char *who, const srm_model *m, const int32_t *h_offsets, int N, size_t workspace_bytes,
                          int64_t &max_rows, int &pmax)
{
    if (h_offsets[0] < 0) return fail(SRM_EINVAL, "%s: offsets[0] is negative", who);
    // rows the workspace holds (largest r with row_bytes(r) <= workspace_bytes)
    int64_t lo = 0, hi = (1 << 30) - 1;
    while (lo < hi) {
        const int64_t mid = (lo + hi + 1) / 2;
        if (row_bytes(m, mid) <= workspace_bytes) lo = mid; else hi = mid - 1;
    }
    max_rows = lo;
    pmax = 0;
    for (int n = 0; n < N; ++n) {
        const int64_t len = (int64_t)h_offsets[n + 1] - h_offsets[n];
        if (len < 1 || len > m->cfg.n_ctx)
            return fail(SRM_EINVAL, "%s: prompt %d has length %lld outside [1, n_ctx = %d]", who, n, (long long)len,
                        m->cfg.n_ctx);
        if (len > max_rows)
            return fail(SRM_ENOMEM, "%s: workspace %zu < %zu bytes (prompt %d of %lld tokens)", who, workspace_bytes,
                        row_bytes(m, len), n, (long long)len);
        pmax = std::max(pmax, (int)len);
    }
    return SRM_OK;
}

extern "C" int srm_prefill_ragged(srm_model *m, const int32_t *d_tokens, const int32_t *h_offsets,
                                  const int32_t *d_offsets, int32_t N, int32_t fanout_k, const int32_t *d_slot,
                                  int64_t state_batch, void *d_state, int32_t *d_next_tok, int32_t *d_pos,
                                  float *d_logits, void *d_workspace, size_t workspace_bytes, void *hip_stream)
{
    const char *who = "srm_prefill_ragged";
    if (!m || !d_tokens || !h_offsets || !d_offsets || !d_state || !d_next_tok || !d_workspace)
        return fail(SRM_EINVAL, "%s: null argument", who);
    if (N <= 0 || fanout_k <= 0) return fail(SRM_EINVAL, "%s: N and fanout_k must be positive", who);
    if (d_slot && fanout_k != 1) return fail(SRM_EINVAL, "%s: a slot list needs fanout_k = 1", who);
    if (state_batch <= 0 || state_batch >= (1 << 30)) return fail(SRM_EINVAL, "%s: state_batch out of range", who);
    if (!d_slot && (int64_t)N * fanout_k > state_batch)
        return fail(SRM_EINVAL, "%s: N * fanout_k = %lld exceeds state_batch = %lld", who, (long long)N * fanout_k,
                    (long long)state_batch);
    int64_t max_rows = 0;
    int pmax = 0;
    SRM_TRY(ragged_lengths(who, m, h_offsets, N, workspace_bytes, max_rows, pmax));
    const RaggedPlan plan = plan_ragged(m, h_offsets, N, max_rows, pmax);
    if (!plan.chunk && (size_t)2 * m->Hs * pmax * sizeof(float) > 64 * 1024)   // the sequential scan's coefficient stage
        return fail(SRM_EINVAL, "%s: n_heads * longest prompt too large for the coefficient stage", who);
    SRM_TRY(check_device(m));
    hipStream_t st = as_stream(hip_stream);
    return m->wsize == 2 ? prefill_ragged_impl<bf16>(m, d_tokens, h_offsets, d_offsets, N, fanout_k, d_slot,
                                                     state_batch, d_state, d_next_tok, d_pos, d_logits, d_workspace,
                                                     plan, pmax, st)
                         : prefill_ragged_impl<float>(m, d_tokens, h_offsets, d_offsets, N, fanout_k, d_slot,
                                                      state_batch, d_state, d_next_tok, d_pos, d_logits, d_workspace,
                                                      plan, pmax, st);
}

extern "C" size_t srm_workspace_bytes_config(const srm_config *cfg, int64_t rows)
{
    if (!cfg || rows <= 0) return 0;
    srm_model m;
    if (model_geometry("srm_workspace_bytes_config", cfg, &m) != SRM_OK) return 0;
    return srm_workspace_bytes(&m, rows);
}

extern "C" int srm_prefill_ragged_plan(const srm_config *cfg, const int32_t *h_offsets, int32_t N,
                                       size_t workspace_bytes, srm_prefill_plan *out)
{
    const char *who = "srm_prefill_ragged_plan";
    if (!cfg || !h_offsets || !out) return fail(SRM_EINVAL, "%s: null argument", who);
    if (N <= 0) return fail(SRM_EINVAL, "%s: N must be positive", who);
    srm_model m;
    SRM_TRY(model_geometry(who, cfg, &m));
    int64_t max_rows = 0;
    int pmax = 0;
    SRM_TRY(ragged_lengths(who, &m, h_offsets, N, workspace_bytes, max_rows, pmax));
    const RaggedPlan plan = plan_ragged(&m, h_offsets, N, max_rows, pmax);
    out->passes = (int32_t)plan.first.size() - 1;
    out->chunk_len = plan.chunk;
    out->chunk_len_by_shape = plan.chunk_by_shape;
    out->n_chunks = plan.chunk_by_shape ? (int32_t)cdiv(pmax, plan.chunk_by_shape) : 1;
    out->scratch_need = plan.need;
    out->scratch_room = plan.room;
    return SRM_OK;
}

// ------------------------------------------------------------------ parallel form
template <typename T>
static int parallel_impl(srm_model *m, const int32_t *tok, int B, int T_, float *hidden, float *logits, void *ws,
                         int64_t per_pass, hipStream_t st)
{
    const int d = m->d;
    for (int64_t b0 = 0; b0 < B; b0 += per_pass) {
        const int64_t nc = std::min<int64_t>(per_pass, B - b0);
        const int64_t rows = nc * T_;
        Workspace w = carve(m, ws, rows);
        SRM_TRY((layernorm<T, true>(m, nullptr, 0, tok + b0 * T_, w.x, m->layers[0].ln1_g, m->layers[0].ln1_b,
                                    w.a, rows, st)));
        auto mix = [&](int l) {
            return mixer_parallel<T, false>(m, m->layers[l], w, T_, nc, PrefillSeqs{}, st);
        };
        for (int l = 0; l < m->L; ++l) SRM_TRY((block<T>(m, l, w, rows, (int64_t)B * T_, st, mix, true)));
        HIP_TRY(hipMemcpyAsync(hidden + (size_t)b0 * T_ * d, w.x, (size_t)rows * d * 4, hipMemcpyDeviceToDevice, st));
        if (logits)
            SRM_TRY((linear<EPI_F32, T>(w.a, m->head, nullptr, rows, m->V, d, logits + (size_t)b0 * T_ * m->V, st, nullptr, nullptr, 64,
                                        nullptr, Sampling(), MixArgs(), (int64_t)B * T_)));
    }
    return SRM_OK;
}

extern "C" int srm_parallel_forward(srm_model *m, const int32_t *d_tok, int32_t B, int32_t T, float *d_hidden,
                                    float *d_logits, void *d_workspace, size_t workspace_bytes, void *hip_stream)
{
    if (!m || !d_tok || !d_hidden || !d_workspace) return fail(SRM_EINVAL, "srm_parallel_forward: null argument");
    if (B <= 0 || T <= 0) return fail(SRM_EINVAL, "srm_parallel_forward: B and T must be positive");
    if (T > m->cfg.n_ctx) return fail(SRM_EINVAL, "srm_parallel_forward: T = %d exceeds n_ctx = %d", T, m->cfg.n_ctx);
    if ((size_t)T * sizeof(float) > 32 * 1024) return fail(SRM_EINVAL, "srm_parallel_forward: T too large");
    if (B > 65535) return fail(SRM_EINVAL, "srm_parallel_forward: B > 65535");
    const int64_t max_seqs = std::max<int64_t>(1, ((1 << 30) - 1) / T);
    int64_t per_pass = seqs_per_pass(m, workspace_bytes, T, std::min<int64_t>(B, max_seqs));
    if (per_pass < 1)
        return fail(SRM_ENOMEM, "srm_parallel_forward: workspace %zu < %zu bytes (one sequence)", workspace_bytes,
                    row_bytes(m, T));
    SRM_TRY(check_device(m));
    hipStream_t st = as_stream(hip_stream);
    return m->wsize == 2
               ? parallel_impl<bf16>(m, d_tok, B, T, d_hidden, d_logits, d_workspace, per_pass, st)
               : parallel_impl<float>(m, d_tok, B, T, d_hidden, d_logits, d_workspace, per_pass, st);
}

// ------------------------------------------------------------------ kernel-level entry points
extern "C" int srm_mixer_update(srm_model *m, int32_t layer, int32_t pos, int64_t B, const void *d_u,
                                void *d_state_layer, void *d_m, void *hip_stream)
{
    if (!m || !d_u || !d_state_layer || !d_m) return fail(SRM_EINVAL, "srm_mixer_update: null argument");
    if (layer < 0 || layer >= m->L) return fail(SRM_EINVAL, "srm_mixer_update: layer %d outside [0, %d)", layer, m->L);
    if (pos < 0 || pos >= m->cfg.n_ctx) return fail(SRM_EINVAL, "srm_mixer_update: pos %d outside [0, %d)", pos, m->cfg.n_ctx);
    if (B <= 0 || B >= (1 << 30)) return fail(SRM_EINVAL, "srm_mixer_update: batch out of range");
    SRM_TRY(check_device(m));
    hipStream_t st = as_stream(hip_stream);
    return m->wsize == 2 ? state_update<bf16>(m, layer, pos, B, d_u, d_state_layer, d_m, st)
                         : state_update<float>(m, layer, pos, B, d_u, d_state_layer, d_m, st);
}

extern "C" int srm_mixer_project_update(srm_model *m, int32_t layer, int32_t pos, int64_t B, const void *d_a,
                                        void *d_state_layer, void *d_m, void *hip_stream)
{
    if (!m || !d_a || !d_state_layer || !d_m) return fail(SRM_EINVAL, "srm_mixer_project_update: null argument");
    if (m->noproj) return fail(SRM_EINVAL, "srm_mixer_project_update: the model has no head projections");
    if (layer < 0 || layer >= m->L)
        return fail(SRM_EINVAL, "srm_mixer_project_update: layer %d outside [0, %d)", layer, m->L);
    if (pos < 0 || pos >= m->cfg.n_ctx)
        return fail(SRM_EINVAL, "srm_mixer_project_update: pos %d outside [0, %d)", pos, m->cfg.n_ctx);
    if (B <= 0 || B >= (1 << 30)) return fail(SRM_EINVAL, "srm_mixer_project_update: batch out of range");
    SRM_TRY(check_device(m));
    hipStream_t st = as_stream(hip_stream);
    const LayerDev &y = m->layers[layer];
    const MixArgs mx{d_state_layer, y.alpha, y.beta, y.lam, m->cfg.n_ctx, m->hrow, m->dm / m->Hs, m->shalf ? 1 : 0};
    Sampling where;
    where.pos = pos;
    return m->wsize == 2 ? linear<EPI_MIX, bf16>(d_a, y.w_in, y.b_in, B, m->dm, m->d, d_m, st, nullptr, nullptr, 64,
                                                 nullptr, where, mx)
                         : linear<EPI_MIX, float>(d_a, y.w_in, y.b_in, B, m->dm, m->d, d_m, st, nullptr, nullptr, 64,
                                                  nullptr, where, mx);
}

extern "C" int srm_mixer_block(srm_model *m, int32_t layer, int32_t pos, const int32_t *d_pos_rows, int64_t B,
                               float *d_x, void *d_state_layer, void *d_norm_out, float *d_slabs, void *hip_stream)
{
    if (!m || !d_x || !d_state_layer || !d_norm_out || !d_slabs) return fail(SRM_EINVAL, "srm_mixer_block: null argument");
    if (!token_mix_shape_ok(m))
        return fail(SRM_EINVAL, "srm_mixer_block: needs bf16 weights, head projections of width d and d = 256 or 512");
    if (layer < 0 || layer >= m->L) return fail(SRM_EINVAL, "srm_mixer_block: layer %d outside [0, %d)", layer, m->L);
    if (!d_pos_rows && (pos < 0 || pos >= m->cfg.n_ctx))
        return fail(SRM_EINVAL, "srm_mixer_block: pos %d outside [0, %d)", pos, m->cfg.n_ctx);
    if (B <= 0 || B >= (1 << 26)) return fail(SRM_EINVAL, "srm_mixer_block: batch out of range");
    SRM_TRY(check_device(m));
    hipStream_t st = as_stream(hip_stream);
    Sampling where;
    where.pos = pos;
    where.pos_rows = d_pos_rows;
    SRM_TRY(token_mix(m, layer, TokMixCall{d_x, d_state_layer, where, d_slabs}, B, st));
    const LayerDev &y = m->layers[layer];
    return layernorm<bf16, false>(m, d_x, m->d, nullptr, d_x, y.ln2_g, y.ln2_b, d_norm_out, B, st, nullptr, 0, 0, d_slabs,
                                  m->d / kTokMixCols);
}

extern "C" int srm_sample_logits(const float *d_logits, int64_t rows, int32_t vocab, float temperature, float top_p,
                                 uint32_t seed, int32_t pos, int32_t *d_tok_out, void *hip_stream)
{
    if (!d_logits || !d_tok_out) return fail(SRM_EINVAL, "srm_sample_logits: null argument");
    if (rows <= 0 || rows >= (1 << 30) || vocab <= 0) return fail(SRM_EINVAL, "srm_sample_logits: sizes out of range");
    if (!(temperature > 0.0f)) return fail(SRM_EINVAL, "srm_sample_logits: temperature must be > 0");
    if (!(top_p > 0.0f)) return fail(SRM_EINVAL, "srm_sample_logits: top_p must be > 0");
    hipLaunchKernelGGL((nucleus_kernel<256, true, false>), dim3((unsigned)rows), dim3(256), 0, as_stream(hip_stream),
                       d_logits, (int64_t)vocab, vocab, temperature, top_p, seed, pos, nullptr, nullptr, d_tok_out,
                       nullptr, nullptr, (int64_t)0, nullptr, nullptr, nullptr, 0u);
    HIP_TRY(hipGetLastError());
    return SRM_OK;
}

extern "C" int srm_probe_copy(void *d_dst, const void *d_src, size_t bytes, int32_t streaming, void *hip_stream)
{
    if (!d_dst || !d_src) return fail(SRM_EINVAL, "srm_probe_copy: null argument");
    if (bytes == 0 || bytes % 16 || ((uintptr_t)d_dst | (uintptr_t)d_src) % 16)
        return fail(SRM_EINVAL, "srm_probe_copy: size and pointers must be multiples of 16 bytes");
    constexpr int U = 4;
    const int64_t n16 = (int64_t)(bytes / 16);
    const int64_t blocks = cdiv(n16, 256 * U);
    if (blocks >= (1ll << 31)) return fail(SRM_EINVAL, "srm_probe_copy: at most 32 TiB per call");
    if (streaming)
        hipLaunchKernelGGL((probe_copy_kernel<U, true>), dim3((unsigned)blocks), dim3(256), 0, as_stream(hip_stream),
                           (const u32x4_t *)d_src, (u32x4_t *)d_dst, n16);
    else
        hipLaunchKernelGGL((probe_copy_kernel<U, false>), dim3((unsigned)blocks), dim3(256), 0, as_stream(hip_stream),
                           (const u32x4_t *)d_src, (u32x4_t *)d_dst, n16);
    HIP_TRY(hipGetLastError());
    return SRM_OK;
}

extern "C" int srm_probe_mfma(float *d_out, int32_t blocks, int32_t iters, int32_t random_operands, double *flop,
                              void *hip_stream)
{
    if (!d_out) return fail(SRM_EINVAL, "srm_probe_mfma: null argument");
    if (blocks <= 0 || blocks > (1 << 20) || iters <= 0 || iters > (1 << 20))
        return fail(SRM_EINVAL, "srm_probe_mfma: blocks and iters must lie in [1, 2^20]");
    hipLaunchKernelGGL(probe_mfma_kernel, dim3((unsigned)blocks), dim3(256), 0, as_stream(hip_stream), d_out, iters, 1.0f,
                       random_operands ? 1 : 0);
    HIP_TRY(hipGetLastError());
    if (flop) *flop = (double)blocks * 4 /*wavefronts*/ * iters * 8 /*tiles*/ * (2.0 * 16 * 16 * 32);
    return SRM_OK;
}

extern "C" void srm_linear_timeline_probe(void *d_u64, int64_t blocks)
{
    g_clock_probe = blocks > 0 ? static_cast<unsigned long long *>(d_u64) : nullptr;
    g_clock_blocks = g_clock_probe ? blocks : 0;
}

extern "C" size_t srm_linear_scratch_bytes(int64_t M, int32_t N)
{
    if (M <= 0 || N <= 0) return 0;
    return align_up((size_t)M * cdiv(N, 64) * 4, 256) * 2;
}

template <typename T>
static int linear_entry(int epilogue, const void *A, const void *W, const float *bias, int64_t M, int N, int K,
                        void *out, int32_t *amax, void *scratch, hipStream_t st)
{
    switch (epilogue) {
    case 0: return linear<EPI_STORE, T>(A, W, bias, M, N, K, out, st);
    case 1: return linear<EPI_GELU, T>(A, W, bias, M, N, K, out, st);
    case 2: return linear<EPI_RESID, T>(A, W, bias, M, N, K, out, st);
    case 3: {
        float *pv = static_cast<float *>(scratch);
        int32_t *pi = reinterpret_cast<int32_t *>(static_cast<unsigned char *>(scratch) +
                                                  align_up((size_t)M * cdiv(N, 64) * 4, 256));
        int nparts = 0;
        SRM_TRY((linear<EPI_ARGMAX, T>(A, W, bias, M, N, K, out, st, pv, pi, 64, &nparts)));
        return argmax_finalize(pv, pi, M, nparts, amax, 0, 1, N, st);
    }
    case 4: return linear<EPI_F32, T>(A, W, bias, M, N, K, out, st);
    default: return fail(SRM_EINVAL, "srm_linear: unknown epilogue %d", epilogue);
    }
}

// ------------------------------------------------------------------ entry point that allocates nothing
// Scratch of srm_linear_argmax_noalloc: the per-column-tile (max, index) partials of the LM-head form,
// [M][ceil(N / 64)] fp32 then the same of int32, in a file-scope device array instead of a caller's
// workspace.  Every GPU the library runs on holds its own copy until the process ends.  In host code the
// array's name is only a handle: its device address is looked up once per device and used from then on.
constexpr size_t kNoallocScratch = (size_t)8 << 20;
static __device__ __align__(256) unsigned char scratch[kNoallocScratch];
constexpr int kNoallocMaxDevices = 64;
static void *g_noalloc_ptr[kNoallocMaxDevices];
static std::mutex g_noalloc_mutex;

static int noalloc_scratch(void **out)
{
    int dev = -1;
    HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= kNoallocMaxDevices) return fail(SRM_EINVAL, "srm_linear_argmax_noalloc: device %d out of range", dev);
    std::lock_guard<std::mutex> lock(g_noalloc_mutex);
    if (!g_noalloc_ptr[dev]) {
        void *ptr = nullptr;
        HIP_TRY(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
        if (!ptr) return fail(SRM_EHIP, "srm_linear_argmax_noalloc: no address for the scratch array on device %d", dev);
        g_noalloc_ptr[dev] = ptr;
    }
    *out = g_noalloc_ptr[dev];
    return SRM_OK;
}

extern "C" size_t srm_linear_argmax_noalloc_max_bytes(void) { return kNoallocScratch; }

extern "C" int srm_linear_argmax_noalloc(int32_t dtype, const void *d_A, const void *d_W, const float *d_bias,
                                         int64_t M, int32_t N, int32_t K, int32_t *d_argmax, void *hip_stream)
{
    const char *who = "srm_linear_argmax_noalloc";
    if (!d_A || !d_W || !d_argmax) return fail(SRM_EINVAL, "%s: null argument", who);
    if (M <= 0 || N <= 0 || K <= 0) return fail(SRM_EINVAL, "%s: sizes must be positive", who);
    const size_t need = srm_linear_scratch_bytes(M, N);
    if (need > kNoallocScratch)
        return fail(SRM_EINVAL, "%s: M = %lld rows x N = %d columns need %zu bytes of partial results, the built-in "
                                "scratch holds %zu (use srm_linear with a workspace)", who, (long long)M, N, need,
                    kNoallocScratch);
    void *ptr = nullptr;
    SRM_TRY(noalloc_scratch(&ptr));
    hipStream_t st = as_stream(hip_stream);
    if (dtype == SRM_BF16) return linear_entry<bf16>(3, d_A, d_W, d_bias, M, N, K, nullptr, d_argmax, ptr, st);
    if (dtype == SRM_FP32) return linear_entry<float>(3, d_A, d_W, d_bias, M, N, K, nullptr, d_argmax, ptr, st);
    return fail(SRM_EINVAL, "%s: unknown dtype %d", who, dtype);
}

extern "C" int srm_linear(int32_t dtype, int32_t epilogue, const void *d_A, const void *d_W, const float *d_bias,
                          int64_t M, int32_t N, int32_t K, void *d_out, int32_t *d_argmax, void *d_scratch,
                          void *hip_stream)
{
    if (!d_A || !d_W) return fail(SRM_EINVAL, "srm_linear: null operand");
    // epilogue codes >= 100 pin a bf16 tile, (tile + 1) * 100 + epilogue, for tile sweeps
    int forced = -1;
    if (epilogue >= 100) {
        forced = epilogue / 100 - 1;
        epilogue %= 100;
        if (forced >= kNumTiles || dtype != SRM_BF16) return fail(SRM_EINVAL, "srm_linear: unknown tile code");
    }
    if (epilogue == 3 ? (!d_argmax || !d_scratch) : !d_out) return fail(SRM_EINVAL, "srm_linear: null output");
    if (M <= 0 || N <= 0 || K <= 0) return fail(SRM_EINVAL, "srm_linear: sizes must be positive");
    hipStream_t st = as_stream(hip_stream);
    g_force_tile = forced;
    int rc;
    if (dtype == SRM_BF16) rc = linear_entry<bf16>(epilogue, d_A, d_W, d_bias, M, N, K, d_out, d_argmax, d_scratch, st);
    else if (dtype == SRM_FP32) rc = linear_entry<float>(epilogue, d_A, d_W, d_bias, M, N, K, d_out, d_argmax, d_scratch, st);
    else rc = fail(SRM_EINVAL, "srm_linear: unknown dtype %d", dtype);
    g_force_tile = -1;
    return rc;
}

// ------------------------------------------------------------------ few samples: steps as one kernel
// (Included here so that its kernels come last in the code object: with 0.3 MB of them in front, the chains of short launches
// of the others were up to 1 % slower, by where their own code then lies: sequence form 4 x 256 of the fp32 model 191.8 | 193.5 us.)
#include "few.hpp"

constexpr int kFewGroupColumns = 8, kFewGroupBlocks = kFewGroups * 256 / kFewGroupColumns, kFewCuLds = 84 * 1024;
constexpr int64_t kFewGroupRows = kFewGroups * 4;    // samples of a call at most
static size_t few_group_words_bytes(const srm_model *m, int64_t B, int mb)
{
    return (align_up((size_t)B, mb) * ((size_t)2 * m->d + m->ff) + (size_t)kFewGroupBlocks * (2 * mb + 1)) * sizeof(few_word) + 256;
}

// Whether a model gets the packed copies: where some call can use them on this device (current when the model is made).
static bool few_packable(const srm_model *m)
{
    return few_max_rows(m) > 0 && (!m->noproj || m->L >= 6) && !few_off() && m->device < kFewDevices &&
           align_up(m->d / few_columns(m), kFewShare) <= (size_t)device_cus();
}

// The packed copies of a model's matrices and, in front of them, its table of layers: one allocation of whole 2 MB pages (a table
// of its own and the odd size went with decode steps of 65536 samples up to 1 % slower, 27119 against 26849 us before there were
// copies; 26735 against 26723 this way).
static int few_pack(srm_model *m)
{
    const size_t d = m->d, ff = m->ff, s = m->wsize, proj = m->noproj ? 0 : d * d * s, mlp = d * ff * s;
    const size_t head = align_up((size_t)m->V, 4) * d * s, table = align_up(sizeof(FewLayer) * m->L, 256);
    const size_t words = m->wsize == 4 ? few_group_words_bytes(m, kFewGroupRows, kFewGroupRows / kFewGroups) : 0;
    const size_t total = align_up(table + m->L * (2 * proj + 2 * mlp) + head + words, (size_t)2 << 20);
    hipError_t e = hipMalloc(&m->few_slab, total);
    if (e == hipErrorOutOfMemory) {                  // the step kernels do all that these are for
        (void)hipGetLastError();
        m->few_slab = nullptr;
        return SRM_OK;
    }
    if (e != hipSuccess) return fail(SRM_EHIP, "srm_init_weights: hipMalloc(%zu): %s", total, hipGetErrorString(e));
    m->few_layers = static_cast<FewLayer *>(m->few_slab);
    unsigned char *at = static_cast<unsigned char *>(m->few_slab) + table;
    auto pack = [&](const void *W, size_t N, size_t K) {
        const int64_t n = (int64_t)(align_up(N, 4) * K * s / 16);
        hipLaunchKernelGGL(few_pack_kernel, dim3((unsigned)cdiv(n, 256)), dim3(256), 0, nullptr, static_cast<const u32x4_t *>(W),
                           reinterpret_cast<u32x4_t *>(at), (int)N, (int)(K * s / 16));
        const void *p = at;
        at += n * 16;
        return p;
    };
    std::vector<FewLayer> fl(m->L);
    for (int l = 0; l < m->L; ++l) {
        const LayerDev &y = m->layers[l];
        fl[l] = FewLayer{{y.ln1_g, y.ln1_b, y.ln2_g, y.ln2_b}, y.b_in, y.alpha, y.beta, y.lam, y.b_out, y.b_up, y.b_down,
                         nullptr, nullptr, pack(y.w_up, ff, d), pack(y.w_down, d, ff)};
        if (!m->noproj) {
            fl[l].w_in = pack(y.w_in, d, d);
            fl[l].w_out = pack(y.w_out, d, d);
        }
    }
    m->few_head = pack(m->head, m->V, d);
    if (words) m->few_words = at;                    // (the copies are whole multiples of 256 bytes)
    e = hipGetLastError();
    if (e == hipSuccess) e = hipMemcpy(m->few_layers, fl.data(), sizeof(FewLayer) * m->L, hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipDeviceSynchronize();
    return e == hipSuccess ? SRM_OK : fail(SRM_EHIP, "srm_init_weights: packed matrices: %s", hipGetErrorString(e));
}

// x and mx of a pass's last rows (LastRows) into w.g, in front of the MLP's activations; w becomes the workspace of those rows.
template <typename T>
static int gather_last_rows(const srm_model *m, Workspace &w, const LastRows &lr, int64_t rows, hipStream_t st)
{
    unsigned char *p = static_cast<unsigned char *>(w.g);
    const size_t xb = align_up((size_t)lr.n * m->d * 4, 256), mb = align_up((size_t)lr.n * m->dm * sizeof(T), 256);
    if (xb + mb + (size_t)lr.n * m->ff * sizeof(T) > (size_t)rows * m->ff * sizeof(T))
        return fail(SRM_EINVAL, "gather_last_rows: no room");
    float *x = reinterpret_cast<float *>(p);
    T *mx = reinterpret_cast<T *>(p + xb);
    hipLaunchKernelGGL((last_rows_kernel<T>), dim3((unsigned)lr.n), dim3(256), 0, st, w.x, static_cast<const T *>(w.mx), x, mx,
                       m->d, m->dm, lr.len, lr.seq_end, lr.base, rows);
    HIP_TRY(hipGetLastError());
    w.x = x;
    w.mx = mx;
    w.g = p + xb + mb;
    return SRM_OK;
}

// The launch.  Its work-groups wait for each other, so all of them must become resident: of this process's kernels of this kind
// only as many run at a time on a device as have a CU for each work-group (two of d = 1024, four of the others), whatever their
// streams, and other kernels end by themselves.  The CUs are counted in shares of 64, each with the event of its latest kernel;
// a launch takes the shares that its stream had before, else unused ones, else those used longest ago, and waits for their
// events.  What this cannot see (other processes' kernels of this kind, cooperative kernels that fill the device) is what the
// arrival is for.  A cooperative launch costs 20 us instead of 5 (a step of 16 layers, d = 1024: 211 | 195 us) and, once used,
// makes the later launches of the process slower (36 launches, 315 us: by 1 to 2 %).
// us per step of 1 | 2 | 4 | 8 streams at once, a thread each, all streams together: d = 512, 1 row: one kernel at a time 73 | 76 |
// 76 | 76, this 73 | 41 | 24 | 28, step kernels 134 | 77 | 42 | 41; 4 rows 97 | 99 | 99 | 99, 97 | 51 | 31 | 36, 137 | 75 | 43 | 42;
// d = 1024, 1 row 198 | 200 | 200 | 199, 198 | 123 | 124 | 128, 348 | 209 | 127 | 164; 4 rows 289 | 291 | 290 | 291, 288 | 168 | 171 |
// 177, 354 | 213 | 130 | 131: there the step kernels are the better ones from four streams on.
struct FewShare { hipEvent_t ev; hipStream_t st; unsigned long long used; };         // st: only a preference
// events are kept until the process ends; met: the latest launch that found one of another stream
struct FewDevice { FewShare share[kFewShares]; hipEvent_t events[kFewShares]; unsigned long long met; };
static std::mutex few_lock;
static FewDevice few_devices[kFewDevices];
static unsigned long long few_launches;
// How many other streams have a kernel of this kind running or waiting (0.3 us for each; none to ask where one stream launches
// them).  None has at the moment, but one had in the latest few launches: one, which is between two steps.  Streams that launch
// in turn, each behind a wait for the other, never meet.
static int few_others(int device, hipStream_t st)
{
    const std::lock_guard<std::mutex> hold(few_lock);
    FewDevice &d = few_devices[device];
    hipStream_t seen[kFewShares];
    int n = 0;
    bool recent = false;
    for (const FewShare &s : d.share) {
        if (!s.used || s.st == st || std::find(seen, seen + n, s.st) != seen + n) continue;
        recent = recent || few_launches - s.used < kFewShares;
        // (the question belongs to no capture that this thread has begun)
        hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
        if (refused(hipThreadExchangeStreamCaptureMode(&mode))) continue;
        const hipError_t e = hipEventQuery(s.ev);
        (void)hipThreadExchangeStreamCaptureMode(&mode);
        if (e == hipErrorNotReady) seen[n++] = s.st;
        else (void)refused(e);
    }
    if (n) d.met = few_launches + 1;
    else if (recent && d.met && few_launches + 1 - d.met < kFewShares) return 1;
    return n;
}
// reset(): what is to stand between the kernels that the launch waits for and its own.
template <typename F>
static int few_launch(int device, const void *kern, int blocks, int threads, int lds, void **args, hipStream_t st, F &&reset)
{
    const std::lock_guard<std::mutex> hold(few_lock);
    FewDevice &d = few_devices[device];
    const int need = (int)cdiv(blocks, kFewShare), all = std::min(device_cus() / kFewShare, kFewShares) / need * need;
    if (need < 1 || all < need) return fail(SRM_EINVAL, "few_launch: %d work-groups", blocks);
    int at = 0;
    auto rank = [&](int i) {                         // of the shares from i on: smaller is better
        unsigned long long latest = 0;
        bool mine = true;
        for (int k = i; k < i + need; ++k) {
            latest = std::max(latest, d.share[k].used);
            mine = mine && d.share[k].used && d.share[k].st == st;
        }
        return mine ? 0 : latest + 1;
    };
    for (int i = need; i < all; i += need)
        if (rank(i) < rank(at)) at = i;
    // an event that no other share's kernel is known by (there are as many events as shares)
    auto others_have = [&](hipEvent_t e) {
        for (int k = 0; k < kFewShares; ++k)
            if ((k < at || k >= at + need) && d.share[k].used && d.share[k].ev == e) return true;
        return false;
    };
    hipEvent_t *own = d.events;
    while (*own && others_have(*own)) ++own;
    if (!*own) HIP_TRY(hipEventCreateWithFlags(own, hipEventDisableTiming));
    const hipEvent_t ev = *own;
    hipEvent_t waited = nullptr;
    for (int k = at; k < at + need; ++k) {
        const hipEvent_t before = d.share[k].ev;
        if (before && before != waited) HIP_TRY(hipStreamWaitEvent(st, before, 0));
        waited = before;
    }
    SRM_TRY(reset());
    HIP_TRY(hipExtLaunchKernel(kern, dim3((unsigned)blocks), dim3((unsigned)threads), args, (size_t)lds, st, nullptr, ev, 0));
    ++few_launches;
    for (int k = at; k < at + need; ++k) d.share[k] = FewShare{ev, st, few_launches};
    return SRM_OK;
}

// How often an arrival is asked for before it is given up, some 8 ms: longer than any other kernel of this library keeps CUs
// from it, and about what one work-group alone then takes for a step (us per step, together | alone: d = 1024, 16 layers, 1 row
// 195 | 7040, 4 rows 290 | 7310, without projections 149 | 5990; d = 512, 8 layers 75 | 960; fp32, d = 256, 8 rows 52 | 410).  The
// arrival itself costs 0.3 to 0.7 us per launch (195.5 | 196.2; d = 512 74.8 | 75.1).
constexpr unsigned few_arrive_polls = 1u << 13;
// Of the groups of few_group_rows, some 0.1 ms (64 times that until a whole group has started): see stack_arrive_polls.  (Three processes
// that generate with the toy model at a time, us per token: 8 rows 120, 32 rows 124; step kernels 99 and 124; one work-group alone
// behind 8 ms 1793 and 1866.)
constexpr unsigned few_group_polls = 1u << 9;

static const void *few_group_kernel(int mb)
{
    return mb == 1 ? reinterpret_cast<const void *>(few_rows_kernel<float, 256, kFewGroupColumns, 1, true, true>)
           : mb == 2 ? reinterpret_cast<const void *>(few_rows_kernel<float, 256, kFewGroupColumns, 2, true, true>)
                     : reinterpret_cast<const void *>(few_rows_kernel<float, 256, kFewGroupColumns, 4, true, true>);
}
template <typename TW, int D, int NWC, bool PROJ>
static const void *few_kernel(int mb)
{
    switch (mb) {
    case 1: return reinterpret_cast<const void *>(few_rows_kernel<TW, D, NWC, 1, PROJ>);
    case 2: return reinterpret_cast<const void *>(few_rows_kernel<TW, D, NWC, 2, PROJ>);
    case 4: return reinterpret_cast<const void *>(few_rows_kernel<TW, D, NWC, 4, PROJ>);
    }
    if constexpr (sizeof(TW) == 4) return reinterpret_cast<const void *>(few_rows_kernel<TW, D, NWC, 8, PROJ>);
    else return nullptr;
}

// fp32 steps in groups of rows, each by the work-groups of one XCD, whose exchanges stay in its L2: the rows of a group (0: not
// that way).  Every XCD reads all weights, at 0.95 TB/s; what is left beside that is the exchanges, some 1 us each.  Generation with the
// toy model (d = 256, 4 layers, 4096 tokens), us per token, 64 work-groups over all XCDs (from 9 rows on step kernels) | groups: 1 row
// 31.5 | 26.2, 2: 32.9 | 26.2, 4: 38.1 | 29.4, 8: 52.7 | 30.3, 9: 84 | 33, 16: 86 | 34, 17: 92 | 37, 32: 97 | 38.  Up to 8 rows both have the
// same bits, and where other streams launch such steps side by side the small grids, of which four fit the device, get more done
// (8 rows, us per token of 1 | 2 | 4 streams: groups 30 | 30 | 30, small grids 52 | 27 | 14); more rows
// hold the device for their call, whatever their streams, and get more done than the step kernels all the same (16 rows, 2 | 4
// streams, step kernels 49 | 143, groups 34 | 35; 32 rows 56 | 206, 38 | 39).  Single steps of more than 8 rows
// keep the sums of the step kernels.
// Their words, more than the arrays of as many rows, are the model's own, so that the way of a call does not depend on its
// workspace.  Kernels that take the whole device never run side by side, whatever their streams (few_launch).
static int few_group_rows(const srm_model *m, int64_t B, int64_t G)
{
    if (!m->few_words || B > kFewGroupRows || (G == 1 && B > few_max_rows(m))) return 0;
    if (device_cus() < kFewGroupBlocks || device_cus() >= 2 * kFewGroupBlocks) return 0;
    return B <= kFewGroups ? 1 : B <= 2 * kFewGroups ? 2 : 4;
}
static int few_run(srm_model *m, int64_t B, int pos0, int G, const int32_t *tok_in, int32_t *tok_out, int32_t *store,
                   void *state, float temperature, uint32_t seed, float *logits, float *hidden, void *ws, hipStream_t st)
{
    const int D = m->d;
    st = few_stream(st);
    int gmb = few_group_rows(m, B, G);
    if (gmb && B <= few_max_rows(m) && few_others(m->device, st)) gmb = 0;
    const int mb = gmb ? gmb : few_bucket(B), nwc = gmb ? kFewGroupColumns : few_columns(m), nb = gmb ? kFewGroupBlocks : D / nwc;
    const void *kern = gmb ? few_group_kernel(gmb)
                       : m->wsize == 4 ? few_kernel<float, 256, 4, true>(mb)
                       : m->noproj ? (D == 512 ? few_kernel<bf16, 512, 8, false>(mb) : few_kernel<bf16, 1024, 8, false>(mb))
                                   : (D == 512 ? few_kernel<bf16, 512, 8, true>(mb) : few_kernel<bf16, 1024, 8, true>(mb));
    if (!kern) return fail(SRM_EINVAL, "few_run: no kernel for %lld rows", (long long)B);
    FewArgs a{};
    a.layers = m->few_layers;
    a.embed = m->embed; a.head = m->few_head;
    a.lnf_g = m->lnf_g; a.lnf_b = m->lnf_b;
    a.V = m->V; a.L = m->L; a.dh = m->dm / m->Hs; a.hrow = m->hrow; a.n_ctx = m->cfg.n_ctx;
    a.eps = m->cfg.ln_eps;
    a.B = a.Bs = (int)B; a.row0 = 0; a.pos0 = pos0; a.G = G;
    a.tok_in = tok_in; a.tok_out = tok_out; a.store = store;
    a.state = state; a.state_half = m->shalf ? 1 : 0;
    a.logits = logits; a.hidden = hidden;
    a.temp = temperature; a.seed = seed;
    unsigned char *base = gmb ? m->few_words : static_cast<unsigned char *>(ws) + few_list_bytes(B);
    a.xw = reinterpret_cast<few_word *>(base);
    const size_t rows = gmb ? align_up(B, mb) : mb;
    a.mw = a.xw + rows * D;
    a.gw = a.mw + rows * D;
    a.pw = a.gw + rows * (m->wsize == 2 ? m->ff / 2 : m->ff);
    few_word *const here = a.pw + (size_t)mb * nb * 2;           // (of groups, see few_rows_kernel)
    a.flag = reinterpret_cast<unsigned *>(here + (gmb ? nb : 0));
    a.max_polls = poll_bound(1u << 21);              // a second or two
    a.arrive_polls = gmb ? few_group_polls : few_arrive_polls;
    // words of the arrivals of work-groups that are withdrawn from the start
    int w0 = 0, w1 = 0;
    const char *sw = getenv("SRM_ONE_KERNEL_STEP");
    if (sw && sw[0] == '2') {
        const few_word *const words = reinterpret_cast<const few_word *>(base);
        w0 = gmb ? (int)(here - words) + (sw[1] == ':' ? atoi(sw + 2) : 0) : (int)(a.pw - words) + (nb - 1) * mb * 2;
        w1 = gmb ? (int)(here - words) + nb : w0 + 1;
    }
    if (sw && sw[0] == '3') a.arrive_polls = sw[1] == ':' ? (unsigned)atoi(sw + 2) : 0;
    a.scattered = sw && sw[0] == '4';
    const int n = (int)((gmb ? few_group_words_bytes(m, B, mb) : few_words_bytes(m, B)) / 16), n_store = store ? (int)B * G : 0;
    auto reset = [&] {
        hipLaunchKernelGGL(few_reset_kernel, dim3((unsigned)std::min<int64_t>(64, cdiv(n, 256))), dim3(256), 0, st,
                           reinterpret_cast<u32x4_t *>(base), n, w0, w1, static_cast<int *>(ws), store, n_store);
        HIP_TRY(hipGetLastError());
        return (int)SRM_OK;
    };
    if (!gmb) SRM_TRY(reset());
    // (groups: a CU for each work-group)
    const int lds = std::max(few_lds_bytes((int)m->wsize, D, nwc, mb), gmb ? kFewCuLds : 0);
    HIP_TRY(hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds));
    void *args[] = {&a};
    return few_launch(m->device, kern, nb, (kFewGather + nwc) * 64, lds, args, st, [&] { return gmb ? reset() : (int)SRM_OK; });
}

// ------------------------------------------------------------------ some dozens of samples and more: all layers as one kernel
#include "stack.hpp"

// How the rows of a step are cut: groups of at least 16.  Up to 64 rows of a group all its members share one tile of rows, 16
// columns each; above, they are 16 pairs that share 32 columns and take the tiles of up to 64 rows in turn.
struct StackPlan {
    int per, cw, rb, tiles;  // rows of a group; columns of a member; 16-row blocks of a tile; tiles of a group
};
static StackPlan stack_plan(int64_t rows)
{
    StackPlan s;
    s.per = (int)std::max<int64_t>(16, cdiv(rows, kStackGroups));
    s.cw = s.per <= 64 ? 16 : 32;
    s.tiles = s.per <= 64 ? 1 : 2 * (int)cdiv(s.per, 128);
    s.rb = (int)cdiv(cdiv(s.per, s.tiles), 16);
    return s;
}
// Its memory in the workspace: x and a where they always are, the rest from the array of u on, over what only the step kernels
// or the head behind it use.  Of one group m lies where g does: each is written behind a wait for the last to have read the other.
// (So five rows find room in the arrays of a small vocabulary too; those of several groups do not wait for each other.)
struct StackMem {
    unsigned char *words;
    float2 *stats;
    bf16 *m, *g;
    size_t bytes;            // from u on
};
static StackMem stack_carve(const srm_model *m, const Workspace &w, const StackPlan &s, int64_t rows)
{
    StackMem r;
    unsigned char *p = static_cast<unsigned char *>(w.u);
    size_t off = 0;
    auto take = [&](size_t bytes) {
        unsigned char *q = p + off;
        off += align_up(bytes, 256);
        return q;
    };
    const size_t used = (size_t)cdiv(rows, s.per) * s.tiles * s.rb * 16;
    r.words = take(kStackWordBytes);
    r.stats = reinterpret_cast<float2 *>(take((size_t)rows * (m->d / s.cw) * sizeof(float2)));
    if (rows > s.per) r.m = reinterpret_cast<bf16 *>(take(used * m->d * 2));
    r.g = reinterpret_cast<bf16 *>(take(used * m->ff * 2));
    if (rows <= s.per) r.m = r.g;
    r.bytes = off;
    return r;
}
// Which steps.  Measured per decode step with logits (us, step kernels | layers as one kernel), d = 512, 8 layers, 32000 tokens: 5
// rows 139 | 120, 9: 170 | 122, 37: 182 | 122, 128: 190 | 133, 129: 204 | 154, 300: 241 | 178, 512: 256 | 207, 513: 293 | 222, 1024: 316 |
// 256, 1025: 376 | 334, 1536: 407 | 343, 1537: 416 | 418, 1700: 428 | 416, 2048: 437 | 408, 2304: 525 | 476; then a group's six tiles are of
// four blocks and not of three: 2305: 532 | 565, 2560: 536 | 579, 3000: 579 | 582, 3072: 574 | 578.  Up to four rows few.hpp's steps are
// shorter (98).  A width of 512 is what the kernel's registers and LDS were laid out for; at 1024 every XCD would read 21 MB of
// weights per layer, 22 us at the 0.95 TB/s an XCD gets, where a layer of 37 rows takes 25.  Six layers: as in few_ok, for the
// results of shallower models.  (A width of 256, models without projections and combined heads would be forms of its own, which
// have not been made or measured.)
// Streams that launch such steps side by side take half or a quarter of the work-groups each (few_others), same bits.  us per step, no
// logits, all streams together, of 1 | 2 | 4 streams, a thread each: 37 rows 119 | 91 | 75 to 137, step kernels 178 | 99 | 61 to 99 (how the
// runtime deals the streams to its queues); 300: 169 | 145 | 119, 231 | 132 | 92; 1024: 235 | 213 | 190, 300 | 215 | 205.  In turn, each
// behind a wait for the one before: 37 rows 136 | 137 | 136 (by half and by a quarter 186 | 284), 300: 186 | 185 | 184 (271 | 438), 1024:
// 250 | 250 | 250 (370 | 609).  Larger steps take the whole device one after the other: of 2 | 3 | 4 streams, shared | this, 1100 rows -
// | 314 | 444, - | 302 | 303; 1536: - | 330 | 261, - | 300 | 299; 2048: 346 | 396 | 319 to 555, 358 | 358 | 359; 3000: - | 574 | 803, - | 504 | 506.
// Beside other work of the process (300 rows, us per step and calls per second of the other stream, step kernels | this; large model):
// prefills of 256 x 128 3666 and 93 | 554 and 67; decode steps of 16384 samples 3065 and 149 | 555 and 106; of 3001 with top-p 594
// and 437 | 235 and 171; no arrival was given up (longest step 1.5 ms).
constexpr int64_t kStackSharedRows = 1024;
constexpr int64_t kStackMinRows = 5, kStackMaxRows = 2304;
static_assert(kStackMaxRows <= (int64_t)kStackGroups * kStackMaxPer, "their positions are kept in LDS");
// Polls of the arrival, some 0.1 ms: beside other work of the process as good as any longer (300 rows beside prefills, us per step with
// 7 | 0.8 | 0.2 | 0.1 | 0.04 | 0.01 ms: 564 | 561 | 560 | 560 | 593 | 593, 1024 rows beside 3001 with top-p 279 | 279 | 278 | 278 | 282 | 351).  It
// counts where other processes run such steps, and each gets some of the CUs (300 rows, three processes: 7216 | 1381 | 787 | 617 | 593 |
// 593, step kernels 329; two: 340 | - | 336 | - | 336, 280; waiting for all, and one alone otherwise, three took 29242).
constexpr unsigned stack_arrive_polls = 1u << 9;
static bool stack_ok(const srm_model *m, int64_t rows, size_t ws_bytes, hipStream_t st)
{
    if (!m->few_layers || m->wsize != 2 || m->d != 512 || m->noproj || m->L < 6 || rows < kStackMinRows || rows > kStackMaxRows) return false;
    if (device_cus() < kStackBlocks || few_off()) return false;
    if (getenv("SRM_TOKEN_MIX") || getenv("SRM_FUSE_MIXER") || getenv("SRM_LN_ON_LOAD")) return false;
    // (the last 256 bytes: srm_generate's counters)
    const Workspace w = carve(m, reinterpret_cast<void *>(256), rows);
    const size_t at = reinterpret_cast<size_t>(w.u) - 256;
    if (at + stack_carve(m, w, stack_plan(rows), rows).bytes + 256 > ws_bytes) return false;
    return one_kernel_stream(few_stream(st));
}

template <int CW, int RB, bool MULTI>
static const void *stack_kernel_of()
{
    return reinterpret_cast<const void *>(stack_kernel<512, CW, RB, MULTI>);
}
static int stack_layers(srm_model *m, const DecodeArgs &d, const Workspace &w, int64_t b0, int64_t nb, hipStream_t st, const unsigned **dead)
{
    const StackPlan s = stack_plan(nb);
    const StackMem mem = stack_carve(m, w, s, nb);
    st = few_stream(st);
    const void *kern = s.cw == 16 ? (s.rb == 1 ? stack_kernel_of<16, 1, false>() : s.rb == 2 ? stack_kernel_of<16, 2, false>()
                                     : s.rb == 3 ? stack_kernel_of<16, 3, false>() : stack_kernel_of<16, 4, false>())
                       : s.tiles == 2 ? (s.rb == 3 ? stack_kernel_of<32, 3, false>() : stack_kernel_of<32, 4, false>())
                                      : (s.rb == 3 ? stack_kernel_of<32, 3, true>() : stack_kernel_of<32, 4, true>());
    StackArgs a{};
    a.layers = m->few_layers;
    a.lnf_g = m->lnf_g; a.lnf_b = m->lnf_b;
    a.L = m->L; a.dh = m->dm / m->Hs; a.hrow = m->hrow; a.n_ctx = m->cfg.n_ctx;
    a.eps = m->cfg.ln_eps;
    a.rows = (int)nb; a.per = s.per; a.tiles = s.tiles;
    a.pos = d.pos; a.pos_dev = d.pos_dev; a.pos_rows = d.pos_rows ? d.pos_rows + b0 : nullptr;
    a.state = static_cast<unsigned char *>(d.state) + (size_t)b0 * m->dm * m->ssize;
    a.layer_bytes = (size_t)d.B * m->dm * m->ssize;
    a.state_half = m->shalf ? 1 : 0;
    a.x = w.x; a.stats = mem.stats; a.m = mem.m; a.g = mem.g;
    a.a = static_cast<bf16 *>(w.a);
    a.hidden = d.hidden ? d.hidden + (size_t)b0 * m->d : nullptr;
    a.here = reinterpret_cast<few_word *>(mem.words);
    a.count = reinterpret_cast<unsigned *>(mem.words + kStackBlocks * 8);
    a.left = reinterpret_cast<unsigned *>(mem.words + kStackBlocks * 8 + kStackGroups * 128);
    a.dead = d.gave_up ? d.gave_up : a.left + 1;     // (that of a call stays set)
    a.max_polls = poll_bound(1u << 21, d.step);      // a second or two
    a.arrive_polls = stack_arrive_polls;
    const int others = nb > kStackSharedRows ? 0 : few_others(m->device, st), blocks = kStackBlocks / (others == 0 ? 1 : others == 1 ? 2 : 4);
    int starting = kStackBlocks;                     // work-groups that are not withdrawn from the start
    const char *sw = getenv("SRM_ONE_KERNEL_STEP");
    if (sw && sw[0] == '2') starting = sw[1] == ':' ? atoi(sw + 2) : 0;
    if (sw && sw[0] == '3') a.arrive_polls = sw[1] == ':' ? (unsigned)atoi(sw + 2) : 0;
    a.scattered = sw && sw[0] == '4';
    *dead = a.dead;
    auto begin = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)cdiv(nb, 4)), dim3(256), 0, st, d.tok_in + b0, static_cast<const bf16 *>(m->embed),
                           m->V, w.x, mem.stats, (int)nb, reinterpret_cast<u32x4_t *>(mem.words), starting, b0 == 0 ? d.advance_ctr : nullptr);
        return hipGetLastError();
    };
    HIP_TRY(s.cw == 16 ? begin(stack_begin_kernel<512, 16>) : begin(stack_begin_kernel<512, 32>));
    const int lds = stack_lds_bytes(512, s.cw, s.rb);
    HIP_TRY(hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, std::max(lds, kFewCuLds)));
    void *args[] = {&a};
    return few_launch(m->device, kern, blocks, kStackThreads, std::max(lds, kFewCuLds), args, st, [] { return (int)SRM_OK; });
}
