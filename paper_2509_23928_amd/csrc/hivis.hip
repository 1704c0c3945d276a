// Host side of the HiViS draft-verify library: context, state machine, launch sequences.
// The C ABI is declared and documented in include/hivis.h.
#include "hivis.h"
#include "hivis_sizes.h"
#include "hivis_kernels.h"
#include "hivis_gemm.h"
#include "hivis_fused.h"
#include "hivis_stream.h"
#include "hivis_tile.h"
#include "hivis_attn.h"
#include "hivis_tree.h"

#include <hip/hip_ext.h>
#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <cstdlib>
#include <map>
#include <mutex>
#include <string>
#include <vector>

using namespace hivis;

// Scratch memory of hivis_draft_noalloc: a file-scope device array instead of an allocation.  Every GPU the library runs on
// holds its own copy at its own address until the process ends.  In host code the name `scratch` is only a stand-in for
// the symbol: the device address is looked up once per device with hipGetSymbolAddress (scratch_for_device below) and that
// pointer, never the name, is what kernels receive.
#define HIVIS_SCRATCH_BYTES HIVIS_NOALLOC_SCRATCH_BYTES
static __device__ __align__(256) unsigned char scratch[HIVIS_SCRATCH_BYTES];

namespace {

enum State { ST_CREATED = 0, ST_READY, ST_DRAFTED, ST_VERIFIED, ST_TREE_DRAFTED, ST_TREE_VERIFIED };

// Rows of a draft tree (null pointers: ordinary causal rows)
struct TreeRows { const int* pos_delta = nullptr; const unsigned long long* mask = nullptr; };

struct LayerDev {
    void* norm1 = nullptr; void* norm2 = nullptr;   // [d] storage dtype
    uint4* wqkv = nullptr;                          // packed [d] -> [q_dim + 2 kv_dim]
    uint4* wo = nullptr;                            // packed [q_dim] -> [d]
    uint4* wgu = nullptr;                           // packed [d] -> [2 ffn]  (gate | up)
    uint4* wd = nullptr;                            // packed [ffn] -> [d]
    float* bqkv = nullptr;                          // optional q/k/v projection biases [q_dim + 2 kv_dim], in wqkv's column order
};

struct KVDev { void* k = nullptr; void* v = nullptr; int maxL = 0; };   // [B][Hkv][maxL][hd]

}  // namespace

struct hivis_ctx {
    hivis_config cfg{};
    hipStream_t stream = nullptr;
    int state = ST_CREATED;
    std::string err;
    int esize = 4;
    int num_cu = 256;

    // weights
    void* embed = nullptr; void* final_norm = nullptr; void* rho = nullptr;
    uint4* lm_head = nullptr; uint4* fuse_w = nullptr;
    uint4* fuse_w1 = nullptr;            // rows [0, d) of the fusion FC, packed on their own (K = d), and
    bool lm_ext = false;                 // the packed LM head is followed by w1's tiles in one buffer (lm_head .. lm_head + (V + d) d)
    float* emb_w2 = nullptr;             // [V][d] fp32: Embed(token) . w2, the embedding half of the fusion FC per token
    std::vector<LayerDev> layers; LayerDev draft;
    std::vector<KVDev> tkv; KVDev dkv;

    // per-sequence state (device) + host mirrors
    int* tlen = nullptr; int* dlen = nullptr; int* zeros = nullptr;
    int32_t* text = nullptr; int text_stride = 0;
    std::vector<int> h_tlen, h_dlen;
    int v = 0, K = 0;

    // activations (fp32)
    float *x = nullptr, *a = nullptr, *qkv = nullptr, *att = nullptr, *proj = nullptr, *gu = nullptr, *act = nullptr;
    float *catT = nullptr;      // [MAX_ROWS][2d]: verify features g | embeddings of the following tokens
    float *catD = nullptr;      // [B][2d]: drafter hidden f' | embedding of the drafted token
    float *u = nullptr, *dout = nullptr;
    // phase programs on row fragments (bf16 models with the fusion FC's table, one launch per phase)
    bool stream_rows = false;
    uint4* catDf = nullptr;              // the rows of catD as row fragments (of batch rows)
    uint4* vfrag = nullptr;              // features of a verify program's rows
    // up to 16 rows of a prefill: residual rows times a gain, attention rows (or features), MLP rows; sums of squares
    uint4 *st_frag = nullptr, *st_att = nullptr, *st_act = nullptr; float* st_ssq = nullptr;
    uint4* tcatf = nullptr;              // hidden rows of a tree level, or of a tree's re-feed
    float *feat = nullptr;      // [B][max_text][d] true features of prompt text rows (prefill only)
    float *attn_ws = nullptr; size_t attn_ws_floats = 0;
    int* rows_cnt = nullptr; int rows_cnt_n = 0;      // arrival counters of the key-split attention launched outside a phase program (zero between launches)
    float *logits_v = nullptr, *logits_d = nullptr, *logits_p = nullptr;
    int32_t *row_tok = nullptr, *drafts = nullptr, *ttok = nullptr, *nacc = nullptr, *out_tok = nullptr, *next_tok = nullptr;
    float* am_v = nullptr; int* am_i = nullptr;      // greedy candidates per row and segment (launch_argmax)
    int32_t* h_result = nullptr;         // pinned host mirror of [nacc | out_tok | abort flag | bad-logits flag]
    int* bad = nullptr;                  // device flag: a greedy-token kernel met a row without a finite maximum (cleared by hivis_prefill)
    bool rng_seeded = false; unsigned long long rng_seed = 0, rng_calls = 0;   // device-side uniforms (hivis_rng_seed): Philox key and draw-call count
    float* u_tree = nullptr;             // [TREE_MAX_DEPTH + 1] uniforms of hivis_tree_accept_sample, one per depth
    float *u_draft = nullptr, *u_acc = nullptr, *u_res = nullptr;   // uniform numbers of the sampling calls: [B][k_max], [B][k_max] (row stride K), [B]
    float inv_temp = 1.0f; bool drafts_sampled = false;             // set by hivis_draft_sample; hivis_accept_sample needs the drafter's distributions
    void* vis = nullptr;        // staging for vis_embeds [B][max_vis][d]
    // whole-prompt prefill buffers (bf16 models): all v+l rows of one or several sequences per layer
    int pf_rows = 0;
    hivis::PrefillSizes pf_sizes{};
    int tall_cw = 0;
    float *pf_x = nullptr, *pf_xt = nullptr, *pf_a = nullptr, *pf_qkv = nullptr, *pf_att = nullptr, *pf_proj = nullptr, *pf_gu = nullptr;
    uint4 *pf_frag = nullptr, *pf_frag2 = nullptr;      // activation fragments: of d / q_dim wide rows, and of the MLP's inner rows
    std::vector<int32_t> h_ids;

    // phase programs (fused_rows_ok: how many rows they take)
    bool fused = false;
    int fused_grid = 0; size_t fused_lds = 0, fused_lds_w = 0;      // LDS of a phase launch; of the bf16w kernels
    float* rope_tab = nullptr; float* pm = nullptr; int* pi = nullptr; unsigned* bar = nullptr;
    float* fattn_ws = nullptr; size_t fattn_ws_floats = 0;
    struct Program { hivis::Phase* dev = nullptr; int n = 0; std::vector<hivis::Phase>* host = nullptr; };
    int attn_shared_min = 128;           // rows per sequence from which a causal pass uses the shared-tile attention kernel (128 rows per workgroup)
    int keys_per_split = 192;            // attention: cached keys per workgroup (one or two 16-key tiles per wavefront) before the key range is split further
    bool keys_forced = false;            // HIVIS_KEYS_PER_SPLIT: of half-precision caches as well (attn_block_splits otherwise)
    bool attn_elect = true;              // key splits merged by the workgroup that arrives last (false: by a merge launch)
    int attn_flags = 3;                  // AttnShape::flags of the phase programs
    bool persistent = false;             // HIVIS_PERSISTENT=1: one cooperative launch per pass instead of one launch per phase
    std::map<int, Program> programs;     // key = kind * 64 + K
    unsigned long long* prof = nullptr; int prof_left = 0;   // developer aid: HIVIS_PROF=n dumps per-phase times of n verify passes

    // draft tree (batch 1): device arrays are allocated by the first hivis_tree_draft call, for the limits below
    hivis::TreeDev tree{}; bool tree_ready = false;
    int tk = 0, tdepth = 0, tn = 0;                       // top-k, depth, candidates of the current tree
    int vrows = 0;                                        // rows of the last verify pass (chain: B*(K+1); tree: N+1)
    float *tH = nullptr, *tlogits = nullptr, *tcat = nullptr, *troll = nullptr;
    int32_t* ttok_rows = nullptr;                         // tokens of a level's rows
    float* tree_pool = nullptr;                           // buffers of tree_rows_program
    float *tcand_v = nullptr, *tseg = nullptr; int32_t* tcand_i = nullptr; int tnseg = 0;   // per-segment top-k candidates and (max, sum) partials   // hidden rows, their logits, level inputs, re-feed inputs
    void** kv_ptrs = nullptr; void* kv_staging = nullptr;
    float* splitk_ws = nullptr; size_t splitk_floats = 0;      // K-slice partials (splitk_space)
    // passes that no phase program takes: split-K layers from wide_min rows on (with stand-alone kernels on both sides 10 rows were faster
    // on the skinny ones, 12 on the split-K layer); HIVIS_WIDE_GEMM=0: never
    bool no_wide_gemm = false; int wide_min = 11;
    int32_t* h_tree_result = nullptr;                     // pinned [1 + TREE_MAX_DEPTH + 1]

    // timing
    int ktime_epi = -1;                                  // GEMM epilogue kind whose verify launches are event-timed (-1: none)
    int ktime_stride = 8; int64_t ktime_seen = 0;        // every ktime_stride-th such launch is timed (an event pair costs ~8 us of idle queue)
    std::vector<hipEvent_t> kev; size_t kev_used = 0;     // event pairs recorded since the last accept
    double kms = 0; int64_t klaunches = 0; double kbytes = 0;
    bool timing = false;
    // phase timing: event pairs recorded without waiting, resolved at the next point where the stream is synchronised anyway
    std::vector<hipEvent_t> pev; std::vector<int> pev_phase; size_t pev_used = 0;
    double phase_ms[4] = {0, 0, 0, 0}; int64_t phase_calls[4] = {0, 0, 0, 0};
    std::vector<void*> allocs;
    // hivis_draft_noalloc: this device's address of the static scratch array, and host storage for its phase list
    // (reserved at create, so the call itself allocates nothing on the host either)
    void* scratch_dev = nullptr;
    std::vector<hivis::Phase> na_phases;
};

namespace {

int fail(hivis_ctx* c, int code, const char* fmt, ...) {
    char buf[512];
    va_list ap; va_start(ap, fmt); vsnprintf(buf, sizeof buf, fmt, ap); va_end(ap);
    if (c) c->err = buf;
    return code;
}

#define HIP_TRY(c, expr)                                                                              \
    do {                                                                                              \
        hipError_t e_ = (expr);                                                                       \
        if (e_ != hipSuccess) return fail((c), HIVIS_EHIP, "%s failed: %s", #expr, hipGetErrorString(e_)); \
    } while (0)

// Device address of the static scratch array on device `dev` (which must be the current device): looked up once per
// device, then kept for the life of the process.
constexpr int MAX_DEVICES = 64;
void* g_scratch_ptr[MAX_DEVICES] = {};
std::mutex g_scratch_mu;
int scratch_for_device(hivis_ctx* c, int dev) {
    if (dev < 0 || dev >= MAX_DEVICES) return fail(c, HIVIS_EINVAL, "device index %d outside [0,%d)", dev, MAX_DEVICES);
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* ptr = nullptr;
        HIP_TRY(c, hipGetSymbolAddress((void**)&ptr, HIP_SYMBOL(scratch)));
        if (!ptr) return fail(c, HIVIS_EHIP, "hipGetSymbolAddress(scratch) returned a null address");
        g_scratch_ptr[dev] = ptr;
    }
    c->scratch_dev = g_scratch_ptr[dev];
    return HIVIS_OK;
}

template <typename T> int dev_alloc(hivis_ctx* c, T** p, size_t count) {
    void* q = nullptr;
    HIP_TRY(c, hipMalloc(&q, std::max<size_t>(count, 1) * sizeof(T)));
    c->allocs.push_back(q);
    *p = (T*)q;
    return HIVIS_OK;
}

// ---- weight upload + re-layout -------------------------------------------------------------
template <typename WT>
int pack_matrix(hivis_ctx* c, const void* const* srcs, const int* ncols, int nsrc, int K, int transposed, void* staging,
                uint4** out, int mode = PACK_PLAIN) {
    int N = 0;
    PackSrc ps{};
    char* st = (char*)staging;
    for (int i = 0; i < 3; ++i) { ps.p[i] = nullptr; ps.n[i] = 0; }
    for (int i = 0; i < nsrc; ++i) {
        const size_t bytes = (size_t)K * ncols[i] * sizeof(WT);
        HIP_TRY(c, hipMemcpy(st, srcs[i], bytes, hipMemcpyHostToDevice));
        ps.p[i] = st; ps.n[i] = ncols[i];
        st += (bytes + 255) & ~(size_t)255;
        N += ncols[i];
    }
    ps.transposed = transposed; ps.mode = mode; ps.hd = c->cfg.head_dim;
    const size_t n16 = (size_t)K * N * sizeof(WT) / 16;
    if (int rc = dev_alloc(c, out, n16)) return rc;
    const int blocks = (int)std::min<size_t>((n16 + 255) / 256, 65535);
    hipLaunchKernelGGL(pack_weights_kernel<WT>, dim3(blocks), dim3(256), 0, c->stream, ps, K, N, *out);
    HIP_TRY(c, hipGetLastError());
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    return HIVIS_OK;
}

template <typename WT>
int upload_vec(hivis_ctx* c, const void* src, size_t count, void** out) {
    WT* p = nullptr;
    if (int rc = dev_alloc(c, &p, count)) return rc;
    HIP_TRY(c, hipMemcpy(p, src, count * sizeof(WT), hipMemcpyHostToDevice));
    *out = p;
    return HIVIS_OK;
}

template <typename WT>
int upload_layer(hivis_ctx* c, const hivis_layer_weights& w, void* staging, LayerDev& L) {
    const hivis_config& g = c->cfg;
    const int qd = g.n_q_heads * g.head_dim, kd = g.n_kv_heads * g.head_dim;
    if (!w.norm1 || !w.wq || !w.wk || !w.wv || !w.wo || !w.norm2 || !w.wg || !w.wu || !w.wd)
        return fail(c, HIVIS_EINVAL, "null layer weight pointer");
    if (int rc = upload_vec<WT>(c, w.norm1, g.d, &L.norm1)) return rc;
    if (int rc = upload_vec<WT>(c, w.norm2, g.d, &L.norm2)) return rc;
    { const void* s[3] = {w.wq, w.wk, w.wv}; int n[3] = {qd, kd, kd};
      if (int rc = pack_matrix<WT>(c, s, n, 3, g.d, 0, staging, &L.wqkv, PACK_QKV)) return rc; }
    { const void* s[1] = {w.wo}; int n[1] = {g.d};
      if (int rc = pack_matrix<WT>(c, s, n, 1, qd, 0, staging, &L.wo)) return rc; }
    { const void* s[2] = {w.wg, w.wu}; int n[2] = {g.ffn, g.ffn};
      if (int rc = pack_matrix<WT>(c, s, n, 2, g.d, 0, staging, &L.wgu, PACK_GATEUP)) return rc; }
    { const void* s[1] = {w.wd}; int n[1] = {g.d};
      if (int rc = pack_matrix<WT>(c, s, n, 1, g.ffn, 0, staging, &L.wd)) return rc; }
    if (w.bq || w.bk || w.bv) {
        if (!w.bq || !w.bk || !w.bv) return fail(c, HIVIS_EINVAL, "q/k/v biases: give all three or none");
        // the fused qkv columns: [q heads | k heads | v heads], inside every q and k head the rotary pair (i, i + hd/2)
        // in adjacent columns (2i, 2i+1): the biases follow their columns
        const int hd = g.head_dim, half = hd / 2;
        std::vector<float> b((size_t)qd + 2 * kd);
        auto val = [](const void* p, size_t i) -> float {
            if (sizeof(WT) == 2) { const uint32_t u = (uint32_t)((const uint16_t*)p)[i] << 16; float f; memcpy(&f, &u, 4); return f; }
            return ((const float*)p)[i];
        };
        for (int part = 0; part < 2; ++part) {
            const void* src = part == 0 ? w.bq : w.bk;
            const int n = part == 0 ? qd : kd, off = part == 0 ? 0 : qd;
            for (int col = 0; col < n; ++col) {
                const int h = col / hd, pc = col % hd;
                b[(size_t)off + col] = val(src, (size_t)h * hd + ((pc & 1) ? pc / 2 + half : pc / 2));
            }
        }
        for (int col = 0; col < kd; ++col) b[(size_t)qd + kd + col] = val(w.bv, col);
        if (int rc = dev_alloc(c, &L.bqkv, b.size())) return rc;
        HIP_TRY(c, hipMemcpy(L.bqkv, b.data(), b.size() * sizeof(float), hipMemcpyHostToDevice));
    }
    return HIVIS_OK;
}

// column chunks per row for the row-wise kernels: few rows -> split every row over several workgroups
static inline int row_chunks(int rows) { return rows >= 256 ? 1 : std::max(1, std::min(8, 256 / std::max(rows, 1))); }

int launch_pack(hivis_ctx* c, const float* A, int lda, int M, int K, uint4** out);
int wide_gemm(hivis_ctx* c, const uint4* frag, int M, int K, const uint4* Wp, int N, float* Y, int ldy, hivis::Parts* defer = nullptr);
template <typename WT>
int layer_forward_wide(hivis_ctx* c, const LayerDev& L, const KVDev& kv, float* h, hivis::Parts pending, const int* base,
                       int offset, int seq0, int nseq, int m, TreeRows tr, hivis::Parts* out_pending);

// ---- launches --------------------------------------------------------------------------------
// greedy token of each of `rows` rows of logits: row r's to out[(r / m) * sseq + r % m]
void launch_argmax(hivis_ctx* c, const float* logits, int rows, int32_t* out, int m, int sseq) {
    const int V = c->cfg.vocab, nseg = (V + ARGMAX_SEG - 1) / ARGMAX_SEG;
    hipLaunchKernelGGL(argmax_part_kernel, dim3(rows, nseg), dim3(256), 0, c->stream, logits, V, c->am_v, c->am_i);
    hipLaunchKernelGGL(argmax_final_kernel, dim3(rows), dim3(64), 0, c->stream, (const float*)c->am_v, (const int*)c->am_i, nseg, V, out, m, sseq, c->bad);
}

template <typename WT>
int gemm(hivis_ctx* c, const float* A, int lda, int M, int K, const uint4* Wp, int N, float* Y, int ldy, int epi) {
    if (M < 1 || M > MAX_ROWS) return fail(c, HIVIS_EINVAL, "gemm rows %d out of range", M);
    if (sizeof(WT) == 2 && M >= c->wide_min && c->pf_frag && c->pf_rows >= MAX_ROWS && ldy == N && epi == EPI_STORE && !c->no_wide_gemm) {
        uint4* frag = nullptr;
        if (int rc = launch_pack(c, A, lda, M, K, &frag)) return rc;
        return wide_gemm(c, frag, M, K, Wp, N, Y, ldy);
    }
    if (M > CHAIN_MAX_ROWS) {            // wider passes (tree verify)
        // fp32 models, and bf16 ones with HIVIS_WIDE_GEMM=0 or less than 64 rows of room: one launch per 32 rows
        for (int r0 = 0; r0 < M; r0 += CHAIN_MAX_ROWS)
            if (int rc = gemm<WT>(c, A + (size_t)r0 * lda, lda, std::min(CHAIN_MAX_ROWS, M - r0), K, Wp, N, Y + (size_t)r0 * ldy, ldy, epi)) return rc;
        return HIVIS_OK;
    }
    const int ntiles = N / 16;
    const int grid = std::min(ntiles, c->num_cu);
    constexpr int ROWS = WTraits<WT>::ROWS;
    const int T = (M + ROWS - 1) / ROWS;
    // dynamic LDS = cross-wavefront reduction buffer [NW][G][T][64][RPL] floats
#define HIVIS_SKINNY(T_, KBW_, G_, NW_) HIVIS_SKINNY_(T_, KBW_, G_, NW_, false)
#define HIVIS_SKINNY_(T_, KBW_, G_, NW_, UP_)                                                                      \
    do {                                                                                                           \
        constexpr size_t lds_ = (size_t)NW_ * G_ * T_ * 64 * WTraits<WT>::RPL * sizeof(float);                     \
        static bool attr_done_ = false;                                                                            \
        if (!attr_done_ && lds_ > 64 * 1024) {                                                                     \
            HIP_TRY(c, hipFuncSetAttribute((const void*)gemm_skinny_kernel<WT, T_, KBW_, G_, NW_, UP_>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_)); \
            attr_done_ = true;                                                                                     \
        }                                                                                                          \
        hipLaunchKernelGGL((gemm_skinny_kernel<WT, T_, KBW_, G_, NW_, UP_>), dim3(grid), dim3(NW_ * 64), lds_, c->stream, A, lda, M, K, Wp, N, Y, ldy, epi); \
    } while (0)
    if constexpr (sizeof(WT) == 2) {
        if (T == 1) HIVIS_SKINNY(1, 4, 8, 16);
        // 8 wavefronts for the wider row counts: every wavefront may use 256 registers (raw rows + fragments + accumulators
        // spill at 128)
        else if (T == 2) HIVIS_SKINNY(2, 4, 4, 8);
        else HIVIS_SKINNY_(4, 2, 4, 8, true);     // all 4 tiles' weights of a pass in flight together
    } else {
        if (T == 1) HIVIS_SKINNY(1, 4, 4, 16);
        else HIVIS_SKINNY(2, 4, 2, 16);
    }
#undef HIVIS_SKINNY
#undef HIVIS_SKINNY_
    HIP_TRY(c, hipGetLastError());
    return HIVIS_OK;
}

template <typename WT>
int attention(hivis_ctx* c, const float* q, int ldq, const KVDev& kv, const int* base, int offset, int seq0, int nseq,
              int m, int max_keys, float* out, int ldo, const unsigned long long* tmask = nullptr, int qrows = 0) {
    typedef typename KVType<WT>::type KT;
    const hivis_config& g = c->cfg;
    AttnShape sh{};
    sh.Hq = g.n_q_heads; sh.Hkv = g.n_kv_heads; sh.m = m;
    const int group = g.n_q_heads / g.n_kv_heads;
    if (m >= ATT_RMAX) { sh.mi = ATT_RMAX; sh.gh = 1; }
    else { sh.mi = m; sh.gh = std::max(1, std::min(group, ATT_RMAX / m)); }
    sh.seq0 = seq0; sh.offset = offset; sh.maxL = kv.maxL; sh.ldq = ldq; sh.qrows = qrows; sh.nwaves = 4; sh.tmask = tmask;
    // enough workgroups to occupy the chip, at most one 64-key tile per wavefront slot; and half as many (head,row) pairs per item, again and again,
    // as long as that leaves one workgroup to a CU at most: an item's rows go one after the other (32 rows x 4 heads of 64 over 100 keys, us: 8 items of 16 rows
    // 24.8 and 5.7 to merge, 128 items of one row 6.1 and under 4).  What an item reads of the cache comes from L2; beyond a workgroup per CU nothing is idle.
    const int tiles = (max_keys + 63) / 64;
    int items = 0, nsplit = 0;
    for (;; sh.gh > 1 ? sh.gh = (sh.gh + 1) / 2 : sh.mi = (sh.mi + 1) / 2) {
        sh.n_hblk = (group + sh.gh - 1) / sh.gh; sh.n_rblk = (m + sh.mi - 1) / sh.mi;
        items = nseq * g.n_kv_heads * sh.n_hblk * sh.n_rblk;
        nsplit = std::max(1, std::min({(2 * c->num_cu + items - 1) / items, (tiles + 3) / 4, 16}));
        if (sh.mi * sh.gh == 1 || 2 * items * nsplit > c->num_cu) break;
    }
    sh.nsplit = nsplit;
    const size_t need = (size_t)items * nsplit * 4 * ATT_RMAX * (g.head_dim + 2);
    if (need > c->attn_ws_floats) return fail(c, HIVIS_EINVAL, "attention workspace too small (%zu > %zu)", need, c->attn_ws_floats);
    const int rows = sh.mi * sh.gh;              // an item's (head,row) pairs at most
#define HIVIS_ATTN_PARTIAL(HD_, RC_) hipLaunchKernelGGL((attn_partial_kernel<KT, HD_, RC_>), dim3(items, nsplit), dim3(256), 0, c->stream, q, (const KT*)kv.k, (const KT*)kv.v, base, sh, c->attn_ws)
#define HIVIS_ATTN_STANDALONE(HD_)                                                                                                       \
    do {                                                                                                                                 \
        if (rows <= 1) HIVIS_ATTN_PARTIAL(HD_, 1);                                                                                       \
        else if (rows <= 2) HIVIS_ATTN_PARTIAL(HD_, 2);                                                                                  \
        else if (rows <= 4) HIVIS_ATTN_PARTIAL(HD_, 4);                                                                                  \
        else if (rows <= 8) HIVIS_ATTN_PARTIAL(HD_, 8);                                                                                  \
        else HIVIS_ATTN_PARTIAL(HD_, ATT_RMAX);                                                                                          \
        hipLaunchKernelGGL((attn_merge_kernel<HD_>), dim3(items), dim3(256), 0, c->stream, c->attn_ws, base, sh, out, ldo);              \
    } while (0)
    if (g.head_dim == 128) HIVIS_ATTN_STANDALONE(128); else HIVIS_ATTN_STANDALONE(64);
#undef HIVIS_ATTN_STANDALONE
#undef HIVIS_ATTN_PARTIAL
    HIP_TRY(c, hipGetLastError());
    return HIVIS_OK;
}

AttnShape fused_attn_shape(hivis_ctx* c, int nseq, int m, int offset, int maxL, int ldq, bool alone, int* items_out);

int key_splits(const hivis_ctx* c, int keys, int most, bool half) { return half && !c->keys_forced ? attn_block_splits(keys, most) : attn_splits(keys, most, c->keys_per_split); }

// One launch of attention over half-precision caches, in blocks of keys (attn_split_kernel) or in tiles (attn_tiles_kernel) as attn_walks has it.  rm: (head,row) pairs an item
// may hold, 8 or 16 (the partials' and the kernel's); keys: cached rows of the longest sequence, with those of the pass; once: cached rows with the non-temporal hint.
int launch_attn_half(hivis_ctx* c, const AttnShape& sh, int items, int rm, int keys, const float* q, const void* kc, const void* vc, const int* base, const AttnOut& out,
                     uint4* frag_out, float* ws, int* cnt, bool once, unsigned long long* prof2 = nullptr, unsigned long long* prof3 = nullptr, hipEvent_t ev0 = nullptr, hipEvent_t ev1 = nullptr) {
    const int hd = c->cfg.head_dim, heads = items / sh.n_rblk;
    const dim3 grid = (sh.flags & 2) ? dim3(8, sh.nsplit, (heads + 7) / 8 * sh.n_rblk) : dim3(sh.nsplit, items);
    const FastDiv by_rblk = FastDiv::by(sh.n_rblk), by_hblk = FastDiv::by(sh.n_hblk), by_hkv = FastDiv::by(sh.Hkv);
#define HIVIS_ATTN_FORMS(LAUNCH_)                                                                                                             \
    if (rm > FUSED_RMAX) { if (hd == 128) LAUNCH_(128, ATTN_ROWS_RM, false); else LAUNCH_(64, ATTN_ROWS_RM, false); }                         \
    else if (hd == 128) { if (once) LAUNCH_(128, FUSED_RMAX, true); else LAUNCH_(128, FUSED_RMAX, false); }                                   \
    else { if (once) LAUNCH_(64, FUSED_RMAX, true); else LAUNCH_(64, FUSED_RMAX, false); }
    if (attn_walks(c->num_cu, hd, items, rm, attn_blocks(keys, sh.nsplit))) {
        AttnTilesArgs a{};
        a.q = q; a.kc = (const f16_t*)kc; a.vc = (const f16_t*)vc; a.base = base; a.ws = ws; a.cnt = cnt; a.out = out; a.out.afrag = frag_out; a.items = items;
        a.by_rblk = by_rblk; a.by_hblk = by_hblk; a.by_hkv = by_hkv; a.sh = sh; a.prof2 = prof2; a.prof3 = prof3;
#define HIVIS_TILES(HD_, RM_, ONCE_)                                                                                                          \
        do { constexpr int lds_ = (int)(fused_attn_mfma_lds_floats(HD_, FUSED_NW, RM_) * sizeof(float));                                      \
             hipExtLaunchKernelGGL((attn_tiles_kernel<HD_, RM_, ONCE_>), grid, dim3(FUSED_NT), lds_, c->stream, ev0, ev1, 0, a); } while (0)
        HIVIS_ATTN_FORMS(HIVIS_TILES)
#undef HIVIS_TILES
    } else {
        AttnArgs a{};
        a.q = q; a.kc = (const f16_t*)kc; a.vc = (const f16_t*)vc; a.base = base; a.tmask = sh.tmask; a.ws = ws; a.cnt = cnt;
        a.y = out.y; a.ldo = out.ldo; a.rows_out = out.frag; a.rows = out.rows; a.frag_out = frag_out;
        a.ldq = sh.ldq; a.maxL = sh.maxL; a.offset = sh.offset; a.seq0 = sh.seq0; a.m = sh.m; a.qrows = sh.qrows; a.mi = sh.mi; a.gh = sh.gh; a.Hkv = sh.Hkv;
        a.group = sh.Hq / sh.Hkv; a.n_rblk = sh.n_rblk; a.n_hblk = sh.n_hblk; a.items = items; a.nsplit = sh.nsplit; a.flags = sh.flags; a.nbase = sh.nbase;
        a.by_rblk = by_rblk; a.by_hblk = by_hblk; a.by_hkv = by_hkv; a.by_split = FastDiv::by(sh.nsplit); a.by_mi = FastDiv::by(sh.mi);
        for (int b = 0; b < sh.nbase; ++b) a.base_val[b] = sh.base_val[b];
        a.prof2 = prof2; a.prof3 = prof3;
#define HIVIS_SPLIT(HD_, RM_, ONCE_)                                                                                                          \
        do { constexpr int lds_ = AttnSplitCfg<HD_, RM_>::LDS;                                                                                \
             hipExtLaunchKernelGGL((attn_split_kernel<HD_, RM_, ONCE_>), grid, dim3(FUSED_NT), lds_, c->stream, ev0, ev1, 0, a); } while (0)
        HIVIS_ATTN_FORMS(HIVIS_SPLIT)
#undef HIVIS_SPLIT
    }
#undef HIVIS_ATTN_FORMS
    HIP_TRY(c, hipGetLastError());
    return HIVIS_OK;
}

// Attention of nseq x m rows on the matrix cores, outside a phase program (prefill; passes with more rows than one MFMA
// tile): long causal row ranges through the shared-tile kernel, others through the verify pass's kernel in one launch over all items.  Rows of sequence seq0 + s sit at positions base[seq0 + s] + offset + i.
template <typename WT>
int attention_rows_mfma(hivis_ctx* c, const float* q, int ldq, const KVDev& kv, const int* base, int offset, int seq0, int nseq, int m,
                        float* out, int ldo, const unsigned long long* tmask = nullptr, uint4* frag_out = nullptr, bool* wrote_frag = nullptr, int qrows = 0, uint4* row_frag = nullptr) {
    // row_frag (optional, up to 16 rows): the rows go there as row fragments.
    // frag_out / wrote_frag (optional): where the kernel chosen can, the rows go out as A fragments of the next GEMM
    // (K = ldo) instead of fp32 rows, and *wrote_frag says so
    if (wrote_frag) *wrote_frag = false;
    const hivis_config& g = c->cfg;
    typedef typename KVType<WT>::type KT;
    if constexpr (std::is_same<KT, f16_t>::value) {
        // long causal row ranges (prefill): key tiles shared by a workgroup through LDS.  Too few such workgroups leave CUs idle
        // (the last 128 of 3008 rows, 32 heads: 240 us): 16 rows per workgroup then.
        const long items2 = (long)nseq * g.n_q_heads * ((m + 127) / 128);
        if (m >= c->attn_shared_min && 2 * items2 >= c->num_cu && tmask == nullptr && frag_out && wrote_frag) {
            // two workgroups of 128 rows fit a CU; where there are fewer of them, 64 rows each (640 rows x 32 heads: 35 us, 46 with 128)
            const bool large = items2 >= 2 * c->num_cu;
            const int rows = large ? 128 : 64, nw = rows / 16;
            AttnShape sh{};
            sh.Hq = g.n_q_heads; sh.Hkv = g.n_kv_heads; sh.m = m; sh.mi = rows; sh.gh = 1;
            sh.n_hblk = g.n_q_heads / g.n_kv_heads; sh.n_rblk = (m + rows - 1) / rows;
            sh.seq0 = seq0; sh.offset = offset; sh.maxL = kv.maxL; sh.ldq = ldq; sh.qrows = qrows; sh.nwaves = nw; sh.nsplit = 1; sh.tmask = nullptr;
            const int items = nseq * g.n_q_heads * sh.n_rblk;
            const size_t lds = attn_shared_lds_bytes(g.head_dim);
#define HIVIS_SHARED(HD_, NW_)                                                                                                             \
    hipLaunchKernelGGL((attn_rows_shared_kernel<HD_, NW_>), dim3(items), dim3(64 * NW_), lds, c->stream, q, (const f16_t*)kv.k,            \
                       (const f16_t*)kv.v, base, sh, ldo, frag_out)
            if (g.head_dim == 128) { if (large) HIVIS_SHARED(128, 8); else HIVIS_SHARED(128, 4); }
            else { if (large) HIVIS_SHARED(64, 8); else HIVIS_SHARED(64, 4); }
#undef HIVIS_SHARED
            *wrote_frag = true;
            HIP_TRY(c, hipGetLastError());
            return HIVIS_OK;
        }
        AttnShape sh{};
        int items = 0, rm = FUSED_RMAX;
        if (m > FUSED_RMAX) {
            // many rows per sequence: 16 (head,row) pairs per work item, which reads every cached key half as often
            rm = ATTN_ROWS_RM;
            sh.Hq = g.n_q_heads; sh.Hkv = g.n_kv_heads; sh.m = m;
            const int group = g.n_q_heads / g.n_kv_heads;
            if (m >= rm) { sh.mi = rm; sh.gh = 1; }
            else { sh.mi = m; sh.gh = std::max(1, std::min(group, rm / m)); }
            sh.n_hblk = (group + sh.gh - 1) / sh.gh; sh.n_rblk = (m + sh.mi - 1) / sh.mi;
            sh.offset = offset; sh.maxL = kv.maxL; sh.ldq = ldq;
            items = nseq * g.n_kv_heads * sh.n_hblk * sh.n_rblk;
        } else sh = fused_attn_shape(c, nseq, m, offset, kv.maxL, ldq, false, &items);
        sh.seq0 = seq0; sh.tmask = tmask; sh.flags = c->attn_flags; sh.qrows = qrows; sh.nsplit = 1;
        if (base == c->zeros && nseq <= 8) sh.nbase = nseq;             // (base_val: zeros)
        float* ws = nullptr; int* cnt = nullptr;
        // (the host mirrors the cache lengths that `base` holds)
        const std::vector<int>* hl = base == c->tlen ? &c->h_tlen : base == c->dlen ? &c->h_dlen : nullptr;
        int max_keys = 0;
        for (int s = 0; s < nseq; ++s) max_keys = std::max(max_keys, (hl ? (*hl)[seq0 + s] : 0) + offset + m);
        if (c->attn_elect && items <= c->rows_cnt_n) {
            // the key range of an item is split over workgroups and the last one to arrive merges (as in the phase programs).  No more workgroups than CUs: with
            // more, 160 items of 32 rows got slower (8.8 -> 9.6 ms per verify).
            const int wgs = (sh.flags & 2) ? (items / sh.n_rblk + 7) / 8 * 8 * sh.n_rblk : items;
            int nsplit = key_splits(c, max_keys, std::min(ATTN_MAX_SPLITS, std::max(1, c->fused_grid / wgs)), true);
            while (nsplit > 1 && (size_t)items * nsplit * rm * (g.head_dim + 2) > c->attn_ws_floats) --nsplit;
            if (nsplit > 1) { sh.nsplit = nsplit; ws = c->attn_ws; cnt = c->rows_cnt; }
        }
        uint4* frag = (frag_out && wrote_frag && ldo % 32 == 0) ? frag_out : nullptr;
        if (frag) *wrote_frag = true;
        return launch_attn_half(c, sh, items, rm, max_keys, q, kv.k, kv.v, base, AttnOut{out, ldo, row_frag, nseq * m}, frag, ws, cnt, false);
    }
    return fail(c, HIVIS_EINVAL, "attention on the matrix cores needs half-precision caches");
}

void launch_attn_f32(hivis_ctx* c, const Phase& ph, int rows, unsigned long long* prof2, unsigned long long* prof3, hipEvent_t ev0, hipEvent_t ev1) {
    AttnF32Args a{};
    a.q = ph.A; a.kc = (const float*)ph.kc; a.vc = (const float*)ph.vc; a.base = ph.base; a.ws = ph.ws; a.cnt = ph.cnt; a.y = ph.Y; a.rows_out = ph.F;
    a.ldo = ph.ldy; a.rows = rows; a.items = ph.att_items; a.sh = ph.att; a.prof2 = prof2; a.prof3 = prof3;
    a.by_rblk = FastDiv::by(a.sh.n_rblk); a.by_hblk = FastDiv::by(a.sh.n_hblk); a.by_hkv = FastDiv::by(a.sh.Hkv);
    const dim3 grid = (a.sh.flags & 2) ? dim3(8, a.sh.nsplit, (a.items + 7) / 8) : dim3(a.items, a.sh.nsplit);
    const bool one = a.sh.gh * a.sh.mi == 1;         // (head,row) pairs an item holds at most: one for a draft step of one query head per key head, else up to 8
#define HIVIS_ATTN_F32(HD_, RC_) hipExtLaunchKernelGGL((attn_f32_kernel<HD_, RC_>), grid, dim3(FUSED_NT), 0, c->stream, ev0, ev1, 0, a)
    if (c->cfg.head_dim == 128) { if (one) HIVIS_ATTN_F32(128, 1); else HIVIS_ATTN_F32(128, FUSED_RMAX); }
    else if (one) HIVIS_ATTN_F32(64, 1);
    else HIVIS_ATTN_F32(64, FUSED_RMAX);
#undef HIVIS_ATTN_F32
}

// One decoder layer on M = nseq*m rows.  h: residual stream [M][d] (in place).  `pending` (may be null) is a delta
// from the previous layer that has not been added to h yet; on return *pending_out is this layer's MLP output, still
// to be added by the caller (the next layer's first norm, or a final norm/add, fuses that addition).
template <typename WT>
int layer_forward(hivis_ctx* c, const LayerDev& L, const KVDev& kv, float* h, const float* pending, const int* base,
                  int offset, int seq0, int nseq, int m, int max_keys, TreeRows tr = TreeRows()) {
    typedef typename KVType<WT>::type KT;
    const hivis_config& g = c->cfg;
    const int M = nseq * m, d = g.d, qd = g.n_q_heads * g.head_dim, kd = g.n_kv_heads * g.head_dim, F = g.ffn;
    const int nqkv = qd + 2 * kd;
    hipLaunchKernelGGL((add_rmsnorm_kernel<WT>), dim3(M), dim3(256), 0, c->stream, h, d, pending, d, (const WT*)L.norm1, c->a, d, d, g.rms_eps);
    if (int rc = gemm<WT>(c, c->a, d, M, d, L.wqkv, nqkv, c->qkv, nqkv, EPI_STORE)) return rc;
    hipLaunchKernelGGL((rope_append_kernel<KT>), dim3(M, row_chunks(M)), dim3(256), 0, c->stream, c->qkv, g.n_q_heads, g.n_kv_heads, g.head_dim, base, offset, seq0, m, (KT*)kv.k, (KT*)kv.v, kv.maxL, g.rope_theta, tr.pos_delta, (const float*)L.bqkv, (const float*)c->rope_tab, g.max_vis + g.max_text);
    if (c->fused && std::is_same<KT, f16_t>::value) { if (int rc = attention_rows_mfma<WT>(c, c->qkv, nqkv, kv, base, offset, seq0, nseq, m, c->att, qd, tr.mask)) return rc; }
    else if (int rc = attention<WT>(c, c->qkv, nqkv, kv, base, offset, seq0, nseq, m, max_keys, c->att, qd, tr.mask)) return rc;
    if (int rc = gemm<WT>(c, c->att, qd, M, qd, L.wo, d, c->proj, d, EPI_STORE)) return rc;
    hipLaunchKernelGGL((add_rmsnorm_kernel<WT>), dim3(M), dim3(256), 0, c->stream, h, d, (const float*)c->proj, d, (const WT*)L.norm2, c->a, d, d, g.rms_eps);
    if (int rc = gemm<WT>(c, c->a, d, M, d, L.wgu, 2 * F, c->gu, 2 * F, EPI_STORE)) return rc;
    hipLaunchKernelGGL(silu_mul_kernel, dim3(M, row_chunks(M)), dim3(256), 0, c->stream, (const float*)c->gu, c->act, F);
    if (int rc = gemm<WT>(c, c->act, F, M, F, L.wd, d, c->proj, d, EPI_STORE)) return rc;
    HIP_TRY(c, hipGetLastError());
    return HIVIS_OK;   // c->proj holds the MLP delta, not yet added to h
}

// Target pass over M = nseq*m rows already in c->x; leaves post-final-norm features in out (row stride ldo)
// for rows >= first_out_row (pointer arithmetic done by the caller through first_out_row).
template <typename WT>
int target_forward(hivis_ctx* c, int seq0, int nseq, int m, const int* base, int offset, int max_keys, float* out, int ldo,
                   int first_out_row, TreeRows tr = TreeRows()) {
    const hivis_config& g = c->cfg;
    const int M = nseq * m;
    const float* pending = nullptr;
    if constexpr (sizeof(WT) == 2) {
        if (M >= c->wide_min && M <= MAX_ROWS && c->fused && c->pf_frag && c->pf_rows >= MAX_ROWS && g.d <= 8192 && !c->no_wide_gemm) {
            Parts pend{nullptr, 0, 0};
            for (int l = 0; l < g.n_layers; ++l)
                if (int rc = layer_forward_wide<WT>(c, c->layers[l], c->tkv[l], c->x, pend, base, offset, seq0, nseq, m, tr, &pend)) return rc;
            if (pend.n > 1) hipLaunchKernelGGL(splitk_reduce_kernel, dim3(M, row_chunks(M)), dim3(256), 0, c->stream, pend, g.d, g.d, c->proj, g.d);
            const int nout_w = M - first_out_row;
            if (nout_w > 0)
                hipLaunchKernelGGL((add_rmsnorm_kernel<WT>), dim3(nout_w), dim3(256), 0, c->stream, c->x + (size_t)first_out_row * g.d, g.d,
                                   (const float*)c->proj + (size_t)first_out_row * g.d, g.d, (const WT*)c->final_norm, out, ldo, g.d, g.rms_eps);
            HIP_TRY(c, hipGetLastError());
            return HIVIS_OK;
        }
    }
    for (int l = 0; l < g.n_layers; ++l) {
        // KV of layer l for all sequences
        if (int rc = layer_forward<WT>(c, c->layers[l], c->tkv[l], c->x, pending, base, offset, seq0, nseq, m, max_keys, tr)) return rc;
        pending = c->proj;
    }
    const int nout = M - first_out_row;
    if (nout > 0)
        hipLaunchKernelGGL((add_rmsnorm_kernel<WT>), dim3(nout), dim3(256), 0, c->stream, c->x + (size_t)first_out_row * g.d, g.d,
                           pending + (size_t)first_out_row * g.d, g.d, (const WT*)c->final_norm, out, ldo, g.d, g.rms_eps);
    HIP_TRY(c, hipGetLastError());
    return HIVIS_OK;
}

// Drafter: fusion FC on cat rows [M][2d] + rho_idx, then its single layer; output rows (h + mlp delta) to out.
template <typename WT>
int drafter_forward(hivis_ctx* c, const float* cat, int seq0, int nseq, int m, int rho_idx, int offset, int max_keys,
                    float* out, int ldo, TreeRows tr = TreeRows()) {
    const hivis_config& g = c->cfg;
    const int M = nseq * m, d = g.d;
    if (int rc = gemm<WT>(c, cat, 2 * d, M, 2 * d, c->fuse_w, d, c->u, d, EPI_STORE)) return rc;
    hipLaunchKernelGGL((add_rho_kernel<WT>), dim3(M), dim3(256), 0, c->stream, c->u, d, (const WT*)c->rho, rho_idx, d);
    bool wide = false;
    if constexpr (sizeof(WT) == 2) wide = M >= c->wide_min && M <= MAX_ROWS && c->fused && c->pf_frag && c->pf_rows >= MAX_ROWS && d <= 8192 && !c->no_wide_gemm;
    if (wide) {
        if constexpr (sizeof(WT) == 2) {
            Parts pend{nullptr, 0, 0};
            if (int rc = layer_forward_wide<WT>(c, c->draft, c->dkv, c->u, pend, c->dlen, offset, seq0, nseq, m, tr, &pend)) return rc;
            if (pend.n > 1) hipLaunchKernelGGL(splitk_reduce_kernel, dim3(M, row_chunks(M)), dim3(256), 0, c->stream, pend, d, d, c->proj, d);
        }
    } else if (int rc = layer_forward<WT>(c, c->draft, c->dkv, c->u, nullptr, c->dlen, offset, seq0, nseq, m, max_keys, tr)) return rc;
    hipLaunchKernelGGL(add_rows_kernel, dim3(M), dim3(256), 0, c->stream, (const float*)c->u, d, (const float*)c->proj, d, out, ldo, d);
    HIP_TRY(c, hipGetLastError());
    return HIVIS_OK;
}


// ---- persistent-kernel path --------------------------------------------------------------------
enum { PROG_VERIFY = 0, PROG_DRAFT = 1, PROG_ROLL = 2, PROG_DRAFT_SAMPLE = 3 };

// Rows a phase program takes: one MFMA tile; bf16 models, one launch per phase: up to 16, through the bf16w kernels.  Measured with
// two target layers against the stand-alone kernels (9 and 10 rows) and K slices (from 11 on), us per call, before -> now:
//                                    verify 9 rows   12 rows      16 rows      re-feed 9 rows  16 rows      draft round, 9 sequences, K = 2
//   d 4096, ffn 11008, vocab  32000  397 -> 314      397 -> 330   419 -> 347   214 -> 156      221 -> 176   325 -> 273
//   d 5120, ffn 13824, vocab  32000  492 -> 405      484 -> 415   499 -> 426   278 -> 206      278 -> 214   407 -> 337
//   d 3584, ffn 18944, vocab 152064  760 -> 497      730 -> 520   795 -> 547   227 -> 178      231 -> 202   757 -> 577
//   d 2048, ffn  5632, vocab  32000  224 -> 173      249 -> 184   266 -> 191   121 ->  98      152 -> 105   168 -> 152
template <typename WT>
bool fused_rows_ok(const hivis_ctx* c, int M) { return M <= (sizeof(WT) == 2 && !c->persistent ? WTraits<bf16w_t>::ROWS : WTraits<WT>::ROWS); }

// alone (fp32 caches only; the rule: attn_alone): each head and row an item of its own, if there are CUs for them.  (The matrix cores of the
// bf16 models take all rows of an item at once.)
AttnShape fused_attn_shape(hivis_ctx* c, int nseq, int m, int offset, int maxL, int ldq, bool alone, int* items_out) {
    const hivis_config& g = c->cfg;
    AttnShape sh{};
    sh.Hq = g.n_q_heads; sh.Hkv = g.n_kv_heads; sh.m = m;
    const AttnCut cut = attn_cut(nseq, m, g.n_q_heads, g.n_kv_heads, alone && nseq * g.n_q_heads * m <= c->fused_grid);
    sh.mi = cut.mi; sh.gh = cut.gh; sh.n_hblk = cut.n_hblk; sh.n_rblk = cut.n_rblk;
    sh.seq0 = 0; sh.offset = offset; sh.maxL = maxL; sh.ldq = ldq; sh.nwaves = FUSED_NW;
    const int items = cut.items;
    // (with the splits of an item on one XCD the grid holds whole rounds of eight items: more workgroups than CUs would take two turns,
    // 14.4 -> 23.5 us for 28 items in nine splits)
    sh.nsplit = std::min(ATTN_MAX_SPLITS, std::max(1, c->fused_grid / ((c->attn_flags & 2) ? (items + 7) / 8 * 8 : items)));
    *items_out = items;
    return sh;
}

// Bump allocator for the per-phase output buffers of one program (first pass counts, second pass hands out).
struct Pool {
    float* base = nullptr; size_t used = 0;
    float* take(size_t floats) {
        floats = (floats + 63) & ~(size_t)63;            // 256-byte granules: buffers never share a cache line
        float* p = base ? base + used : nullptr;
        used += floats;
        return p;
    }
};

// phases of one decoder layer on rows h [M][d]; returns the buffer holding h + attention + MLP.  Every phase
// writes into a buffer of its own (see the memory discipline in hivis_fused.h).  dst: optional fixed destination
// of the layer output (row stride ldd).
template <typename WT>
float* layer_phases(hivis_ctx* c, std::vector<Phase>& P, Pool& pool, const LayerDev& L, const KVDev& kv, float* h, const int* base,
                    int offset, int nseq, int m, float* dst, int ldd, int* ld_out, bool persistent, bool elect, bool alone) {
    const hivis_config& g = c->cfg;
    const int M = nseq * m;
    const int d = g.d, qd = g.n_q_heads * g.head_dim, kd = g.n_kv_heads * g.head_dim, F = g.ffn, nqkv = qd + 2 * kd;
    float* qkv = pool.take((size_t)M * nqkv);
    float* att = pool.take((size_t)M * qd);
    float* h1 = pool.take((size_t)M * d);
    float* act = pool.take((size_t)M * F);
    float* h2 = dst ? dst : pool.take((size_t)M * d);
    const int ld2 = dst ? ldd : d;
    Phase q{}; q.type = PH_GEMM; q.pro = PRO_RMS; q.epi = FEPI_QKV; q.K = d; q.N = nqkv; q.W = L.wqkv; q.A = h; q.lda = d;
    q.gain = L.norm1; q.Y = qkv; q.ldy = nqkv; q.kc = kv.k; q.vc = kv.v; q.maxL = kv.maxL; q.base = base; q.offset = offset; q.rope = c->rope_tab; q.bias = L.bqkv;
    P.push_back(q);
    Phase a{}; a.type = PH_ATTN; a.A = qkv; a.lda = nqkv; a.kc = kv.k; a.vc = kv.v; a.maxL = kv.maxL; a.base = base; a.offset = offset;
    a.att = fused_attn_shape(c, nseq, m, offset, kv.maxL, nqkv, false, &a.att_items);
    int items = a.att_items;                           // (of the launch with the most, and the most partials)
    if (alone) { (void)fused_attn_shape(c, nseq, m, offset, kv.maxL, nqkv, true, &items); a.att_alone = items > a.att_items; }
    a.ws = pool.take(std::max(attn_partials(c->fused_grid, a.att_items), attn_partials(c->fused_grid, items)) * FUSED_RMAX * (g.head_dim + 2));
    if (persistent || elect) {
        a.cnt = (int*)pool.take((size_t)items);        // zero from the pool's memset; the merging workgroup re-zeroes it
        a.Y = att; a.ldy = qd;
        P.push_back(a);
    } else {
        // key splits merged by a launch of their own
        a.cnt = nullptr; a.Y = att; a.ldy = qd;
        P.push_back(a);
        Phase mg = a; mg.type = PH_ATTN_MERGE; mg.Y = att; mg.ldy = qd;
        P.push_back(mg);
    }
    Phase o{}; o.type = PH_GEMM; o.pro = PRO_PLAIN; o.epi = FEPI_ADD_TO; o.K = qd; o.N = d; o.W = L.wo; o.A = att; o.lda = qd;
    o.Y = h1; o.ldy = d; o.R = h; o.ldr = d;
    P.push_back(o);
    Phase gu{}; gu.type = PH_GEMM; gu.pro = PRO_RMS; gu.epi = FEPI_SILU; gu.K = d; gu.N = 2 * F; gu.W = L.wgu; gu.A = h1; gu.lda = d;
    gu.gain = L.norm2; gu.Y = act; gu.ldy = F;
    P.push_back(gu);
    Phase dn{}; dn.type = PH_GEMM; dn.pro = PRO_PLAIN; dn.epi = FEPI_ADD_TO; dn.K = F; dn.N = d; dn.W = L.wd; dn.A = act; dn.lda = F;
    dn.Y = h2; dn.ldy = ld2; dn.R = h1; dn.ldr = d;
    P.push_back(dn);
    *ld_out = ld2;
    return h2;
}

// Residual rows of a pass on row fragments: fp32 rows h [M][d]; F: the rows times the next norm's gain, ssq: their sums of squares in
// nssq parts per row.  (F null: the first phase adds table rows to fp32 rows itself.)
struct StreamRows { float* h; uint4* F; float* ssq; int nssq; };

// layer_phases on row fragments.  out: where the layer's rows go (h, F, ssq: null for what nobody reads); out_gain: gain for out.F.
template <typename WT>
void layer_stream(hivis_ctx* c, std::vector<Phase>& P, Pool& pool, const LayerDev& L, const KVDev& kv, StreamRows in, const int* base, int offset, int nseq, int m,
                  StreamRows out, const void* out_gain, bool elect) {
    const hivis_config& g = c->cfg;
    const int M = nseq * m;
    const int d = g.d, qd = g.n_q_heads * g.head_dim, kd = g.n_kv_heads * g.head_dim, F = g.ffn, nqkv = qd + 2 * kd;
    float* qrows = pool.take((size_t)M * qd);
    uint4* attF = (uint4*)pool.take((size_t)M * qd);
    float* h1 = pool.take((size_t)M * d);
    uint4* h1F = (uint4*)pool.take((size_t)M * d);
    float* h1s = pool.take((size_t)M * ssq_stride(d / 16));
    uint4* actF = (uint4*)pool.take((size_t)M * F);
    Phase q{}; q.type = PH_GEMM; q.pro = PRO_RMS; q.epi = FEPI_QKV; q.K = d; q.N = nqkv; q.W = L.wqkv; q.A = in.h; q.lda = d;
    q.gain = L.norm1; q.Y = qrows; q.ldy = qd; q.kc = kv.k; q.vc = kv.v; q.maxL = kv.maxL; q.base = base; q.offset = offset; q.rope = c->rope_tab; q.bias = L.bqkv;
    q.Af = in.F; q.ssq = in.ssq; q.nssq = in.nssq;
    P.push_back(q);
    Phase a{}; a.type = PH_ATTN; a.A = qrows; a.lda = qd; a.kc = kv.k; a.vc = kv.v; a.maxL = kv.maxL; a.base = base; a.offset = offset;
    a.att = fused_attn_shape(c, nseq, m, offset, kv.maxL, qd, false, &a.att_items);
    a.ws = pool.take(attn_partials(c->fused_grid, a.att_items) * FUSED_RMAX * (g.head_dim + 2));
    a.F = attF; a.ldy = qd;
    if (elect) a.cnt = (int*)pool.take((size_t)a.att_items);       // zero from the pool's memset; the merging workgroup re-zeroes it
    P.push_back(a);
    if (!elect) { Phase mg = a; mg.type = PH_ATTN_MERGE; P.push_back(mg); }
    Phase o{}; o.type = PH_GEMM; o.pro = PRO_PLAIN; o.epi = FEPI_ADD_TO; o.K = qd; o.N = d; o.W = L.wo; o.Af = attF;
    o.Y = h1; o.ldy = d; o.R = in.h; o.ldr = d; o.F = h1F; o.fgain = L.norm2; o.ssq_out = h1s;
    P.push_back(o);
    Phase gu{}; gu.type = PH_GEMM; gu.pro = PRO_RMS; gu.epi = FEPI_SILU; gu.K = d; gu.N = 2 * F; gu.W = L.wgu; gu.Af = h1F; gu.ssq = h1s; gu.nssq = d / 16;
    gu.F = actF;
    P.push_back(gu);
    Phase dn{}; dn.type = PH_GEMM; dn.pro = PRO_PLAIN; dn.epi = FEPI_ADD_TO; dn.K = F; dn.N = d; dn.W = L.wd; dn.Af = actF;
    dn.Y = out.h; dn.ldy = d; dn.R = h1; dn.ldr = d; dn.F = out.F; dn.fgain = out_gain; dn.ssq_out = out.ssq;
    P.push_back(dn);
}

// bytes of the weights that a draft step reads: the drafter's layer, the LM head, the fusion FC's w1
double draft_step_bytes(const hivis_ctx* c) {
    const hivis_config& g = c->cfg;
    const double qd = g.n_q_heads * g.head_dim, kd = g.n_kv_heads * g.head_dim;
    return c->esize * (double)g.d * (2 * qd + 2 * kd + 3.0 * g.ffn + g.vocab + g.d);
}

// greedy candidates per row of an LM-head phase: its workgroups (a single-launch program always runs the whole grid)
int lm_candidates(const hivis_ctx* c, int N, bool persistent) { return persistent ? c->fused_grid : std::min(c->fused_grid, N / 16); }

template <typename WT>
void build_phases(hivis_ctx* c, int kind, int K, Pool& pool, std::vector<Phase>& P, bool persistent, bool elect, bool stream, bool lm_ext, bool alone) {
    const hivis_config& g = c->cfg;
    const int B = g.batch, d = g.d, V = g.vocab, G = c->fused_grid;
    int ld = d;
    // Launch-per-phase programs fold two small phases away: the gather of Embed(x) into the fusion FC (its activation
    // columns [d, 2d) come straight from the embedding table), and, with `elect`, the greedy-token reduction into the
    // LM-head phase (the workgroup that arrives last reduces the candidates).  The single-launch program keeps both phases.
    const bool fold = !persistent;
    const bool lm_elect = elect && !persistent;
    auto rows_of = [&](int M, bool sums) {
        StreamRows r{};
        r.h = pool.take((size_t)M * d); r.F = (uint4*)pool.take((size_t)M * d);
        if (sums) { r.ssq = pool.take((size_t)M * ssq_stride(d / 16)); r.nssq = d / 16; }
        return r;
    };
    if (stream && kind == PROG_VERIFY) {
        const int m = K + 1, M = B * m;
        StreamRows x = rows_of(M, false);
        x.ssq = pool.take((size_t)M * ssq_stride(1)); x.nssq = 1;
        Phase pr{}; pr.type = PH_PREP; pr.ids = c->row_tok; pr.id_sseq = m; pr.id_srow = 1; pr.gain = c->embed; pr.Y = x.h; pr.ldy = d;
        pr.F = x.F; pr.fgain = c->layers[0].norm1; pr.ssq_out = x.ssq;
        P.push_back(pr);
        for (int l = 0; l < g.n_layers; ++l) {
            const bool end = l + 1 == g.n_layers;
            StreamRows y = end ? StreamRows{pool.take((size_t)M * d), nullptr, nullptr, 0} : rows_of(M, true);
            layer_stream<WT>(c, P, pool, c->layers[l], c->tkv[l], x, c->tlen, 0, B, m, y, end ? nullptr : c->layers[l + 1].norm1, elect);
            x = y;
        }
        Phase nr{}; nr.type = PH_NORM_ROWS; nr.A = x.h; nr.lda = d; nr.gain = c->final_norm; nr.Y = c->catT; nr.ldy = 2 * d; nr.F = c->vfrag;
        P.push_back(nr);
        Phase lm{}; lm.type = PH_GEMM; lm.pro = PRO_PLAIN; lm.epi = FEPI_LOGITS; lm.K = d; lm.N = V; lm.W = c->lm_head; lm.Af = c->vfrag;
        lm.Y = c->logits_v; lm.ldy = V; lm.pm = pool.take((size_t)M * G); lm.pi = (int*)pool.take((size_t)M * G);
        lm.tok_out = c->ttok; lm.o_sseq = g.k_max + 1; lm.o_srow = 1;
        if (lm_elect) lm.cnt = (int*)pool.take(1);
        P.push_back(lm);
        if (!lm_elect) {
            Phase am{}; am.type = PH_ARGMAX; am.tok_out = c->ttok; am.o_sseq = g.k_max + 1; am.o_srow = 1; am.pm = lm.pm; am.pi = lm.pi; am.N = lm_candidates(c, lm.N, false);
            P.push_back(am);
        }
    } else if (stream && kind != PROG_ROLL) {
        const uint4* f = c->catDf;            // the drafter's hidden rows
        for (int i = 1; i <= K; ++i) {
            Phase lm{}; lm.type = PH_GEMM; lm.pro = PRO_PLAIN; lm.epi = FEPI_LOGITS; lm.K = d; lm.N = V; lm.W = c->lm_head; lm.Af = f;
            lm.Y = c->logits_d + (size_t)(i - 1) * B * V; lm.ldy = V; lm.pm = pool.take((size_t)B * G); lm.pi = (int*)pool.take((size_t)B * G);
            lm.tok_out = c->drafts + (i - 1); lm.o_sseq = g.k_max; lm.o_srow = 0;
            // greedy token of step i: reduced by the phase that follows (as below), by the LM head's last workgroup, or by a phase of its own
            // The fusion FC on the LM-head launch, and a staged q|k|v that adds the table rows, for one or two sequences; for more, an FC phase and
            // q|k|v on row fragments.  Rounds of 7 steps, FC phase -> on the LM head, one to four sequences: 2560 wide 594 -> 553, 597 -> 572, 602 ->
            // 592, 605 -> 611 us; 4096 wide 889 -> 856, 891 -> 874, 897 -> 909, 905 -> 932; 5120 wide 1225 -> 1211, 1233 -> 1229, 1240 -> 1260, 1247 -> 1287;
            // 2048 wide 440 -> 414, 444 -> 454, 447 -> 457, 449 -> 473.
            const bool later = kind == PROG_DRAFT && i < K, ext = later && lm_ext && B <= 2;
            const bool in_lm = !later && lm_elect && kind == PROG_DRAFT;
            float* u_part = ext ? pool.take((size_t)B * d) : nullptr;
            if (ext) { lm.N = V + d; lm.Y2 = u_part; lm.ldy2 = d; lm.vec = c->rho; lm.vec_idx = std::min(i, g.n_resid - 1); }
            if (in_lm) lm.cnt = (int*)pool.take(1);
            P.push_back(lm);
            const int ncand = lm_candidates(c, lm.N, false);
            if (!in_lm && !later) {
                Phase am{}; am.type = PH_ARGMAX; am.tok_out = lm.tok_out; am.o_sseq = g.k_max; am.o_srow = 0; am.pm = lm.pm; am.pi = lm.pi; am.N = ncand;
                if (kind == PROG_DRAFT_SAMPLE) { am.type = PH_SAMPLE; am.A = lm.Y; am.lda = V; am.u = c->u_draft; am.u_sseq = g.k_max; am.u_idx = i - 1; }
                P.push_back(am);
            }
            if (i == K) break;
            StreamRows u{};
            if (ext) u.h = pool.take((size_t)B * d);
            else {
                u = rows_of(B, true);
                Phase fu{}; fu.type = PH_GEMM; fu.pro = PRO_PLAIN; fu.epi = FEPI_ADDVEC; fu.K = d; fu.N = d; fu.W = c->fuse_w1; fu.Af = f;
                fu.Y = u.h; fu.ldy = d; fu.vec = c->rho; fu.vec_idx = std::min(i, g.n_resid - 1); fu.add_rows = c->emb_w2;
                fu.F = u.F; fu.fgain = c->draft.norm1; fu.ssq_out = u.ssq;
                if (later) { fu.pm = lm.pm; fu.pi = lm.pi; fu.ncand = ncand; fu.tok_out = lm.tok_out; fu.o_sseq = g.k_max; fu.o_srow = 0; }
                else { fu.tok = c->drafts + (i - 1); fu.tok_sseq = g.k_max; fu.tok_srow = 0; }
                P.push_back(fu);
            }
            const size_t qi = P.size();
            uint4* fn = (uint4*)pool.take((size_t)B * d);
            layer_stream<WT>(c, P, pool, c->draft, c->dkv, u, c->dlen, i - 1, B, 1, StreamRows{nullptr, fn, nullptr, 0}, nullptr, elect);
            if (ext) {      // the layer's first phase (QKV): rows = u_part + table[token], tokens from this step's candidates, u written back
                Phase& q = P[qi];
                q.A = u_part; q.lda = d; q.add_rows = c->emb_w2; q.wb = u.h; q.tok = nullptr; q.pm = lm.pm; q.pi = lm.pi; q.ncand = ncand;
                q.tok_out = lm.tok_out; q.o_sseq = g.k_max; q.o_srow = 0;
            }
            f = fn;
        }
    } else if (stream) {
        // the re-fed rows are the verify pass's features, whose fragments it left
        const int m = K + 1, M = B * m;
        StreamRows u = rows_of(M, true);
        Phase fu{}; fu.type = PH_GEMM; fu.pro = PRO_PLAIN; fu.epi = FEPI_ADDVEC; fu.K = d; fu.N = d; fu.W = c->fuse_w1; fu.Af = c->vfrag;
        fu.Y = u.h; fu.ldy = d; fu.vec = c->rho; fu.vec_idx = 0; fu.add_rows = c->emb_w2; fu.tok = c->next_tok; fu.tok_sseq = g.k_max + 1; fu.tok_srow = 1;
        fu.F = u.F; fu.fgain = c->draft.norm1; fu.ssq_out = u.ssq;
        P.push_back(fu);
        layer_stream<WT>(c, P, pool, c->draft, c->dkv, u, c->dlen, 0, B, m, StreamRows{c->dout, nullptr, nullptr, 0}, nullptr, elect);
    } else if (kind == PROG_VERIFY) {
        const int m = K + 1, M = B * m;
        float* x = pool.take((size_t)M * d);
        Phase pr{}; pr.type = PH_PREP; pr.ids = c->row_tok; pr.id_sseq = m; pr.id_srow = 1; pr.gain = c->embed; pr.Y = x; pr.ldy = d;
        pr.base = c->tlen; pr.offset = 0;
        P.push_back(pr);
        for (int l = 0; l < g.n_layers; ++l) x = layer_phases<WT>(c, P, pool, c->layers[l], c->tkv[l], x, c->tlen, 0, B, m, nullptr, 0, &ld, persistent, elect, alone);
        Phase nr{}; nr.type = PH_NORM_ROWS; nr.A = x; nr.lda = d; nr.gain = c->final_norm; nr.Y = c->catT; nr.ldy = 2 * d;
        P.push_back(nr);
        Phase lm{}; lm.type = PH_GEMM; lm.pro = PRO_PLAIN; lm.epi = FEPI_LOGITS; lm.K = d; lm.N = V; lm.W = c->lm_head; lm.A = c->catT; lm.lda = 2 * d;
        lm.Y = c->logits_v; lm.ldy = V; lm.pm = pool.take((size_t)M * G); lm.pi = (int*)pool.take((size_t)M * G);
        lm.tok_out = c->ttok; lm.o_sseq = g.k_max + 1; lm.o_srow = 1;
        if (lm_elect) lm.cnt = (int*)pool.take(1);         // zero from the pool's memset; the reducing workgroup re-zeroes it
        P.push_back(lm);
        if (!lm_elect) {
            Phase am{}; am.type = PH_ARGMAX; am.tok_out = c->ttok; am.o_sseq = g.k_max + 1; am.o_srow = 1; am.pm = lm.pm; am.pi = lm.pi; am.N = lm_candidates(c, lm.N, persistent);
            P.push_back(am);
        }
    } else if (kind == PROG_DRAFT || kind == PROG_DRAFT_SAMPLE) {
        // cat: [B][2d] = drafter hidden f' | embedding of the token drafted from it; a fresh buffer per step
        float* cat = c->catD;
        for (int i = 1; i <= K; ++i) {
            Phase lm{}; lm.type = PH_GEMM; lm.pro = PRO_PLAIN; lm.epi = FEPI_LOGITS; lm.K = d; lm.N = V; lm.W = c->lm_head; lm.A = cat; lm.lda = 2 * d;
            lm.Y = c->logits_d + (size_t)(i - 1) * B * V; lm.ldy = V; lm.pm = pool.take((size_t)B * G); lm.pi = (int*)pool.take((size_t)B * G);
            lm.tok_out = c->drafts + (i - 1); lm.o_sseq = g.k_max; lm.o_srow = 0;
            // greedy token of step i: reduced by the fusion FC that follows (steps before the last), by the LM head's last
            // workgroup (last step, with `elect`), or by a phase of its own
            const bool in_fc = fold && kind == PROG_DRAFT && i < K;
            // ... and with the extended LM head there is no FC phase: this LM-head launch also computes f' w1 + rho for the
            // next step (d extra columns), and the next step's QKV phase reduces the token and adds the table row of it
            // (the QKV variants that add the table rows stage two or four rows; fp32, rounds of 7 steps of one and four sequences: 256 wide 270 -> 232,
            // 295 -> 265 us, 2048 wide 847 -> 809, 903 -> 882)
            const bool ext = in_fc && lm_ext && B <= 4;
            float* u_part = ext ? pool.take((size_t)B * d) : nullptr;
            if (ext) { lm.N = V + d; lm.Y2 = u_part; lm.ldy2 = d; lm.vec = c->rho; lm.vec_idx = std::min(i, g.n_resid - 1); }
            const bool in_lm = !in_fc && lm_elect && kind == PROG_DRAFT;
            if (in_lm) lm.cnt = (int*)pool.take(1);
            P.push_back(lm);
            if (!in_lm && !in_fc) {
                Phase am{}; am.type = PH_ARGMAX; am.tok_out = c->drafts + (i - 1); am.o_sseq = g.k_max; am.o_srow = 0; am.pm = lm.pm; am.pi = lm.pi; am.N = lm_candidates(c, lm.N, persistent);
                if (kind == PROG_DRAFT_SAMPLE) {     // the token is drawn from softmax(logits / T) instead (uniforms [B][k_max], column i-1)
                    am.type = PH_SAMPLE; am.A = lm.Y; am.lda = V; am.u = c->u_draft; am.u_sseq = g.k_max; am.u_idx = i - 1;
                }
                P.push_back(am);
            }
            if (i < K) {
                float* u = pool.take((size_t)B * d);
                float* cat_next = pool.take((size_t)B * 2 * d);
                Phase fu{}; fu.type = PH_GEMM; fu.pro = PRO_PLAIN; fu.epi = FEPI_ADDVEC; fu.K = 2 * d; fu.N = d; fu.W = c->fuse_w; fu.A = cat; fu.lda = 2 * d;
                fu.Y = u; fu.ldy = d; fu.vec = c->rho; fu.vec_idx = std::min(i, g.n_resid - 1);
                if (fold) {
                    fu.emb = c->embed; fu.tok = c->drafts + (i - 1); fu.tok_sseq = g.k_max; fu.tok_srow = 0;
                    if (c->emb_w2) { fu.emb = nullptr; fu.add_rows = c->emb_w2; fu.K = d; fu.W = c->fuse_w1; }     // embedding half from the table
                    if (in_fc) { fu.tok = nullptr; fu.pm = lm.pm; fu.pi = lm.pi; fu.ncand = lm_candidates(c, lm.N, persistent); fu.tok_out = c->drafts + (i - 1); fu.o_sseq = g.k_max; fu.o_srow = 0; }
                }
                else {
                    Phase pr{}; pr.type = PH_PREP; pr.ids = c->drafts + (i - 1); pr.id_sseq = g.k_max; pr.id_srow = 0; pr.gain = c->embed;
                    pr.Y = cat + d; pr.ldy = 2 * d; pr.base = c->dlen; pr.offset = i - 1;
                    P.push_back(pr);
                }
                if (!ext) P.push_back(fu);
                const size_t qi = P.size();
                const int ncand = lm_candidates(c, lm.N, persistent);
                layer_phases<WT>(c, P, pool, c->draft, c->dkv, u, c->dlen, i - 1, B, 1, cat_next, 2 * d, &ld, persistent, elect, alone);
                if (ext) {      // the layer's first phase (QKV): rows = u_part + table[token], tokens from this step's candidates, u written back
                    Phase& q = P[qi];
                    q.A = u_part; q.lda = d; q.add_rows = c->emb_w2; q.wb = u; q.tok = nullptr; q.pm = lm.pm; q.pi = lm.pi; q.ncand = ncand;
                    q.tok_out = c->drafts + (i - 1); q.o_sseq = g.k_max; q.o_srow = 0;
                }
                cat = cat_next;
            }
        }
    } else {
        const int m = K + 1, M = B * m;
        float* u = pool.take((size_t)M * d);
        Phase fu{}; fu.type = PH_GEMM; fu.pro = PRO_PLAIN; fu.epi = FEPI_ADDVEC; fu.K = 2 * d; fu.N = d; fu.W = c->fuse_w; fu.A = c->catT; fu.lda = 2 * d;
        fu.Y = u; fu.ldy = d; fu.vec = c->rho; fu.vec_idx = 0;
        if (fold) {
            fu.emb = c->embed; fu.tok = c->next_tok; fu.tok_sseq = g.k_max + 1; fu.tok_srow = 1;
            if (c->emb_w2) { fu.emb = nullptr; fu.add_rows = c->emb_w2; fu.K = d; fu.W = c->fuse_w1; }
        }
        else {
            Phase pr{}; pr.type = PH_PREP; pr.ids = c->next_tok; pr.id_sseq = g.k_max + 1; pr.id_srow = 1; pr.gain = c->embed;
            pr.Y = c->catT + d; pr.ldy = 2 * d; pr.base = c->dlen; pr.offset = 0;
            P.push_back(pr);
        }
        P.push_back(fu);
        layer_phases<WT>(c, P, pool, c->draft, c->dkv, u, c->dlen, 0, B, m, c->dout, d, &ld, persistent, elect, alone);
    }
    // chain the GEMM phases for the cross-barrier weight prefetch
    for (size_t i = 0; i < P.size(); ++i) {
        if (P[i].type != PH_GEMM) continue;
        for (size_t j = i + 1; j < P.size(); ++j)
            if (P[j].type == PH_GEMM) { P[i].next_W = P[j].W; P[i].next_K = P[j].K; P[i].next_N = P[j].N; break; }
    }
}

template <typename WT>
int get_program(hivis_ctx* c, int kind, int K, hivis_ctx::Program* out) {
    const int key = kind * 64 + K;
    auto it = c->programs.find(key);
    if (it != c->programs.end()) { *out = it->second; return HIVIS_OK; }
    std::vector<Phase> P;
    Pool count;
    const bool alone = std::is_same<WT, float>::value && !c->persistent;
    build_phases<WT>(c, kind, K, count, P, c->persistent, c->attn_elect, c->stream_rows, c->lm_ext, alone);           // sizes only
    Pool pool;
    if (int rc = dev_alloc(c, &pool.base, count.used)) return rc;
    HIP_TRY(c, hipMemsetAsync(pool.base, 0, count.used * sizeof(float), c->stream));      // (on the stream of the passes that count on it)
    P.clear();
    build_phases<WT>(c, kind, K, pool, P, c->persistent, c->attn_elect, c->stream_rows, c->lm_ext, alone);
    hivis_ctx::Program pg;
    pg.n = (int)P.size();
    if (int rc = dev_alloc(c, &pg.dev, P.size())) return rc;
    HIP_TRY(c, hipMemcpy(pg.dev, P.data(), P.size() * sizeof(Phase), hipMemcpyHostToDevice));
    pg.host = new std::vector<Phase>(P);
    c->programs[key] = pg;
    *out = pg;
    return HIVIS_OK;
}

// One launch per phase (the default way a pass runs): grids sized to the phase's work.  phases: host array of n phases.
template <typename WT>
int launch_phases(hivis_ctx* c, const Phase* phases, int n, int kind, int K, const PassParams& pp, bool do_prof) {
    const hivis_config& g = c->cfg;
    // one launch per phase; grids sized to the phase's work
    // key splits per attention item: enough workgroups to fill the chip for long caches, a single workgroup (and no
    // merge launch) for short ones; the program was sized for the largest split count
    int max_keys = 0;
    for (int b = 0; b < g.batch; ++b) max_keys = std::max(max_keys, (kind == PROG_VERIFY ? c->h_tlen[b] : c->h_dlen[b]) + K + 1);
    // Cached rows of all target layers that the memory-side cache (256 MB) does not hold from pass to pass are read with the non-temporal
    // hint, where one workgroup reads each: 3010 keys x 4 layers (394 MB) 24.7 -> 23.1 us per layer.  Rows that it does hold are not: the
    // weights, read with the hint, leave them there (650 keys x 8 layers, 170 MB: 11.6 us, 12.8 with the hint; the drafter's layer 7.2 and 8.4).
    const bool once = !std::is_same<WT, float>::value && kind == PROG_VERIFY &&
                      (double)g.n_layers * g.batch * g.n_kv_heads * max_keys * g.head_dim * 8.0 > 256.0e6;
    // Weights of a draft round (or of a tree's levels), read once per step: without the hint where that cache holds all of a step's.  A round of
    // 12 steps, one sequence, with the hint -> without: 1024 wide, 32000 columns (97 MB) 569 -> 530 us, 1536 wide (160 MB) 665 -> 622, 2048 wide
    // (229 MB) 755 -> 713; but 2560 wide (336 MB) 974 -> 1040, 2048 wide with 50272 columns (348 MB) 963 -> 1044.  (With plain loads and
    // staged rows 547, 655, 738, 1079 and 1052.)  Rows of up to 2048 values, where that was measured.
    const bool keep = !std::is_same<WT, float>::value && (kind == PROG_DRAFT || kind == PROG_DRAFT_SAMPLE) && K > 1 && g.d <= STREAM_SHORT_K && draft_step_bytes(c) <= 256.0e6;
    for (int p = 0; p < n; ++p) {
        Phase ph = phases[p];
        ph.next_W = nullptr;                       // nothing is prefetched across a kernel boundary (pulling the next launch's
                                                   // first units into L2 during the epilogue was measured: 3% slower)
        if (ph.type == PH_ATTN || ph.type == PH_ATTN_MERGE) {
            ph.att.nsplit = key_splits(c, max_keys, ph.att.nsplit, !std::is_same<WT, float>::value);
            if (ph.att_alone) {
                int items = 0;
                AttnShape one = fused_attn_shape(c, pp.nseq, pp.m, ph.offset, ph.maxL, ph.att.ldq, true, &items);
                one.nsplit = attn_splits(max_keys, one.nsplit, c->keys_per_split);
                if (attn_alone(pp.nseq, pp.m, g.n_q_heads, g.n_kv_heads, g.head_dim, max_keys, one.nsplit, ph.att.nsplit)) { ph.att = one; ph.att_items = items; }
            }
            ph.att.flags = c->attn_flags;
        }
        if (ph.type == PH_ATTN || ph.type == PH_ATTN_MERGE || (ph.type == PH_GEMM && ph.epi == FEPI_QKV)) {
            if (g.batch <= 8 && ph.att.seq0 == 0) {          // the lengths the device arrays hold right now, by value
                ph.att.nbase = g.batch;
                for (int b = 0; b < g.batch; ++b) ph.att.base_val[b] = kind == PROG_VERIFY ? c->h_tlen[b] : c->h_dlen[b];
            }
            if (ph.type == PH_ATTN_MERGE && ph.att.nsplit == 1) continue;
        }
        int grid = c->fused_grid;
        if (ph.type == PH_ATTN_MERGE) grid = std::min(grid, ph.att_items);
        else if (ph.type == PH_PREP) grid = std::min(grid, pp.M);
        else if (ph.type == PH_NORM_ROWS) grid = std::min(grid, pp.M);
        else if (ph.type == PH_ARGMAX) grid = std::min(grid, (pp.M + FUSED_NW - 1) / FUSED_NW);
        else if (ph.type == PH_SAMPLE) grid = std::min(grid, pp.M);
        else if (ph.type == PH_GEMM) grid = std::min(grid, ph.N / 16);      // (the LM head's number of greedy candidates per row: lm_candidates)
        PassParams ppl = pp;
        if (do_prof) { ppl.prof2 = pp.prof2 + (size_t)p * 8; if (p >= n / 2 && p < n / 2 + 8) ppl.prof3 = c->prof + 4096 * 11 + (size_t)(p - n / 2) * PROF_WGS * 4; }
        // kev0/kev1 (null unless this launch is timed) are attached to the dispatch itself: they read the kernel's own
        // start and end timestamps, with no marker packets before or after it in the queue
        // (bf16w has GEMM kernels only: the other phases work on fp32 rows)
        typedef typename std::conditional<std::is_same<WT, bf16w_t>::value, bf16_t, WT>::type RT;
        const size_t lds = ph.type == PH_GEMM && std::is_same<WT, bf16w_t>::value ? c->fused_lds_w : c->fused_lds;
#define HIVIS_LAUNCH(TY, EP) do { typedef typename std::conditional<TY == PH_GEMM, WT, RT>::type KT_; \
                              constexpr bool may_ = TY == PH_GEMM && (std::is_same<WT, float>::value || EP == FEPI_ADD_TO || EP == FEPI_ADDVEC);     /* (the rule of `single`) */ \
                              if (may_ && single) hipExtLaunchKernelGGL((phase_kernel<KT_, TY, EP, may_>), dim3(grid), dim3(FUSED_NT), lds, c->stream, kev0, kev1, 0, ph, ppl); \
                              else hipExtLaunchKernelGGL((phase_kernel<KT_, TY, EP, false>), dim3(grid), dim3(FUSED_NT), lds, c->stream, kev0, kev1, 0, ph, ppl); } while (0)
#define HIVIS_LAUNCH_KEEP(EP) hipExtLaunchKernelGGL((phase_kernel<bf16_t, PH_GEMM, EP, false, true>), dim3(grid), dim3(FUSED_NT), lds, c->stream, kev0, kev1, 0, ph, ppl)
        // one tile per workgroup at most.  (q|k|v, gate|up and LM head: fp32 models only, whose matrices are that small; 256 wide: 7.7 -> 7.0, 7.2 -> 6.0 and 9.0 -> 7.8 us; q|k|v 1024 wide 8.7 -> 7.4, 2048 wide 11.0 -> 10.7)
        const bool single = ph.type == PH_GEMM && ph.N / 16 <= grid &&
                            (std::is_same<WT, float>::value || (ph.epi != FEPI_LOGITS && ph.epi != FEPI_SILU && ph.epi != FEPI_QKV));
        const bool kmatch = kind == PROG_VERIFY && ph.type == PH_GEMM && ph.epi == c->ktime_epi;
        const int64_t kseq = kmatch ? c->ktime_seen++ : 0;
        const bool ktimed = kmatch && (kseq % c->ktime_stride) == 0;
        hipEvent_t kev0 = nullptr, kev1 = nullptr;
        if (ktimed) {
            if (c->kev_used + 2 > c->kev.size()) { hipEvent_t e0, e1; HIP_TRY(c, hipEventCreate(&e0)); HIP_TRY(c, hipEventCreate(&e1)); c->kev.push_back(e0); c->kev.push_back(e1); }
            kev0 = c->kev[c->kev_used]; kev1 = c->kev[c->kev_used + 1];
            c->kev_used += 2;
            c->kbytes = (double)ph.K * ph.N * c->esize;
        }
        if constexpr (!std::is_same<WT, float>::value) {
            if (ph.type == PH_GEMM && ph.Af) {
                // tiles of a workgroup in groups of at most 8, as even as they come (a kernel of fewer tiles takes more groups).  Nine for the 8-row
                // LM head: 4096 wide, 32000 columns and w1's (2256 tiles) 47.6 us in one group of nine, 49.7 in two of five.  (Measured at that width only;
                // ten tiles, 5120 wide, are two groups of five.)
                const int most = (ph.N / 16 + grid - 1) / grid, upto = std::is_same<WT, bf16_t>::value && ph.epi == FEPI_LOGITS && ph.K > STREAM_SHORT_K ? 9 : 8;
                const int ngroups = (most + upto - 1) / upto, group = (most + ngroups - 1) / ngroups;
                const bool sh = ph.K <= STREAM_SHORT_K;
                if constexpr (std::is_same<WT, bf16w_t>::value) {
                    // 9..16 rows and at most half as many tiles as CUs: a second workgroup per tile, each with half the rows in the 8-row form
                    // (half the fragments through a CU's address pipeline; the tile's weights come from the L2 once).  2048 columns, 12 rows:
                    // down (K = 5632) 14.1 -> 10.8 us, O 6.6 -> 6.0.
                    if ((ph.epi == FEPI_ADD_TO || ph.epi == FEPI_ADDVEC) && 2 * grid <= c->fused_grid && grid == ph.N / 16) {
#define HIVIS_HALVES_(EP, SH_, KP_) hipExtLaunchKernelGGL((stream_kernel<bf16_t, EP, 1, SH_, KP_>), dim3(2 * grid), dim3(FUSED_NT), stream_lds_floats(1, WTraits<bf16_t>::RPL) * sizeof(float), c->stream, kev0, kev1, 0, ph, ppl)
#define HIVIS_HALVES(EP, SH_) do { if (keep) HIVIS_HALVES_(EP, SH_, true); else HIVIS_HALVES_(EP, SH_, false); } while (0)
                        if (ph.epi == FEPI_ADD_TO) { if (sh) HIVIS_HALVES(FEPI_ADD_TO, true); else HIVIS_HALVES(FEPI_ADD_TO, false); }
                        else { if (sh) HIVIS_HALVES(FEPI_ADDVEC, true); else HIVIS_HALVES(FEPI_ADDVEC, false); }
#undef HIVIS_HALVES
#undef HIVIS_HALVES_
                        continue;
                    }
                }
#define HIVIS_STREAM_(EP, G_, SH_, KP_) hipExtLaunchKernelGGL((stream_kernel<WT, EP, G_, SH_, KP_>), dim3(grid), dim3(FUSED_NT), stream_lds_floats(G_, WTraits<WT>::RPL) * sizeof(float), c->stream, kev0, kev1, 0, ph, ppl)
#define HIVIS_STREAM(EP, G_) HIVIS_STREAM_(EP, G_, false, false)
#define HIVIS_STREAM2(EP, G_) do { if (sh && keep) HIVIS_STREAM_(EP, G_, true, true); else if (sh) HIVIS_STREAM_(EP, G_, true, false); else HIVIS_STREAM_(EP, G_, false, false); } while (0)
#define HIVIS_STREAM1(EP) do { if (!sh && keep) HIVIS_STREAM_(EP, 1, false, true); else HIVIS_STREAM2(EP, 1); } while (0)      // (rows of the MLP's inner width)
                switch (ph.epi) {
                case FEPI_ADD_TO: if (group <= 1) HIVIS_STREAM1(FEPI_ADD_TO); else HIVIS_STREAM(FEPI_ADD_TO, 2); break;
                case FEPI_ADDVEC: if (group <= 1) HIVIS_STREAM2(FEPI_ADDVEC, 1); else HIVIS_STREAM(FEPI_ADDVEC, 2); break;
                case FEPI_QKV: if (group <= 1) HIVIS_STREAM2(FEPI_QKV, 1); else if (group <= 2) HIVIS_STREAM2(FEPI_QKV, 2); else if (group <= 3) HIVIS_STREAM(FEPI_QKV, 3); else HIVIS_STREAM(FEPI_QKV, 4); break;
                case FEPI_SILU:
                    if (group <= 2) HIVIS_STREAM2(FEPI_SILU, 2); else if (group <= 3) HIVIS_STREAM2(FEPI_SILU, 3); else if (group <= 4) HIVIS_STREAM(FEPI_SILU, 4);
                    else if (group <= 6) HIVIS_STREAM(FEPI_SILU, 6); else HIVIS_STREAM(FEPI_SILU, 8);
                    break;
                case FEPI_LOGITS: if (group <= 2) HIVIS_STREAM2(FEPI_LOGITS, 2); else if (group <= 4) HIVIS_STREAM2(FEPI_LOGITS, 4); else if (group <= 6) HIVIS_STREAM2(FEPI_LOGITS, 6);
                    else {
                        if constexpr (std::is_same<WT, bf16_t>::value) { if (group > 8) { HIVIS_STREAM(FEPI_LOGITS, 9); break; } }
                        HIVIS_STREAM2(FEPI_LOGITS, 8);
                    }
                    break;
                default: return fail(c, HIVIS_EINVAL, "phase %d: no kernel for epilogue %d", p, ph.epi);
                }
#undef HIVIS_STREAM1
#undef HIVIS_STREAM2
#undef HIVIS_STREAM
#undef HIVIS_STREAM_
                continue;
            }
            if (ph.type == PH_NORM_ROWS && ph.F) {
                hipExtLaunchKernelGGL(stream_norm_kernel, dim3(pp.M), dim3(FUSED_NT), 0, c->stream, kev0, kev1, 0, ph, ppl);
                continue;
            }
            if (ph.type == PH_PREP && ph.F) {
                hipExtLaunchKernelGGL(stream_prep_kernel, dim3(pp.M), dim3(FUSED_NT), 0, c->stream, kev0, kev1, 0, ph, ppl);
                continue;
            }
        }
        if constexpr (std::is_same<WT, float>::value) {
            // fp32, one tile per workgroup and one pass over K: the wavefronts share K evenly, in kernels for as many blocks as they then have.  (The
            // fusion FC only with the table.)
            const int kblks = ph.K / 16;
            if (single && kblks <= TILE_MAX_BLOCKS && (ph.epi != FEPI_ADDVEC || ph.add_rows) && !(ph.epi == FEPI_QKV && (ph.pos_delta || (ph.add_rows && pp.M > 4)))) {
                const int per = (kblks + FUSED_NW - 1) / FUSED_NW;
#define HIVIS_TILE_(EP, U_) hipExtLaunchKernelGGL((tile_kernel<EP, U_>), dim3(grid), dim3(FUSED_NT), 0, c->stream, kev0, kev1, 0, ph, ppl)
#define HIVIS_TILE(EP) do { if (per <= 2) HIVIS_TILE_(EP, 2); else if (per <= 4) HIVIS_TILE_(EP, 4); else if (per <= 6) HIVIS_TILE_(EP, 6); else HIVIS_TILE_(EP, 8); } while (0)
                switch (ph.epi) {
                case FEPI_ADD_TO: HIVIS_TILE(FEPI_ADD_TO); break;
                case FEPI_ADDVEC: HIVIS_TILE(FEPI_ADDVEC); break;
                case FEPI_QKV: if (ph.add_rows) HIVIS_TILE(FEPI_QKV_TAB); else HIVIS_TILE(FEPI_QKV); break;
                case FEPI_SILU: HIVIS_TILE(FEPI_SILU); break;
                case FEPI_LOGITS: HIVIS_TILE(FEPI_LOGITS); break;
                default: return fail(c, HIVIS_EINVAL, "phase %d: no kernel for epilogue %d", p, ph.epi);
                }
#undef HIVIS_TILE
#undef HIVIS_TILE_
                continue;
            }
        }
        switch (ph.type) {
        case PH_GEMM:
            switch (ph.epi) {
            case FEPI_ADD_TO: HIVIS_LAUNCH(PH_GEMM, FEPI_ADD_TO); break;
            case FEPI_ADDVEC: HIVIS_LAUNCH(PH_GEMM, FEPI_ADDVEC); break;
            case FEPI_QKV:
                if constexpr (std::is_same<WT, bf16_t>::value) {        // rows of a draft tree: the 16-row form knows their positions
                    if (ph.pos_delta) {
                        hipExtLaunchKernelGGL((phase_kernel<bf16w_t, PH_GEMM, FEPI_QKV, false>), dim3(grid), dim3(FUSED_NT), c->fused_lds_w, c->stream, kev0, kev1, 0, ph, ppl);
                        break;
                    }
                }
                if constexpr (!std::is_same<WT, bf16w_t>::value) {      // (table rows are added for at most four sequences)
                    if (ph.add_rows && pp.M <= 2) { if (keep) HIVIS_LAUNCH_KEEP(FEPI_QKV_TAB); else HIVIS_LAUNCH(PH_GEMM, FEPI_QKV_TAB); break; }
                    if (ph.add_rows) { HIVIS_LAUNCH(PH_GEMM, FEPI_QKV_TAB4); break; }
                }
                HIVIS_LAUNCH(PH_GEMM, FEPI_QKV);
                break;
            case FEPI_SILU: HIVIS_LAUNCH(PH_GEMM, FEPI_SILU); break;
            case FEPI_LOGITS: HIVIS_LAUNCH(PH_GEMM, FEPI_LOGITS); break;
            default: return fail(c, HIVIS_EINVAL, "phase %d: no kernel for epilogue %d", p, ph.epi);
            }
            break;
        case PH_ATTN:
            if constexpr (std::is_same<WT, float>::value) launch_attn_f32(c, ph, pp.M, ppl.prof2, ppl.prof3, kev0, kev1);
            else if (int rc = launch_attn_half(c, ph.att, ph.att_items, FUSED_RMAX, max_keys, ph.A, ph.kc, ph.vc, ph.base, AttnOut{ph.Y, ph.ldy, ph.F, pp.M}, nullptr, ph.ws, ph.cnt,
                                                once && ph.att.n_hblk == 1 && ph.att.n_rblk == 1, ppl.prof2, ppl.prof3, kev0, kev1)) return rc;
            break;
        case PH_ATTN_MERGE: HIVIS_LAUNCH(PH_ATTN_MERGE, 0); break;
        case PH_PREP: HIVIS_LAUNCH(PH_PREP, 0); break;
        case PH_NORM_ROWS: HIVIS_LAUNCH(PH_NORM_ROWS, 0); break;
        case PH_SAMPLE: HIVIS_LAUNCH(PH_SAMPLE, 0); break;
        case PH_ARGMAX: HIVIS_LAUNCH(PH_ARGMAX, 0); break;
        default: return fail(c, HIVIS_EINVAL, "phase %d: unknown type %d", p, ph.type);
        }
#undef HIVIS_LAUNCH_KEEP
#undef HIVIS_LAUNCH
    }
    HIP_TRY(c, hipGetLastError());
    return HIVIS_OK;
}

template <typename WT>
int run_program(hivis_ctx* c, int kind, int K, int nseq, int m) {
    hivis_ctx::Program pg;
    if (int rc = get_program<WT>(c, kind, K, &pg)) return rc;
    const hivis_config& g = c->cfg;
    PassParams pp{};
    pp.phases = pg.dev; pp.nphases = pg.n;
    pp.M = nseq * m; pp.nseq = nseq; pp.m = m;
    pp.d = g.d; pp.Hq = g.n_q_heads; pp.Hkv = g.n_kv_heads; pp.hd = g.head_dim; pp.F = g.ffn; pp.V = g.vocab;
    pp.eps = g.rms_eps; pp.theta = g.rope_theta; pp.inv_temp = c->inv_temp;
    pp.bar = c->bar; pp.bad = c->bad;
    pp.spin_limit = 1u << 22;
    const bool do_prof = c->prof && kind == PROG_VERIFY && c->prof_left > 0;
    pp.prof = do_prof ? c->prof : nullptr;
    pp.prof2 = do_prof ? c->prof + 4096 * 3 : nullptr;
    if (!c->persistent) {
        if constexpr (std::is_same<WT, bf16_t>::value) {
            if (pp.M > WTraits<WT>::ROWS) { if (int rc = launch_phases<bf16w_t>(c, pg.host->data(), pg.n, kind, K, pp, do_prof)) return rc; }
            else if (int rc = launch_phases<WT>(c, pg.host->data(), pg.n, kind, K, pp, do_prof)) return rc;
        } else if (int rc = launch_phases<WT>(c, pg.host->data(), pg.n, kind, K, pp, do_prof)) return rc;
        if (do_prof) {
            // developer aid: timestamps (100 MHz) that workgroup 0 of each launch wrote, for one layer in the middle
            std::vector<unsigned long long> t2((size_t)pg.n * 8);
            HIP_TRY(c, hipStreamSynchronize(c->stream));
            HIP_TRY(c, hipMemcpy(t2.data(), pp.prof2, t2.size() * 8, hipMemcpyDeviceToHost));
            const int p0 = std::min(pg.n / 2, pg.n - 1);
            const auto after = [](unsigned long long t, unsigned long long from) { return ((double)t - (double)from) * 0.01; };
            for (int p = p0; p < std::min(pg.n, p0 + 14); ++p) {
                const Phase& P = (*pg.host)[p];
                const unsigned long long* m = &t2[(size_t)p * 8];
                int before = p - 1;                                        // (row kernels write no marks)
                while (before >= 0 && !t2[(size_t)before * 8]) --before;
                if (!m[0] || before < 0) { fprintf(stderr, "[hivis prof] phase %d type %d epi %d: no marks\n", p, P.type, P.epi); continue; }
                fprintf(stderr, "[hivis prof] phase %d type %d epi %d: entry %+.2f us after the entry of phase %d;", p, P.type, P.epi, after(m[0], t2[(size_t)before * 8]), before);
                for (int k = 1; k < 7; ++k) if (m[k]) fprintf(stderr, " m%d %+.2f", k, after(m[k], m[0]));
                fprintf(stderr, "\n");
            }
            // per-workgroup entry/exit of the same launches: spread of the exits, the latest workgroups and where they ran
            std::vector<unsigned long long> t3((size_t)8 * 4096);
            HIP_TRY(c, hipMemcpy(t3.data(), c->prof + 4096 * 11, t3.size() * 8, hipMemcpyDeviceToHost));
            for (int p = p0; p < std::min(pg.n, p0 + 8); ++p) {
                const Phase& P = (*pg.host)[p];
                const unsigned long long* w = t3.data() + (size_t)(p - p0) * PROF_WGS * 4;
                std::vector<std::pair<double, int>> ends; double s0 = 1e300, s1 = 0;
                const auto ran = [&](int b) { return w[b * 4] && w[b * 4 + 1]; };          // (not workgroups without an item)
                for (int b = 0; b < PROF_WGS; ++b) if (ran(b)) { s0 = std::min(s0, (double)w[b * 4]); s1 = std::max(s1, (double)w[b * 4]); }
                for (int b = 0; b < PROF_WGS; ++b) if (ran(b)) ends.push_back({((double)w[b * 4 + 1] - s0) * 0.01, b});
                if (ends.empty()) continue;
                std::sort(ends.begin(), ends.end());
                const size_t n = ends.size();
                fprintf(stderr, "[hivis wg] phase %d type %d epi %d: %zu workgroups, entries within %.2f us; exits min %.2f p10 %.2f p50 %.2f p90 %.2f max %.2f us; latest:", p, P.type, P.epi, n,
                        (s1 - s0) * 0.01, ends[0].first, ends[n / 10].first, ends[n / 2].first, ends[n * 9 / 10].first, ends[n - 1].first);
                for (size_t k = n > 6 ? n - 6 : 0; k < n; ++k) {
                    const unsigned long long id = w[ends[k].second * 4 + 2];
                    fprintf(stderr, " wg%d(xcc%llu se%llu cu%llu)", ends[k].second, id >> 32, (id >> 13) & 7, (id >> 8) & 15);
                }
                double xs[8] = {}; int xn[8] = {};
                for (auto& e : ends) { const int x = (int)(w[e.second * 4 + 2] >> 32) & 7; xs[x] += e.first; xn[x]++; }
                if (t2[p * 8] && ran(0)) fprintf(stderr, "; wg0: entry->mark0 %.2f, mark0->exit %.2f us", after(t2[p * 8], w[0]), after(w[1], t2[p * 8]));
                fprintf(stderr, "; mean exit per xcc:");
                for (int x = 0; x < 8; ++x) fprintf(stderr, " %.1f(%d)", xn[x] ? xs[x] / xn[x] : 0.0, xn[x]);
                fprintf(stderr, "\n");
            }
            HIP_TRY(c, hipMemset(c->prof + 4096 * 3, 0, (size_t)16 * 4096 * 8));
            c->prof_left--;
        }
        return HIVIS_OK;
    }
    hipLaunchKernelGGL(set_ints_kernel, dim3(1), dim3(64), 0, c->stream, (int*)c->bar, 1, 0);
    void* args[] = {&pp};
    HIP_TRY(c, hipLaunchCooperativeKernel((const void*)fused_pass_kernel<WT>, dim3(c->fused_grid), dim3(FUSED_NT), args, c->fused_lds, c->stream));
    if (do_prof) {
        std::vector<unsigned long long> t((size_t)pg.n * 3), t2((size_t)pg.n * 8);
        std::vector<Phase> P(pg.n);
        HIP_TRY(c, hipStreamSynchronize(c->stream));
        HIP_TRY(c, hipMemcpy(t.data(), c->prof, t.size() * 8, hipMemcpyDeviceToHost));
        HIP_TRY(c, hipMemcpy(P.data(), pg.dev, P.size() * sizeof(Phase), hipMemcpyDeviceToHost));
        HIP_TRY(c, hipMemcpy(t2.data(), c->prof + 4096 * 3, t2.size() * 8, hipMemcpyDeviceToHost));
        for (int p = 7; p < 13 && p < pg.n; ++p) if (P[p].type == PH_GEMM)
            fprintf(stderr, "[hivis prof2] phase %d epi %d: entry+%.2f  staged+%.2f  pass0+%.2f  allpass+%.2f  reduced+%.2f  end+%.2f | work %.2f wait %.2f us\n", p, P[p].epi,
                    (t2[p*8]-t[p*3])*0.01, (t2[p*8+1]-t2[p*8])*0.01, (t2[p*8+2]-t2[p*8+1])*0.01, (t2[p*8+3]-t2[p*8+2])*0.01, (t2[p*8+4]-t2[p*8+3])*0.01, (t2[p*8+5]-t2[p*8+4])*0.01, (t[p*3+1]-t[p*3])*0.01, (t[p*3+2]-t[p*3+1])*0.01);
        double tot[8][8] = {}, bar[8][8] = {}; int cnt[8][8] = {};
        for (int p = 0; p < pg.n; ++p) {
            const int ty = P[p].type, ep = P[p].type == PH_GEMM ? P[p].epi : 0;
            tot[ty][ep] += (t[p * 3 + 1] - t[p * 3]) * 0.01; bar[ty][ep] += (t[p * 3 + 2] - t[p * 3 + 1]) * 0.01; cnt[ty][ep]++;
        }
        fprintf(stderr, "[hivis prof] verify pass %.1f us (workgroup 0 view)\n", (t[pg.n * 3 - 1] - t[0]) * 0.01);
        for (int ty = 0; ty < 8; ++ty) for (int ep = 0; ep < 8; ++ep) if (cnt[ty][ep])
            fprintf(stderr, "[hivis prof]   type %d epi %d: n=%3d  work %7.2f us avg, barrier wait %7.2f us avg\n", ty, ep, cnt[ty][ep], tot[ty][ep] / cnt[ty][ep], bar[ty][ep] / cnt[ty][ep]);
        c->prof_left--;
    }
    return HIVIS_OK;
}

// Phases a draft program of K steps needs at most (LM head, token, prep, fusion FC, QKV, attention, merge, O, gate|up, down)
static inline size_t draft_phase_capacity(int k_max) { return (size_t)k_max * 10 + 4; }

// The draft round of do_draft with every intermediate buffer inside the static scratch array: the same phase list and
// the same kernels (always one launch per phase), built into host storage reserved at create; no allocation of any kind.
template <typename WT>
int draft_noalloc(hivis_ctx* c, int K) {
    const hivis_config& g = c->cfg;
    std::vector<Phase>& P = c->na_phases;
    if (draft_phase_capacity(K) > P.capacity()) return fail(c, HIVIS_ECAP, "phase list of K=%d exceeds the storage reserved at create", K);
    // Accepted is what fits as the plain list: fp32 rows between the phases, and for fp32 models a launch of the fusion FC per step and
    // attention items that share their keys.  Row fragments, and for fp32 models items of one row and the FC on the LM-head launch,
    // where they fit as well.
    auto size = [&](bool stream, bool ext, bool alone) {
        P.clear();
        Pool count;
        build_phases<WT>(c, PROG_DRAFT, K, count, P, false, false, stream, ext, alone);            // sizes only
        return count.used * sizeof(float);
    };
    const bool bf16 = sizeof(WT) == 2;
    const size_t need = size(false, bf16 && c->lm_ext, false);
    const bool alone = !bf16 && size(false, false, true) <= (size_t)HIVIS_SCRATCH_BYTES;
    const bool ext = c->lm_ext && (bf16 || size(false, true, alone) <= (size_t)HIVIS_SCRATCH_BYTES);
    const bool stream = c->stream_rows && size(true, ext, alone) <= (size_t)HIVIS_SCRATCH_BYTES;
    if (need > (size_t)HIVIS_SCRATCH_BYTES)
        return fail(c, HIVIS_ECAP, "draft round of K=%d needs %zu bytes of scratch, the static array holds %u", K, need, (unsigned)HIVIS_SCRATCH_BYTES);
    P.clear();
    Pool pool; pool.base = (float*)c->scratch_dev;                  // the looked-up device address, not the array's name
    build_phases<WT>(c, PROG_DRAFT, K, pool, P, false, false, stream, ext, alone);
    PassParams pp{};
    pp.phases = nullptr; pp.nphases = (int)P.size();
    pp.M = g.batch; pp.nseq = g.batch; pp.m = 1;
    pp.d = g.d; pp.Hq = g.n_q_heads; pp.Hkv = g.n_kv_heads; pp.hd = g.head_dim; pp.F = g.ffn; pp.V = g.vocab;
    pp.eps = g.rms_eps; pp.theta = g.rope_theta; pp.inv_temp = c->inv_temp;
    pp.bar = c->bar; pp.bad = c->bad; pp.spin_limit = 1u << 22;
    return launch_phases<WT>(c, P.data(), (int)P.size(), PROG_DRAFT, K, pp, false);
}

template <typename WT>
int fused_setup(hivis_ctx* c) {
    typedef WTraits<WT> TR;
    const hivis_config& g = c->cfg;
    const char* env = getenv("HIVIS_FUSED");
    if (env && env[0] == '0') { c->fused = false; return HIVIS_OK; }
    const size_t gemm_f = fused_gemm_lds_floats(FusedCfg<WT>::NW, FusedCfg<WT>::G, TR::RPL, FusedCfg<WT>::KBW, FUSED_CHUNK<WT>);
    const size_t attn_f = std::max(fused_attn_lds_floats(g.head_dim, FUSED_NW, FUSED_RMAX), fused_attn_mfma_lds_floats(g.head_dim, FUSED_NW, FUSED_RMAX));
    c->fused_lds = std::max(gemm_f, attn_f) * sizeof(float);
    // the attribute is per kernel, not per context: contexts with different head sizes may be alive together, so it only grows
    static size_t lds_limit = 0;
    lds_limit = std::max(lds_limit, c->fused_lds);
    HIP_TRY(c, hipFuncSetAttribute((const void*)fused_pass_kernel<WT>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_limit));
    {
        const void* ks[] = {(const void*)phase_kernel<WT, PH_GEMM, FEPI_ADD_TO, false>,
                            (const void*)phase_kernel<WT, PH_GEMM, FEPI_ADDVEC, false>, (const void*)phase_kernel<WT, PH_GEMM, FEPI_QKV, false>,
                            (const void*)phase_kernel<WT, PH_GEMM, FEPI_QKV_TAB, false>, (const void*)phase_kernel<WT, PH_GEMM, FEPI_QKV_TAB4, false>,
                            (const void*)phase_kernel<WT, PH_GEMM, FEPI_SILU, false>, (const void*)phase_kernel<WT, PH_GEMM, FEPI_LOGITS, false>,
                            (const void*)phase_kernel<WT, PH_GEMM, FEPI_ADD_TO, true>,
                            (const void*)phase_kernel<WT, PH_GEMM, FEPI_ADDVEC, true>,
                            (const void*)phase_kernel<WT, PH_ATTN_MERGE, 0, false>,
                            (const void*)phase_kernel<WT, PH_PREP, 0, false>, (const void*)phase_kernel<WT, PH_NORM_ROWS, 0, false>,
                            (const void*)phase_kernel<WT, PH_ARGMAX, 0, false>, (const void*)phase_kernel<WT, PH_SAMPLE, 0, false>};
        for (const void* k : ks) HIP_TRY(c, hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_limit));
    }
    if constexpr (std::is_same<WT, float>::value) {
        const void* ks[] = {(const void*)phase_kernel<WT, PH_GEMM, FEPI_QKV, true>, (const void*)phase_kernel<WT, PH_GEMM, FEPI_QKV_TAB, true>,
                            (const void*)phase_kernel<WT, PH_GEMM, FEPI_QKV_TAB4, true>, (const void*)phase_kernel<WT, PH_GEMM, FEPI_SILU, true>,
                            (const void*)phase_kernel<WT, PH_GEMM, FEPI_LOGITS, true>};
        for (const void* k : ks) HIP_TRY(c, hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_limit));
    }
    if constexpr (std::is_same<WT, bf16_t>::value) {
        const void* kk[] = {(const void*)phase_kernel<bf16_t, PH_GEMM, FEPI_QKV_TAB, false, true>};
        for (const void* k : kk) HIP_TRY(c, hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_limit));
        typedef FusedCfg<bf16w_t> CW;
        c->fused_lds_w = fused_gemm_lds_floats(CW::NW, CW::G, WTraits<bf16w_t>::RPL, CW::KBW, FUSED_CHUNK<bf16w_t>) * sizeof(float);
        const void* ks[] = {(const void*)phase_kernel<bf16w_t, PH_GEMM, FEPI_ADD_TO, false>, (const void*)phase_kernel<bf16w_t, PH_GEMM, FEPI_ADD_TO, true>,
                            (const void*)phase_kernel<bf16w_t, PH_GEMM, FEPI_ADDVEC, false>, (const void*)phase_kernel<bf16w_t, PH_GEMM, FEPI_ADDVEC, true>,
                            (const void*)phase_kernel<bf16w_t, PH_GEMM, FEPI_QKV, false>, (const void*)phase_kernel<bf16w_t, PH_GEMM, FEPI_SILU, false>,
                            (const void*)phase_kernel<bf16w_t, PH_GEMM, FEPI_LOGITS, false>};
        for (const void* k : ks) HIP_TRY(c, hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)c->fused_lds_w));
    }
    if constexpr (std::is_same<WT, bf16_t>::value) {
        // (the only stream kernels beyond 64 KB of LDS)
        const void* ks[] = {(const void*)stream_kernel<bf16w_t, FEPI_SILU, 8, false>, (const void*)stream_kernel<bf16w_t, FEPI_LOGITS, 8, false>, (const void*)stream_kernel<bf16w_t, FEPI_LOGITS, 8, true>,
                            (const void*)stream_kernel<bf16w_t, FEPI_LOGITS, 8, true, true>};
        for (const void* k : ks) HIP_TRY(c, hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)(stream_lds_floats(8, WTraits<bf16w_t>::RPL) * sizeof(float))));
    }
    { const char* pe = getenv("HIVIS_PERSISTENT"); c->persistent = pe && pe[0] == '1'; }
    { const char* we = getenv("HIVIS_WIDE_GEMM"); c->no_wide_gemm = we && we[0] == '0'; }
    { const char* we = getenv("HIVIS_WIDE_MIN"); if (we && atoi(we) >= 1) c->wide_min = atoi(we); }
    { const char* ke = getenv("HIVIS_ATTN_SHARED_MIN"); if (ke && atoi(ke) >= 1) c->attn_shared_min = atoi(ke); }
    { const char* ke = getenv("HIVIS_KEYS_PER_SPLIT"); if (ke && atoi(ke) >= 16) { c->keys_per_split = atoi(ke); c->keys_forced = true; } }
    { const char* ee = getenv("HIVIS_ATTN_ELECT"); if (ee) c->attn_elect = ee[0] == '1'; }
    { const char* fe = getenv("HIVIS_ATTN_FLAGS"); if (fe) c->attn_flags = atoi(fe); }
    int nb = 0;
    HIP_TRY(c, hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, (const void*)fused_pass_kernel<WT>, FUSED_NT, c->fused_lds));
    if (nb < 1) return fail(c, HIVIS_EHIP, "persistent kernel does not fit on a compute unit");
    c->fused_grid = c->num_cu;
    int rc;
    if ((rc = dev_alloc(c, &c->bar, 2))) return rc;
    HIP_TRY(c, hipMemset(c->bar, 0, 2 * sizeof(unsigned)));
    if (const char* pe = getenv("HIVIS_PROF")) { c->prof_left = atoi(pe); if (c->prof_left > 0) { if ((rc = dev_alloc(c, &c->prof, (size_t)4096 * 19))) return rc; HIP_TRY(c, hipMemset(c->prof, 0, (size_t)4096 * 19 * 8)); } }
    c->fused = true;
    return HIVIS_OK;
}


// ---- GEMMs on activation fragments (bf16 models) --------------------------------------------------------------
// Room for K-slice partials: up to SPLITK_RESERVE floats from create on (allocating more takes a context longer than it saves);
// when a pass needs more, they are replaced once by all that any pass of this context can need.  (Growing step by step cost each
// longer prompt up to 5 ms and left the smaller buffers behind.)  The partials of one product are consumed before the next one
// starts, so nothing refers to the old buffer.  False: no device memory, and the caller does without slices.
// HIVIS_SPLITK_RESERVE=n: MB instead of 128, 0 for none.
constexpr size_t SPLITK_RESERVE = (size_t)32 << 20;
bool splitk_alloc(hivis_ctx* c, size_t floats) {
    void* q = nullptr;
    if (hipMalloc(&q, floats * sizeof(float)) != hipSuccess) { (void)hipGetLastError(); return false; }
    c->allocs.push_back(q);
    c->splitk_ws = (float*)q; c->splitk_floats = floats;
    return true;
}
size_t splitk_most(const hivis_ctx* c) {
    const hivis_config& g = c->cfg;
    return hivis::splitk_floats(c->num_cu, g.d, g.n_q_heads * g.head_dim, g.n_kv_heads * g.head_dim, g.ffn, c->pf_rows);
}
bool splitk_space(hivis_ctx* c, size_t floats) {
    if (floats <= c->splitk_floats) return true;
    if (hipStreamSynchronize(c->stream) != hipSuccess) return false;
    if (c->splitk_ws) {
        c->allocs.erase(std::find(c->allocs.begin(), c->allocs.end(), (void*)c->splitk_ws));
        (void)hipFree(c->splitk_ws);
        c->splitk_ws = nullptr; c->splitk_floats = 0;
    }
    return splitk_alloc(c, std::max(floats, splitk_most(c))) || splitk_alloc(c, floats);
}
// rows of fp32 -> fragments, in the buffer that holds them (*out)
int launch_pack(hivis_ctx* c, const float* A, int lda, int M, int K, uint4** out) {
    const int which = frag_buffer(c->pf_sizes, M, K);
    if (!which) return fail(c, HIVIS_EINVAL, "no buffer holds the fragments of %d rows of %d values", M, K);
    *out = which == 1 ? c->pf_frag : c->pf_frag2;
    const size_t chunks = frag_values(M, K) / 8;
    hipLaunchKernelGGL(pack_afrag_kernel, dim3((unsigned)std::min<size_t>((chunks + 255) / 256, 65535)), dim3(256), 0, c->stream, A, lda, M, K / 32, *out);
    return HIVIS_OK;
}

// the plan of a GEMM whose K range may be cut into slices, with room for them
TallPlan sliced_plan(hivis_ctx* c, int M, int K, int N) {
    TallPlan pl = tall_plan(c->num_cu, M, K / 32, N / 16, true, c->tall_cw);
    if (pl.ksplit > 1 && !splitk_space(c, (size_t)pl.ksplit * M * N)) pl = tall_plan(c->num_cu, M, K / 32, N / 16, false, c->tall_cw);
    return pl;
}

template <int EPI>
int launch_tall(hivis_ctx* c, const TallPlan& pl, const uint4* frag, int M, int K, const uint4* Wp, int N, TallOut o) {
    const int kblks = K / 32, row_tiles = (M + 15) / 16, ntiles = N / 16;
    if (pl.ksplit > 1) o.part = c->splitk_ws;
    const int tiles = ((M + TALL_ROWS - 1) / TALL_ROWS) * ((ntiles + 2 * pl.cw - 1) / (2 * pl.cw)) * pl.ksplit;
#define HIVIS_TALL(CW_)                                                                                                                    \
    hipLaunchKernelGGL((gemm_tall_kernel<CW_, EPI>), dim3(8 * ((tiles + 7) / 8)), dim3(TALL_THREADS), tall_lds_bytes<CW_>(), c->stream,    \
                       (const v4u_t*)frag, row_tiles, kblks, (const v4u_t*)Wp, ntiles, M, pl.ksplit, o)
    if (pl.cw == 8) HIVIS_TALL(8);
    else if (pl.cw == 7) HIVIS_TALL(7);
    else HIVIS_TALL(6);
#undef HIVIS_TALL
    HIP_TRY(c, hipGetLastError());
    return HIVIS_OK;
}
// the whole-prompt kernels that use more LDS than a launch gets without asking
int prefill_lds_setup(hivis_ctx* c) {
    struct { const void* k; size_t bytes; } ks[] = {
#define HIVIS_TALL_LDS(EPI_) {(const void*)gemm_tall_kernel<8, EPI_>, (size_t)tall_lds_bytes<8>()}, {(const void*)gemm_tall_kernel<7, EPI_>, (size_t)tall_lds_bytes<7>()}, \
                             {(const void*)gemm_tall_kernel<6, EPI_>, (size_t)tall_lds_bytes<6>()}
        HIVIS_TALL_LDS(TALL_STORE), HIVIS_TALL_LDS(TALL_SILU), HIVIS_TALL_LDS(TALL_QKV),
#undef HIVIS_TALL_LDS
#define HIVIS_WIDE_LDS(RT_, KW_, CT_) {(const void*)gemm_wide_kernel<RT_, KW_, CT_, WIDE_STORE>, (size_t)WideCfg<RT_, KW_, CT_>::LDS}, \
                                      {(const void*)gemm_wide_kernel<RT_, KW_, CT_, WIDE_SILU>, (size_t)WideCfg<RT_, KW_, CT_>::LDS}
        HIVIS_WIDE_LDS(2, 4, 2), HIVIS_WIDE_LDS(2, 4, 3), HIVIS_WIDE_LDS(2, 2, 2), HIVIS_WIDE_LDS(2, 4, 5), HIVIS_WIDE_LDS(2, 2, 3), HIVIS_WIDE_LDS(2, 2, 4), HIVIS_WIDE_LDS(2, 2, 5),
        HIVIS_WIDE_LDS(4, 4, 2), HIVIS_WIDE_LDS(4, 4, 3), HIVIS_WIDE_LDS(4, 2, 2), HIVIS_WIDE_LDS(4, 4, 5), HIVIS_WIDE_LDS(4, 2, 3), HIVIS_WIDE_LDS(4, 2, 4),
#undef HIVIS_WIDE_LDS
#define HIVIS_SPLIT_LDS(HD_, RM_, ONCE_) {(const void*)attn_split_kernel<HD_, RM_, ONCE_>, (size_t)AttnSplitCfg<HD_, RM_>::LDS}, \
                                         {(const void*)attn_tiles_kernel<HD_, RM_, ONCE_>, fused_attn_mfma_lds_floats(HD_, FUSED_NW, RM_) * sizeof(float)}
        HIVIS_SPLIT_LDS(128, ATTN_ROWS_RM, false), HIVIS_SPLIT_LDS(64, ATTN_ROWS_RM, false), HIVIS_SPLIT_LDS(128, FUSED_RMAX, true), HIVIS_SPLIT_LDS(128, FUSED_RMAX, false),
        HIVIS_SPLIT_LDS(64, FUSED_RMAX, true), HIVIS_SPLIT_LDS(64, FUSED_RMAX, false),
#undef HIVIS_SPLIT_LDS
        {(const void*)attn_rows_shared_kernel<128, 8>, attn_shared_lds_bytes(128)}, {(const void*)attn_rows_shared_kernel<128, 4>, attn_shared_lds_bytes(128)},
        {(const void*)attn_rows_shared_kernel<64, 8>, attn_shared_lds_bytes(64)}, {(const void*)attn_rows_shared_kernel<64, 4>, attn_shared_lds_bytes(64)}};
    for (const auto& k : ks) HIP_TRY(c, hipFuncSetAttribute(k.k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)k.bytes));
    return HIVIS_OK;
}

// Up to 64 rows in ONE pass over the weights (gemm_wide_kernel): the 11..64-row passes that no phase program takes, and a prefill's
// products of up to 64 rows.
template <int EPI>
int launch_wide(hivis_ctx* c, const WidePlan& pl, const uint4* frag, int M, int K, const uint4* Wp, int N, float* Y, int ldy, uint4* frag_out, int kblks_out) {
    const int ntiles = N / 16;
    const dim3 grid(pl.ksplit, (ntiles + pl.tiles - 1) / pl.tiles);
#define HIVIS_WIDE(RT_, KW_, CT_)                                                                                                              \
    {                                                                                                                                          \
        constexpr int lds_ = WideCfg<RT_, KW_, CT_>::LDS;                                                                                      \
        hipLaunchKernelGGL((gemm_wide_kernel<RT_, KW_, CT_, EPI>), grid, dim3(WIDE_THREADS), lds_, c->stream, frag, (M + 15) / 16, K / 32, pl.kper, Wp, ntiles, M, \
                           Y, ldy, pl.ksplit > 1 ? c->splitk_ws : nullptr, frag_out, kblks_out);                                               \
    } break
    if (M <= 32) switch (pl.form) {
        case 0: HIVIS_WIDE(2, 4, 2); case 1: HIVIS_WIDE(2, 4, 3); case 2: HIVIS_WIDE(2, 2, 2); case 3: HIVIS_WIDE(2, 4, 5);
        case 4: HIVIS_WIDE(2, 2, 3); case 5: HIVIS_WIDE(2, 2, 4); case 6: HIVIS_WIDE(2, 2, 5);
    } else switch (pl.form) {
        case 0: HIVIS_WIDE(4, 4, 2); case 1: HIVIS_WIDE(4, 4, 3); case 2: HIVIS_WIDE(4, 2, 2); case 3: HIVIS_WIDE(4, 4, 5);
        case 4: HIVIS_WIDE(4, 2, 3); case 5: HIVIS_WIDE(4, 2, 4);
    }
#undef HIVIS_WIDE
    HIP_TRY(c, hipGetLastError());
    return HIVIS_OK;
}
// defer != nullptr: the slice partials are not reduced here; *defer describes them for the consuming row kernel.
int wide_gemm(hivis_ctx* c, const uint4* frag, int M, int K, const uint4* Wp, int N, float* Y, int ldy, Parts* defer) {
    WidePlan pl = wide_plan(c->num_cu, M, K / 32, N / 16, true);
    if (pl.ksplit > 1 && !splitk_space(c, (size_t)pl.ksplit * M * ldy)) pl = wide_plan(c->num_cu, M, K / 32, N / 16, false);
    if (int rc = launch_wide<WIDE_STORE>(c, pl, frag, M, K, Wp, N, Y, ldy, nullptr, 0)) return rc;
    const Parts res{pl.ksplit > 1 ? c->splitk_ws : Y, pl.ksplit, (size_t)M * ldy};
    if (defer) *defer = res;
    else if (pl.ksplit > 1) hipLaunchKernelGGL(splitk_reduce_kernel, dim3(M, row_chunks(M)), dim3(256), 0, c->stream, res, N, ldy, Y, ldy);
    HIP_TRY(c, hipGetLastError());
    return HIVIS_OK;
}

// Any number of rows; the result is *out: K slices, or the one result in Y (row stride N).
int rows_gemm(hivis_ctx* c, const uint4* frag, int M, int K, const uint4* Wp, int N, float* Y, Parts* out) {
    if (M <= MAX_ROWS) return wide_gemm(c, frag, M, K, Wp, N, Y, N, out);
    const TallPlan pl = sliced_plan(c, M, K, N);
    TallOut o{}; o.Y = Y; o.ldy = N;
    if (int rc = launch_tall<TALL_STORE>(c, pl, frag, M, K, Wp, N, o)) return rc;
    *out = Parts{pl.ksplit > 1 ? c->splitk_ws : Y, pl.ksplit, (size_t)M * N};
    return HIVIS_OK;
}

// whether a product of M > 64 rows ends in the GEMM itself (TALL_QKV / TALL_SILU), and its plan then
bool ends_in_gemm(hivis_ctx* c, int M, int K, int N, TallPlan* pl) {
    if (M <= MAX_ROWS) return false;
    *pl = tall_plan(c->num_cu, M, K / 32, N / 16, false, c->tall_cw);
    // (room for the slices is asked for only where they are wanted: those of gate|up are the largest)
    return tall_fused(*pl, tall_plan(c->num_cu, M, K / 32, N / 16, true, c->tall_cw)) || sliced_plan(c, M, K, N).ksplit == 1;
}

// M = nseq * m rows: q (rotated) to q_out [M][q_dim], k and v of sequence seq0 + s to its cache rows base[seq0 + s] + offset ..
template <typename WT>
int rows_qkv(hivis_ctx* c, const LayerDev& L, const KVDev& kv, const uint4* frag, const int* base, int offset, int seq0, int nseq, int m,
             TreeRows tr, float* scratch, float* q_out) {
    typedef typename KVType<WT>::type KT;
    const hivis_config& g = c->cfg;
    const int M = nseq * m, d = g.d, qd = g.n_q_heads * g.head_dim, kd = g.n_kv_heads * g.head_dim, nqkv = qd + 2 * kd, npos = g.max_vis + g.max_text;
    TallPlan pl;
    if (base == c->zeros && offset == 0 && !tr.pos_delta && ends_in_gemm(c, M, d, nqkv, &pl)) {
        TallOut o{};
        o.Y = q_out; o.ldy = qd; o.bias = L.bqkv; o.rope = c->rope_tab; o.npos = npos; o.seq0 = seq0; o.m = m;
        o.qd = qd; o.kd = kd; o.HD = g.head_dim; o.Hkv = g.n_kv_heads; o.maxL = kv.maxL; o.kc = (f16_t*)kv.k; o.vc = (f16_t*)kv.v;
        return launch_tall<TALL_QKV>(c, pl, frag, M, d, L.wqkv, nqkv, o);
    }
    Parts p{};
    if (int rc = rows_gemm(c, frag, M, d, L.wqkv, nqkv, scratch, &p)) return rc;
    hipLaunchKernelGGL((wide_rope_append_kernel<KT>), dim3(M, M <= MAX_ROWS ? 8 : row_chunks(M)), dim3(256), 0, c->stream, p, q_out, qd, g.n_q_heads, g.n_kv_heads, g.head_dim,
                       base, offset, seq0, m, (KT*)kv.k, (KT*)kv.v, kv.maxL, g.rope_theta, tr.pos_delta, (const float*)L.bqkv, (const float*)c->rope_tab, npos);
    HIP_TRY(c, hipGetLastError());
    return HIVIS_OK;
}

// gate|up product and SiLU(gate) * up of M rows: fragments (in the layout of the down projection) to frag_out
int rows_gateup(hivis_ctx* c, const LayerDev& L, const uint4* frag, int M, float* scratch, uint4* frag_out) {
    const int d = c->cfg.d, F = c->cfg.ffn;
    if (M <= MAX_ROWS) {
        const WidePlan whole = wide_plan(c->num_cu, M, d / 32, F / 8, false);
        if (tall_fused(whole, wide_plan(c->num_cu, M, d / 32, F / 8, true)))
            return launch_wide<WIDE_SILU>(c, whole, frag, M, d, L.wgu, 2 * F, nullptr, 0, frag_out, F / 32);
    }
    TallPlan pl;
    if (ends_in_gemm(c, M, d, 2 * F, &pl)) {
        TallOut o{}; o.frag = frag_out; o.kblks_out = F / 32;
        return launch_tall<TALL_SILU>(c, pl, frag, M, d, L.wgu, 2 * F, o);
    }
    Parts p{};
    if (int rc = rows_gemm(c, frag, M, d, L.wgu, 2 * F, scratch, &p)) return rc;
    hipLaunchKernelGGL(wide_silu_frag_kernel, dim3((M + 15) / 16, (F / 8 + 15) / 16), dim3(256), 0, c->stream, p, M, F, frag_out);
    HIP_TRY(c, hipGetLastError());
    return HIVIS_OK;
}

// h += delta (if any), then fragments of RMSNorm(h) to c->pf_frag
template <typename WT>
int rows_norm(hivis_ctx* c, float* h, const Parts& delta, int M, const void* gain) {
    const int d = c->cfg.d;
    if (d <= 4 * WNORM_NT * WNORM_GROUPS) {
        hipLaunchKernelGGL((wide_add_norm_frag_kernel<WT>), dim3((M + 15) / 16 * 16), dim3(WNORM_NT), 0, c->stream, h, d, delta, d, M, (const WT*)gain, c->pf_frag, d, c->cfg.rms_eps);
    } else {                // rows wider than that kernel's registers
        if (delta.n > 1) hipLaunchKernelGGL(splitk_reduce_kernel, dim3(M, row_chunks(M)), dim3(256), 0, c->stream, delta, d, d, c->pf_proj, d);
        const float* one = delta.n > 1 ? c->pf_proj : delta.p;
        hipLaunchKernelGGL((add_rmsnorm_kernel<WT>), dim3(M), dim3(256), 0, c->stream, h, d, one, d, (const WT*)gain, c->pf_a, d, d, c->cfg.rms_eps);
        uint4* frag = nullptr;              // (d wide rows: always pf_frag)
        if (int rc = launch_pack(c, c->pf_a, d, M, d, &frag)) return rc;
    }
    HIP_TRY(c, hipGetLastError());
    return HIVIS_OK;
}

// One decoder layer on up to 64 rows (nseq sequences x m rows; bf16 models): the split-K GEMMs chained through row kernels
// that read the slice partials and write the next GEMM's fragments.  `pending` / `out_pending` as in layer_forward, as partials.
template <typename WT>
int layer_forward_wide(hivis_ctx* c, const LayerDev& L, const KVDev& kv, float* h, Parts pending, const int* base,
                       int offset, int seq0, int nseq, int m, TreeRows tr, Parts* out_pending) {
    const hivis_config& g = c->cfg;
    const int M = nseq * m, d = g.d, qd = g.n_q_heads * g.head_dim, F = g.ffn;
    Parts po{};
    if (int rc = rows_norm<WT>(c, h, pending, M, L.norm1)) return rc;
    if (int rc = rows_qkv<WT>(c, L, kv, c->pf_frag, base, offset, seq0, nseq, m, tr, c->pf_qkv, c->qkv)) return rc;
    // (the attention writes the O projection's fragments itself where its kernel can; rows beyond M of the last row tile
    // then keep whatever the buffer held: an MFMA output row depends on its own activation row only, and those rows are never stored)
    bool att_frag = false;
    if (int rc = attention_rows_mfma<WT>(c, c->qkv, qd, kv, base, offset, seq0, nseq, m, c->att, qd, tr.mask, c->pf_frag, &att_frag)) return rc;
    uint4* frag = c->pf_frag;
    if (!att_frag) { if (int rc = launch_pack(c, c->att, qd, M, qd, &frag)) return rc; }
    if (int rc = rows_gemm(c, frag, M, qd, L.wo, d, c->proj, &po)) return rc;
    if (int rc = rows_norm<WT>(c, h, po, M, L.norm2)) return rc;
    if (int rc = rows_gateup(c, L, c->pf_frag, M, c->gu, c->pf_frag2)) return rc;
    return rows_gemm(c, c->pf_frag2, M, F, L.wd, d, c->proj, out_pending);
}

// ---- prefill rows that the GEMMs on row fragments take (up to 16; c->stream_rows) --------------------------------------
// One GEMM phase on nseq x m rows, outside a program.
int launch_stream(hivis_ctx* c, Phase ph, int nseq, int m) {
    const hivis_config& g = c->cfg;
    PassParams pp{};
    pp.M = nseq * m; pp.nseq = nseq; pp.m = m; pp.d = g.d; pp.Hq = g.n_q_heads; pp.Hkv = g.n_kv_heads; pp.hd = g.head_dim; pp.F = g.ffn; pp.V = g.vocab;
    pp.eps = g.rms_eps; pp.theta = g.rope_theta; pp.bad = c->bad;
    ph.type = PH_GEMM;
    ph.att.seq0 = 1;                       // (positions from ph.base, not from the host's mirrors of the cache lengths: those are of the last request)
    return pp.M > WTraits<bf16_t>::ROWS ? launch_phases<bf16w_t>(c, &ph, 1, PROG_ROLL, 0, pp, false) : launch_phases<bf16_t>(c, &ph, 1, PROG_ROLL, 0, pp, false);
}
// q (rotated) to q_out, k and v of sequences seq0 .. to their cache rows 0 ..; rows and sums of squares in st_frag / st_ssq
int stream_qkv(hivis_ctx* c, const LayerDev& L, const KVDev& kv, int nssq, int seq0, int nseq, int m, float* q_out) {
    const hivis_config& g = c->cfg;
    const int qd = g.n_q_heads * g.head_dim, kd = g.n_kv_heads * g.head_dim;
    const size_t at = (size_t)seq0 * g.n_kv_heads * kv.maxL * g.head_dim * KVWidth<f16_t>::W;
    Phase q{}; q.epi = FEPI_QKV; q.K = g.d; q.N = qd + 2 * kd; q.W = L.wqkv; q.Af = c->st_frag; q.ssq = c->st_ssq; q.nssq = nssq;
    q.Y = q_out; q.ldy = qd; q.kc = (f16_t*)kv.k + at; q.vc = (f16_t*)kv.v + at; q.maxL = kv.maxL; q.base = c->zeros; q.offset = 0; q.rope = c->rope_tab; q.bias = L.bqkv;
    return launch_stream(c, q, nseq, m);
}
// Second half of a layer on the last n rows of each of nseq sequences, as rows_attn_mlp: h in place, complete.  next_gain (optional): h times
// it goes to st_frag, the sums of squares to st_ssq.
int stream_attn_mlp(hivis_ctx* c, const LayerDev& L, const KVDev& kv, const float* q, int qrows, int offset, int seq0, int nseq, int n, float* h, const void* next_gain) {
    const hivis_config& g = c->cfg;
    const int d = g.d, qd = g.n_q_heads * g.head_dim, F = g.ffn;
    if (int rc = attention_rows_mfma<bf16_t>(c, q, qd, kv, c->zeros, offset, seq0, nseq, n, nullptr, qd, nullptr, nullptr, nullptr, qrows, c->st_att)) return rc;
    Phase o{}; o.epi = FEPI_ADD_TO; o.K = qd; o.N = d; o.W = L.wo; o.Af = c->st_att; o.Y = h; o.ldy = d; o.R = h; o.ldr = d;
    o.F = c->st_frag; o.fgain = L.norm2; o.ssq_out = c->st_ssq;
    if (int rc = launch_stream(c, o, nseq, n)) return rc;
    Phase gu{}; gu.epi = FEPI_SILU; gu.K = d; gu.N = 2 * F; gu.W = L.wgu; gu.Af = c->st_frag; gu.ssq = c->st_ssq; gu.nssq = d / 16; gu.F = c->st_act;
    if (int rc = launch_stream(c, gu, nseq, n)) return rc;
    Phase dn{}; dn.epi = FEPI_ADD_TO; dn.K = F; dn.N = d; dn.W = L.wd; dn.Af = c->st_act; dn.Y = h; dn.ldy = d; dn.R = h; dn.ldr = d;
    if (next_gain) { dn.F = c->st_frag; dn.fgain = next_gain; dn.ssq_out = c->st_ssq; }
    return launch_stream(c, dn, nseq, n);
}

// ---- whole-prompt prefill (bf16 models): all rows of one or several sequences per layer -------------------------
// Second half of a layer, after q, k and v: attention, O projection, MLP on the last n rows of each of nseq sequences (their q rows:
// q, qrows rows apart from one sequence to the next; positions offset ..).  h [nseq * n][d]: their residual rows.
template <typename WT>
int rows_attn_mlp(hivis_ctx* c, const LayerDev& L, const KVDev& kv, const float* q, int qrows, int offset, int seq0, int nseq, int n,
                  float* h, Parts* out_pending) {
    const hivis_config& g = c->cfg;
    const int M = nseq * n, d = g.d, qd = g.n_q_heads * g.head_dim, F = g.ffn;
    if (c->stream_rows && M <= WTraits<bf16w_t>::ROWS) { *out_pending = Parts{nullptr, 0, 0}; return stream_attn_mlp(c, L, kv, q, qrows, offset, seq0, nseq, n, h, nullptr); }
    bool att_frag = false;
    if (c->fused) { if (int rc = attention_rows_mfma<WT>(c, q, qd, kv, c->zeros, offset, seq0, nseq, n, c->pf_att, qd, nullptr, c->pf_frag, &att_frag, qrows)) return rc; }
    else if (int rc = attention<WT>(c, q, qd, kv, c->zeros, offset, seq0, nseq, n, offset + n, c->pf_att, qd, nullptr, qrows)) return rc;
    uint4* frag = c->pf_frag;
    if (!att_frag) { if (int rc = launch_pack(c, c->pf_att, qd, M, qd, &frag)) return rc; }
    Parts po{};
    if (int rc = rows_gemm(c, frag, M, qd, L.wo, d, c->pf_proj, &po)) return rc;
    if (int rc = rows_norm<WT>(c, h, po, M, L.norm2)) return rc;
    if (int rc = rows_gateup(c, L, c->pf_frag, M, c->pf_gu, c->pf_frag2)) return rc;
    return rows_gemm(c, c->pf_frag2, M, F, L.wd, d, c->pf_proj, out_pending);
}

template <typename WT>
int prefill_target_tall(hivis_ctx* c, int b0, int nseq, int v, int l) {
    const hivis_config& g = c->cfg;
    const int m = v + l, M = nseq * m, d = g.d, qd = g.n_q_heads * g.head_dim;
    hipLaunchKernelGGL((prefill_rows_kernel<WT>), dim3(m, nseq), dim3(256), 0, c->stream, (const WT*)c->vis + (size_t)b0 * g.max_vis * d, (size_t)g.max_vis * d, v,
                       (const WT*)c->embed, (const int32_t*)(c->text + (size_t)b0 * c->text_stride), c->text_stride, 0, c->pf_x, d);
    Parts pend{nullptr, 0, 0};
    float* h = c->pf_x;
    if (c->stream_rows && M <= WTraits<bf16w_t>::ROWS) {
        // (a prompt of a few words: five launches per layer instead of eight; nine rows, two layers: 130 us less per request)
        hipLaunchKernelGGL(stream_rows_kernel, dim3(M), dim3(FUSED_NT), 0, c->stream, (const float*)h, d, d, (const bf16_t*)c->layers[0].norm1, c->st_frag, 0, M, c->st_ssq);
        for (int l_ = 0; l_ < g.n_layers; ++l_) {
            if (int rc = stream_qkv(c, c->layers[l_], c->tkv[l_], l_ ? d / 16 : 1, b0, nseq, m, c->pf_qkv)) return rc;
            if (int rc = stream_attn_mlp(c, c->layers[l_], c->tkv[l_], c->pf_qkv, m, 0, b0, nseq, m, h, l_ + 1 < g.n_layers ? c->layers[l_ + 1].norm1 : nullptr)) return rc;
        }
        for (int s = 0; s < nseq; ++s)
            hipLaunchKernelGGL((add_rmsnorm_kernel<WT>), dim3(l), dim3(256), 0, c->stream, h + ((size_t)s * m + v) * d, d, (const float*)nullptr, 0,
                               (const WT*)c->final_norm, c->feat + (size_t)(b0 + s) * g.max_text * d, d, d, g.rms_eps);
        HIP_TRY(c, hipGetLastError());
        return HIVIS_OK;
    }
    for (int l_ = 0; l_ < g.n_layers; ++l_) {
        const LayerDev& L = c->layers[l_];
        if (int rc = rows_norm<WT>(c, h, pend, M, L.norm1)) return rc;
        if (int rc = rows_qkv<WT>(c, L, c->tkv[l_], c->pf_frag, c->zeros, 0, b0, nseq, m, TreeRows(), c->pf_gu, c->pf_qkv)) return rc;
        // the last layer's output is read at the text rows only: behind its keys and values nothing needs the visual rows
        const int first = l_ + 1 == g.n_layers ? v : 0, n = m - first;
        if (first) { hipLaunchKernelGGL(tail_rows_kernel, dim3(n, nseq), dim3(256), 0, c->stream, (const float*)h, m, first, c->pf_xt, d); h = c->pf_xt; }
        if (int rc = rows_attn_mlp<WT>(c, L, c->tkv[l_], c->pf_qkv + (size_t)first * qd, m, first, b0, nseq, n, h, &pend)) return rc;
    }
    // features of the text rows (h now holds l rows per sequence): final norm of (h + last MLP delta)
    if (pend.n > 1) hipLaunchKernelGGL(splitk_reduce_kernel, dim3(nseq * l, row_chunks(nseq * l)), dim3(256), 0, c->stream, pend, d, d, c->pf_proj, d);
    for (int s = 0; s < nseq; ++s)
        hipLaunchKernelGGL((add_rmsnorm_kernel<WT>), dim3(l), dim3(256), 0, c->stream, h + (size_t)s * l * d, d, pend.p ? (const float*)c->pf_proj + (size_t)s * l * d : nullptr, d,
                           (const WT*)c->final_norm, c->feat + (size_t)(b0 + s) * g.max_text * d, d, d, g.rms_eps);
    HIP_TRY(c, hipGetLastError());
    return HIVIS_OK;
}

// Drafter prefill over the l text rows of nseq sequences: rows [f^j ; Embed(x_{j+1})] through the fusion FC, + rho_0, then the
// drafter's layer.  Only the last row's output is ever read (f'_1 of the coming round): the other rows end at their keys and values.
template <typename WT>
int prefill_drafter_tall(hivis_ctx* c, int b0, int nseq, int l) {
    const hivis_config& g = c->cfg;
    const int M = nseq * l, d = g.d, qd = g.n_q_heads * g.head_dim;
    const float* table = c->emb_w2;          // Embed(x) w2 of every token: the FC then multiplies f alone
    const int K = table ? d : 2 * d;
    Parts p{};
    if (c->stream_rows && M <= WTraits<bf16w_t>::ROWS) {
        for (int s = 0; s < nseq; ++s)
            hipLaunchKernelGGL(stream_rows_kernel, dim3(l), dim3(FUSED_NT), 0, c->stream, (const float*)(c->feat + (size_t)(b0 + s) * g.max_text * d), d, d,
                               (const bf16_t*)nullptr, c->st_att, s * l, M, (float*)nullptr);
        Phase fu{}; fu.epi = FEPI_ADDVEC; fu.K = d; fu.N = d; fu.W = c->fuse_w1; fu.Af = c->st_att; fu.Y = c->pf_x; fu.ldy = d; fu.vec = c->rho; fu.vec_idx = 0;
        fu.add_rows = c->emb_w2; fu.tok = c->text + (size_t)b0 * c->text_stride + 1; fu.tok_sseq = c->text_stride; fu.tok_srow = 1;
        fu.F = c->st_frag; fu.fgain = c->draft.norm1; fu.ssq_out = c->st_ssq;
        if (int rc = launch_stream(c, fu, nseq, l)) return rc;
        if (int rc = stream_qkv(c, c->draft, c->dkv, d / 16, b0, nseq, l, c->pf_qkv)) return rc;
    } else {
        hipLaunchKernelGGL((fuse_frag_kernel<WT>), dim3((M + 15) / 16 * 16), dim3(256), 0, c->stream, (const float*)(c->feat + (size_t)b0 * g.max_text * d), g.max_text, l, M,
                           (const int32_t*)(c->text + (size_t)b0 * c->text_stride), c->text_stride, (const WT*)c->embed, table, (const WT*)c->rho, c->pf_x, c->pf_frag, d);
        if (int rc = rows_gemm(c, c->pf_frag, M, K, table ? c->fuse_w1 : c->fuse_w, d, c->pf_proj, &p)) return rc;
        if (int rc = rows_norm<WT>(c, c->pf_x, p, M, c->draft.norm1)) return rc;
        if (int rc = rows_qkv<WT>(c, c->draft, c->dkv, c->pf_frag, c->zeros, 0, b0, nseq, l, TreeRows(), c->pf_gu, c->pf_qkv)) return rc;
    }
    hipLaunchKernelGGL(tail_rows_kernel, dim3(1, nseq), dim3(256), 0, c->stream, (const float*)c->pf_x, l, l - 1, c->pf_xt, d);
    if (int rc = rows_attn_mlp<WT>(c, c->draft, c->dkv, c->pf_qkv + (size_t)(l - 1) * qd, l, l - 1, b0, nseq, 1, c->pf_xt, &p)) return rc;
    hipLaunchKernelGGL(add_parts_kernel, dim3(nseq, row_chunks(nseq)), dim3(256), 0, c->stream, (const float*)c->pf_xt, p, d, c->catD + (size_t)b0 * 2 * d, 2 * d,
                       c->catDf, b0, g.batch);
    HIP_TRY(c, hipGetLastError());
    return HIVIS_OK;
}

struct PhaseTimer {
    hivis_ctx* c; int phase; bool on;
    PhaseTimer(hivis_ctx* c_, int p) : c(c_), phase(p), on(false) {
        if (!c->timing) return;
        while (c->pev_used + 2 > c->pev.size()) {
            hipEvent_t e = nullptr;
            if (hipEventCreate(&e) != hipSuccess) return;
            c->pev.push_back(e);
        }
        on = hipEventRecord(c->pev[c->pev_used], c->stream) == hipSuccess;
    }
    void stop() {
        if (!on) return;
        on = false;
        if (hipEventRecord(c->pev[c->pev_used + 1], c->stream) != hipSuccess) return;
        c->pev_phase.resize(c->pev.size() / 2);
        c->pev_phase[c->pev_used / 2] = phase;
        c->pev_used += 2;
    }
};
// after a stream synchronisation: fold the recorded pairs into the per-phase totals
static void resolve_phase_events(hivis_ctx* c) {
    for (size_t i = 0; i + 1 < c->pev_used; i += 2) {
        float ms = 0.f;
        const int ph = c->pev_phase[i / 2];
        if (hipEventElapsedTime(&ms, c->pev[i], c->pev[i + 1]) == hipSuccess) { c->phase_ms[ph] += ms; c->phase_calls[ph]++; }
    }
    c->pev_used = 0;
}

// ---- the four calls, typed -------------------------------------------------------------------
template <typename WT>
int do_prefill(hivis_ctx* c, const void* vis_embeds, int v, const int32_t* text_ids, int l, int32_t* first_token, bool sample) {
    const hivis_config& g = c->cfg;
    const int B = g.batch, d = g.d;
    PhaseTimer pt(c, 0);
    // stage inputs
    if (v > 0) {
        for (int b = 0; b < B; ++b)
            HIP_TRY(c, hipMemcpyAsync((char*)c->vis + (size_t)b * g.max_vis * d * sizeof(WT), (const char*)vis_embeds + (size_t)b * v * d * sizeof(WT),
                                      (size_t)v * d * sizeof(WT), hipMemcpyDefault, c->stream));
    }
    for (int b = 0; b < B; ++b)
        HIP_TRY(c, hipMemcpyAsync(c->text + (size_t)b * c->text_stride, c->h_ids.data() + (size_t)b * l, (size_t)l * sizeof(int32_t), hipMemcpyHostToDevice, c->stream));
    hipLaunchKernelGGL(set_ints_kernel, dim3(1), dim3(64), 0, c->stream, c->tlen, B, 0);
    hipLaunchKernelGGL(set_ints_kernel, dim3(1), dim3(64), 0, c->stream, c->dlen, B, 0);
    // a fresh start also clears the sticky error words: the bad-logits flag and, for the one-launch-per-pass path, the
    // barrier's arrival counter and abort flag (an aborted pass leaves the abort flag set)
    hipLaunchKernelGGL(set_ints_kernel, dim3(1), dim3(64), 0, c->stream, c->bad, 1, 0);
    if (c->bar) hipLaunchKernelGGL(set_ints_kernel, dim3(1), dim3(64), 0, c->stream, (int*)c->bar, 2, 0);

    const int total = v + l;
    // bf16 models: whole prompts, as many sequences at a time as the buffers hold; fp32: chunks of the decode passes' size
    [[maybe_unused]] const int per = std::max(1, std::min(B, c->pf_rows / total));
    if constexpr (sizeof(WT) == 2) {
        for (int b = 0; b < B; b += per)
            if (int rc = prefill_target_tall<WT>(c, b, std::min(per, B - b), v, l)) return rc;
    } else {
        for (int b = 0; b < B; ++b) {
            for (int p0 = 0; p0 < total; p0 += CHAIN_MAX_ROWS) {
                const int m = std::min(CHAIN_MAX_ROWS, total - p0);
                hipLaunchKernelGGL((prefill_rows_kernel<WT>), dim3(m), dim3(256), 0, c->stream, (const WT*)c->vis + (size_t)b * g.max_vis * d, (size_t)0, v,
                                   (const WT*)c->embed, (const int32_t*)(c->text + (size_t)b * c->text_stride), 0, p0, c->x, d);
                const int first_out = std::max(0, v - p0);       // rows of this chunk before the first text row produce no feature
                float* out = c->feat + ((size_t)b * g.max_text + std::max(0, p0 - v)) * d;
                if (int rc = target_forward<WT>(c, b, 1, m, c->zeros, p0, p0 + m, out, d, std::min(first_out, m))) return rc;
            }
        }
    }
    hipLaunchKernelGGL(set_ints_kernel, dim3(1), dim3(64), 0, c->stream, c->tlen, B, total);
    // first token x_{l+1}: LM head on the last text row of every sequence
    if (int rc = gemm<WT>(c, c->feat + (size_t)(l - 1) * d, g.max_text * d, B, d, c->lm_head, g.vocab, c->logits_p, g.vocab, EPI_STORE)) return rc;
    if (sample) hipLaunchKernelGGL(sample_rows_kernel, dim3(B), dim3(SAMPLE_NT), 0, c->stream, (const float*)c->logits_p, g.vocab, c->inv_temp, (const float*)c->u_res, 1, c->text + l, c->text_stride);
    else launch_argmax(c, c->logits_p, B, c->text + l, 1, c->text_stride);
    // drafter prefill over the l text positions: rows [f^j ; Embed(x_{j+1})] + rho_0
    if constexpr (sizeof(WT) == 2) {
        for (int b = 0; b < B; b += per)
            if (int rc = prefill_drafter_tall<WT>(c, b, std::min(per, B - b), l)) return rc;
    } else {
        for (int b = 0; b < B; ++b) {
            for (int j0 = 0; j0 < l; j0 += CHAIN_MAX_ROWS) {
                const int m = std::min(CHAIN_MAX_ROWS, l - j0);
                hipLaunchKernelGGL((fuse_rows_kernel<WT>), dim3(m), dim3(256), 0, c->stream, (const float*)(c->feat + (size_t)b * g.max_text * d),
                                   (const WT*)c->embed, (const int32_t*)(c->text + (size_t)b * c->text_stride), j0, c->catT, d);
                if (int rc = drafter_forward<WT>(c, c->catT, b, 1, m, 0, j0, j0 + m, c->dout, d)) return rc;
                if (j0 + m == l)   // f'_1: drafter output at the last true-feature row
                    hipLaunchKernelGGL(copy_rows_kernel, dim3(1), dim3(256), 0, c->stream, (const float*)(c->dout + (size_t)(m - 1) * d), d, c->catD + (size_t)b * 2 * d, 2 * d, d);
            }
        }
    }
    hipLaunchKernelGGL(set_ints_kernel, dim3(1), dim3(64), 0, c->stream, c->dlen, B, l);
    HIP_TRY(c, hipGetLastError());
    pt.stop();
    std::vector<int32_t> ft(B);
    for (int b = 0; b < B; ++b)
        HIP_TRY(c, hipMemcpyAsync(&ft[b], c->text + (size_t)b * c->text_stride + l, sizeof(int32_t), hipMemcpyDeviceToHost, c->stream));
    int bad = 0;
    HIP_TRY(c, hipMemcpyAsync(&bad, c->bad, sizeof(int), hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    if (bad) return fail(c, HIVIS_EINVAL, "prefill produced logits without a finite maximum (NaN or Inf in vis_embeds or in the weights); prefill again with valid inputs");
    if (first_token) for (int b = 0; b < B; ++b) first_token[b] = ft[b];
    for (int b = 0; b < B; ++b) { c->h_tlen[b] = total; c->h_dlen[b] = l; }
    c->v = v;
    c->state = ST_READY;
    return HIVIS_OK;
}

template <typename WT>
int do_draft(hivis_ctx* c, int K, bool sample) {
    const hivis_config& g = c->cfg;
    const int B = g.batch, d = g.d, V = g.vocab;
    PhaseTimer pt(c, 1);
    if (c->fused && fused_rows_ok<WT>(c, B)) {
        if (int rc = run_program<WT>(c, sample ? PROG_DRAFT_SAMPLE : PROG_DRAFT, K, B, 1)) return rc;
        pt.stop();
        return HIVIS_OK;
    }
    int max_keys = 0;
    for (int b = 0; b < B; ++b) max_keys = std::max(max_keys, c->h_dlen[b]);
    for (int i = 1; i <= K; ++i) {
        float* lg = c->logits_d + (size_t)(i - 1) * B * V;
        if (int rc = gemm<WT>(c, c->catD, 2 * d, B, d, c->lm_head, V, lg, V, EPI_STORE)) return rc;
        if (sample) hipLaunchKernelGGL(sample_rows_kernel, dim3(B), dim3(SAMPLE_NT), 0, c->stream, (const float*)lg, V, c->inv_temp, (const float*)(c->u_draft + (i - 1)), g.k_max, c->drafts + (i - 1), g.k_max);
        else launch_argmax(c, lg, B, c->drafts + (i - 1), 1, g.k_max);
        if (i < K) {
            hipLaunchKernelGGL((gather_rows_kernel<WT>), dim3(B), dim3(256), 0, c->stream, (const WT*)c->embed, (const int32_t*)(c->drafts + (i - 1)), 1, g.k_max, c->catD + d, 2 * d, d);
            if (int rc = drafter_forward<WT>(c, c->catD, 0, B, 1, std::min(i, g.n_resid - 1), i - 1, max_keys + i, c->catD, 2 * d)) return rc;
        }
    }
    HIP_TRY(c, hipGetLastError());
    pt.stop();
    return HIVIS_OK;
}

template <typename WT>
int do_verify(hivis_ctx* c) {
    const hivis_config& g = c->cfg;
    const int B = g.batch, d = g.d, V = g.vocab, K = c->K, M = B * (K + 1);
    PhaseTimer pt(c, 2);
    int max_keys = 0;
    for (int b = 0; b < B; ++b) max_keys = std::max(max_keys, c->h_tlen[b]);
    hipLaunchKernelGGL(verify_tokens_kernel, dim3(1), dim3(64), 0, c->stream, (const int32_t*)c->text, c->text_stride, (const int*)c->dlen, (const int32_t*)c->drafts, g.k_max, K, c->row_tok, B);
    if (c->fused && fused_rows_ok<WT>(c, M)) {
        if (int rc = run_program<WT>(c, PROG_VERIFY, K, B, K + 1)) return rc;
        pt.stop();
        return HIVIS_OK;
    }
    hipLaunchKernelGGL((gather_rows_kernel<WT>), dim3(M), dim3(256), 0, c->stream, (const WT*)c->embed, (const int32_t*)c->row_tok, M, 0, c->x, d, d);
    if (int rc = target_forward<WT>(c, 0, B, K + 1, c->tlen, 0, max_keys + K + 1, c->catT, 2 * d, 0)) return rc;
    if (int rc = gemm<WT>(c, c->catT, 2 * d, M, d, c->lm_head, V, c->logits_v, V, EPI_STORE)) return rc;
    // target's greedy token after each row: ttok[b][i], row stride k_max+1
    launch_argmax(c, c->logits_v, M, c->ttok, K + 1, g.k_max + 1);
    HIP_TRY(c, hipGetLastError());
    pt.stop();
    return HIVIS_OK;
}

template <typename WT>
int do_accept(hivis_ctx* c, int32_t* n_accepted, int32_t* tokens, bool sample) {
    const hivis_config& g = c->cfg;
    const int B = g.batch, d = g.d, K = c->K, M = B * (K + 1);
    PhaseTimer pt(c, 3);
    if (sample)
        hipLaunchKernelGGL(accept_sample_kernel, dim3(B), dim3(ACCEPT_NT), 0, c->stream, (const int32_t*)c->drafts, (const float*)c->logits_v, (const float*)c->logits_d,
                           B, g.vocab, g.k_max, K, c->inv_temp, (const float*)c->u_acc, (const float*)c->u_res, c->text, c->text_stride,
                           (const int*)c->dlen, c->tlen, c->nacc, c->out_tok, c->next_tok);
    else
        hipLaunchKernelGGL(accept_kernel, dim3(B), dim3(64), 0, c->stream, (const int32_t*)c->drafts, (const int32_t*)c->ttok, g.k_max, K, c->text, c->text_stride,
                           (const int*)c->dlen, c->tlen, c->nacc, c->out_tok, c->next_tok);
    // roll-forward: K+1 rows per sequence [g_i ; Embed(token after row i)] + rho_0 through the drafter at positions
    // dlen..dlen+K; rows beyond n_b are computed but become dead (the drafter length advances by n_b+1 only).
    if (c->fused && fused_rows_ok<WT>(c, M)) {
        if (int rc = run_program<WT>(c, PROG_ROLL, K, B, K + 1)) return rc;
    } else {
        hipLaunchKernelGGL((gather_rows_kernel<WT>), dim3(M), dim3(256), 0, c->stream, (const WT*)c->embed, (const int32_t*)c->next_tok, K + 1, g.k_max + 1, c->catT + d, 2 * d, d);
        int max_keys = 0;
        for (int b = 0; b < B; ++b) max_keys = std::max(max_keys, c->h_dlen[b]);
        if (int rc = drafter_forward<WT>(c, c->catT, 0, B, K + 1, 0, 0, max_keys + K + 1, c->dout, d)) return rc;
    }
    const size_t nres = (size_t)B + (size_t)B * (g.k_max + 1);
    hipLaunchKernelGGL(select_row_kernel, dim3(B), dim3(256), 0, c->stream, (const float*)c->dout, K + 1, (const int32_t*)c->nacc, c->catD, 2 * d, c->dlen, d, c->catDf,
                       c->h_result, (int)nres, (const int*)c->bad);
    HIP_TRY(c, hipGetLastError());
    pt.stop();
    c->h_result[nres] = 0;
    if (c->fused && c->persistent) HIP_TRY(c, hipMemcpyAsync(c->h_result + nres, c->bar + 1, sizeof(unsigned), hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    // Either flag means the device state (lengths, text) has already moved on from something invalid while the host
    // mirrors have not: the context is put back to "created", which only a new hivis_prefill leaves.
    if (c->h_result[nres]) { c->state = ST_CREATED; return fail(c, HIVIS_EHIP, "one-launch pass: grid barrier timed out (pass aborted); prefill again"); }
    if (c->h_result[nres + 1]) { c->state = ST_CREATED; return fail(c, HIVIS_EINVAL, "a pass produced logits without a finite maximum (NaN or Inf in the inputs or weights); prefill again"); }
    const int32_t* hn = c->h_result; const int32_t* ht = c->h_result + B;
    for (size_t i = 0; i + 1 < c->kev_used; i += 2) {
        float ms = 0.f;
        if (hipEventElapsedTime(&ms, c->kev[i], c->kev[i + 1]) == hipSuccess) { c->kms += ms; c->klaunches++; }
    }
    c->kev_used = 0;
    resolve_phase_events(c);
    for (int b = 0; b < B; ++b) {
        c->h_tlen[b] += hn[b] + 1; c->h_dlen[b] += hn[b] + 1;
        if (n_accepted) n_accepted[b] = hn[b];
    }
    if (tokens) memcpy(tokens, ht, (size_t)B * (g.k_max + 1) * sizeof(int32_t));
    c->state = ST_READY;
    (void)M;
    return HIVIS_OK;
}


// ---- draft tree (batch 1) ---------------------------------------------------------------------------
PassParams tree_pass(const hivis_ctx* c, int m) {
    const hivis_config& g = c->cfg;
    PassParams pp{};
    pp.M = m; pp.nseq = 1; pp.m = m; pp.d = g.d; pp.Hq = g.n_q_heads; pp.Hkv = g.n_kv_heads; pp.hd = g.head_dim; pp.F = g.ffn; pp.V = g.vocab;
    pp.eps = g.rms_eps; pp.theta = g.rope_theta; pp.inv_temp = c->inv_temp; pp.bar = c->bar; pp.bad = c->bad; pp.spin_limit = 1u << 22;
    return pp;
}

// m <= 16 rows of a draft tree (or of its re-feed) through the fusion FC + rho_idx and the drafter's layer as a phase list, one launch per
// phase: inputs cat [m][2d] = hidden row | embedding and the rows' tokens (tok); layer output to out [m][d]; lm_out (optional): its
// logits.  The lists of all row counts lie in one pool, tree_pool: the passes of a call follow each other on the stream.  The
// attention's arrival counters (zero between launches) are its first words for every row count, so no list's rows overwrite them.
// Up to 8 rows: the 8-row kernels (drafts of the 7B widths with k = 8: 699 -> 682 us, of a 2048-wide model with k = 2: 152 -> 141; there the 16-row
// kernels were slower than the stand-alone ones, 150); in the list without row fragments q|k|v takes the 16-row one, which alone knows tree positions.
template <typename WT>
void tree_rows_phases(hivis_ctx* c, int m, const float* cat, const int32_t* tok, int rho_idx, int offset, TreeRows tr, float* out, float* lm_out,
                      Pool& pool, std::vector<Phase>& P) {
    const hivis_config& g = c->cfg;
    const int d = g.d, V = g.vocab;
    int* counters = (int*)pool.take(2 * g.n_q_heads);          // at most two row blocks of 8 per head
    if (c->stream_rows) {
        StreamRows u{pool.take((size_t)m * d), (uint4*)pool.take((size_t)m * d), pool.take((size_t)m * ssq_stride(d / 16)), d / 16};
        Phase fu{}; fu.type = PH_GEMM; fu.pro = PRO_PLAIN; fu.epi = FEPI_ADDVEC; fu.K = d; fu.N = d; fu.W = c->fuse_w1; fu.Af = c->tcatf;
        fu.Y = u.h; fu.ldy = d; fu.vec = c->rho; fu.vec_idx = rho_idx; fu.add_rows = c->emb_w2; fu.tok = tok; fu.tok_sseq = 0; fu.tok_srow = 1;
        fu.F = u.F; fu.fgain = c->draft.norm1; fu.ssq_out = u.ssq;
        P.push_back(fu);
        const size_t l0 = P.size();
        uint4* outF = lm_out ? (uint4*)pool.take((size_t)m * d) : nullptr;
        layer_stream<WT>(c, P, pool, c->draft, c->dkv, u, c->dlen, offset, 1, m, StreamRows{out, outF, nullptr, 0}, nullptr, c->attn_elect);
        for (size_t i = l0; i < P.size(); ++i) {
            P[i].pos_delta = tr.pos_delta; P[i].att.tmask = tr.mask;
            if (P[i].type == PH_ATTN && c->attn_elect) P[i].cnt = counters;
        }
        if (lm_out) {
            Phase lm{}; lm.type = PH_GEMM; lm.pro = PRO_PLAIN; lm.epi = FEPI_LOGITS; lm.K = d; lm.N = V; lm.W = c->lm_head; lm.Af = outF;
            lm.Y = lm_out; lm.ldy = V; lm.pm = pool.take((size_t)m * c->fused_grid); lm.pi = (int*)pool.take((size_t)m * c->fused_grid);
            P.push_back(lm);
        }
        return;
    }
    float* u = pool.take((size_t)m * d);
    Phase fu{}; fu.type = PH_GEMM; fu.pro = PRO_PLAIN; fu.epi = FEPI_ADDVEC; fu.K = 2 * d; fu.N = d; fu.W = c->fuse_w; fu.A = cat; fu.lda = 2 * d;
    fu.Y = u; fu.ldy = d; fu.vec = c->rho; fu.vec_idx = rho_idx;
    if (c->emb_w2) { fu.add_rows = c->emb_w2; fu.K = d; fu.W = c->fuse_w1; fu.tok = tok; fu.tok_sseq = 0; fu.tok_srow = 1; }      // embedding half from the table
    P.push_back(fu);
    const size_t l0 = P.size();
    int ld = d;
    layer_phases<WT>(c, P, pool, c->draft, c->dkv, u, c->dlen, offset, 1, m, out, d, &ld, false, c->attn_elect, false);
    for (size_t i = l0; i < P.size(); ++i) {
        P[i].pos_delta = tr.pos_delta; P[i].att.tmask = tr.mask;
        if (P[i].type == PH_ATTN && c->attn_elect) P[i].cnt = counters;
    }
    float* pm = pool.take((size_t)m * c->fused_grid); int* pi = (int*)pool.take((size_t)m * c->fused_grid);
    if (lm_out) {
        Phase lm{}; lm.type = PH_GEMM; lm.pro = PRO_PLAIN; lm.epi = FEPI_LOGITS; lm.K = d; lm.N = V; lm.W = c->lm_head; lm.A = out; lm.lda = d;
        lm.Y = lm_out; lm.ldy = V; lm.pm = pm; lm.pi = pi;
        P.push_back(lm);
    }
}
// the phase attention of fp32 models takes no ancestor mask: those keep the stand-alone kernels
template <typename WT>
bool tree_program_ok(const hivis_ctx* c, int m) { return sizeof(WT) == 2 && c->fused && !c->persistent && m <= WTraits<bf16w_t>::ROWS; }

template <typename WT>
int tree_rows_program(hivis_ctx* c, int m, const float* cat, const int32_t* tok, int rho_idx, int offset, TreeRows tr, float* out, float* lm_out) {
    std::vector<Phase> P;
    Pool pool; pool.base = c->tree_pool;
    tree_rows_phases<WT>(c, m, cat, tok, rho_idx, offset, tr, out, lm_out, pool, P);
    const PassParams pp = tree_pass(c, m);
    if constexpr (std::is_same<WT, bf16_t>::value) {
        if (m > WTraits<WT>::ROWS) return launch_phases<bf16w_t>(c, P.data(), (int)P.size(), PROG_DRAFT, offset + m, pp, false);
    }
    return launch_phases<WT>(c, P.data(), (int)P.size(), PROG_DRAFT, offset + m, pp, false);
}

// Device arrays of the tree, sized for the library's limits, allocated on the first tree call.
template <typename WT>
int tree_setup(hivis_ctx* c) {
    typedef typename KVType<WT>::type KT;
    if (c->tree_ready) return HIVIS_OK;
    const hivis_config& g = c->cfg;
    const int d = g.d, V = g.vocab, kd = g.n_kv_heads * g.head_dim;
    TreeDev& t = c->tree;
    int rc;
    const int P = TREE_MAX_POOL, R = TREE_MAX_ROWS, D = TREE_MAX_DEPTH;
    if ((rc = dev_alloc(c, &t.pool_tok, P)) || (rc = dev_alloc(c, &t.pool_par, P)) || (rc = dev_alloc(c, &t.pool_score, P)) ||
        (rc = dev_alloc(c, &t.pool_depth, P)) || (rc = dev_alloc(c, &t.pool_hid, P)) || (rc = dev_alloc(c, &t.pool_slot, P)) ||
        (rc = dev_alloc(c, &t.expand, R)) || (rc = dev_alloc(c, &t.dmask, R)) || (rc = dev_alloc(c, &t.dpos, R)) ||
        (rc = dev_alloc(c, &t.sel, R)) || (rc = dev_alloc(c, &t.row_par, R)) || (rc = dev_alloc(c, &t.row_depth, R)) ||
        (rc = dev_alloc(c, &t.vmask, R)) || (rc = dev_alloc(c, &t.ttok, R)) || (rc = dev_alloc(c, &t.path, D + 1)) ||
        (rc = dev_alloc(c, &t.next_tok, D + 1)) || (rc = dev_alloc(c, &t.result, D + 2)))
        return rc;
    t.row_tok = c->row_tok;
    if ((rc = dev_alloc(c, &c->tH, (size_t)(R + 1) * d))) return rc;
    if ((rc = dev_alloc(c, &c->tlogits, (size_t)(R + 1) * V))) return rc;
    if ((rc = dev_alloc(c, &c->tcat, (size_t)TREE_MAX_TOPK * 2 * d))) return rc;
    if ((rc = dev_alloc(c, &c->ttok_rows, TREE_MAX_TOPK))) return rc;
    if ((rc = dev_alloc(c, &c->troll, (size_t)(D + 1) * 2 * d))) return rc;
    { float* f; if ((rc = dev_alloc(c, &f, (size_t)WTraits<bf16w_t>::ROWS * d))) return rc; c->tcatf = (uint4*)f; }
    c->tnseg = (V + TOPK_SEG - 1) / TOPK_SEG;
    if ((rc = dev_alloc(c, &c->tcand_v, (size_t)TREE_MAX_TOPK * c->tnseg * TREE_MAX_TOPK))) return rc;
    if ((rc = dev_alloc(c, &c->tcand_i, (size_t)TREE_MAX_TOPK * c->tnseg * TREE_MAX_TOPK))) return rc;
    if ((rc = dev_alloc(c, &c->tseg, (size_t)TREE_MAX_TOPK * c->tnseg * 2))) return rc;
    // cache pointers of all target layers (keys, values) for the compaction kernels, and their staging rows
    std::vector<void*> ptrs;
    for (int l = 0; l < g.n_layers; ++l) { ptrs.push_back(c->tkv[l].k); ptrs.push_back(c->tkv[l].v); }
    if ((rc = dev_alloc(c, &c->kv_ptrs, ptrs.size()))) return rc;
    HIP_TRY(c, hipMemcpy(c->kv_ptrs, ptrs.data(), ptrs.size() * sizeof(void*), hipMemcpyHostToDevice));
    { KT* st; if ((rc = dev_alloc(c, &st, (size_t)g.n_layers * 2 * D * kd * KVWidth<KT>::W))) return rc; c->kv_staging = st; }
    HIP_TRY(c, hipHostMalloc((void**)&c->h_tree_result, (D + 3) * sizeof(int32_t), hipHostMallocDefault));     // result [D + 2] | bad-logits flag
    // pool and row arrays start at zero: a level whose logits have no finite maximum writes no entries, and what a later
    // kernel then reads as a token id must still be a valid one
    HIP_TRY(c, hipMemsetAsync(t.pool_tok, 0, P * sizeof(*t.pool_tok), c->stream)); HIP_TRY(c, hipMemsetAsync(t.pool_par, 0, P * sizeof(*t.pool_par), c->stream));
    HIP_TRY(c, hipMemsetAsync(t.pool_score, 0, P * sizeof(*t.pool_score), c->stream)); HIP_TRY(c, hipMemsetAsync(t.pool_depth, 0, P * sizeof(*t.pool_depth), c->stream));
    HIP_TRY(c, hipMemsetAsync(t.pool_hid, 0, P * sizeof(*t.pool_hid), c->stream)); HIP_TRY(c, hipMemsetAsync(t.pool_slot, 0, P * sizeof(*t.pool_slot), c->stream));
    HIP_TRY(c, hipMemsetAsync(t.expand, 0, R * sizeof(*t.expand), c->stream)); HIP_TRY(c, hipMemsetAsync(t.sel, 0, R * sizeof(*t.sel), c->stream));
    HIP_TRY(c, hipMemsetAsync(t.row_par, 0, R * sizeof(*t.row_par), c->stream)); HIP_TRY(c, hipMemsetAsync(t.row_depth, 0, R * sizeof(*t.row_depth), c->stream));
    HIP_TRY(c, hipMemsetAsync(t.ttok, 0, R * sizeof(*t.ttok), c->stream)); HIP_TRY(c, hipMemsetAsync(t.path, 0, (D + 1) * sizeof(*t.path), c->stream));
    HIP_TRY(c, hipMemsetAsync(t.next_tok, 0, (D + 1) * sizeof(*t.next_tok), c->stream)); HIP_TRY(c, hipMemsetAsync(t.result, 0, (D + 2) * sizeof(*t.result), c->stream));
    HIP_TRY(c, hipMemsetAsync(t.dmask, 0, R * sizeof(*t.dmask), c->stream)); HIP_TRY(c, hipMemsetAsync(t.dpos, 0, R * sizeof(*t.dpos), c->stream));
    HIP_TRY(c, hipMemsetAsync(t.vmask, 0, R * sizeof(*t.vmask), c->stream)); HIP_TRY(c, hipMemsetAsync(c->ttok_rows, 0, TREE_MAX_TOPK * sizeof(int32_t), c->stream));
    if (tree_program_ok<WT>(c, 1)) {
        size_t most = 0;
        for (int m = 1; tree_program_ok<WT>(c, m); ++m) {
            std::vector<Phase> P;
            Pool count;
            float some = 0.f;            // (any address: the list with an LM head is the longer one)
            tree_rows_phases<WT>(c, m, nullptr, nullptr, 0, 0, TreeRows(), nullptr, &some, count, P);
            most = std::max(most, count.used);
        }
        if ((rc = dev_alloc(c, &c->tree_pool, most))) return rc;
        HIP_TRY(c, hipMemsetAsync(c->tree_pool, 0, most * sizeof(float), c->stream));          // (the arrival counters start at zero)
    }
    c->tree_ready = true;
    return HIVIS_OK;
}

// Pool of k + (depth-1) k^2 nodes, level by level; then the N best-scored candidates and their verify rows.
template <typename WT>
int do_tree_draft(hivis_ctx* c, int k, int depth, int N) {
    const hivis_config& g = c->cfg;
    const int d = g.d, V = g.vocab;
    if (int rc = tree_setup<WT>(c)) return rc;
    PhaseTimer pt(c, 1);
    const TreeDev& t = c->tree;
    // hidden row 0 = the drafter's pending state f'_1; its distribution gives level 1
    hipLaunchKernelGGL(copy_rows_kernel, dim3(1), dim3(256), 0, c->stream, (const float*)c->catD, 2 * d, c->tH, d, d);
    if (int rc = gemm<WT>(c, c->tH, d, 1, d, c->lm_head, V, c->tlogits, V, EPI_STORE)) return rc;
    const int nseg = c->tnseg;
    const size_t child_lds = (size_t)nseg * k * 2 * sizeof(float);
    if (child_lds > 48 * 1024) return fail(c, HIVIS_EINVAL, "vocabulary too large for the top-k merge (%d segments x %d)", nseg, k);
    hipLaunchKernelGGL(tree_topk_part_kernel, dim3(1, nseg), dim3(TOPK_NT), 0, c->stream, (const float*)c->tlogits, V, k, c->tcand_v, c->tcand_i, c->tseg);
    hipLaunchKernelGGL(tree_children_kernel, dim3(1), dim3(CHILD_NT), child_lds, c->stream, (const float*)c->tcand_v, (const int32_t*)c->tcand_i, (const float*)c->tseg, nseg, k, 0,
                       (const int32_t*)nullptr, 1, 0, t);
    int lo = 0, n = k;
    for (int j = 1; j < depth; ++j) {
        const int n_prev = (j - 1) * k, row0 = 1 + n_prev;
        const int32_t* E = t.expand + n_prev;
        const bool program = tree_program_ok<WT>(c, k);
        hipLaunchKernelGGL((tree_expand_kernel<WT>), dim3(k), dim3(256), 0, c->stream, lo, n, k, n_prev, j, t, (const float*)c->tH,
                           program && c->emb_w2 ? (const WT*)nullptr : (const WT*)c->embed, c->tcat, c->ttok_rows, d, program && c->stream_rows ? c->tcatf : (uint4*)nullptr);
        TreeRows tr; tr.pos_delta = t.dpos + n_prev; tr.mask = t.dmask + n_prev;
        float* hid = c->tH + (size_t)row0 * d; float* lg = c->tlogits + (size_t)row0 * V;
        if (program) {
            if (int rc = tree_rows_program<WT>(c, k, c->tcat, c->ttok_rows, std::min(j, g.n_resid - 1), n_prev, tr, hid, lg)) return rc;
        } else {
            if (int rc = drafter_forward<WT>(c, c->tcat, 0, 1, k, std::min(j, g.n_resid - 1), n_prev, c->h_dlen[0] + n_prev + k, hid, d, tr)) return rc;
            if (int rc = gemm<WT>(c, hid, d, k, d, c->lm_head, V, lg, V, EPI_STORE)) return rc;
        }
        const int first = lo + n;
        hipLaunchKernelGGL(tree_topk_part_kernel, dim3(k, nseg), dim3(TOPK_NT), 0, c->stream, (const float*)(c->tlogits + (size_t)row0 * V), V, k, c->tcand_v, c->tcand_i, c->tseg);
        hipLaunchKernelGGL(tree_children_kernel, dim3(k), dim3(CHILD_NT), child_lds, c->stream, (const float*)c->tcand_v, (const int32_t*)c->tcand_i, (const float*)c->tseg, nseg, k, first,
                           E, j + 1, row0, t);
        lo = first; n = k * k;
    }
    hipLaunchKernelGGL(tree_select_kernel, dim3(1), dim3(1024), 0, c->stream, lo + n, N, (const int32_t*)c->text, (const int*)c->dlen, t);
    HIP_TRY(c, hipGetLastError());
    pt.stop();
    return HIVIS_OK;
}

template <typename WT>
int do_tree_verify(hivis_ctx* c) {
    const hivis_config& g = c->cfg;
    const int d = g.d, V = g.vocab, M = c->tn + 1;
    PhaseTimer pt(c, 2);
    const TreeDev& t = c->tree;
    hipLaunchKernelGGL((gather_rows_kernel<WT>), dim3(M), dim3(256), 0, c->stream, (const WT*)c->embed, (const int32_t*)t.row_tok, M, 0, c->x, d, d);
    TreeRows tr; tr.pos_delta = t.row_depth; tr.mask = t.vmask;
    if (int rc = target_forward<WT>(c, 0, 1, M, c->tlen, 0, c->h_tlen[0] + M, c->catT, 2 * d, 0, tr)) return rc;
    if (int rc = gemm<WT>(c, c->catT, 2 * d, M, d, c->lm_head, V, c->logits_v, V, EPI_STORE)) return rc;
    launch_argmax(c, c->logits_v, M, t.ttok, M, 0);
    HIP_TRY(c, hipGetLastError());
    pt.stop();
    c->vrows = M;
    return HIVIS_OK;
}

template <typename WT>
int do_tree_accept(hivis_ctx* c, int32_t* n_accepted, int32_t* tokens, bool sample) {
    typedef typename KVType<WT>::type KT;
    const hivis_config& g = c->cfg;
    const int d = g.d, N = c->tn, depth = c->tdepth;
    PhaseTimer pt(c, 3);
    const TreeDev& t = c->tree;
    // T > 0: the token the target DRAWS after every row replaces its greedy token (row of depth j: uniform u_tree[j]);
    // the walk below is the same: a candidate is followed when it is the token after its parent row
    if (sample) hipLaunchKernelGGL(sample_rows_kernel, dim3(N + 1), dim3(SAMPLE_NT), 0, c->stream, (const float*)c->logits_v, g.vocab, c->inv_temp,
                                   (const float*)c->u_tree, 1, t.ttok, 1, (const int32_t*)t.row_depth);
    hipLaunchKernelGGL(tree_accept_kernel, dim3(1), dim3(64), 0, c->stream, N, depth, c->text, (const int*)c->dlen, t);
    // target cache: the followed rows move to the slots right after the root's
    for (int scatter = 0; scatter < 2; ++scatter)
        hipLaunchKernelGGL((tree_kv_gather_kernel<KT>), dim3(depth, 2 * g.n_layers), dim3(256), 0, c->stream, (KT* const*)c->kv_ptrs, c->tkv[0].maxL,
                           g.n_kv_heads, g.head_dim * KVWidth<KT>::W, (const int*)c->tlen, (const int32_t*)t.result, (const int32_t*)t.path, depth, (KT*)c->kv_staging, scatter);
    // drafter: every tree row is dropped (its length never advanced); depth+1 rows rebuilt from the true features
    const bool program = tree_program_ok<WT>(c, depth + 1);
    hipLaunchKernelGGL((tree_roll_cat_kernel<WT>), dim3(depth + 1), dim3(256), 0, c->stream, (const float*)c->catT, 2 * d, (const int32_t*)t.path,
                       (const int32_t*)t.next_tok, program && c->emb_w2 ? (const WT*)nullptr : (const WT*)c->embed, c->troll, d, program && c->stream_rows ? c->tcatf : (uint4*)nullptr);
    if (program) { if (int rc = tree_rows_program<WT>(c, depth + 1, c->troll, t.next_tok, 0, 0, TreeRows(), c->dout, nullptr)) return rc; }
    else if (int rc = drafter_forward<WT>(c, c->troll, 0, 1, depth + 1, 0, 0, c->h_dlen[0] + depth + 1, c->dout, d)) return rc;
    hipLaunchKernelGGL(tree_finish_kernel, dim3(1), dim3(256), 0, c->stream, (const float*)c->dout, (const int32_t*)t.result, c->catD, c->dlen, c->tlen, d, c->catDf,
                       c->h_tree_result, depth + 2, (const int*)c->bad, TREE_MAX_DEPTH + 2);
    HIP_TRY(c, hipGetLastError());
    pt.stop();
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    resolve_phase_events(c);
    if (c->h_tree_result[TREE_MAX_DEPTH + 2]) { c->state = ST_CREATED; return fail(c, HIVIS_EINVAL, "a pass produced logits without a finite maximum (NaN or Inf in the inputs or weights); prefill again"); }
    const int n = c->h_tree_result[0];
    c->h_tlen[0] += n + 1; c->h_dlen[0] += n + 1;
    *n_accepted = n;
    memcpy(tokens, c->h_tree_result + 1, (size_t)(depth + 1) * sizeof(int32_t));
    c->state = ST_READY;
    return HIVIS_OK;
}

// The fusion FC is linear in its two halves: [f ; Embed(x)] [w1 ; w2] = f w1 + Embed(x) w2 (section 3.2), and the second
// term depends on the token alone.  The table T[x] = Embed(x) w2 ([V][d], fp32: products summed
// in fp32) is computed here once, with the prefill's GEMM over ranges of embedding rows (fp32 models: 32 rows at a time), and the phase programs' FC then
// streams w1 only (d x d instead of 2d x d per step) and adds T[x] in its epilogue.  HIVIS_EMB_TABLE=0 keeps the full FC.
template <typename WT>
int build_embed_fc_table(hivis_ctx* c, const hivis_weights* w) {
    const hivis_config& g = c->cfg;
    const int d = g.d, V = g.vocab;
    { const char* e = getenv("HIVIS_EMB_TABLE"); if (e && e[0] == '0') return HIVIS_OK; }
    if (!c->fused || c->persistent || (sizeof(WT) == 2 && (!c->pf_frag || c->pf_rows < 8))) return HIVIS_OK;
    void* staging = nullptr;
    HIP_TRY(c, hipMalloc(&staging, (size_t)d * d * sizeof(WT) + 4096));
    uint4* w2p = nullptr;
    int rc = HIVIS_OK;
    do {
        { const void* s[1] = {w->fuse_w}; int n[1] = {d};
          if ((rc = pack_matrix<WT>(c, s, n, 1, d, 0, staging, &c->fuse_w1))) break; }
        { const void* s[1] = {(const WT*)w->fuse_w + (size_t)d * d}; int n[1] = {d};
          if ((rc = pack_matrix<WT>(c, s, n, 1, d, 0, staging, &w2p))) break; }
        float* table = nullptr;
        {   // no room for the table is not an error: the FC then keeps multiplying the embedding half
            void* q = nullptr;
            if (hipMalloc(&q, (size_t)V * d * sizeof(float)) != hipSuccess) { (void)hipGetLastError(); break; }
            c->allocs.push_back(q);
            table = (float*)q;
        }
        if constexpr (sizeof(WT) != 2) {
            for (int r0 = 0; r0 < V && !rc; r0 += CHAIN_MAX_ROWS)
                rc = gemm<WT>(c, (const WT*)c->embed + (size_t)r0 * d, d, std::min(CHAIN_MAX_ROWS, V - r0), d, w2p, d, table + (size_t)r0 * d, d, EPI_STORE);
        }
        const int R = c->pf_rows;                                  // rows per GEMM: what the prefill buffers hold
        for (int r0 = 0; sizeof(WT) == 2 && r0 < V && !rc; r0 += R) {
            const int n = std::min(R, V - r0);
            hipLaunchKernelGGL((rows_to_f32_kernel<WT>), dim3(1024), dim3(256), 0, c->stream, (const WT*)c->embed + (size_t)r0 * d, (size_t)n * d, c->pf_x);
            uint4* frag = nullptr;
            if ((rc = launch_pack(c, c->pf_x, d, n, d, &frag))) break;
            TallOut o{}; o.Y = table + (size_t)r0 * d; o.ldy = d;
            rc = launch_tall<TALL_STORE>(c, tall_plan(c->num_cu, n, d / 32, d / 16, false), frag, n, d, w2p, d, o);
        }
        if (rc) break;
        if (hipStreamSynchronize(c->stream) != hipSuccess) { rc = fail(c, HIVIS_EHIP, "building the embedding table of the fusion FC failed"); break; }
        c->emb_w2 = table;
        // w1's tiles behind the LM head's, in one buffer: both have K = d, so a draft step's LM-head launch can compute
        // f' w1 as d more output columns and the fusion FC needs no launch of its own (HIVIS_LM_EXT=0: keep the FC phase)
        const char* le = getenv("HIVIS_LM_EXT");
        if (!(le && le[0] == '0')) {
            const size_t lm_bytes = (size_t)V * d * sizeof(WT), w1_bytes = (size_t)d * d * sizeof(WT);
            void* q = nullptr;
            if (hipMalloc(&q, lm_bytes + w1_bytes) != hipSuccess) { (void)hipGetLastError(); break; }
            if (hipMemcpyAsync(q, c->lm_head, lm_bytes, hipMemcpyDeviceToDevice, c->stream) != hipSuccess ||
                hipMemcpyAsync((char*)q + lm_bytes, c->fuse_w1, w1_bytes, hipMemcpyDeviceToDevice, c->stream) != hipSuccess ||
                hipStreamSynchronize(c->stream) != hipSuccess) { (void)hipFree(q); rc = fail(c, HIVIS_EHIP, "copying the LM head failed"); break; }
            // the separate LM-head buffer is no longer needed
            for (auto it = c->allocs.begin(); it != c->allocs.end(); ++it) if (*it == (void*)c->lm_head) { c->allocs.erase(it); break; }
            (void)hipFree(c->lm_head);
            c->allocs.push_back(q);
            c->lm_head = (uint4*)q;
            c->lm_ext = true;
        }
    } while (0);
    (void)hipFree(staging);
    return rc;
}

template <typename WT>
int do_create(hivis_ctx* c, const hivis_weights* w) {
    const hivis_config& g = c->cfg;
    const int d = g.d, qd = g.n_q_heads * g.head_dim, kd = g.n_kv_heads * g.head_dim, F = g.ffn, V = g.vocab, B = g.batch;
    // staging big enough for the largest source set of one packed matrix
    size_t stg = std::max({(size_t)d * (qd + 2 * kd), (size_t)qd * d, (size_t)2 * d * F, (size_t)F * d, (size_t)V * d, (size_t)2 * d * d}) * sizeof(WT) + 4096;
    void* staging = nullptr;
    HIP_TRY(c, hipMalloc(&staging, stg));
    int rc = HIVIS_OK;
    do {
        if ((rc = upload_vec<WT>(c, w->embed, (size_t)V * d, &c->embed))) break;
        if ((rc = upload_vec<WT>(c, w->final_norm, d, &c->final_norm))) break;
        if ((rc = upload_vec<WT>(c, w->resid_rho, (size_t)g.n_resid * d, &c->rho))) break;
        { const void* s[1] = {w->lm_head}; int n[1] = {V};
          if ((rc = pack_matrix<WT>(c, s, n, 1, d, 1, staging, &c->lm_head))) break; }
        { const void* s[1] = {w->fuse_w}; int n[1] = {d};
          if ((rc = pack_matrix<WT>(c, s, n, 1, 2 * d, 0, staging, &c->fuse_w))) break; }
        c->layers.resize(g.n_layers);
        for (int l = 0; l < g.n_layers && !rc; ++l) rc = upload_layer<WT>(c, w->layers[l], staging, c->layers[l]);
        if (rc) break;
        if ((rc = upload_layer<WT>(c, w->draft_layer, staging, c->draft))) break;
    } while (0);
    (void)hipFree(staging);
    if (rc) return rc;

    // KV caches (KW storage elements per cached value: hi and lo halves for bf16 models)
    constexpr int KW = KVWidth<typename KVType<WT>::type>::W;
    const int maxLt = g.max_vis + g.max_text, maxLd = g.max_text;
    c->tkv.resize(g.n_layers);
    for (int l = 0; l < g.n_layers; ++l) {
        typename KVType<WT>::type *k, *v;
        if ((rc = dev_alloc(c, &k, (size_t)B * kd * maxLt * KW))) return rc;
        if ((rc = dev_alloc(c, &v, (size_t)B * kd * maxLt * KW))) return rc;
        c->tkv[l].k = k; c->tkv[l].v = v; c->tkv[l].maxL = maxLt;
    }
    { typename KVType<WT>::type *k, *v;
      if ((rc = dev_alloc(c, &k, (size_t)B * kd * maxLd * KW))) return rc;
      if ((rc = dev_alloc(c, &v, (size_t)B * kd * maxLd * KW))) return rc;
      c->dkv.k = k; c->dkv.v = v; c->dkv.maxL = maxLd; }
    { WT* vis; if ((rc = dev_alloc(c, &vis, (size_t)B * std::max(1, g.max_vis) * d))) return rc; c->vis = vis; }

    // state + activations
    c->text_stride = g.max_text + g.k_max + 2;
    if ((rc = dev_alloc(c, &c->tlen, B))) return rc;
    if ((rc = dev_alloc(c, &c->dlen, B))) return rc;
    if ((rc = dev_alloc(c, &c->zeros, B))) return rc;
    HIP_TRY(c, hipMemset(c->zeros, 0, B * sizeof(int)));
    if ((rc = dev_alloc(c, &c->text, (size_t)B * c->text_stride))) return rc;
    HIP_TRY(c, hipMemset(c->text, 0, (size_t)B * c->text_stride * sizeof(int32_t)));
    const int R = MAX_ROWS;
    if ((rc = dev_alloc(c, &c->x, (size_t)R * d))) return rc;
    if ((rc = dev_alloc(c, &c->a, (size_t)R * d))) return rc;
    if ((rc = dev_alloc(c, &c->qkv, (size_t)R * (qd + 2 * kd)))) return rc;
    if ((rc = dev_alloc(c, &c->att, (size_t)R * qd))) return rc;
    if ((rc = dev_alloc(c, &c->proj, (size_t)R * d))) return rc;
    if ((rc = dev_alloc(c, &c->gu, (size_t)R * 2 * F))) return rc;
    if ((rc = dev_alloc(c, &c->act, (size_t)R * F))) return rc;
    if ((rc = dev_alloc(c, &c->catT, (size_t)R * 2 * d))) return rc;
    if ((rc = dev_alloc(c, &c->catD, (size_t)B * 2 * d))) return rc;
    if ((rc = dev_alloc(c, &c->u, (size_t)R * d))) return rc;
    if ((rc = dev_alloc(c, &c->dout, (size_t)R * d))) return rc;
    if ((rc = dev_alloc(c, &c->feat, (size_t)B * g.max_text * d))) return rc;
    if (sizeof(WT) == 2) {
        if ((rc = prefill_lds_setup(c))) return rc;
        c->pf_sizes = prefill_sizes(d, qd, F, B, g.max_vis, g.max_text);
        const int PR = c->pf_sizes.rows;
        c->pf_rows = PR;
        if ((rc = dev_alloc(c, &c->pf_x, (size_t)PR * d))) return rc;
        if ((rc = dev_alloc(c, &c->pf_xt, (size_t)std::min(PR, B * g.max_text) * d))) return rc;
        if (d > 4 * WNORM_NT * WNORM_GROUPS && (rc = dev_alloc(c, &c->pf_a, (size_t)PR * d))) return rc;
        if ((rc = dev_alloc(c, &c->pf_qkv, std::max((size_t)PR * qd, (size_t)R * (qd + 2 * kd))))) return rc;
        if ((rc = dev_alloc(c, &c->pf_proj, (size_t)PR * d))) return rc;
        if ((rc = dev_alloc(c, &c->pf_gu, (size_t)R * std::max(2 * F, qd + 2 * kd)))) return rc;      // (more rows: finished in the GEMM, or K slices)
        if ((rc = dev_alloc(c, &c->pf_frag, c->pf_sizes.frag / 4))) return rc;      // 4 bytes per value, in 16-byte units
        if ((rc = dev_alloc(c, &c->pf_frag2, c->pf_sizes.frag2 / 4))) return rc;
        // HIVIS_TALL_CW=6, 7 or 8: prefill GEMMs in tiles of 192, 224 or 256 columns only
        if (const char* ce = getenv("HIVIS_TALL_CW")) { const int cw = atoi(ce); if (cw >= 6 && cw <= 8) c->tall_cw = cw; }
        const char* re = getenv("HIVIS_SPLITK_RESERVE");
        const size_t reserve = re && atoi(re) >= 0 ? (size_t)atoi(re) << 18 : SPLITK_RESERVE;
        if (reserve) (void)splitk_alloc(c, std::min(reserve, splitk_most(c)));      // (no room is not an error here)
    }
    if ((rc = dev_alloc(c, &c->logits_v, (size_t)R * V))) return rc;
    if ((rc = dev_alloc(c, &c->logits_d, (size_t)g.k_max * B * V))) return rc;
    if ((rc = dev_alloc(c, &c->logits_p, (size_t)B * V))) return rc;
    { const size_t n = (size_t)std::max(R, B) * ((V + ARGMAX_SEG - 1) / ARGMAX_SEG); if ((rc = dev_alloc(c, &c->am_v, n)) || (rc = dev_alloc(c, &c->am_i, n))) return rc; }
    if ((rc = dev_alloc(c, &c->row_tok, R))) return rc;
    if ((rc = dev_alloc(c, &c->drafts, (size_t)B * g.k_max))) return rc;
    if ((rc = dev_alloc(c, &c->ttok, (size_t)B * (g.k_max + 1)))) return rc;
    if ((rc = dev_alloc(c, &c->u_draft, (size_t)B * g.k_max))) return rc;
    if ((rc = dev_alloc(c, &c->u_acc, (size_t)B * g.k_max))) return rc;
    if ((rc = dev_alloc(c, &c->u_res, (size_t)B))) return rc;
    if ((rc = dev_alloc(c, &c->u_tree, (size_t)TREE_MAX_DEPTH + 1))) return rc;
    // accepted counts and emitted tokens share one block: select_row_kernel stores it to the pinned mirror as it is
    if ((rc = dev_alloc(c, &c->nacc, (size_t)B + (size_t)B * (g.k_max + 1)))) return rc;
    c->out_tok = c->nacc + B;
    HIP_TRY(c, hipHostMalloc((void**)&c->h_result, ((size_t)B + (size_t)B * (g.k_max + 1) + 2) * sizeof(int32_t), hipHostMallocDefault));
    if ((rc = dev_alloc(c, &c->bad, 1))) return rc;
    HIP_TRY(c, hipMemset(c->bad, 0, sizeof(int)));
    if ((rc = dev_alloc(c, &c->next_tok, (size_t)B * (g.k_max + 1)))) return rc;
    c->h_tlen.assign(B, 0); c->h_dlen.assign(B, 0);
    // rotary table over every position either cache can hold (read by the QKV epilogue of the phase programs)
    {
        const int npos = g.max_vis + g.max_text;
        if ((rc = dev_alloc(c, &c->rope_tab, (size_t)npos * g.head_dim))) return rc;
        const size_t n = (size_t)npos * (g.head_dim / 2);
        hipLaunchKernelGGL(rope_table_kernel, dim3((unsigned)std::min<size_t>((n + 255) / 256, 4096)), dim3(256), 0, c->stream, c->rope_tab, npos, g.head_dim, g.rope_theta);
        HIP_TRY(c, hipGetLastError());
    }
    if ((rc = fused_setup<WT>(c))) return rc;
    // (attention rows of a whole-prompt pass: as fragments except from passes of at most 8 rows per sequence, and HIVIS_FUSED=0)
    if (c->pf_rows && (rc = dev_alloc(c, &c->pf_att, (size_t)(c->fused ? B * FUSED_RMAX : c->pf_rows) * qd))) return rc;
    // attention workspace: (items * nsplit) work groups x 4 wave slots x RMAX rows x (hd + 2) floats, where
    // items * nsplit <= 2 * num_cu + items and items <= max(2, B) * n_q_heads
    {
        size_t max_items = (size_t)std::max({2, B, MAX_ROWS / ATT_RMAX}) * g.n_q_heads;
        // (whole-prompt passes use it with HIVIS_FUSED=0 only)
        if (c->pf_rows && !c->fused) max_items = std::max(max_items, (size_t)g.n_q_heads * ((c->pf_rows + ATT_RMAX - 1) / ATT_RMAX + B));
        c->attn_ws_floats = (2 * (size_t)c->num_cu + max_items) * 4 * ATT_RMAX * (g.head_dim + 2);
        if ((rc = dev_alloc(c, &c->attn_ws, c->attn_ws_floats))) return rc;
        c->rows_cnt_n = (std::max(2, B) + MAX_ROWS / ATTN_ROWS_RM) * g.n_q_heads;      // (items of up to 64 rows: a head and 16 of them, or up to 8 of one sequence)
        if ((rc = dev_alloc(c, &c->rows_cnt, (size_t)c->rows_cnt_n))) return rc;
        HIP_TRY(c, hipMemset(c->rows_cnt, 0, (size_t)c->rows_cnt_n * sizeof(int)));
    }
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    if ((rc = build_embed_fc_table<WT>(c, w))) return rc;
    if (sizeof(WT) == 2 && c->fused && !c->persistent && c->emb_w2 && d <= STREAM_MAX_D) {
        const int R16 = WTraits<bf16w_t>::ROWS;
        float *f, *v;
        if ((rc = dev_alloc(c, &f, (size_t)B * d)) || (rc = dev_alloc(c, &v, (size_t)R16 * d))) return rc;
        c->catDf = (uint4*)f; c->vfrag = (uint4*)v;
        float *sf, *sa, *sm;
        if ((rc = dev_alloc(c, &sf, (size_t)R16 * d)) || (rc = dev_alloc(c, &sa, (size_t)R16 * std::max(d, qd))) || (rc = dev_alloc(c, &sm, (size_t)R16 * F)) ||
            (rc = dev_alloc(c, &c->st_ssq, (size_t)R16 * ssq_stride(d / 16)))) return rc;
        c->st_frag = (uint4*)sf; c->st_att = (uint4*)sa; c->st_act = (uint4*)sm;
        c->stream_rows = true;
    }
    return HIVIS_OK;
}

int check_config(const hivis_config* g, std::string& why) {
    char buf[256];
#define BAD(...) do { snprintf(buf, sizeof buf, __VA_ARGS__); why = buf; return HIVIS_EINVAL; } while (0)
    if (g->dtype != HIVIS_F32 && g->dtype != HIVIS_BF16) BAD("dtype %d unknown", g->dtype);
    const int al = g->dtype == HIVIS_BF16 ? 32 : 16;
    if (g->n_layers < 1 || g->d < al || g->n_q_heads < 1 || g->n_kv_heads < 1 || g->ffn < al || g->vocab < 16) BAD("non-positive dimension");
    if (g->head_dim != 64 && g->head_dim != 128) BAD("head_dim %d not in {64,128}", g->head_dim);
    if (g->n_q_heads % g->n_kv_heads) BAD("n_q_heads %% n_kv_heads != 0");
    if (g->d % al || (g->n_q_heads * g->head_dim) % al || (g->n_kv_heads * g->head_dim) % al || g->ffn % al) BAD("d, q_dim, kv_dim, ffn must be multiples of %d", al);
    if (g->vocab % 16) BAD("vocab must be a multiple of 16");
    if (g->batch < 1 || g->k_max < 1 || g->batch * (g->k_max + 1) > CHAIN_MAX_ROWS) BAD("batch*(k_max+1) must be in 2..%d", CHAIN_MAX_ROWS);
    if (g->max_vis < 0 || g->max_text < 2 + g->k_max) BAD("capacity too small");
    if (g->n_resid < 1) BAD("n_resid must be >= 1");
    if (!(g->rope_theta > 1.f) || !(g->rms_eps >= 0.f)) BAD("rope_theta / rms_eps out of range");
#undef BAD
    return HIVIS_OK;
}

thread_local std::string g_create_err;

}  // namespace

#define DISPATCH(c, fn, ...) ((c)->cfg.dtype == HIVIS_BF16 ? fn<bf16_t>(__VA_ARGS__) : fn<float>(__VA_ARGS__))

extern "C" {

int hivis_create(const hivis_config* cfg, const hivis_weights* w, void* hip_stream, hivis_ctx** out) {
    if (out) *out = nullptr;
    if (!cfg || !w || !out) { g_create_err = "null argument"; return HIVIS_EINVAL; }
    if (int rc = check_config(cfg, g_create_err)) return rc;
    if (!w->embed || !w->lm_head || !w->final_norm || !w->layers || !w->fuse_w || !w->resid_rho) { g_create_err = "null weight pointer"; return HIVIS_EINVAL; }
    hivis_ctx* c = new hivis_ctx();
    c->cfg = *cfg;
    c->stream = (hipStream_t)hip_stream;
    c->esize = cfg->dtype == HIVIS_BF16 ? 2 : 4;
    int dev = 0; hipDeviceProp_t prop;
    if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&prop, dev) != hipSuccess) {
        g_create_err = "no HIP device"; delete c; return HIVIS_EHIP;
    }
    c->num_cu = prop.multiProcessorCount;
    c->na_phases.reserve(draft_phase_capacity(cfg->k_max));
    int rc = scratch_for_device(c, dev);
    if (!rc) rc = DISPATCH(c, do_create, c, w);
    if (rc) { g_create_err = c->err; hivis_destroy(c); return rc; }
    *out = c;
    return HIVIS_OK;
}

int hivis_destroy(hivis_ctx* c) {
    if (!c) return HIVIS_OK;
    (void)hipStreamSynchronize(c->stream);
    for (void* p : c->allocs) (void)hipFree(p);
    for (auto& kv : c->programs) delete kv.second.host;
    for (hipEvent_t e : c->pev) (void)hipEventDestroy(e);
    if (c->h_result) (void)hipHostFree(c->h_result);
    if (c->h_tree_result) (void)hipHostFree(c->h_tree_result);
    for (hipEvent_t e : c->kev) (void)hipEventDestroy(e);
    delete c;
    return HIVIS_OK;
}

int hivis_prefill(hivis_ctx* c, const void* vis_embeds, int32_t v, const int32_t* text_ids, int32_t l, int32_t* first_token) {
    if (!c) return HIVIS_EINVAL;
    const hivis_config& g = c->cfg;
    if (!text_ids || v < 0 || l < 1 || (v > 0 && !vis_embeds)) return fail(c, HIVIS_EINVAL, "bad prefill arguments (v=%d, l=%d)", v, l);
    if (v > g.max_vis || l + g.k_max + 2 > g.max_text) return fail(c, HIVIS_ECAP, "prompt exceeds capacity (v=%d/%d, l=%d/%d)", v, g.max_vis, l, g.max_text);
    c->h_ids.resize((size_t)g.batch * l);
    HIP_TRY(c, hipMemcpy(c->h_ids.data(), text_ids, c->h_ids.size() * sizeof(int32_t), hipMemcpyDefault));
    for (int32_t id : c->h_ids)
        if (id < 0 || id >= g.vocab) return fail(c, HIVIS_EINVAL, "token id %d outside [0,%d)", id, g.vocab);
    c->state = ST_CREATED;
    return DISPATCH(c, do_prefill, c, vis_embeds, v, text_ids, l, first_token, false);
}

static int check_uniforms(hivis_ctx* c, const float* u, size_t n, const char* what);

// Fills the uniform arrays of one sampling call on the device (up to two arrays share the call's number).
static int rng_fill(hivis_ctx* c, float* uA, int nA, int rowA, int strideA, unsigned purposeA, float* uB, int nB, unsigned purposeB) {
    if (!c->rng_seeded) return fail(c, HIVIS_ESTATE, "null uniform arrays need hivis_rng_seed first");
    const unsigned long long n = c->rng_calls++;
    const int total = nA + nB;
    hipLaunchKernelGGL(rng_fill_kernel, dim3((total + 255) / 256), dim3(256), 0, c->stream, uA, nA, std::max(rowA, 1), strideA, purposeA, uB, nB, purposeB,
                       (unsigned)(c->rng_seed & 0xFFFFFFFFull), (unsigned)(c->rng_seed >> 32), (unsigned)(n & 0xFFFFFFFFull), (unsigned)(n >> 32));
    HIP_TRY(c, hipGetLastError());
    return HIVIS_OK;
}

int hivis_rng_seed(hivis_ctx* c, uint64_t seed, uint64_t* calls_so_far) {
    if (!c) return HIVIS_EINVAL;
    if (calls_so_far) *calls_so_far = c->rng_calls;
    c->rng_seeded = true; c->rng_seed = seed; c->rng_calls = 0;
    return HIVIS_OK;
}

int hivis_prefill_sample(hivis_ctx* c, const void* vis_embeds, int32_t v, const int32_t* text_ids, int32_t l, float temperature,
                         const float* u_first, int32_t* first_token) {
    if (!c) return HIVIS_EINVAL;
    const hivis_config& g = c->cfg;
    if (!text_ids || v < 0 || l < 1 || (v > 0 && !vis_embeds)) return fail(c, HIVIS_EINVAL, "bad prefill arguments (v=%d, l=%d)", v, l);
    if (!(temperature > 0.0f)) return fail(c, HIVIS_EINVAL, "temperature must be positive");
    if (!u_first && !c->rng_seeded) return fail(c, HIVIS_ESTATE, "null u_first needs hivis_rng_seed first");
    if (u_first) { if (int rc = check_uniforms(c, u_first, (size_t)g.batch, "u_first")) return rc; }
    if (v > g.max_vis || l + g.k_max + 2 > g.max_text) return fail(c, HIVIS_ECAP, "prompt exceeds capacity (v=%d/%d, l=%d/%d)", v, g.max_vis, l, g.max_text);
    c->h_ids.resize((size_t)g.batch * l);
    HIP_TRY(c, hipMemcpy(c->h_ids.data(), text_ids, c->h_ids.size() * sizeof(int32_t), hipMemcpyDefault));
    for (int32_t id : c->h_ids)
        if (id < 0 || id >= g.vocab) return fail(c, HIVIS_EINVAL, "token id %d outside [0,%d)", id, g.vocab);
    if (u_first) { HIP_TRY(c, hipMemcpyAsync(c->u_res, u_first, (size_t)g.batch * sizeof(float), hipMemcpyHostToDevice, c->stream)); }
    else if (int rc = rng_fill(c, c->u_res, g.batch, 1, 1, 0u, nullptr, 0, 0u)) return rc;
    c->inv_temp = 1.0f / temperature;
    c->state = ST_CREATED;
    return DISPATCH(c, do_prefill, c, vis_embeds, v, text_ids, l, first_token, true);
}

static int check_room(hivis_ctx* c, int K) {
    const hivis_config& g = c->cfg;
    for (int b = 0; b < g.batch; ++b) {
        if (c->h_dlen[b] + K + 2 > g.max_text) return fail(c, HIVIS_ECAP, "sequence %d: text length %d + K + 2 exceeds max_text %d", b, c->h_dlen[b], g.max_text);
        if (c->h_tlen[b] + K + 1 > g.max_vis + g.max_text) return fail(c, HIVIS_ECAP, "sequence %d: target cache full", b);
    }
    return HIVIS_OK;
}

int hivis_draft(hivis_ctx* c, int32_t K) {
    if (!c) return HIVIS_EINVAL;
    if (c->state != ST_READY) return fail(c, HIVIS_ESTATE, "hivis_draft needs a prefilled/accepted context");
    if (K < 1 || K > c->cfg.k_max) return fail(c, HIVIS_EINVAL, "K=%d outside [1,%d]", K, c->cfg.k_max);
    if (int rc = check_room(c, K)) return rc;
    int rc = DISPATCH(c, do_draft, c, K, false);
    if (rc) return rc;
    c->K = K; c->state = ST_DRAFTED; c->drafts_sampled = false;
    return HIVIS_OK;
}

int hivis_draft_noalloc(hivis_ctx* c, int32_t K) {
    if (!c) return HIVIS_EINVAL;
    const hivis_config& g = c->cfg;
    if (c->state != ST_READY) return fail(c, HIVIS_ESTATE, "hivis_draft_noalloc needs a prefilled/accepted context");
    if (K < 1 || K > g.k_max) return fail(c, HIVIS_EINVAL, "K=%d outside [1,%d]", K, g.k_max);
    const int max_rows = g.dtype == HIVIS_BF16 ? WTraits<bf16_t>::ROWS : WTraits<float>::ROWS;
    if (!c->fused || g.batch > max_rows)
        return fail(c, HIVIS_EINVAL, "hivis_draft_noalloc needs the phase programs (HIVIS_FUSED not 0) and batch <= %d", max_rows);
    if (!c->scratch_dev) return fail(c, HIVIS_EHIP, "the static scratch array was not resolved at create");
    if (int rc = check_room(c, K)) return rc;
    int rc = DISPATCH(c, draft_noalloc, c, K);
    if (rc) return rc;
    c->K = K; c->state = ST_DRAFTED; c->drafts_sampled = false;
    return HIVIS_OK;
}

static int check_uniforms(hivis_ctx* c, const float* u, size_t n, const char* what) {
    if (!u) return fail(c, HIVIS_EINVAL, "null %s", what);
    for (size_t i = 0; i < n; ++i)
        if (!(u[i] >= 0.0f && u[i] < 1.0f)) return fail(c, HIVIS_EINVAL, "%s[%zu] = %g outside [0, 1)", what, i, (double)u[i]);
    return HIVIS_OK;
}

int hivis_draft_sample(hivis_ctx* c, int32_t K, float temperature, const float* u) {
    if (!c) return HIVIS_EINVAL;
    if (c->state != ST_READY) return fail(c, HIVIS_ESTATE, "hivis_draft_sample needs a prefilled/accepted context");
    if (K < 1 || K > c->cfg.k_max) return fail(c, HIVIS_EINVAL, "K=%d outside [1,%d]", K, c->cfg.k_max);
    if (!(temperature > 0.0f)) return fail(c, HIVIS_EINVAL, "temperature must be positive");
    const int B = c->cfg.batch;
    if (!u && !c->rng_seeded) return fail(c, HIVIS_ESTATE, "null u needs hivis_rng_seed first");
    if (u) { if (int rc = check_uniforms(c, u, (size_t)B * K, "u")) return rc; }
    if (int rc = check_room(c, K)) return rc;
    if (u) {
        for (int b = 0; b < B; ++b)
            HIP_TRY(c, hipMemcpyAsync(c->u_draft + (size_t)b * c->cfg.k_max, u + (size_t)b * K, K * sizeof(float), hipMemcpyHostToDevice, c->stream));
    } else if (int rc = rng_fill(c, c->u_draft, B * K, K, c->cfg.k_max, 1u, nullptr, 0, 0u)) return rc;
    c->inv_temp = 1.0f / temperature;
    int rc = DISPATCH(c, do_draft, c, K, true);
    if (rc) return rc;
    c->K = K; c->state = ST_DRAFTED; c->drafts_sampled = true;
    return HIVIS_OK;
}

int hivis_set_drafts(hivis_ctx* c, const int32_t* tokens, int32_t K) {
    if (!c) return HIVIS_EINVAL;
    if (c->state != ST_READY) return fail(c, HIVIS_ESTATE, "hivis_set_drafts needs a prefilled/accepted context");
    if (!tokens || K < 1 || K > c->cfg.k_max) return fail(c, HIVIS_EINVAL, "bad planted drafts (K=%d)", K);
    if (int rc = check_room(c, K)) return rc;
    for (int i = 0; i < c->cfg.batch * K; ++i)
        if (tokens[i] < 0 || tokens[i] >= c->cfg.vocab) return fail(c, HIVIS_EINVAL, "planted token %d outside vocab", tokens[i]);
    for (int b = 0; b < c->cfg.batch; ++b)
        HIP_TRY(c, hipMemcpyAsync(c->drafts + (size_t)b * c->cfg.k_max, tokens + (size_t)b * K, K * sizeof(int32_t), hipMemcpyHostToDevice, c->stream));
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    c->K = K; c->state = ST_DRAFTED; c->drafts_sampled = false;
    return HIVIS_OK;
}

int hivis_verify(hivis_ctx* c) {
    if (!c) return HIVIS_EINVAL;
    if (c->state != ST_DRAFTED) return fail(c, HIVIS_ESTATE, "hivis_verify needs drafts");
    int rc = DISPATCH(c, do_verify, c);
    if (rc) return rc;
    c->state = ST_VERIFIED; c->vrows = c->cfg.batch * (c->K + 1);
    return HIVIS_OK;
}

int hivis_accept(hivis_ctx* c, int32_t* n_accepted, int32_t* tokens) {
    if (!c) return HIVIS_EINVAL;
    if (c->state != ST_VERIFIED) return fail(c, HIVIS_ESTATE, "hivis_accept needs a verified context");
    if (!n_accepted || !tokens) return fail(c, HIVIS_EINVAL, "null output pointer");
    return DISPATCH(c, do_accept, c, n_accepted, tokens, false);
}

int hivis_accept_sample(hivis_ctx* c, float temperature, const float* u_accept, const float* u_resample, int32_t* n_accepted, int32_t* tokens) {
    if (!c) return HIVIS_EINVAL;
    if (c->state != ST_VERIFIED) return fail(c, HIVIS_ESTATE, "hivis_accept_sample needs a verified context");
    if (!c->drafts_sampled) return fail(c, HIVIS_ESTATE, "hivis_accept_sample needs drafts drawn by hivis_draft_sample (their distributions)");
    if (!n_accepted || !tokens) return fail(c, HIVIS_EINVAL, "null output pointer");
    if (!(temperature > 0.0f)) return fail(c, HIVIS_EINVAL, "temperature must be positive");
    const int B = c->cfg.batch, K = c->K;
    if ((u_accept == nullptr) != (u_resample == nullptr)) return fail(c, HIVIS_EINVAL, "u_accept and u_resample must both be given or both be null");
    if (u_accept) {
        if (int rc = check_uniforms(c, u_accept, (size_t)B * K, "u_accept")) return rc;
        if (int rc = check_uniforms(c, u_resample, (size_t)B, "u_resample")) return rc;
        HIP_TRY(c, hipMemcpyAsync(c->u_acc, u_accept, (size_t)B * K * sizeof(float), hipMemcpyHostToDevice, c->stream));
        HIP_TRY(c, hipMemcpyAsync(c->u_res, u_resample, (size_t)B * sizeof(float), hipMemcpyHostToDevice, c->stream));
    } else if (int rc = rng_fill(c, c->u_acc, B * K, K, K, 2u, c->u_res, B, 3u)) return rc;
    c->inv_temp = 1.0f / temperature;
    return DISPATCH(c, do_accept, c, n_accepted, tokens, true);
}

int hivis_tree_draft(hivis_ctx* c, int32_t top_k, int32_t depth, int32_t n_nodes) {
    if (!c) return HIVIS_EINVAL;
    const hivis_config& g = c->cfg;
    if (g.batch != 1) return fail(c, HIVIS_EINVAL, "tree drafting needs batch 1 (got %d)", g.batch);
    if (c->state != ST_READY) return fail(c, HIVIS_ESTATE, "hivis_tree_draft needs a prefilled/accepted context");
    if (top_k < 1 || top_k > TREE_MAX_TOPK || depth < 1 || depth > TREE_MAX_DEPTH) return fail(c, HIVIS_EINVAL, "top_k=%d outside [1,%d] or depth=%d outside [1,%d]", top_k, TREE_MAX_TOPK, depth, TREE_MAX_DEPTH);
    const int P = top_k + (depth - 1) * top_k * top_k;
    if (P > TREE_MAX_POOL || (depth - 1) * top_k > TREE_MAX_ROWS) return fail(c, HIVIS_EINVAL, "tree too large: pool %d > %d or expanded rows %d > %d", P, TREE_MAX_POOL, (depth - 1) * top_k, TREE_MAX_ROWS);
    if (n_nodes < 1 || n_nodes > P || n_nodes + 1 > TREE_MAX_ROWS) return fail(c, HIVIS_EINVAL, "n_nodes=%d outside [1, min(pool %d, %d)]", n_nodes, P, TREE_MAX_ROWS - 1);
    if (c->h_dlen[0] + std::max((depth - 1) * top_k, depth + 1) + 2 > g.max_text) return fail(c, HIVIS_ECAP, "text length %d + tree rows exceeds max_text %d", c->h_dlen[0], g.max_text);
    if (c->h_tlen[0] + n_nodes + 1 > g.max_vis + g.max_text) return fail(c, HIVIS_ECAP, "target cache full");
    int rc = DISPATCH(c, do_tree_draft, c, top_k, depth, n_nodes);
    if (rc) return rc;
    c->tk = top_k; c->tdepth = depth; c->tn = n_nodes; c->state = ST_TREE_DRAFTED;
    return HIVIS_OK;
}

int hivis_tree_set(hivis_ctx* c, int32_t n_nodes, const int32_t* tokens, const int32_t* parents) {
    if (!c) return HIVIS_EINVAL;
    const hivis_config& g = c->cfg;
    if (g.batch != 1) return fail(c, HIVIS_EINVAL, "tree drafting needs batch 1 (got %d)", g.batch);
    if (c->state != ST_READY) return fail(c, HIVIS_ESTATE, "hivis_tree_set needs a prefilled/accepted context");
    if (!tokens || !parents || n_nodes < 1 || n_nodes + 1 > TREE_MAX_ROWS) return fail(c, HIVIS_EINVAL, "bad planted tree (n_nodes=%d)", n_nodes);
    // verify rows 1..n_nodes: parents are row indices (0 = root) and precede their children
    std::vector<int32_t> tok(n_nodes + 1, 0), par(n_nodes + 1, -1), dep(n_nodes + 1, 0);
    std::vector<unsigned long long> mask(n_nodes + 1, 1ull);
    int depth = 1;
    for (int i = 1; i <= n_nodes; ++i) {
        const int p = parents[i - 1], t = tokens[i - 1];
        if (p < 0 || p >= i) return fail(c, HIVIS_EINVAL, "planted row %d: parent %d outside [0,%d)", i, p, i);
        if (t < 0 || t >= g.vocab) return fail(c, HIVIS_EINVAL, "planted token %d outside vocab", t);
        tok[i] = t; par[i] = p; dep[i] = dep[p] + 1; mask[i] = mask[p] | (1ull << i);
        depth = std::max(depth, dep[i]);
    }
    if (depth > TREE_MAX_DEPTH) return fail(c, HIVIS_EINVAL, "planted tree depth %d > %d", depth, TREE_MAX_DEPTH);
    if (c->h_dlen[0] + depth + 3 > g.max_text) return fail(c, HIVIS_ECAP, "text length %d + tree rows exceeds max_text %d", c->h_dlen[0], g.max_text);
    if (c->h_tlen[0] + n_nodes + 1 > g.max_vis + g.max_text) return fail(c, HIVIS_ECAP, "target cache full");
    if (int rc = DISPATCH(c, tree_setup, c)) return rc;
    const TreeDev& t = c->tree;
    // row 0's token: the last known text token (device to device)
    HIP_TRY(c, hipMemcpyAsync(t.row_tok + 1, tok.data() + 1, n_nodes * sizeof(int32_t), hipMemcpyHostToDevice, c->stream));
    HIP_TRY(c, hipMemcpyAsync(t.row_tok, c->text + c->h_dlen[0], sizeof(int32_t), hipMemcpyDeviceToDevice, c->stream));
    HIP_TRY(c, hipMemcpyAsync(t.row_par, par.data(), (n_nodes + 1) * sizeof(int32_t), hipMemcpyHostToDevice, c->stream));
    HIP_TRY(c, hipMemcpyAsync(t.row_depth, dep.data(), (n_nodes + 1) * sizeof(int32_t), hipMemcpyHostToDevice, c->stream));
    HIP_TRY(c, hipMemcpyAsync(t.vmask, mask.data(), (n_nodes + 1) * sizeof(unsigned long long), hipMemcpyHostToDevice, c->stream));
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    c->tk = 0; c->tdepth = depth; c->tn = n_nodes; c->state = ST_TREE_DRAFTED;
    return HIVIS_OK;
}

int hivis_tree_verify(hivis_ctx* c) {
    if (!c) return HIVIS_EINVAL;
    if (c->state != ST_TREE_DRAFTED) return fail(c, HIVIS_ESTATE, "hivis_tree_verify needs a drafted tree");
    int rc = DISPATCH(c, do_tree_verify, c);
    if (rc) return rc;
    c->state = ST_TREE_VERIFIED;
    return HIVIS_OK;
}

int hivis_tree_accept(hivis_ctx* c, int32_t* n_accepted, int32_t* tokens) {
    if (!c) return HIVIS_EINVAL;
    if (c->state != ST_TREE_VERIFIED) return fail(c, HIVIS_ESTATE, "hivis_tree_accept needs a verified tree");
    if (!n_accepted || !tokens) return fail(c, HIVIS_EINVAL, "null output pointer");
    return DISPATCH(c, do_tree_accept, c, n_accepted, tokens, false);
}

int hivis_tree_accept_sample(hivis_ctx* c, float temperature, const float* u, int32_t* n_accepted, int32_t* tokens) {
    if (!c) return HIVIS_EINVAL;
    if (c->state != ST_TREE_VERIFIED) return fail(c, HIVIS_ESTATE, "hivis_tree_accept_sample needs a verified tree");
    if (!n_accepted || !tokens) return fail(c, HIVIS_EINVAL, "null output pointer");
    if (!(temperature > 0.0f)) return fail(c, HIVIS_EINVAL, "temperature must be positive");
    const int n = c->tdepth + 1;
    if (u) {
        if (int rc = check_uniforms(c, u, (size_t)n, "u")) return rc;
        HIP_TRY(c, hipMemcpyAsync(c->u_tree, u, (size_t)n * sizeof(float), hipMemcpyHostToDevice, c->stream));
    } else if (int rc = rng_fill(c, c->u_tree, n, 1, 1, 4u, nullptr, 0, 0u)) return rc;
    c->inv_temp = 1.0f / temperature;
    return DISPATCH(c, do_tree_accept, c, n_accepted, tokens, true);
}

int hivis_tree_get(hivis_ctx* c, int32_t* pool_tokens, int32_t* pool_parents, float* pool_scores, int32_t* expand, int32_t* selected,
                   int32_t* row_tokens, int32_t* row_parents, int32_t* row_depths, int32_t* target_tokens) {
    if (!c) return HIVIS_EINVAL;
    if (!c->tree_ready || c->tn < 1) return fail(c, HIVIS_ESTATE, "no tree drafted yet");
    const TreeDev& t = c->tree;
    const int k = c->tk, P = k + (c->tdepth - 1) * k * k, N = c->tn;
    if (k == 0 && (pool_tokens || pool_parents || pool_scores || expand || selected)) return fail(c, HIVIS_ESTATE, "the last tree was planted: it has no pool");
#define GET(dst, src, n) do { if (dst) HIP_TRY(c, hipMemcpyAsync(dst, src, (size_t)(n) * 4, hipMemcpyDeviceToHost, c->stream)); } while (0)
    GET(pool_tokens, t.pool_tok, P); GET(pool_parents, t.pool_par, P); GET(pool_scores, t.pool_score, P);
    GET(expand, t.expand, (c->tdepth - 1) * k); GET(selected, t.sel, N);
    GET(row_tokens, t.row_tok, N + 1); GET(row_parents, t.row_par, N + 1); GET(row_depths, t.row_depth, N + 1);
    if (target_tokens) {
        if (c->state != ST_TREE_VERIFIED && c->state != ST_READY) return fail(c, HIVIS_ESTATE, "tree not verified yet");
        GET(target_tokens, t.ttok, N + 1);
    }
#undef GET
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    return HIVIS_OK;
}

int hivis_tree_get_logits(hivis_ctx* c, float* out) {
    if (!c || !out) return HIVIS_EINVAL;
    if (!c->tree_ready || c->tn < 1 || c->tk < 1) return fail(c, HIVIS_ESTATE, "no tree drafted yet");
    const size_t rows = 1 + (size_t)(c->tdepth - 1) * c->tk;
    HIP_TRY(c, hipMemcpyAsync(out, c->tlogits, rows * c->cfg.vocab * sizeof(float), hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    return HIVIS_OK;
}

int hivis_get_logits(hivis_ctx* c, int32_t which, float* out) {
    if (!c || !out) return HIVIS_EINVAL;
    const hivis_config& g = c->cfg;
    const float* src; size_t n;
    if (which == 0) { if ((c->state != ST_VERIFIED && c->state != ST_TREE_VERIFIED && c->state != ST_READY) || c->vrows < 1) return fail(c, HIVIS_ESTATE, "no verify logits"); src = c->logits_v; n = (size_t)c->vrows * g.vocab; }
    else if (which == 1) { src = c->logits_d; n = (size_t)c->K * g.batch * g.vocab; }
    else if (which == 2) { src = c->logits_p; n = (size_t)g.batch * g.vocab; }
    else return fail(c, HIVIS_EINVAL, "which=%d", which);
    if (c->state == ST_CREATED) return fail(c, HIVIS_ESTATE, "nothing computed yet");
    HIP_TRY(c, hipMemcpyAsync(out, src, n * sizeof(float), hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    return HIVIS_OK;
}

int hivis_get_hidden(hivis_ctx* c, int32_t which, float* out) {
    if (!c || !out) return HIVIS_EINVAL;
    const hivis_config& g = c->cfg;
    if (c->state == ST_CREATED) return fail(c, HIVIS_ESTATE, "nothing computed yet");
    const int d = g.d;
    if (which == 0) {
        if (c->vrows < 1) return fail(c, HIVIS_ESTATE, "no verify pass yet");
        HIP_TRY(c, hipMemcpy2DAsync(out, d * sizeof(float), c->catT, 2 * d * sizeof(float), d * sizeof(float), (size_t)c->vrows, hipMemcpyDeviceToHost, c->stream));
    } else if (which == 1) {
        HIP_TRY(c, hipMemcpy2DAsync(out, d * sizeof(float), c->catD, 2 * d * sizeof(float), d * sizeof(float), (size_t)g.batch, hipMemcpyDeviceToHost, c->stream));
    } else return fail(c, HIVIS_EINVAL, "which=%d", which);
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    return HIVIS_OK;
}

int hivis_kv_lengths(hivis_ctx* c, int32_t* target_len, int32_t* drafter_len) {
    if (!c) return HIVIS_EINVAL;
    const int B = c->cfg.batch;
    if (target_len) HIP_TRY(c, hipMemcpyAsync(target_len, c->tlen, B * sizeof(int), hipMemcpyDeviceToHost, c->stream));
    if (drafter_len) HIP_TRY(c, hipMemcpyAsync(drafter_len, c->dlen, B * sizeof(int), hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    return HIVIS_OK;
}

int hivis_get_tokens(hivis_ctx* c, int32_t* drafts, int32_t* target_tokens) {
    if (!c) return HIVIS_EINVAL;
    const hivis_config& g = c->cfg;
    if (c->state == ST_CREATED || c->K < 1) return fail(c, HIVIS_ESTATE, "no draft round yet");
    if (c->state == ST_TREE_DRAFTED || c->state == ST_TREE_VERIFIED) return fail(c, HIVIS_ESTATE, "a tree round is in progress: use hivis_tree_get");
    std::vector<int32_t> hd((size_t)g.batch * g.k_max), ht((size_t)g.batch * (g.k_max + 1));
    HIP_TRY(c, hipMemcpyAsync(hd.data(), c->drafts, hd.size() * sizeof(int32_t), hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(c, hipMemcpyAsync(ht.data(), c->ttok, ht.size() * sizeof(int32_t), hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    for (int b = 0; b < g.batch; ++b) {
        if (drafts) for (int i = 0; i < c->K; ++i) drafts[b * c->K + i] = hd[(size_t)b * g.k_max + i];
        if (target_tokens) for (int i = 0; i <= c->K; ++i) target_tokens[b * (c->K + 1) + i] = ht[(size_t)b * (g.k_max + 1) + i];
    }
    return HIVIS_OK;
}

int hivis_timing(hivis_ctx* c, int32_t enable) {
    if (!c) return HIVIS_EINVAL;
    c->timing = enable != 0;
    return HIVIS_OK;
}

int hivis_kernel_timing(hivis_ctx* c, int32_t gemm_kind) {
    if (!c || gemm_kind < -1 || gemm_kind > 5) return HIVIS_EINVAL;
    c->ktime_epi = gemm_kind; c->kms = 0; c->klaunches = 0; c->kev_used = 0; c->ktime_seen = 0;
    return HIVIS_OK;
}

int hivis_kernel_ms(hivis_ctx* c, double* total_ms, int64_t* launches, double* bytes_per_launch) {
    if (!c) return HIVIS_EINVAL;
    if (total_ms) *total_ms = c->kms;
    if (launches) *launches = c->klaunches;
    if (bytes_per_launch) *bytes_per_launch = c->kbytes;
    c->kms = 0; c->klaunches = 0;
    return HIVIS_OK;
}

int hivis_phase_ms(hivis_ctx* c, int32_t phase, double* total_ms, int64_t* calls) {
    if (!c || phase < 0 || phase > 3) return HIVIS_EINVAL;
    if (c->pev_used) { HIP_TRY(c, hipStreamSynchronize(c->stream)); resolve_phase_events(c); }
    if (total_ms) *total_ms = c->phase_ms[phase];
    if (calls) *calls = c->phase_calls[phase];
    c->phase_ms[phase] = 0; c->phase_calls[phase] = 0;
    return HIVIS_OK;
}

int hivis_algorithmic_bytes(hivis_ctx* c, double* verify_bytes, double* draft_step_bytes) {
    if (!c) return HIVIS_EINVAL;
    const hivis_config& g = c->cfg;
    const double b = c->esize, d = g.d, qd = (double)g.n_q_heads * g.head_dim, kd = (double)g.n_kv_heads * g.head_dim, F = g.ffn, V = g.vocab;
    const double w_layer = (2 * d * qd + 2 * d * kd + 3 * d * F) * b;
    double kv_t = 0, kv_d = 0;
    for (int s = 0; s < g.batch; ++s) { kv_t += 2.0 * c->h_tlen[s] * kd * b * g.n_layers; kv_d += 2.0 * c->h_dlen[s] * kd * b; }
    if (verify_bytes) *verify_bytes = g.n_layers * w_layer + V * d * b + kv_t;
    // (the method's bytes: the fusion FC as [2d x d] weights, also where the library reads only w1 and a table row per sequence)
    if (draft_step_bytes) *draft_step_bytes = w_layer + 2 * d * d * b + V * d * b + kv_d;
    return HIVIS_OK;
}

int32_t hivis_clamp_token(int32_t id, int32_t vocab) { return clamp_token(id, vocab); }

int hivis_calib_stream(void* hip_stream, int64_t buffer_bytes, int32_t n_buffers, int32_t passes, int32_t workgroups, double* gb_per_s,
                       double* us_per_launch) {
    if (buffer_bytes < (1 << 20) || n_buffers < 1 || n_buffers > 64 || passes < 1 || workgroups < 1 || workgroups > 65535) return HIVIS_EINVAL;
    hipStream_t st = (hipStream_t)hip_stream;
    const size_t n16 = (size_t)buffer_bytes / 16;
    const size_t trips = n16 / 4096;
    if (trips == 0) return HIVIS_EINVAL;
    std::vector<void*> bufs;
    unsigned* sink = nullptr;
    std::vector<hipEvent_t> ev;
    int rc = HIVIS_OK;
    auto cleanup = [&]() {
        for (void* b : bufs) (void)hipFree(b);
        if (sink) (void)hipFree(sink);
        for (hipEvent_t e : ev) (void)hipEventDestroy(e);
    };
#define CAL_TRY(expr) do { if ((expr) != hipSuccess) { cleanup(); return HIVIS_EHIP; } } while (0)
    CAL_TRY(hipMalloc((void**)&sink, sizeof(unsigned)));
    for (int i = 0; i < n_buffers; ++i) {
        void* b = nullptr;
        CAL_TRY(hipMalloc(&b, n16 * 16));
        bufs.push_back(b);
        CAL_TRY(hipMemsetAsync(b, 0x5A, n16 * 16, st));
    }
    // Timed like the dominant GEMM in hivis_kernel_timing: start / stop events attached to the dispatch itself read the
    // kernel's own begin and end (events recorded around a batch of short launches measure the host's launch rate
    // instead: 12 us per launch for a 6.8 us kernel).  At most 256 launches carry events (every k-th beyond that).
    const int total = passes * n_buffers;
    const int stride = (total + 255) / 256;
    const int timed = (total + stride - 1) / stride;
    ev.resize((size_t)2 * timed, nullptr);
    for (hipEvent_t& e : ev) CAL_TRY(hipEventCreate(&e));
    // one untimed round over all buffers, then `passes` timed rounds; the buffers rotate so that nothing read comes from a cache
    for (int i = 0; i < n_buffers; ++i) hipLaunchKernelGGL(calib_stream_kernel, dim3(workgroups), dim3(512), 0, st, (const uint4*)bufs[i], n16, sink);
    for (int l = 0, t = 0; l < total; ++l) {
        hipEvent_t a = nullptr, b = nullptr;
        if (l % stride == 0) { a = ev[2 * t]; b = ev[2 * t + 1]; ++t; }
        hipExtLaunchKernelGGL(calib_stream_kernel, dim3(workgroups), dim3(512), 0, st, a, b, 0, (const uint4*)bufs[l % n_buffers], n16, sink);
    }
    CAL_TRY(hipStreamSynchronize(st));
    CAL_TRY(hipGetLastError());
    double ms_sum = 0.0;
    for (int t = 0; t < timed; ++t) {
        float ms = 0.f;
        CAL_TRY(hipEventElapsedTime(&ms, ev[2 * t], ev[2 * t + 1]));
        ms_sum += ms;
    }
#undef CAL_TRY
    const double bytes = (double)trips * 4096 * 16.0;                 // what one launch reads
    const double us = ms_sum * 1e3 / timed;                           // average duration of one launch
    if (gb_per_s) *gb_per_s = bytes / (us * 1e-6) / 1e9;
    if (us_per_launch) *us_per_launch = us;
    cleanup();
    return rc;
}

const char* hivis_last_error(hivis_ctx* c) { return c ? c->err.c_str() : g_create_err.c_str(); }
const char* hivis_version(void) { return "hivis-gfx950 0.1"; }

}  // extern "C"
