// Draft-tree kernels (section 4 inference setting: top-k tree expanded to a fixed depth, the best-scored candidates
// verified in one pass; section 2.1 names the tree structure).  Batch 1.
//
// Pool layout (P = k + (depth-1) k^2 nodes): level 1 = the k most probable tokens after the drafter's pending hidden
// state; level j+1 = k children of each of the k rows expanded at level j, row by row, rank by rank.  A node's score
// is the sum of the log-probabilities along its path.  Everything that decides an index (top-k, expansion set,
// candidate set, acceptance walk) orders by (score descending, index ascending), so results are unique.
#pragma once
#include "hivis_gemm.h"

namespace hivis {

constexpr int TREE_MAX_TOPK = 16;       // k
constexpr int TREE_MAX_ROWS = 64;       // verify rows (root + candidates); drafter tree rows (depth-1)*k: one 64-bit mask each
constexpr int TREE_MAX_DEPTH = 16;
constexpr int TREE_MAX_POOL = 2048;

struct TreeDev {
    int32_t* pool_tok; int32_t* pool_par; float* pool_score; int32_t* pool_depth;   // [P]
    int32_t* pool_hid;                  // [P] hidden row whose distribution the node was taken from
    int32_t* pool_slot;                 // [P] drafter tree row of an expanded node
    int32_t* expand;                    // [depth-1][k] pool indices of the expanded rows
    unsigned long long* dmask;          // [(depth-1) k] ancestor masks of the drafter's tree rows (bit = tree row)
    int32_t* dpos;                      // [(depth-1) k] rotary position of a drafter tree row, relative to the cache length
    int32_t* sel;                       // [N] candidates, ascending pool index
    int32_t* row_tok; int32_t* row_par; int32_t* row_depth;   // [N+1] verify rows (row 0 = root)
    unsigned long long* vmask;          // [N+1] ancestor masks of the verify rows
    int32_t* ttok;                      // [N+1] the target's greedy token after each row
    int32_t* path;                      // [depth+1] rows re-fed after acceptance: root, followed rows, then the last one repeated
    int32_t* next_tok;                  // [depth+1] token that follows each re-fed row
    int32_t* result;                    // [1 + depth+1] accepted length | emitted tokens (-1 padded)
};

// Children of the rows of one level, in two kernels.  Row r of `logits` is the drafter's distribution behind node
// expand_row[r] (or behind the root if expand_row is null); its k most probable tokens (best first) become pool nodes
// first + r k + q with score = parent score + log softmax.
//  1. tree_topk_part_kernel, grid (rows, segments): a workgroup holds one segment of <= 4096 logits in registers (8 per
//     thread, loaded once), writes the segment's (max, sum of exp) and its k best (value, index) pairs.  In every wavefront the
//     lanes' own maxima are ranked by counting; what does not reach the k-th of them cannot be among the k best, and the
//     few survivors of all wavefronts are ranked by counting.
//  2. tree_children_kernel, one workgroup per row: log-normaliser from the segment partials (fixed order), the k best of the
//     segments' candidates by the same two steps, pool entries written.
// (k rounds of a workgroup-wide maximum took 19 us, k rounds of a wavefront's 14; ranking all candidates behind serial loads of
// the partials 12 us for 8 segments and 54 us for 38.)
constexpr int TOPK_NT = 512, TOPK_PER = 8, TOPK_SEG = TOPK_NT * TOPK_PER;
// (value, index) order of everything below: value descending, index ascending
__device__ __forceinline__ bool before(float av, int ai, float bv, int bi) { return av > bv || (av == bv && ai < bi); }
// How many of the n entries (value v[c * stride], index i[c * stride]) in LDS come before (mv, mi).  Eight reads are in flight
// at a time: one per trip waited for each (100 clocks an entry: 5 us for 100 of them).
__device__ __forceinline__ int rank_of(const float* v, const int* i, int n, int stride, float mv, int mi) {
    int rank = 0;
    for (int c = 0; c < n; c += 8) {
        float vv[8]; int ii[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) { const int at = min(c + u, n - 1) * stride; vv[u] = v[at]; ii[u] = i[at]; }
#pragma unroll
        for (int u = 0; u < 8; ++u) rank += (c + u < n && before(vv[u], ii[u], mv, mi)) ? 1 : 0;
    }
    return rank;
}
// ... of consecutive entries, sixteen per trip in 16-byte reads: the arrays are 16-byte aligned and have room for n rounded up to sixteen
__device__ __forceinline__ int rank_of(const float* v, const int* i, int n, float mv, int mi) {
    int rank = 0;
    for (int c = 0; c < n; c += 16) {
        float4 vv[4]; int4 ii[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) { vv[u] = *reinterpret_cast<const float4*>(v + c + 4 * u); ii[u] = *reinterpret_cast<const int4*>(i + c + 4 * u); }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const float x[4] = {vv[u].x, vv[u].y, vv[u].z, vv[u].w};
            const int y[4] = {ii[u].x, ii[u].y, ii[u].z, ii[u].w};
#pragma unroll
            for (int e = 0; e < 4; ++e) rank += (c + 4 * u + e < n && before(x[e], y[e], mv, mi)) ? 1 : 0;
        }
    }
    return rank;
}
// ... entries whose index is their place, for lanes whose mi rise by one from lane to lane (alignment and room as above).  Bound by the comparisons: entries before
// every lane's place or behind every lane's take one (510 entries, one workgroup ranking them all: 28.7 us with the order's three, 13.4 now).
__device__ __forceinline__ int rank_of(const float* v, int n, float mv, int mi) {
    const int first = __builtin_amdgcn_readfirstlane(mi);
    int rank = 0;
    for (int c = 0; c < n; c += 16) {
        float4 vv[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) vv[u] = *reinterpret_cast<const float4*>(v + c + 4 * u);
        float x[16];
#pragma unroll
        for (int u = 0; u < 4; ++u) { x[4 * u] = vv[u].x; x[4 * u + 1] = vv[u].y; x[4 * u + 2] = vv[u].z; x[4 * u + 3] = vv[u].w; }
        if (c + 16 <= first) {
#pragma unroll
            for (int e = 0; e < 16; ++e) rank += x[e] >= mv ? 1 : 0;
        } else if (c >= first + 64 && c + 16 <= n) {
#pragma unroll
            for (int e = 0; e < 16; ++e) rank += x[e] > mv ? 1 : 0;
        } else {
#pragma unroll
            for (int e = 0; e < 16; ++e) rank += (c + e < n && before(x[e], c + e, mv, mi)) ? 1 : 0;
        }
    }
    return rank;
}

__global__ __launch_bounds__(TOPK_NT) void tree_topk_part_kernel(const float* __restrict__ logits, int V, int k,
                                                                 float* __restrict__ cand_v, int32_t* __restrict__ cand_i,
                                                                 float* __restrict__ seg_ms) {
    constexpr int NWV = TOPK_NT / 64, MAXS = NWV * TREE_MAX_TOPK * TOPK_PER;      // survivors: at most k lanes per wavefront
    constexpr int NONE = 0x7FFFFFFF;
    __shared__ float smf[NWV], thr_v[NWV];
    __shared__ __align__(16) float lv[TOPK_NT], sv[MAXS];
    __shared__ __align__(16) int li[TOPK_NT], si[MAXS];
    __shared__ int thr_i[NWV], cnt;
    const int r = blockIdx.x, seg = blockIdx.y, nseg = gridDim.y;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const float* x = logits + (size_t)r * V;
    const int j0 = seg * TOPK_SEG + threadIdx.x;            // element e of a thread: j0 + 512 e
    float v[TOPK_PER];
#pragma unroll
    for (int e = 0; e < TOPK_PER; ++e) v[e] = x[min(j0 + TOPK_NT * e, V - 1)];
    if (threadIdx.x == 0) cnt = 0;
    if (lane == 0) { thr_v[wave] = -INFINITY; thr_i[wave] = NONE; }
    // this thread's best element (a NaN is none)
    float bv = -INFINITY; int bi = NONE;
#pragma unroll
    for (int e = 0; e < TOPK_PER; ++e) {
        const int j = j0 + TOPK_NT * e;
        if (j < V && before(v[e], j, bv, bi)) { bv = v[e]; bi = j; }
    }
    lv[threadIdx.x] = bv; li[threadIdx.x] = bi;
    const float m = block_reduce_max<TOPK_NT>(bv, smf);     // the segment is never empty (the host sizes the grid)
    float sum = 0.f;
#pragma unroll
    for (int e = 0; e < TOPK_PER; ++e) sum += j0 + TOPK_NT * e < V ? expf(v[e] - m) : 0.f;
    sum = wave_sum(sum);
    const int rank = rank_of(lv + wave * 64, li + wave * 64, 64, bv, bi);
    if (rank == k - 1 && bi != NONE) { thr_v[wave] = bv; thr_i[wave] = bi; }
    __syncthreads();
    if (lane == 0) smf[wave] = sum;
    const float tv = thr_v[wave]; const int ti = thr_i[wave];
#pragma unroll
    for (int e = 0; e < TOPK_PER; ++e) {
        const int j = j0 + TOPK_NT * e;
        if (j < V && v[e] == v[e] && !before(tv, ti, v[e], j)) { const int at = atomicAdd(&cnt, 1); sv[at] = v[e]; si[at] = j; }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        float total = 0.f;
        for (int w = 0; w < NWV; ++w) total += smf[w];
        seg_ms[((size_t)r * nseg + seg) * 2] = m; seg_ms[((size_t)r * nseg + seg) * 2 + 1] = total;
    }
    const size_t o = ((size_t)r * nseg + seg) * k;
    const int live = cnt;
    for (int i = threadIdx.x; i < live; i += TOPK_NT) {
        const float mv = sv[i]; const int mi = si[i];
        const int rk = rank_of(sv, si, live, mv, mi);
        if (rk < k) { cand_v[o + rk] = mv; cand_i[o + rk] = mi; }
    }
    // a segment with fewer than k elements pads with (-inf, INT_MAX)
    if ((int)threadIdx.x < k && (int)threadIdx.x >= live) { cand_v[o + threadIdx.x] = -INFINITY; cand_i[o + threadIdx.x] = NONE; }
}

constexpr int CHILD_NT = 256;
__global__ __launch_bounds__(CHILD_NT) void tree_children_kernel(const float* __restrict__ cand_v, const int32_t* __restrict__ cand_i,
                                                                 const float* __restrict__ seg_ms, int nseg, int k, int first,
                                                                 const int32_t* __restrict__ expand_row, int depth, int hid_row0,
                                                                 TreeDev t) {
    // Candidates that reach the k-th best of the segments' maxima lie in at most k segments (with fewer than k segments: in
    // all of them): at most k * k
    constexpr int MAXS = TREE_MAX_TOPK * TREE_MAX_TOPK, NONE = 0x7FFFFFFF;
    extern __shared__ float child_lds[];                     // [nseg k] values, [nseg k] indices
    __shared__ __align__(16) float sv[MAXS];
    __shared__ __align__(16) int si[MAXS];
    __shared__ float thr_v, lz;
    __shared__ int thr_i, cnt;
    const int r = blockIdx.x, n = nseg * k, lane = threadIdx.x & 63;
    float* cv = child_lds; int* ci = reinterpret_cast<int*>(child_lds + n);
    const float* ms = seg_ms + (size_t)r * nseg * 2;
    const int parent = expand_row ? expand_row[r] : -1;      // (requested before anything waits)
    for (int i = threadIdx.x; i < n; i += CHILD_NT) { cv[i] = cand_v[(size_t)r * n + i]; ci[i] = cand_i[(size_t)r * n + i]; }
    if (threadIdx.x == 0) { thr_v = -INFINITY; thr_i = NONE; cnt = 0; }
    const float pscore = parent >= 0 ? t.pool_score[parent] : 0.f;
    if (threadIdx.x < 64) {
        float mx = -INFINITY, sum = 0.f;
        for (int s = lane; s < nseg; s += 64) mx = fmaxf(mx, ms[2 * s]);
        mx = wave_max(mx);
        for (int s = lane; s < nseg; s += 64) sum += ms[2 * s + 1] * expf(ms[2 * s] - mx);
        sum = wave_sum(sum);
        if (lane == 0) lz = mx + logf(sum);
    }
    __syncthreads();
    if (nseg >= k)
        for (int s = threadIdx.x; s < nseg; s += CHILD_NT) {
            const float mv = cv[s * k]; const int mi = ci[s * k];
            const int rank = rank_of(cv, ci, nseg, k, mv, mi);
            if (rank == k - 1 && mi != NONE) { thr_v = mv; thr_i = mi; }
        }
    __syncthreads();
    const float tv = thr_v; const int ti = thr_i;
    for (int i = threadIdx.x; i < n; i += CHILD_NT) {
        const float vi = cv[i]; const int ii = ci[i];
        if (ii == NONE || before(tv, ti, vi, ii)) continue;
        const int at = atomicAdd(&cnt, 1);
        if (at < MAXS) { sv[at] = vi; si[at] = ii; }
    }
    __syncthreads();
    const int live = min(cnt, MAXS);
    for (int i = threadIdx.x; i < live; i += CHILD_NT) {
        const float vi = sv[i]; const int ii = si[i];
        const int rank = rank_of(sv, si, live, vi, ii);
        if (rank < k) {
            const int node = first + r * k + rank;
            t.pool_tok[node] = ii; t.pool_par[node] = parent; t.pool_depth[node] = depth; t.pool_hid[node] = hid_row0 + r;
            t.pool_score[node] = pscore + (vi - lz);
            t.pool_slot[node] = -1;
        }
    }
}

// The k best-scored of the n nodes [lo, lo + n) of one level become the drafter's tree rows n_prev .. n_prev + k - 1
// (rank order), and row rank's fusion input [hidden row the node was drawn from ; Embed(node token)] is written to cat, its token
// to tok.  One workgroup per rank, n <= 256: each ranks all nodes (a launch of its own for that cost more than the k-fold
// counting).  table == nullptr: the embedding half is not needed (it comes from the fusion FC's table).  frag != nullptr: the hidden
// rows go there as row fragments (of k rows) instead of to cat.
template <typename WT>
__global__ __launch_bounds__(256) void tree_expand_kernel(int lo, int n, int k, int n_prev, int level, TreeDev t, const float* __restrict__ H,
                                                          const WT* __restrict__ table, float* __restrict__ cat, int32_t* __restrict__ tok, int d,
                                                          uint4* __restrict__ frag) {
    __shared__ __align__(16) float s[256];
    __shared__ int pick[2];                  // hidden row, token
    const int i = threadIdx.x, want = blockIdx.x;
    // (what a picked node needs is requested by every node's thread before the ranks are known)
    const int node = lo + min(i, n - 1);
    const float si = t.pool_score[node];
    const int parent = t.pool_par[node], hid = t.pool_hid[node], token = t.pool_tok[node];
    const int pslot = t.pool_slot[max(parent, 0)];
    const unsigned long long above = t.dmask[max(pslot, 0)];
    s[i] = i < n ? si : -INFINITY;
    if (i == 0) { pick[0] = 0; pick[1] = 0; }          // (stays so only with NaN scores, where ranks are no permutation)
    __syncthreads();
    if (i < n) {
        const int rank = rank_of(s, n, si, i);
        if (rank == want) {
            const int slot = n_prev + rank;
            t.expand[(level - 1) * k + rank] = node;
            t.pool_slot[node] = slot;
            // (the parent was expanded at the level before, or is the root: its row and mask already exist)
            t.dmask[slot] = (parent >= 0 ? above : 0ull) | (1ull << slot);
            t.dpos[slot] = level - 1;
            pick[0] = hid; pick[1] = token;
            tok[rank] = token;
        }
    }
    __syncthreads();
    const float4* h = reinterpret_cast<const float4*>(H + (size_t)pick[0] * d);
    if (frag) {
        for (int c0 = i; c0 < d / 4; c0 += 4 * 256) {                // four loads in flight
            float4 x[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) x[u] = h[min(c0 + 256 * u, d / 4 - 1)];
#pragma unroll
            for (int u = 0; u < 4; ++u) { const int c = c0 + 256 * u; if (c < d / 4) st_row_quad(frag, k, want, 4 * c, x[u].x, x[u].y, x[u].z, x[u].w); }
        }
        return;
    }
    float* o = cat + (size_t)want * 2 * d;
    for (int c = i; c < d / 4; c += 256) reinterpret_cast<float4*>(o)[c] = h[c];
    if (table) {
        const WT* e = table + (size_t)pick[1] * d;
        for (int c = i; c < d; c += 256) o[d + c] = to_f32(e[c]);
    }
}

// Candidates: the N best-scored pool nodes, in pool order; verify rows 1..N (row 0 = root = the last known token).
// One workgroup of 1024 threads, P <= 2048.
__global__ __launch_bounds__(1024) void tree_select_kernel(int P, int N, const int32_t* __restrict__ text,
                                                           const int* __restrict__ dlen, TreeDev t) {
    __shared__ __align__(16) float s[TREE_MAX_POOL];
    __shared__ short rowof[TREE_MAX_POOL];      // verify row of a pool node, 0 if not a candidate
    __shared__ int count[32];                   // candidates per 64 pool nodes
    for (int i = threadIdx.x; i < P; i += 1024) s[i] = t.pool_score[i];
    __syncthreads();
    bool chosen[2] = {false, false};
    for (int e = 0; e < 2; ++e) {
        const int i = threadIdx.x + e * 1024;
        if (i >= P) continue;
        const float si = s[i];
        chosen[e] = rank_of(s, P, si, i) < N;
    }
    // rows are numbered in pool order: candidates below this one, from the wavefronts' counts and a ballot
    int myrow[2] = {0, 0};
    for (int e = 0; e < 2; ++e) {
        const unsigned long long hit = __ballot(chosen[e]);
        if ((threadIdx.x & 63) == 0) count[e * 16 + (threadIdx.x >> 6)] = (int)__popcll(hit);
        __syncthreads();
        int below = (int)__popcll(hit & ((1ull << (threadIdx.x & 63)) - 1));
        for (int w = 0; w < e * 16 + (int)(threadIdx.x >> 6); ++w) below += count[w];
        if (chosen[e]) myrow[e] = below + 1;
    }
    __syncthreads();
    for (int e = 0; e < 2; ++e) { const int i = threadIdx.x + e * 1024; if (i < P) rowof[i] = (short)myrow[e]; }
    __syncthreads();
    for (int e = 0; e < 2; ++e) {
        const int i = threadIdx.x + e * 1024;
        if (i >= P || !chosen[e]) continue;
        const int row = myrow[e];
        if (row > N) continue;                                    // only with NaN scores (ranks are then not a permutation)
        t.sel[row - 1] = i;
        t.row_tok[row] = t.pool_tok[i];
        t.row_depth[row] = t.pool_depth[i];
        const int parent = t.pool_par[i];
        t.row_par[row] = parent >= 0 ? rowof[parent] : 0;        // the candidate set is closed under ancestors
        unsigned long long m = 1ull;                              // the root
        for (int a = i; a >= 0; a = t.pool_par[a]) m |= 1ull << rowof[a];
        t.vmask[row] = m;
    }
    if (threadIdx.x == 0) { t.row_tok[0] = text[dlen[0]]; t.row_par[0] = -1; t.row_depth[0] = 0; t.vmask[0] = 1ull; }
}

// Greedy acceptance on the tree: from the root, follow the child whose token is the target's greedy token at the
// current row until there is none.  Emits the followed tokens plus the target's token at the last row, appends them
// to the text, and lists the rows whose true features re-condition the drafter.  One wavefront.
__global__ __launch_bounds__(64) void tree_accept_kernel(int N, int depth, int32_t* __restrict__ text, const int* __restrict__ dlen, TreeDev t) {
    const int lane = threadIdx.x;
    int cur = 0, n = 0;
    int mine = 0;                                   // lane e ends up holding re-fed row e (lane 0: the root)
    while (n < depth) {
        const int want = t.ttok[cur];
        int found = 0x7FFFFFFF;
        for (int c = 1 + lane; c <= N; c += 64)
            if (t.row_par[c] == cur && t.row_tok[c] == want) found = min(found, c);
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) found = min(found, __shfl_xor(found, o, 64));
        if (found == 0x7FFFFFFF) break;
        cur = found; ++n;
        if (lane == n) mine = cur;
    }
    if (lane > n) mine = cur;                       // dead rows repeat the last followed row
    const int bonus = t.ttok[cur];
    const int next_row = __shfl(mine, min(lane + 1, 63), 64);
    if (lane <= depth) {
        const int tok = (lane < n) ? t.row_tok[next_row] : bonus;          // token that follows re-fed row `lane`
        t.path[lane] = mine;
        t.next_tok[lane] = tok;
        t.result[1 + lane] = (lane <= n) ? tok : -1;
        if (lane <= n) text[dlen[0] + 1 + lane] = tok;
    }
    if (lane == 0) t.result[0] = n;
}

// Cache compaction after acceptance, for all layers at once: the rows of the followed path move from their tree
// slots base + path[j] to base + j (j = 1..n).  Two kernels (gather into a staging buffer, scatter back) because a
// destination slot of one row can be the source slot of another.
// kv: [n_layers][2] cache pointers; cache layout [Hkv][maxL][HD]; staging [n_layers][2][depth][Hkv*HD], where HD here is
// the STORAGE width of a cached row (head_dim * KVWidth: hi and lo halves of a half-precision cache move together).
template <typename KT>
__global__ void tree_kv_gather_kernel(KT* const* __restrict__ kv, int maxL, int Hkv, int HD, const int* __restrict__ tlen,
                                      const int32_t* __restrict__ result, const int32_t* __restrict__ path, int depth,
                                      KT* __restrict__ staging, int scatter) {
    const int j = blockIdx.x + 1, lk = blockIdx.y;                  // lk = layer * 2 + (0: keys, 1: values)
    const int n = result[0];
    if (j > n) return;
    const int src = path[j];
    if (src == j) return;                                           // already in place
    KT* cache = kv[lk];
    KT* st = staging + ((size_t)lk * depth + (j - 1)) * Hkv * HD;
    const int base = tlen[0];
    for (int idx = threadIdx.x; idx < Hkv * HD; idx += blockDim.x) {
        const int h = idx / HD, c = idx % HD;
        if (scatter) cache[((size_t)h * maxL + base + j) * HD + c] = st[idx];
        else st[idx] = cache[((size_t)h * maxL + base + src) * HD + c];
    }
}

// Re-feed rows after acceptance: [true feature of path row e ; Embed(token after it)], e = 0..depth (rows beyond the
// accepted length repeat the last one and are dead).  g: verify features, row stride ldg.  table, frag as above (gridDim.x rows).
template <typename WT>
__global__ void tree_roll_cat_kernel(const float* __restrict__ g, int ldg, const int32_t* __restrict__ path,
                                     const int32_t* __restrict__ next_tok, const WT* __restrict__ table,
                                     float* __restrict__ cat, int d, uint4* __restrict__ frag) {
    const int e = blockIdx.x;
    const float4* f = reinterpret_cast<const float4*>(g + (size_t)path[e] * ldg);
    if (frag) {
        for (int c = threadIdx.x; c < d / 4; c += blockDim.x) {
            const float4 x = f[c];
            st_row_quad(frag, gridDim.x, e, 4 * c, x.x, x.y, x.z, x.w);
        }
        return;
    }
    float* o = cat + (size_t)e * 2 * d;
    for (int c = threadIdx.x; c < d / 4; c += blockDim.x) reinterpret_cast<float4*>(o)[c] = f[c];
    if (table) {
        const WT* em = table + (size_t)next_tok[e] * d;
        for (int c = threadIdx.x; c < d; c += blockDim.x) o[d + c] = to_f32(em[c]);
    }
}

// After the re-feed: pending hidden state = drafter output at row n; both caches keep n + 1 more rows.
__global__ void tree_finish_kernel(const float* __restrict__ dout, const int32_t* __restrict__ result, float* __restrict__ fnext,
                                   int* __restrict__ dlen, int* __restrict__ tlen, int d, uint4* __restrict__ frag,
                                   int32_t* __restrict__ host, int nres, const int* __restrict__ bad, int bad_at) {
    const int n = result[0];
    // (results and flag straight to the host's pinned mirror, as in select_row_kernel)
    if ((int)threadIdx.x < nres) __hip_atomic_store(&host[threadIdx.x], result[threadIdx.x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    if (threadIdx.x == 255) __hip_atomic_store(&host[bad_at], bad[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    for (int c = 2 * threadIdx.x; c < d; c += 2 * blockDim.x) {
        const float2 x = *reinterpret_cast<const float2*>(dout + (size_t)n * d + c);
        *reinterpret_cast<float2*>(fnext + c) = x;
        if (frag) st_row_pair(frag, 1, 0, c, x.x, x.y);
    }
    if (threadIdx.x == 0) { dlen[0] += n + 1; tlen[0] += n + 1; }
}

// ------------------------------------------------------------------------------------------
// Row-wise kernels around the fragment GEMMs (bf16 models: 11..64-row passes that no phase program takes, and the prefill).
// They read a GEMM result as the sum of its K-slice partials (value = sum over s < nparts of p[s * pstride + index], fixed
// order) and, where the consumer is the next GEMM on fragments, write its A operand directly as activation fragments (layout: hivis_gemm.h), so neither the reduction nor the fragment
// packing is a launch of its own.
// ------------------------------------------------------------------------------------------
// h[row] += delta (sum of partials, optional); fragments of h[row] * gain / sqrt(mean(h^2) + eps).  One workgroup of 1024
// threads per row of the padded row range (rows >= M write zero fragments); d <= 8192, d % 8 == 0.  A thread owns 4
// consecutive columns and requests all slices of them at once (up to 16 loads in flight: with 8 columns per thread and
// 8 slices per trip the kernel paid four memory round trips per row); two neighbouring lanes then hold the 8 values of
// one fragment chunk, exchange them, and the even lane writes the chunk's high parts, the odd lane its low parts.
constexpr int WNORM_NT = 1024, WNORM_GROUPS = 2;
template <typename WT>
__global__ __launch_bounds__(WNORM_NT) void wide_add_norm_frag_kernel(float* __restrict__ h, int ldh, Parts delta, int ldd, int M,
                                                                  const WT* __restrict__ gain, uint4* __restrict__ frag, int d, float eps) {
    __shared__ float part[WNORM_NT / 64];
    constexpr int MAXG = WNORM_GROUPS;              // groups of 4 values per thread
    const int row = blockIdx.x, ng = d / 4, kblks = d / 32;
    const bool live = row < M;
    const int rr = min(row, M - 1);
    float4 x[MAXG];
    float ss = 0.f;
#pragma unroll
    for (int k = 0; k < MAXG; ++k) {
        const int gi = (int)threadIdx.x + WNORM_NT * k;
        x[k] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (gi < ng) {
            float4 a = *reinterpret_cast<const float4*>(h + (size_t)rr * ldh + 4 * gi);
            if (delta.p) {
                const size_t idx = (size_t)rr * ldd + 4 * gi;
                float4 da = *reinterpret_cast<const float4*>(delta.p + idx);
                if (delta.n <= 4) parts_add<3>(da, delta, idx, 1);
                else if (delta.n <= 8) parts_add<7>(da, delta, idx, 1);
                else parts_add<15>(da, delta, idx, 1);        // slices 1..15 in one trip (at most 16 slices)
                a.x += da.x; a.y += da.y; a.z += da.z; a.w += da.w;
                if (live) *reinterpret_cast<float4*>(h + (size_t)rr * ldh + 4 * gi) = a;
            }
            x[k] = a;
            ss += a.x * a.x + a.y * a.y + a.z * a.z + a.w * a.w;
        }
    }
    ss = wave_sum(ss);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = ss;
    __syncthreads();
    float tot = 0.f;
#pragma unroll
    for (int w = 0; w < WNORM_NT / 64; ++w) tot += part[w];
    const float inv = 1.0f / sqrtf(tot / (float)d + eps);
    const int odd = threadIdx.x & 1;
#pragma unroll
    for (int k = 0; k < MAXG; ++k) {
        const int gi = (int)threadIdx.x + WNORM_NT * k;
        // (ng is even, so a lane and its neighbour are in range together; out-of-range lanes still take part in the exchange)
        float4 y = make_float4(0.f, 0.f, 0.f, 0.f);
        if (gi < ng) {
            const WT* gp = gain + 4 * gi;
            y = make_float4(x[k].x * to_f32(gp[0]) * inv, x[k].y * to_f32(gp[1]) * inv, x[k].z * to_f32(gp[2]) * inv, x[k].w * to_f32(gp[3]) * inv);
        }
        const float4 o = make_float4(__shfl_xor(y.x, 1, 64), __shfl_xor(y.y, 1, 64), __shfl_xor(y.z, 1, 64), __shfl_xor(y.w, 1, 64));
        if (gi < ng) {
            const float4 lo4 = odd ? o : y, hi4 = odd ? y : o;        // values 0..3 and 4..7 of the chunk
            uint32_t wh[4], wl[4];
            f32_to_bf16x2_hilo(lo4.x, lo4.y, wh[0], wl[0]);
            f32_to_bf16x2_hilo(lo4.z, lo4.w, wh[1], wl[1]);
            f32_to_bf16x2_hilo(hi4.x, hi4.y, wh[2], wl[2]);
            f32_to_bf16x2_hilo(hi4.z, hi4.w, wh[3], wl[3]);
            const int k0 = 8 * (gi >> 1);
            uint4 w4 = odd ? make_uint4(wl[0], wl[1], wl[2], wl[3]) : make_uint4(wh[0], wh[1], wh[2], wh[3]);
            if (!live) w4 = make_uint4(0u, 0u, 0u, 0u);
            frag[afrag_at(kblks, row, k0) + (odd ? 64 : 0)] = w4;
        }
    }
}

// Fusion FC input of a drafter prefill: row s * l + j (j < l) is [f^j ; Embed(x_{j+1})] of sequence s as fragments, and its
// residual row starts as rho_0 (feat: `fstride` rows per sequence; text: x of the sequence, tstride apart).  With the table
// Embed(x) w2 (tab) the fragments hold f^j alone and the residual row starts as rho_0 + tab[x_{j+1}].  Rows >= M: zero fragments.
template <typename WT>
__global__ void fuse_frag_kernel(const float* __restrict__ feat, int fstride, int l, int M, const int32_t* __restrict__ text, int tstride,
                                 const WT* __restrict__ table, const float* __restrict__ tab, const WT* __restrict__ rho,
                                 float* __restrict__ h, uint4* __restrict__ frag, int d) {
    const int row = blockIdx.x;
    const bool live = row < M;
    const int rr = min(row, M - 1), s = rr / l, j = rr - s * l;
    const float* f = feat + ((size_t)s * fstride + j) * d;
    const int tok = text[(size_t)s * tstride + j + 1];
    const int K = tab ? d : 2 * d;
    for (int k = 8 * threadIdx.x; k < K; k += 8 * blockDim.x) {
        float x[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = k < d ? f[k + e] : to_f32(table[(size_t)tok * d + k - d + e]);
        store_afrag8(frag, K / 32, row, k, x, !live);
    }
    if (live)
        for (int k = threadIdx.x; k < d; k += blockDim.x) h[(size_t)row * d + k] = to_f32(rho[k]) + (tab ? tab[(size_t)tok * d + k] : 0.f);
}

// out row = h row + sum of the partials (optional; d a multiple of 4); frag (optional): the row as row fragments as well, row row0 + r of `rows`
__global__ void add_parts_kernel(const float* __restrict__ h, Parts ps, int d, float* __restrict__ out, int ldo, uint4* __restrict__ frag, int row0, int rows) {
    const int row = blockIdx.x;
    for (int c4 = blockIdx.y * blockDim.x + threadIdx.x; c4 < d / 4; c4 += gridDim.y * blockDim.x) {
        const float4 a = *reinterpret_cast<const float4*>(h + (size_t)row * d + 4 * c4), b = ps.p ? parts_load4(ps, (size_t)row * d + 4 * c4) : make_float4(0.f, 0.f, 0.f, 0.f);
        const float4 y = make_float4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w);
        *reinterpret_cast<float4*>(out + (size_t)row * ldo + 4 * c4) = y;
        if (frag) { st_row_quad(frag, rows, row0 + row, 4 * c4, y.x, y.y, y.z, y.w); }
    }
}

// act = silu(gate) * up from the interleaved gate|up result (sum of partials), written as fragments of the down projection.
// grid (row tiles of 16 rows, column chunks), 256 threads; F % 8 == 0.  Four consecutive threads serve four groups of 8
// activations of one row, 64 threads the 16 rows of a tile: together they read 256 contiguous bytes of a row at a time and write
// whole fragment blocks (a thread per (row, group) in row-major order scattered 16-byte stores over the buffer: 137 us for a
// 3008-row prefill layer).  One trip per thread: with at most 64 chunks (4 row tiles of a 61-row pass x 64 workgroups, a third of
// them with two trips) the 7B verify pass took 5.45 ms, now 5.38.
__global__ void wide_silu_frag_kernel(Parts gu, int M, int F, uint4* __restrict__ frag) {
    const int row = blockIdx.x * 16 + ((threadIdx.x >> 2) & 15), kblks = F / 32;
    const bool live = row < M;
    const int rr = min(row, M - 1);
    const int per = blockDim.x >> 4;
    for (int gi = blockIdx.y * per + (threadIdx.x & 3) + 4 * (threadIdx.x >> 6); gi < F / 8; gi += gridDim.y * per) {
        const size_t o = (size_t)rr * 2 * F + (size_t)gi * 16;
        const float4 g0 = parts_load4(gu, o), g1 = parts_load4(gu, o + 4), u0 = parts_load4(gu, o + 8), u1 = parts_load4(gu, o + 12);
        const float g[8] = {g0.x, g0.y, g0.z, g0.w, g1.x, g1.y, g1.z, g1.w}, u[8] = {u0.x, u0.y, u0.z, u0.w, u1.x, u1.y, u1.z, u1.w};
        float y[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) y[e] = g[e] / (1.0f + expf(-g[e])) * u[e];
        store_afrag8(frag, kblks, row, 8 * gi, y, !live);
    }
}

// rope_append_kernel for rows whose fused QKV result arrives as partials: sums them, rotates q and k, writes q to `q_out`
// (row stride ldq, the buffer the attention reads) and k, v to the cache.  Same position / slot rule and optional bias as
// rope_append_kernel.
template <typename ST>
__global__ void wide_rope_append_kernel(Parts qkv, float* __restrict__ q_out, int ldq, int Hq, int Hkv, int HD, const int* __restrict__ base,
                                        int offset, int seq0, int m, ST* __restrict__ kc, ST* __restrict__ vc, int maxL,
                                        float theta, const int* __restrict__ pos_delta, const float* __restrict__ bias,
                                        const float* __restrict__ rope_tab = nullptr, int npos = 0) {
    const int row = blockIdx.x;
    const int seq = seq0 + row / m;
    const int slot = base[seq] + offset + row % m;
    const int pos = pos_delta ? base[seq] + pos_delta[row] : slot;
    const int half = HD / 2;
    const size_t rbase = (size_t)row * (Hq + 2 * Hkv) * HD;
    const int npair2 = (Hq + Hkv) * half / 2;                 // two pairs (4 adjacent columns) per trip
    for (int idx = blockIdx.y * blockDim.x + threadIdx.x; idx < npair2; idx += gridDim.y * blockDim.x) {
        const int head = (2 * idx) / half, i = (2 * idx) % half;
        float4 x = parts_load4(qkv, rbase + (size_t)head * HD + 2 * i);            // pairs (i, i + hd/2) sit in columns 2i, 2i+1
        if (bias) { const float4 b = *reinterpret_cast<const float4*>(bias + (size_t)head * HD + 2 * i); x.x += b.x; x.y += b.y; x.z += b.z; x.w += b.w; }
        float y[4];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            double s, c;
            if (rope_tab) {
                const float2 t = *reinterpret_cast<const float2*>(rope_tab + ((size_t)min(pos, npos - 1) * half + i + e) * 2);
                c = (double)t.x; s = (double)t.y;
            } else {
                const double inv_freq = exp2(-2.0 * (double)(i + e) / (double)HD * log2((double)theta));
                sincos((double)pos * inv_freq, &s, &c);
            }
            const float x1 = e ? x.z : x.x, x2 = e ? x.w : x.y;
            rotate_pair(x1, x2, c, s, y[2 * e], y[2 * e + 1]);
        }
        if (head < Hq) {
            *reinterpret_cast<float4*>(q_out + (size_t)row * ldq + (size_t)head * HD + 2 * i) = make_float4(y[0], y[1], y[2], y[3]);
        } else {
            ST* dst = kc + (((size_t)seq * Hkv + (head - Hq)) * maxL + slot) * HD * KVWidth<ST>::W;
#pragma unroll
            for (int e = 0; e < 4; ++e) kv_put(dst, HD, 2 * i + e, y[e]);
        }
    }
    for (int idx = blockIdx.y * blockDim.x + threadIdx.x; idx < Hkv * HD / 4; idx += gridDim.y * blockDim.x) {
        const int head = (4 * idx) / HD, c = (4 * idx) % HD;
        float4 v = parts_load4(qkv, rbase + (size_t)(Hq + Hkv) * HD + 4 * idx);
        if (bias) { const float4 b = *reinterpret_cast<const float4*>(bias + (size_t)(Hq + Hkv) * HD + 4 * idx); v.x += b.x; v.y += b.y; v.z += b.z; v.w += b.w; }
        ST* dst = vc + (((size_t)seq * Hkv + head) * maxL + slot) * HD * KVWidth<ST>::W;
        kv_put(dst, HD, c, v.x); kv_put(dst, HD, c + 1, v.y); kv_put(dst, HD, c + 2, v.z); kv_put(dst, HD, c + 3, v.w);
    }
}

}  // namespace hivis
