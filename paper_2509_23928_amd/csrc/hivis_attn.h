// Attention of passes of few rows over half-precision caches (verify, draft steps, roll-forward, draft trees; last rows of a prompt): one (item, key
// split) per workgroup, an item being one key head of a sequence and up to 8 or 16 (query head, row) pairs.
//
// Latency bound: at 650 cached rows a launch moves 21 MB in ten dependent steps.  What the steps are, and what keeps them short:
//   * Item, split and range come from the grid and from reciprocals that the host computes; the first rows are requested after one batch of
//     argument loads.  (Quotients and branches on lengths in memory: 1.8 us before the first request.)
//   * The queries are split into halves once per workgroup, in LDS, while the first keys are under way (every wavefront loading and
//     converting all of them was a third of the CU's address cycles).
//   * 128 keys at a time, 16 per wavefront: scores S^T = K Q^T (mfma 16x16x32 f16; three products of high and low halves in accumulators of their
//     own), the block's maximum through LDS, weights P (high and low) to LDS.
//   * Then a wavefront owns 16 of the head's dims for ALL keys of the block (64-wide heads: half of the keys' tiles), O^T += V^T P^T with the two
//     tiles of a pair side by side in K; V^T comes from the row-major tiles through the transposing LDS read.  So no sums of
//     eight wavefronts are left to merge at the end (1.5 us), only the denominators.
//   * Key splits are merged by the workgroup that arrives last (attn_merge_splits).
// Kernel traces, eight softmaxes merged at the end -> now: 32 heads of 128, 6 rows over 650 keys 11.6 -> 10.6 us, over 3010 (98 MB) 23.1 -> 21.7; a draft step over
// 70..110 keys 7.2 -> 5.9; 28 heads of 4 key heads, 7 rows over 1130 keys 14.2 -> 12.8; two sequences, 64-wide heads, 6 rows over 380 keys 10.5 -> 8.8; items of 16
// pairs, which were not split before: 61 rows over 650 keys 18.8 -> 15.9 (2 splits), 31 rows of 28 heads over 1080 keys 24.4 -> 15.2 (4).  Where a
// workgroup walks many blocks, the two barriers of each cost more than the merge that they save: attn_tiles_kernel below.
#pragma once
#include "hivis_fused.h"

namespace hivis {

// quotient by a launch constant: a * d < 2^31
struct FastDiv {
    unsigned mul;
    static FastDiv by(int d) { return {(1u << 31) / (unsigned)d + 1}; }
    __device__ __forceinline__ int operator()(int a) const { return (int)__umulhi(2u * (unsigned)a, mul); }
};

struct AttnArgs {
    const float* q; const f16_t* kc; const f16_t* vc; const int* base; const unsigned long long* tmask;       // (tmask: rows of a draft tree, or null)
    float* ws; int* cnt;                // partials of the key splits; arrival counter per item (null: merged by a launch of its own)
    float* y; uint4* rows_out; uint4* frag_out;       // the result: fp32 rows, row fragments, or (one split) A fragments of the next GEMM
    int ldq, ldo, maxL, offset, seq0, m, qrows, rows;
    int mi, gh, Hkv, group, n_rblk, n_hblk, items, nsplit, flags, nbase;
    FastDiv by_rblk, by_hblk, by_hkv, by_split, by_mi;
    int base_val[8];
    unsigned long long *prof2, *prof3;  // marks (PassParams)
};

template <int HD, int RM> struct AttnSplitCfg {
    static constexpr int ROWB = HD * 4, VSTRIDE = ROWB + 32, KSTRIDE = ROWB + 16;       // (strides: see attn_wg_mfma)
    static constexpr int V = FUSED_NW * 16 * VSTRIDE, K = FUSED_NW * 16 * KSTRIDE, P = FUSED_NW * 64 * 16, Q = HD * RM * 4;
    static constexpr int LDS = V + K + P + Q + 16 * FUSED_NW * 4 + 16;
    static_assert(K >= 3 * ATTN_MAX_SPLITS * RM * 4 && K >= 4 * 64 * 16 && LDS <= 160 * 1024, "scratch of the merge and of the halves of 64-wide heads");
};

template <int HD, int RM, bool ONCE>
__global__ __launch_bounds__(FUSED_NT) void attn_split_kernel(AttnArgs a) {
    typedef AttnSplitCfg<HD, RM> CF;
    constexpr int NW = FUSED_NW, HALFB = HD * 2, ROWB = CF::ROWB, VSTRIDE = CF::VSTRIDE, KSTRIDE = CF::KSTRIDE;
    constexpr int KS = HD / 32, NB = HD / 16, NCH = ROWB / 16, KPI = 64 / NCH, VT = 16 / KPI, KEYS = 16 * NW;
    static_assert(NB == NW || 2 * NB == NW, "a block of 16 dims per wavefront, or per pair of them");
    extern __shared__ __align__(16) char attn_lds[];
    char* const vt_all = attn_lds;                                       // [NW tiles][16 keys][VSTRIDE]
    char* const kt_all = vt_all + CF::V;                                 // [NW][16][KSTRIDE]
    uint4* const pl = reinterpret_cast<uint4*>(kt_all + CF::K);          // [NW tiles][64 lanes]: weights of 4 keys, high and low halves
    uint4* const ql = pl + CF::P / 16;                                   // [high, low][KS][4][RM]: the queries as operand pieces
    float* const wm = reinterpret_cast<float*>(ql + CF::Q / 16);         // [16 rows][NW]: maxima, at the end denominators
    int* const flag = reinterpret_cast<int*>(wm + 16 * NW);
    // all arguments in one batch of scalar loads (left alone, the compiler loads each just before its first use: ten dependent batches)
    asm volatile("" :: "s"(a.q), "s"(a.kc), "s"(a.vc), "s"(a.base), "s"(a.tmask), "s"(a.ldq), "s"(a.maxL), "s"(a.offset), "s"(a.seq0), "s"(a.m), "s"(a.qrows),
                      "s"(a.rows), "s"(a.mi), "s"(a.gh), "s"(a.Hkv));
    asm volatile("" :: "s"(a.group), "s"(a.n_rblk), "s"(a.n_hblk), "s"(a.items), "s"(a.nsplit), "s"(a.flags), "s"(a.nbase), "s"(a.by_rblk.mul), "s"(a.by_hblk.mul),
                      "s"(a.by_hkv.mul), "s"(a.by_split.mul), "s"(a.by_mi.mul), "s"(a.prof2), "s"(a.prof3));
    asm volatile("" :: "s"(a.ws), "s"(a.cnt), "s"(a.y), "s"(a.rows_out), "s"(a.frag_out), "s"(a.ldo));
    const int wg = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z);
    prof_enter(a.prof3, wg);
#define HIVIS_SMARK(k) if (a.prof2 && wg == 0 && threadIdx.x == 0) a.prof2[k] = wall_clock64();
    HIVIS_SMARK(0)
    // Grid: (8, splits, rounds of 8 heads x row blocks): workgroup b runs on XCD b % 8, so that all row blocks and splits of a head share one
    // (the row blocks of 61 rows otherwise each fetch the head's cache rows: 86 MB per layer for 23); or (splits, heads x row blocks)
    const auto scalar = [](int x) { return __builtin_amdgcn_readfirstlane(x); };         // (what is the same for all lanes stays in scalar registers)
    const bool xcd_map = (a.flags & 2) != 0;
    const int z = scalar(xcd_map ? blockIdx.z : blockIdx.y), split = scalar(xcd_map ? blockIdx.y : blockIdx.x);
    const int zh = scalar(a.by_rblk(z)), rblk = z - zh * a.n_rblk, i1 = scalar(xcd_map ? blockIdx.x + 8 * zh : zh), item = i1 * a.n_rblk + rblk;
    if (item >= a.items) return;
    const int i2 = scalar(a.by_hblk(i1)), hblk = i1 - i2 * a.n_hblk, sl = scalar(a.by_hkv(i2)), kvh = i2 - sl * a.Hkv;
    const int seq = a.seq0 + sl, h0 = hblk * a.gh, nh = min(a.gh, a.group - h0), i0 = rblk * a.mi, ni = min(a.mi, a.m - i0), R = nh * ni;
    int len = 0;                                                         // cached rows before the pass
    if (a.nbase > 0) len = a.base_val[sl];
    else len = __hip_atomic_load(&a.base[seq], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const int pos0 = scalar(len) + a.offset;
    const int nkeys = min(pos0 + i0 + ni, a.maxL);
    const int cs = (scalar(a.by_split(nkeys + a.nsplit - 1)) + 15) & ~15;       // keys per split
    const int k0 = split * cs, k1 = min(nkeys, k0 + cs);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n16 = lane & 15, g = lane >> 4, vks = lane / NCH, vdc = lane % NCH;
    auto pair_of = [&](int r, int& h, int& i) { h = a.by_mi(r); i = r - h * ni; };       // (one head: r < mi; several: all rows in one block, mi = ni)

    // this lane's (head, row) pair (lanes beyond R repeat the last)
    int ph_, pi_;
    pair_of(min(n16, R - 1), ph_, pi_);
    // it sees the keys below `below`, and of a draft tree's (from slot tb on) those of its mask: zero without a tree (no memory access)
    const int tb = pos0 - a.offset, below = a.tmask ? tb : pos0 + i0 + pi_ + 1;
    const unsigned long long tmk = __builtin_bit_cast(unsigned long long, __builtin_amdgcn_raw_buffer_load_b64(buffer_of(a.tmask, a.tmask ? a.rows * 8 : 0), (sl * a.m + i0 + pi_) * 8, 0, 0));
    // ---- queries: one float4 per thread (rows beyond R repeat the last), then the first keys and values of this wavefront (rows clamped into the
    // range: masked below).  Loads return in order and a wait counts them, so nothing is requested under a branch that joins again before the wait.
    const int qr = threadIdx.x / (HD / 4), qc = 4 * (threadIdx.x % (HD / 4));
    int qh_, qi_;
    pair_of(min(qr, R - 1), qh_, qi_);
    const int qrow = sl * (a.qrows ? a.qrows : a.m) + i0 + qi_;
    const float4 qv = *reinterpret_cast<const float4*>(a.q + (size_t)qrow * a.ldq + (size_t)(kvh * a.group + h0 + qh_) * HD + qc);
    const char* kbase = reinterpret_cast<const char*>(a.kc) + ((size_t)seq * a.Hkv + kvh) * a.maxL * ROWB;
    const char* vbase = reinterpret_cast<const char*>(a.vc) + ((size_t)seq * a.Hkv + kvh) * a.maxL * ROWB;
    u32x4_t kr[VT], vr[VT];
    auto load_tile = [&](u32x4_t (&d)[VT], const char* from, int kb_) {
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t = 0; t < VT; ++t) {
            const u32x4_t* p = reinterpret_cast<const u32x4_t*>(from + (size_t)min(kb_ + t * KPI + vks, nkeys - 1) * ROWB + vdc * 16);
            if constexpr (ONCE) d[t] = __builtin_nontemporal_load(p); else d[t] = *p;
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    auto stage_queries = [&]() {
        float4 u = qv;
        asm volatile("" : "+v"(u.x), "+v"(u.y), "+v"(u.z), "+v"(u.w));   // (not before the requests of the keys; waited for by all lanes)
        if (qr >= RM) return;
        const float scale = rsqrtf((float)HD);
        const float x[4] = {u.x * scale, u.y * scale, u.z * scale, u.w * scale};
        f16x4_t hi, lo;
#pragma unroll
        for (int e = 0; e < 4; ++e) { hi[e] = (_Float16)fminf(fmaxf(x[e], -65504.f), 65504.f); lo[e] = (_Float16)(x[e] - (float)hi[e]); }
        f16x4_t* const at = reinterpret_cast<f16x4_t*>(ql + ((qc >> 5) * 4 + ((qc & 31) >> 3)) * RM + qr) + ((qc & 7) >> 2);
        at[0] = hi;
        at[CF::Q / 16] = lo;                                             // (half of the area further)
    };
    int kb = k0 + 16 * wave;
    if (kb < k1) {
        load_tile(kr, kbase, kb);
        load_tile(vr, vbase, kb);
        stage_queries();
        asm volatile("; keys requested");                                // (keeps the two branches apart: joined, the queries would wait for the keys)
    } else {
        stage_queries();
        asm volatile("; none");
    }
    HIVIS_SMARK(1)
    lds_barrier();
    f16x8_t qh[KS], qlo[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        const uint4* at = ql + (ks * 4 + g) * RM + min(n16, RM - 1);
        qh[ks] = __builtin_bit_cast(f16x8_t, at[0]);
        qlo[ks] = __builtin_bit_cast(f16x8_t, at[CF::Q / 32]);
    }

    char* const vt = vt_all + wave * 16 * VSTRIDE;
    char* const kt = kt_all + wave * 16 * KSTRIDE;
    const int blk = wave % NB;                                           // this wavefront's dims [16 blk, + 16)
    float mrun = -INFINITY, lrun = 0.f;
    f32x4_t acc[3];
#pragma unroll
    for (int o = 0; o < 3; ++o) acc[o] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    int kbb = k0;
    // One block of 128 keys.  LAST: the last one, whose later tiles may lie beyond the range and behind which nothing is requested; the others
    // request the next block's keys and values as soon as the registers of this one's are free.
    auto block = [&](auto last_) {
        constexpr bool LAST = decltype(last_)::value;
        const bool mine = !LAST || kb < k1;                              // (uniform)
        float sv[4] = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
        if (mine) {
#pragma unroll
            for (int t = 0; t < VT; ++t) *reinterpret_cast<u32x4_t*>(kt + (t * KPI + vks) * KSTRIDE + vdc * 16) = kr[t];
            if constexpr (!LAST) load_tile(kr, kbase, kb + KEYS);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            // scores, transposed: this lane gets keys kb + 4 g + 0..3 of row n16
            f32x4_t st[3];
#pragma unroll
            for (int o = 0; o < 3; ++o) st[o] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const f16x8_t kh = *reinterpret_cast<const f16x8_t*>(kt + n16 * KSTRIDE + ks * 64 + g * 16);
                const f16x8_t kl = *reinterpret_cast<const f16x8_t*>(kt + n16 * KSTRIDE + HALFB + ks * 64 + g * 16);
                st[0] = __builtin_amdgcn_mfma_f32_16x16x32_f16(kl, qh[ks], st[0], 0, 0, 0);
                st[1] = __builtin_amdgcn_mfma_f32_16x16x32_f16(kh, qlo[ks], st[1], 0, 0, 0);
                st[2] = __builtin_amdgcn_mfma_f32_16x16x32_f16(kh, qh[ks], st[2], 0, 0, 0);
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int key = kb + 4 * g + r;
                const bool sees = (key < below) | (((unsigned)(key - tb) < 64u) & (bool)((tmk >> ((key - tb) & 63)) & 1ull));
                sv[r] = ((key < k1) & sees) ? st[2][r] + (st[0][r] + st[1][r]) : -INFINITY;
            }
        }
        float tmax = fmaxf(fmaxf(sv[0], sv[1]), fmaxf(sv[2], sv[3]));
        tmax = fmaxf(tmax, __shfl_xor(tmax, 16, 64));
        tmax = fmaxf(tmax, __shfl_xor(tmax, 32, 64));
        if (g == 0) wm[n16 * NW + wave] = tmax;
        lds_barrier();                                                   // (also: every wavefront has left the products of the block before)
        const float4 m0 = *reinterpret_cast<const float4*>(wm + n16 * NW), m1 = *reinterpret_cast<const float4*>(wm + n16 * NW + 4);
        const float mnew = fmaxf(mrun, fmaxf(fmaxf(fmaxf(m0.x, m0.y), fmaxf(m0.z, m0.w)), fmaxf(fmaxf(m1.x, m1.y), fmaxf(m1.z, m1.w))));
        const float mref = (mnew == -INFINITY) ? 0.f : mnew;             // nothing visible yet: every exponential below is 0
        const float alpha = __expf(mrun - mref);
        float psum = 0.f;
        f16x4_t pb[2];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float p = __expf(sv[r] - mref);
            psum += p;
            pb[0][r] = (_Float16)p; pb[1][r] = (_Float16)(p - (float)pb[0][r]);
        }
        mrun = mnew;
        lrun = lrun * alpha + psum;
#pragma unroll
        for (int o = 0; o < 3; ++o) acc[o] *= alpha;
        if (mine) {
            const uint2 u0 = __builtin_bit_cast(uint2, pb[0]), u1 = __builtin_bit_cast(uint2, pb[1]);
            pl[wave * 64 + lane] = make_uint4(u0.x, u0.y, u1.x, u1.y);
#pragma unroll
            for (int t = 0; t < VT; ++t) *reinterpret_cast<u32x4_t*>(vt + (t * KPI + vks) * VSTRIDE + vdc * 16) = vr[t];
            if constexpr (!LAST) load_tile(vr, vbase, kb + KEYS);
        }
        lds_barrier();
        // ---- O^T += V^T P^T over the block's tiles, two at a time
        const int nt = min(NW, (k1 - kbb + 15) >> 4);
#pragma unroll
        for (int p = 0; p < NW / 2; ++p) {
            if (2 * p >= nt || (NB < NW && (p & 1) != wave / NB)) continue;       // (uniform)
            const bool both = 2 * p + 1 < nt;
            const int t0 = 2 * p, t1 = both ? t0 + 1 : t0;
            const uint4 w0 = pl[t0 * 64 + lane];
            uint4 w1 = pl[t1 * 64 + lane];
            if (!both) w1 = make_uint4(0u, 0u, 0u, 0u);
            const f16x8_t ph = __builtin_bit_cast(f16x8_t, make_uint4(w0.x, w0.y, w1.x, w1.y)), plo = __builtin_bit_cast(f16x8_t, make_uint4(w0.z, w0.w, w1.z, w1.w));
            f16x8_t v[2];
#pragma unroll
            for (int o = 0; o < 2; ++o) {
                // within a 16-lane group, lane i element e comes from the address of lane 4 e + i / 4, its element i % 4
                const char* src = vt_all + (4 * g + (n16 >> 2)) * VSTRIDE + (blk * 16 + 4 * (n16 & 3)) * 2 + o * HALFB;
                typedef unsigned long long u64x2_t __attribute__((ext_vector_type(2)));
                u64x2_t x;
                x[0] = __builtin_bit_cast(unsigned long long, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4_t*)(src + t0 * 16 * VSTRIDE)));
                x[1] = __builtin_bit_cast(unsigned long long, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4_t*)(src + t1 * 16 * VSTRIDE)));
                v[o] = __builtin_bit_cast(f16x8_t, x);
            }
            acc[0] = __builtin_amdgcn_mfma_f32_16x16x32_f16(v[1], ph, acc[0], 0, 0, 0);
            acc[1] = __builtin_amdgcn_mfma_f32_16x16x32_f16(v[0], plo, acc[1], 0, 0, 0);
            acc[2] = __builtin_amdgcn_mfma_f32_16x16x32_f16(v[0], ph, acc[2], 0, 0, 0);
        }
        kbb += KEYS;
        kb += KEYS;
    };
    while (kbb + KEYS < k1) block(std::false_type());
    if (kbb < k1) block(std::true_type());
    HIVIS_SMARK(3)
    // ---- denominators (and the halves of 64-wide heads) meet in LDS
    float lsum = lrun;
    lsum += __shfl_xor(lsum, 16, 64);
    lsum += __shfl_xor(lsum, 32, 64);
    if (g == 0) wm[n16 * NW + wave] = lsum;                              // (the maxima were read before the last barrier)
    f32x4_t o = acc[2] + (acc[0] + acc[1]);
    f32x4_t* const ex = reinterpret_cast<f32x4_t*>(kt_all);
    if (NB < NW && wave >= NB) ex[(wave - NB) * 64 + lane] = o;
    lds_barrier();
    float l = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) l += wm[n16 * NW + w];
    if (NB < NW && wave < NB) o += ex[wave * 64 + lane];
    const int d0 = blk * 16 + 4 * g;                                     // this lane: dims d0 .. + 3 of row n16
    if (a.nsplit == 1) {
        if (n16 < R && wave < NB) {
            const int row = sl * a.m + i0 + pi_, col = (kvh * a.group + h0 + ph_) * HD + d0;
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] /= l;
            if (a.frag_out) store_afrag4(a.frag_out, a.ldo / 32, row, col, o[0], o[1], o[2], o[3]);
            else if (a.rows_out) st_row_quad(a.rows_out, a.rows, row, col, o[0], o[1], o[2], o[3]);
            else { st_wt2(a.y + (size_t)row * a.ldo + col, o[0], o[1]); st_wt2(a.y + (size_t)row * a.ldo + col + 2, o[2], o[3]); }
        }
    } else {
        // one partial of the workgroup; the workgroup whose partial completes the item merges all of them: partial stored -> stores complete ->
        // arrive on the item's counter -> the last arriver reads the partials.  Every access is an agent-scope atomic (write-through stores, the
        // counter, the loads of the merge): that orders them for every XCD without writing back or invalidating an L2.
        float* const out = a.ws + ((size_t)(item * a.nsplit + split) * RM + n16) * (HD + 2);
        if (n16 < R && wave < NB) {
            st_wt2(out + d0, o[0], o[1]);
            st_wt2(out + d0 + 2, o[2], o[3]);
            if (wave == 0 && g == 0) st_wt2(out + HD, mrun, l);
        }
        if (a.cnt != nullptr) {
            wait_vmem();
            lds_barrier();
            if (threadIdx.x == 0) {
                if (!(a.flags & 1)) __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
                flag[0] = __hip_atomic_fetch_add(&a.cnt[item], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            lds_barrier();
            if (flag[0] == a.nsplit - 1) {
                if (!(a.flags & 1)) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
                AttnShape sh;
                sh.m = a.m;
                attn_merge_splits<HD, RM>(a.ws + (size_t)item * a.nsplit * RM * (HD + 2), a.nsplit, R, ni, kvh * a.group + h0, i0, sl, sh,
                                          reinterpret_cast<float*>(kt_all), AttnOut{a.y, a.ldo, a.rows_out, a.rows, a.frag_out});
                if (threadIdx.x == 0) st_wt(&a.cnt[item], 0);
            }
        }
    }
    HIVIS_SMARK(5)
#undef HIVIS_SMARK
    prof_leave(a.prof3, wg);
}

// One (item, key split) of an fp32 pass per workgroup (attn_wg_partial), launched by itself: its arguments come in one batch of scalar loads and item, head and
// sequence by reciprocals from the host.  (Divisions left: the group of grouped heads, and a split's keys where the splits are no power of two.)  Short passes are a
// chain of such latencies: 4 heads of 64 over 100..180 keys, one row 5.2 -> 4.0 us, five 6.1 -> 4.9 (as a phase of the general launch before).
struct AttnF32Args {
    const float* q; const float* kc; const float* vc; const int* base; float* ws; int* cnt; float* y; uint4* rows_out;
    int ldo, rows, items;
    FastDiv by_rblk, by_hblk, by_hkv;
    AttnShape sh;
    unsigned long long *prof2, *prof3;
};

template <int HD, int RC>
__global__ __launch_bounds__(FUSED_NT) void attn_f32_kernel(AttnF32Args a) {
    __shared__ __align__(16) float lds[FUSED_RMAX * HD + FUSED_NW * FUSED_RMAX * 16 + FUSED_NW * FUSED_RMAX * (HD + 2)];
    asm volatile("" :: "s"(a.q), "s"(a.kc), "s"(a.vc), "s"(a.base), "s"(a.ws), "s"(a.cnt), "s"(a.y), "s"(a.rows_out), "s"(a.ldo), "s"(a.rows), "s"(a.items), "s"(a.by_rblk.mul),
                      "s"(a.by_hblk.mul), "s"(a.by_hkv.mul));
    asm volatile("" :: "s"(a.sh.Hq), "s"(a.sh.Hkv), "s"(a.sh.m), "s"(a.sh.gh), "s"(a.sh.mi), "s"(a.sh.n_hblk), "s"(a.sh.n_rblk), "s"(a.sh.seq0), "s"(a.sh.offset), "s"(a.sh.maxL),
                      "s"(a.sh.nsplit), "s"(a.sh.ldq), "s"(a.sh.qrows), "s"(a.sh.flags), "s"(a.sh.nbase), "s"(a.prof2), "s"(a.prof3));
    const auto scalar = [](int x) { return __builtin_amdgcn_readfirstlane(x); };
    const int wg = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z);
    prof_enter(a.prof3, wg);
    // (grids as in attn_split_kernel)
    const bool xcd_map = (a.sh.flags & 2) != 0;
    const int split = blockIdx.y, item = scalar(xcd_map ? blockIdx.x + 8 * blockIdx.z : blockIdx.x);
    if (item >= a.items) return;
    const int i1 = scalar(a.by_rblk(item)), i2 = scalar(a.by_hblk(i1)), sl = scalar(a.by_hkv(i2));
    const AttnItem it = {item - i1 * a.sh.n_rblk, i1 - i2 * a.sh.n_hblk, i2 - sl * a.sh.Hkv, sl, a.sh.n_hblk == 1 && a.sh.Hq == a.sh.Hkv ? 1 : a.sh.Hq / a.sh.Hkv};
    attn_wg_partial<float, HD, FUSED_RMAX, RC>(a.q, a.kc, a.vc, a.base, a.sh, it, item, split, lds, a.ws, a.cnt, AttnOut{a.y, a.ldo, a.rows_out, a.rows}, wg == 0 ? a.prof2 : nullptr);
    prof_leave(a.prof3, wg);
}

// The same with every wavefront on its own (attn_wg_mfma: tiles of 16 keys, a softmax per wavefront, merged at the end), for workgroups that walk many blocks of 128 keys
// (attn_walks): a prompt's last 128 of 3008 rows, 32 heads, 78 -> 63 us in a traced request.
struct AttnTilesArgs {
    const float* q; const f16_t* kc; const f16_t* vc; const int* base; float* ws; int* cnt;
    AttnOut out;
    int items;
    FastDiv by_rblk, by_hblk, by_hkv;
    AttnShape sh;
    unsigned long long *prof2, *prof3;
};

template <int HD, int RM, bool ONCE>
__global__ __launch_bounds__(FUSED_NT) void attn_tiles_kernel(AttnTilesArgs a) {
    extern __shared__ __align__(16) char attn_lds[];
    const auto scalar = [](int x) { return __builtin_amdgcn_readfirstlane(x); };
    const int wg = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z);
    prof_enter(a.prof3, wg);
    // (grids as in attn_split_kernel)
    const bool xcd_map = (a.sh.flags & 2) != 0;
    const int z = scalar(xcd_map ? blockIdx.z : blockIdx.y), split = scalar(xcd_map ? blockIdx.y : blockIdx.x);
    const int zh = scalar(a.by_rblk(z)), rblk = z - zh * a.sh.n_rblk, i1 = scalar(xcd_map ? blockIdx.x + 8 * zh : zh), item = i1 * a.sh.n_rblk + rblk;
    if (item >= a.items) return;
    const int i2 = scalar(a.by_hblk(i1)), sl = scalar(a.by_hkv(i2));
    const AttnItem it = {rblk, i1 - i2 * a.sh.n_hblk, i2 - sl * a.sh.Hkv, sl, a.sh.Hq == a.sh.Hkv ? 1 : a.sh.Hq / a.sh.Hkv};
    attn_wg_mfma<HD, RM, ONCE>(a.q, a.kc, a.vc, a.base, a.sh, it, item, split, reinterpret_cast<float*>(attn_lds), a.ws, a.cnt, a.out, wg == 0 ? a.prof2 : nullptr);
    prof_leave(a.prof3, wg);
}

}  // namespace hivis
