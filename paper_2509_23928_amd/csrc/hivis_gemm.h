// Dense MFMA GEMM of the prefill (hundreds to thousands of activation rows, bf16 weights) and its operand layout.
#pragma once
#include "hivis_kernels.h"
#include "hivis_sizes.h"

namespace hivis {

// ------------------------------------------------------------------------------------------
// Activation fragments.  Every fp32 activation is split into a bf16 high and a bf16 low part (about 16 mantissa bits).  A
// row tile holds 16 rows; for each block of 32 k-values it has one 1 KiB fragment block of high parts followed by one of
// low parts:
//   frag[((row / 16) * kblks + k / 32) * 2 + part][piece(row % 16, (k / 8) % 4)] (16 bytes, 8 k-values each)
// One weight fragment serves two MFMAs per row tile.
// A row's four pieces of a block are 64 contiguous bytes: the kernels that write fragments work on a row (RMSNorm) or on some
// columns of a few rows, and what they wait for is the number of 64-byte segments their stores touch.  In the MFMA's own lane order
// (row + 16 g, a row's pieces 256 bytes apart) the 61-row verify of the 7B widths took 5.38 ms, now 5.31, the 32-row verify of
// the 13B batch 8.30, now 8.17.  The lane that needs piece (row, g) picks it when it reads LDS; the order of the four pieces
// changes with row / 4, so that the 16 lanes of one g then hit all banks.
// ------------------------------------------------------------------------------------------
__device__ __forceinline__ int afrag_piece(int row, int g) { return 4 * row + (g ^ (row >> 2)); }       // row < 16, g < 4
__device__ __forceinline__ size_t afrag_at(int kblks, int row, int k) {
    return (((size_t)(row >> 4) * kblks + (k >> 5)) * 2) * 64 + afrag_piece(row & 15, (k >> 3) & 3);
}
// 8 consecutive values x[0..8) of row `row` at k (a multiple of 8) -> the high and the low chunk
__device__ __forceinline__ void store_afrag8(uint4* __restrict__ frag, int kblks, int row, int k, const float (&x)[8], bool zero) {
    const size_t at = afrag_at(kblks, row, k);
    uint32_t hi[4], lo[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        f32_to_bf16x2_hilo(x[2 * e], x[2 * e + 1], hi[e], lo[e]);
        if (zero) { hi[e] = 0u; lo[e] = 0u; }
    }
    frag[at] = make_uint4(hi[0], hi[1], hi[2], hi[3]);
    frag[at + 64] = make_uint4(lo[0], lo[1], lo[2], lo[3]);
}
// 4 consecutive values of row `row` at k (a multiple of 4) -> half of the high and of the low chunk
__device__ __forceinline__ void store_afrag4(uint4* __restrict__ frag, int kblks, int row, int k, float a, float b, float c, float d) {
    uint2* at = reinterpret_cast<uint2*>(frag + afrag_at(kblks, row, k)) + ((k >> 2) & 1);
    uint2 hi, lo;
    f32_to_bf16x2_hilo(a, b, hi.x, lo.x);
    f32_to_bf16x2_hilo(c, d, hi.y, lo.y);
    at[0] = hi;
    at[128] = lo;
}

// 2 consecutive values of row `row` at k (even)
__device__ __forceinline__ void store_afrag2(uint4* __restrict__ frag, int kblks, int row, int k, float a, float b) {
    uint32_t* at = reinterpret_cast<uint32_t*>(frag + afrag_at(kblks, row, k)) + ((k >> 1) & 3);
    f32_to_bf16x2_hilo(a, b, at[0], at[256]);
}

// rows of fp32 -> fragments; rows >= M of the last row tile become zeros
__global__ void pack_afrag_kernel(const float* __restrict__ A, int lda, int M, int kblks, uint4* __restrict__ out) {
    const size_t total = (size_t)((M + 15) / 16) * 16 * kblks * 4;        // one thread per chunk of 8 values
    for (size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x; idx < total; idx += (size_t)gridDim.x * blockDim.x) {
        // 16 rows x 4 chunks of one K block are one 1 KiB block: four consecutive threads write 64 contiguous bytes of it
        const int g = (int)(idx & 3), i = (int)((idx >> 2) & 15);
        const size_t blk = idx >> 6;
        const int kb = (int)(blk % (size_t)kblks), row = (int)(blk / (size_t)kblks) * 16 + i, k = kb * 32 + g * 8;
        const float4* p = reinterpret_cast<const float4*>(A + (size_t)min(row, M - 1) * lda + k);
        const float4 x0 = p[0], x1 = p[1];
        const float x[8] = {x0.x, x0.y, x0.z, x0.w, x1.x, x1.y, x1.z, x1.w};
        store_afrag8(out, kblks, row, k, x, row >= M);
    }
}

// A GEMM result as K-slice partials: value = sum over s < n of p[s * stride + index], in that order
struct Parts { const float* p; int n; size_t stride; };

// B slices per trip, their loads issued together (a one-load-per-trip loop costs a memory round trip per slice)
template <int B>
__device__ __forceinline__ void parts_add(float4& a, const Parts& ps, size_t idx, int s0) {
    for (int s = s0; s < ps.n; s += B) {
        float4 v[B];
#pragma unroll
        for (int j = 0; j < B; ++j) v[j] = *reinterpret_cast<const float4*>(ps.p + (size_t)min(s + j, ps.n - 1) * ps.stride + idx);
#pragma unroll
        for (int j = 0; j < B; ++j)
            if (s + j < ps.n) { a.x += v[j].x; a.y += v[j].y; a.z += v[j].z; a.w += v[j].w; }
    }
}
__device__ __forceinline__ float4 parts_load4(const Parts& ps, size_t idx) {
    float4 a = *reinterpret_cast<const float4*>(ps.p + idx);
    if (ps.n <= 4) parts_add<3>(a, ps, idx, 1);       // slices 1..3 in one trip
    else parts_add<8>(a, ps, idx, 1);
    return a;
}

// Y[r][c] = sum of the partials, rows gridDim.x, c < N (N a multiple of 4)
__global__ void splitk_reduce_kernel(Parts ps, int N, int ldp, float* __restrict__ Y, int ldy) {
    const int row = blockIdx.x;
    for (int c4 = blockIdx.y * blockDim.x + threadIdx.x; c4 < N / 4; c4 += gridDim.y * blockDim.x)
        *reinterpret_cast<float4*>(Y + (size_t)row * ldy + 4 * c4) = parts_load4(ps, (size_t)row * ldp + 4 * c4);
}

typedef unsigned v4u_t __attribute__((ext_vector_type(4)));

// One 1 KiB block from memory straight to LDS (no registers): lane l's 16 bytes go to lds[l].
__device__ __forceinline__ void block_to_lds(const v4u_t* src, v4u_t* lds) {
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src, (__attribute__((address_space(3))) void*)lds, 16, 0, 0);
}

// The same from a buffer: lane l's 16 bytes, at byte `off` of the buffer, go to lds[l] (beyond the buffer: no access, LDS undefined)
__device__ __forceinline__ void buffer_to_lds(__amdgpu_buffer_rsrc_t r, v4u_t* lds, int off) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)lds, 16, off, 0, 0, 0);
}

// ------------------------------------------------------------------------------------------
// Tall GEMM: 128 rows x 32 CW columns per workgroup of 8 wavefronts.  They are two groups of four, one wavefront of each
// group per SIMD; the first group multiplies the even K blocks of the tile, the second the odd ones, and at the end they
// exchange halves of their sums through LDS.  The groups work in opposite phases separated by barriers: while one multiplies
// a K block (8 CW MFMAs per wavefront, operands in registers), the other reads its next fragments from LDS and
// requests a later block, so the matrix pipeline of every SIMD always has a wavefront that issues nothing but MFMAs.
// Blocks go from memory to LDS directly (they are in fragment order already) into a ring of four K blocks.  A wavefront
// owns 64 rows x 16 CW columns: 4 x CW accumulator tiles; the weights are the MFMA's A operand, so that a lane ends up with
// four consecutive columns of one row.
// Both parts add into the SAME accumulators (there are no registers for two sets).  That rounds twice as often at the high parts'
// magnitude, but each group's sum has half the K blocks: together the error of the sums alone is that of one sum over all of K with the
// low parts beside it (4.0e-7 of the result for both at K = 4096, 6.7e-7 at K = 11008; the 16 mantissa bits of the operands leave 2.5e-6).
// Bound by power: with random data the MFMAs alone run at 2.0 PFLOP/s on this card (2.46 on zeros), a library product of 8192^3 at 1.13,
// and this kernel's loop takes 136 thousand cycles of a 224-column tile at K = 4096 (115 are MFMAs) whatever the data: 57 us at 2.39 GHz on
// zeros, 77 at 1.76 on random data.  So what the MFMAs switch counts.  640 rows x 22016 columns, launches back to back, by their order: column
// tiles outside, row tiles inside, the part outermost 164.4 us; the same with one operand kept from each to the next 161; both parts of
// an accumulator in turn 158; and a row tile outside, so that each operand changes at every second product, 156.2 (1.48 PFLOP/s).
// 640 rows, K = 4096, high and low parts counted, before the two groups: 22016 columns 249 us, 12288 columns 127; 3008 x 22016: 1090.  The version with the requests
// at the head of the multiplication phase took 203 and 107 us; groups owning row halves instead of K blocks (256-row
// tiles) were no faster at 3008 rows and left too few tiles at 640.
// ------------------------------------------------------------------------------------------
constexpr int TALL_THREADS = 512;
// (a ring of four K blocks; at the end one area of 64 rows x 64 columns per wavefront)
template <int CW> constexpr int tall_lds_bytes() { return 4 * (16 + 2 * CW) > 128 ? 4 * (16 + 2 * CW) * 1024 : 128 * 1024; }

#define HIVIS_PHASE_END(wait_)                               \
    do {                                                     \
        __builtin_amdgcn_sched_barrier(0);                   \
        asm volatile("s_waitcnt " wait_ "\n\ts_barrier" ::: "memory"); \
        __builtin_amdgcn_sched_barrier(0);                   \
    } while (0)

// What becomes of the result:
//   TALL_STORE  fp32 rows; ksplit > 1: the K range is cut into slices, slice s writes its sums to part[s][M][ldy] and the
//               consumer adds them
//   TALL_SILU   W = gate|up (8 + 8 columns per tile): silu(gate) * up leaves as activation fragments of the down projection
//   TALL_QKV    W = q|k|v of whole prompts: bias and rotary embedding applied; q leaves as fp32 rows, k and v go to the cache
//               (row of sequence seq0 + row / m at position row % m)
// (the fp32 rows of gate|up and q|k|v were the largest results of a layer: writing them here and reading them in a row kernel
// cost 20 + 22 us per layer at 640 rows and 112 + 103 us at 3008, beside the GEMMs' own stores)
enum { TALL_STORE = 0, TALL_SILU = 1, TALL_QKV = 2 };
struct TallOut {
    float* Y; int ldy;
    float* part;
    uint4* frag; int kblks_out;
    const float* bias; const float* rope; int npos;       // [q_dim + 2 kv_dim] or null; table of (cos, sin) per position and pair
    int seq0, m, qd, kd, HD, Hkv, maxL;
    f16_t *kc, *vc;
};

// A wavefront's finished 64 rows x NT column tiles, in its own LDS area as [64][4 NT] pieces of four columns (piece p of row
// r at p ^ (r & 15) of 16, so that neither side conflicts), to memory: consecutive lanes take consecutive pieces of a row (for
// fragments its NT column tiles: up to 64 contiguous bytes), so that stores cover whole segments (straight from the
// accumulators a store touched 16 rows, 32 bytes of each in the cache: q|k|v of 640 rows 115 us against 94 us for plain rows).
template <int NT, int EPI>
__device__ __forceinline__ void tall_write(const TallOut& o, const v4u_t* area, int row0, int ct0, int M, int ntiles, float* Y, int lane) {
    if constexpr (EPI == TALL_SILU) {
        for (int it = lane; it < 64 * NT; it += 64) {
            const int r = it / NT, t = it % NT, row = row0 + r;
            f32x4_t p[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) p[e] = __builtin_bit_cast(f32x4_t, area[r * 16 + ((4 * t + e) ^ (r & 15))]);
            if (row < M && ct0 + t < ntiles) {
                float y[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) { const float ga = p[e >> 2][e & 3], up = p[2 + (e >> 2)][e & 3]; y[e] = ga / (1.0f + expf(-ga)) * up; }
                store_afrag8(o.frag, o.kblks_out, row, 8 * (ct0 + t), y, false);
            }
        }
    } else {
        // a lane keeps one piece (four columns) and walks the rows, RPI rows per trip
        constexpr int P = 4 * NT, RPI = 64 / P, TRIPS = (64 + RPI - 1) / RPI;
        const int p = lane % P, col = ct0 * 16 + 4 * p;
        int r = lane / P;
        if (r >= RPI || ct0 + (p >> 2) >= ntiles) return;
        if constexpr (EPI == TALL_STORE) {
#pragma unroll 4
            for (int i = 0; i < TRIPS; ++i, r += RPI)
                if (r < 64 && row0 + r < M) *reinterpret_cast<v4u_t*>(Y + (size_t)(row0 + r) * o.ldy + col) = area[r * 16 + (p ^ (r & 15))];
        } else {
            const bool isq = col < o.qd, isk = !isq && col < o.qd + o.kd;
            const int head = (col - (isq ? 0 : isk ? o.qd : o.qd + o.kd)) / o.HD, c = col % o.HD;
            f32x4_t bias = f32x4_t{0.f, 0.f, 0.f, 0.f};
            if (o.bias) bias = *reinterpret_cast<const f32x4_t*>(o.bias + col);
            int s = (row0 + r) / o.m, pos = row0 + r - s * o.m;
            typedef _Float16 h4_t __attribute__((ext_vector_type(4)));
            // (four rows per trip, their table entries requested together: one memory round trip per row cost 13 us per tile)
            constexpr int U = 4;
            for (int i = 0; i < TRIPS; i += U) {
                f32x4_t t[U], x[U];
                int sq[U], ps[U], rw[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    sq[u] = o.seq0 + s; ps[u] = pos; rw[u] = r;
                    t[u] = *reinterpret_cast<const f32x4_t*>(o.rope + (size_t)min(pos, o.npos - 1) * o.HD + c);
                    x[u] = __builtin_bit_cast(f32x4_t, area[min(r, 63) * 16 + (p ^ (r & 15))]);
                    r += RPI; pos += RPI;
                    while (pos >= o.m) { pos -= o.m; ++s; }
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    if (rw[u] >= 64 || row0 + rw[u] >= M) continue;
                    f32x4_t y = x[u] + bias;
                    if (isq || isk) {
                        // columns 2i, 2i+1 of a head are the rotary pair (i, i + HD/2); two pairs
                        float z[4];
                        rotate_pair(y[0], y[1], t[u][0], t[u][1], z[0], z[1]);
                        rotate_pair(y[2], y[3], t[u][2], t[u][3], z[2], z[3]);
                        y = f32x4_t{z[0], z[1], z[2], z[3]};
                    }
                    if (isq) *reinterpret_cast<f32x4_t*>(o.Y + (size_t)(row0 + rw[u]) * o.ldy + col) = y;
                    else {
                        f16_t* dst = (isk ? o.kc : o.vc) + (((size_t)sq[u] * o.Hkv + head) * o.maxL + ps[u]) * o.HD * 2 + c;
                        h4_t hi, lo;
#pragma unroll
                        for (int e = 0; e < 4; ++e) { hi[e] = (f16_t)fminf(fmaxf(y[e], -65504.f), 65504.f); lo[e] = (f16_t)(y[e] - (float)hi[e]); }
                        *reinterpret_cast<h4_t*>(dst) = hi;
                        *reinterpret_cast<h4_t*>(dst + o.HD) = lo;
                    }
                }
            }
        }
    }
}

template <int CW, int EPI>
__global__ __launch_bounds__(TALL_THREADS, 2) void gemm_tall_kernel(const v4u_t* __restrict__ Af, int row_tiles, int kblks,
                                                                   const v4u_t* __restrict__ Wp, int ntiles, int M, int ksplit, TallOut o) {
    constexpr int RT = TALL_ROWS / 16, CT = 2 * CW;       // row and column tiles of the workgroup
    constexpr int NA = 2 * RT, NBLK = NA + CT;            // blocks of one K block
    constexpr int PER = (NBLK + 3) / 4;                   // blocks each wavefront of a group fetches per K block
    static_assert(PER == 7 || PER == 8, "the counted waits below");
    extern __shared__ __align__(16) v4u_t tall_lds[];     // [4 K blocks][NBLK][64]
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int grp = wave >> 2, w4 = wave & 3;
    const int piece = afrag_piece(lane & 15, lane >> 4);
    // Tiles are numbered so that neighbours share operands (up to 8 row blocks of one column block, then the next column
    // block; K slices outermost) and every XCD (workgroup L runs on XCD L % 8) takes one contiguous range of them: its L2
    // sees a compact patch of row and column blocks.
    const int ncol = (ntiles + CT - 1) / CT, nrow = (row_tiles + RT - 1) / RT;
    const int total = ncol * nrow * ksplit, chunk = (total + 7) / 8;
    const int slot = blockIdx.x / 8, id = (blockIdx.x % 8) * chunk + slot;
    if (slot >= chunk || id >= total) return;
    const int split = id / (ncol * nrow), tid = id % (ncol * nrow);
    const int npanel = (nrow + 7) / 8, prows = (nrow + npanel - 1) / npanel;
    const int panel = tid / (prows * ncol), inp = tid - panel * prows * ncol, pr = min(prows, nrow - panel * prows);
    const int rblk = panel * prows + inp % pr, cblk = inp / pr;
    const int kper = (kblks + ksplit - 1) / ksplit, kbeg = split * kper, nkb = min(kblks, kbeg + kper) - kbeg;
    const int rt_wg = rblk * RT, ct_wg = cblk * CT;

    // the blocks this wavefront fetches per K block: id b < NA is the high / low part b & 1 of row tile b / 2, else column
    // tile b - NA (tiles outside the matrix are replaced by the last one: their results are not stored)
    const v4u_t* src[PER];
    int inc[PER], dst[PER];                               // distance to the same block of the next K block; place in the stage
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int b = min(w4 + 4 * i, NBLK - 1);
        const bool isa = b < NA;
        src[i] = isa ? Af + (((size_t)min(rt_wg + (b >> 1), row_tiles - 1) * kblks + kbeg) * 2 + (b & 1)) * 64
                     : Wp + ((size_t)min(ct_wg + (b - NA), ntiles - 1) * kblks + kbeg) * 64;
        inc[i] = isa ? 128 : 64;
        dst[i] = b * 64;
    }
#define HIVIS_TALL_FETCH(kb_)                                                                                      \
    do {                                                                                                           \
        v4u_t* to_ = tall_lds + (size_t)((kb_) & 3) * NBLK * 64;                                                    \
        _Pragma("unroll") for (int i = 0; i < PER; ++i) block_to_lds(src[i] + (size_t)(kb_) * inc[i] + lane, to_ + dst[i]); \
    } while (0)
    // step s of group g is K block 2 s + g
    const int nsteps = (nkb + 1) / 2, mine = (nkb + 1 - grp) / 2;
    if (grp == 1) {
        HIVIS_TALL_FETCH(0);
        if (nkb > 2) HIVIS_TALL_FETCH(2);
    } else if (nkb > 1) HIVIS_TALL_FETCH(1);

    f32x4_t acc[4][CW];
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int c = 0; c < CW; ++c) acc[r][c] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    const int wr = w4 >> 1, wc = w4 & 1;                  // this wavefront's 4 row tiles and CW column tiles
    v4u_t fa[2][4], fb[CW];

    HIVIS_PHASE_END("vmcnt(0)");
    if (grp == 1) HIVIS_PHASE_END("lgkmcnt(0)");          // the second group runs one phase behind
    for (int s = 0; s < nsteps; ++s) {
        // Memory phase: the fragments of this step, then the request for a block of the OTHER group, whose stage that group
        // read one phase ago.  The block requested in this group's previous memory phase has had three phases to arrive; it is
        // waited for here, one phase before the other group reads it.
        if (s < mine) {
            const v4u_t* at = tall_lds + (size_t)((2 * s + grp) & 3) * NBLK * 64 + lane;
            const v4u_t* aa = tall_lds + (size_t)((2 * s + grp) & 3) * NBLK * 64 + piece;
#pragma unroll
            for (int r = 0; r < 4; ++r) { fa[0][r] = aa[(size_t)(2 * (wr * 4 + r)) * 64]; fa[1][r] = aa[(size_t)(2 * (wr * 4 + r) + 1) * 64]; }
#pragma unroll
            for (int c = 0; c < CW; ++c) fb[c] = at[(size_t)(NA + wc * CW + c) * 64];
        }
        const int nk = 2 * s + 3 + grp;
        __builtin_amdgcn_sched_barrier(0);
        if (nk < nkb) {
            HIVIS_TALL_FETCH(nk);
            if constexpr (PER == 7) HIVIS_PHASE_END("vmcnt(7) lgkmcnt(0)"); else HIVIS_PHASE_END("vmcnt(8) lgkmcnt(0)");
        } else HIVIS_PHASE_END("vmcnt(0) lgkmcnt(0)");
        // multiplication phase
        if (s < mine) {
            __builtin_amdgcn_s_setprio(1);
            // both parts of an accumulator one after the other, and from one product to the next one operand stays (fixed by the fences)
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int c_ = 0; c_ < CW; ++c_)
#pragma unroll
                    for (int p_ = 0; p_ < 2; ++p_) {
                        const int c = (r & 1) ? CW - 1 - c_ : c_, p = ((r * CW + c_) & 1) ? 1 - p_ : p_;
                        acc[r][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, fb[c]), __builtin_bit_cast(bf16x8_t, fa[p][r]), acc[r][c], 0, 0, 0);
                        __builtin_amdgcn_sched_barrier(0);
                    }
            __builtin_amdgcn_s_setprio(0);
        }
        HIVIS_PHASE_END("lgkmcnt(0)");
    }
    if (grp == 0) HIVIS_PHASE_END("lgkmcnt(0)");
#undef HIVIS_TALL_FETCH

    // the groups swap halves of their partial sums: group 0 finishes column tiles [0, CH), group 1 the rest
    constexpr int CH = (CW + 1) / 2;
    v4u_t* ex = tall_lds + lane;
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int c = 0; c < CW; ++c)
            if ((c < CH) == (grp == 1)) ex[(size_t)((w4 * 4 + r) * CW + c) * 64] = __builtin_bit_cast(v4u_t, acc[r][c]);
    HIVIS_PHASE_END("lgkmcnt(0)");
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int c = 0; c < CW; ++c)
            if ((c < CH) == (grp == 0)) acc[r][c] += __builtin_bit_cast(f32x4_t, ex[(size_t)((w4 * 4 + r) * CW + c) * 64]);
    float* const Y = (EPI == TALL_STORE && ksplit > 1) ? o.part + (size_t)split * M * o.ldy : o.Y;
    HIVIS_PHASE_END("lgkmcnt(0)");                        // every exchanged tile has been read
    v4u_t* const area = tall_lds + (size_t)wave * 64 * 16;
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int c = 0; c < CW; ++c)
            if ((c < CH) == (grp == 0)) {
                const int rr = 16 * r + (lane & 15), p = 4 * (c < CH ? c : c - CH) + (lane >> 4);
                area[rr * 16 + (p ^ (rr & 15))] = __builtin_bit_cast(v4u_t, acc[r][c]);
            }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const int row0 = (rt_wg + wr * 4) * 16, ct0 = ct_wg + wc * CW;
    if (grp == 0) tall_write<CH, EPI>(o, area, row0, ct0, M, ntiles, Y, lane);
    else tall_write<CW - CH, EPI>(o, area, row0, ct0 + CH, M, ntiles, Y, lane);
}

// ------------------------------------------------------------------------------------------
// Wide GEMM (up to 64 activation rows: the weights are streamed once).  A workgroup of 8 wavefronts computes all rows x (8 / KW) CT
// column tiles over one K slice (kper K blocks, slice blockIdx.x); slice s writes its sums to part[s][M][ldy] and the consuming row kernel
// adds them.  HBM bound, one workgroup per CU:
//   * A weight block serves one wavefront only, so it goes from memory to that wavefront's registers, NBUF stages of four K blocks ahead
//     (64..192 KB in flight per workgroup); the loop requests a block's successor right behind its products, nothing in it is
//     conditional, and the compiler counts its waits.
//   * The activations go from memory to a ring of R stages in LDS without registers, shared by all wavefronts; one barrier per stage.
//   * A wavefront reads the fragments of every row (8 KB per K block at 64 rows) to multiply CT weight blocks with them, so KW
//     wavefronts share a column group and take 4 / KW K blocks of a stage each: with one column tile per wavefront the reads from LDS were the
//     limit (O, 61 rows: 13.9 us, now 11.2; down 27.2, now 21.6).  They add their sums through LDS at the end.
// The columns of a workgroup decide how often the activations are read (once per column block), the slices how often the sums are written
// and read again: wide_plan.  Against the form before (4 wavefronts, 128 columns, both operands through registers and LDS, up to 16 slices and
// 768 workgroups, whose activations were as many bytes as its weights), us per launch back to back, before -> now; in brackets this kernel
// without activations and products: 61 rows, 7B widths: q|k|v 28.4 -> 22.6 (22.9), O 12.6 -> 11.2 (9.5), gate|up 44.4 -> 34.5 in two slices,
// 39.8 in one with SiLU and the fragments written (34.5), down 25.2 -> 21.6 (18.9), LM head 58.5 -> 49.3, in one slice (48.8).  31 rows, 3584 wide:
// gate|up 54.6 -> 46.8 with SiLU, down 30.3 -> 24.5, LM head of 152064 columns 232 -> 186.  32 rows, 5120 wide: 32 -> 28, 14.2 -> 12.3, 56 -> 47, 29.3 ->
// 24.9, 66 -> 52.5.  Starting the slices' K blocks at different places changed nothing or cost 2-10 us.
// The low parts have accumulators of their own, added at the end: rounded at the high parts' magnitude instead, the K sum's
// error was 1.4 times as large (61 rows, K = 4096 in 3 slices: 3.2e-7 of the result, now 2.2e-7).
//   WIDE_STORE  fp32 rows (Y, row stride ldy; gridDim.x > 1: slices)
//   WIDE_SILU   W = gate|up (8 + 8 columns per tile), one slice: silu(gate) * up leaves as activation fragments (frag, kblks_out K blocks);
//               the row kernel that did it took 8 us and the slices' traffic
// ------------------------------------------------------------------------------------------
constexpr int WIDE_THREADS = 512;
enum { WIDE_STORE = 0, WIDE_SILU = 1 };
template <int RT, int KW, int CT> struct WideCfg {
    static constexpr int SK = WIDE_STAGE, J = SK / KW;                // K blocks of a stage; of it per wavefront
    static constexpr int NBUF = J * CT <= 4 ? 4 : 2;                  // stages of weights in flight
    static constexpr int R = RT == 4 && NBUF == 2 ? 3 : 4;            // stages of activations in LDS
    static constexpr int STAGE = SK * RT * 2 * 64;                    // 16-byte pieces of a stage
    // memory operations requested behind the activations of a stage by the time it is read, at the least: those of R - 2 further stages of
    // activations, and the weights of as many stages as lie between the two points (R - 1) or were requested before the loop (NBUF)
    static constexpr int BEHIND = (NBUF < R - 1 ? NBUF : R - 1) * J * CT + (R - 2) * RT;
    static constexpr int EXCHANGE = (8 / KW) * CT * (KW - 1) * RT * 64;
    static constexpr int LDS = 16 * (R * STAGE > EXCHANGE ? R * STAGE : EXCHANGE);
    static_assert(BEHIND < 64 && LDS <= 160 * 1024 && SK * 2 == WIDE_THREADS / 64, "a wavefront per block of a row tile's stage");
};

template <int RT, int KW, int CT, int EPI>
__global__ __launch_bounds__(WIDE_THREADS) void gemm_wide_kernel(const uint4* __restrict__ Af, int row_tiles, int kblks, int kper, const uint4* __restrict__ Wp,
                                                                int ntiles, int M, float* __restrict__ Y, int ldy, float* __restrict__ part,
                                                                uint4* __restrict__ frag, int kblks_out) {
    typedef WideCfg<RT, KW, CT> CF;
    constexpr int NBUF = CF::NBUF, R = CF::R, SK = CF::SK, J = CF::J;
    extern __shared__ __align__(16) v4u_t tall_lds[];                 // [R][RT][K block, part][64]
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int kg = wave % KW, cg = wave / KW;
    const int piece = afrag_piece(lane & 15, lane >> 4);
    // (blockIdx.x varies fastest: the K slices of a column block on different XCDs)
    const int kb0 = blockIdx.x * kper, nkb = min(kblks - kb0, kper), nst = (nkb + SK - 1) / SK;       // >= 1: no slice is empty
    const int ct0 = (blockIdx.y * (8 / KW) + cg) * CT;
    if (gridDim.x > 1) Y = part + (size_t)blockIdx.x * M * ldy;

    // Activations: wavefront w copies block w (K block w / 2, part w % 2) of every row tile of a stage.  Loads beyond the K slice, the row
    // tiles or the column tiles do not access memory; weights then are zeros, but LDS keeps what it held (a row's Inf or NaN of another
    // K block, say), so the blocks that fill up the last stage are cleared.  (Row tiles that do not exist: rows that are not stored.)
    const __amdgpu_buffer_rsrc_t ra = buffer_of(Af, row_tiles * kblks * 2048);
    int aoff[RT];
#pragma unroll
    for (int i = 0; i < RT; ++i) aoff[i] = i < row_tiles ? (i * kblks + kb0) * 2048 + wave * 1024 : OUT_OF_RANGE;
    auto fetch_rows = [&](int s) {
        v4u_t* const to = tall_lds + (s % R) * CF::STAGE + wave * 64;
        const bool in = SK * s + (wave >> 1) < nkb;
#pragma unroll
        for (int i = 0; i < RT; ++i)
            buffer_to_lds(ra, to + i * SK * 128, (in ? aoff[i] + s * (SK * 2048) : OUT_OF_RANGE) + lane * 16);
        if (!in && s < nst) {
#pragma unroll
            for (int i = 0; i < RT; ++i) to[i * SK * 128 + lane] = v4u_t{0, 0, 0, 0};
        }
    };
    __amdgpu_buffer_rsrc_t rw[CT];
#pragma unroll
    for (int c = 0; c < CT; ++c) rw[c] = buffer_of(Wp + ((size_t)min(ct0 + c, ntiles - 1) * kblks + kb0) * 64, ct0 + c < ntiles ? nkb * 1024 : 0);
    bf16x8_t w[NBUF][J][CT];
    // (the fences keep the weights' requests in the order of their use: a wait is for everything up to a request)
    auto fetch_block = [&](bf16x8_t& d, int s, int j, int c) {
        d = __builtin_bit_cast(bf16x8_t, __builtin_amdgcn_raw_buffer_load_b128(rw[c], lane * 16 + s * (SK * 1024) + kg * (J * 1024) + j * 1024, 0, 2));      // 2: non-temporal
        __builtin_amdgcn_sched_barrier(0x38F);                        // everything but vector memory may pass
    };
    f32x4_t acc[2][RT][CT];
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int r = 0; r < RT; ++r)
#pragma unroll
            for (int c = 0; c < CT; ++c) acc[p][r][c] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < (NBUF > R - 1 ? NBUF : R - 1); ++s) {
        if (s < R - 1) fetch_rows(s);
        __builtin_amdgcn_sched_barrier(0);
        if (s < NBUF) {
#pragma unroll
            for (int j = 0; j < J; ++j)
#pragma unroll
                for (int c = 0; c < CT; ++c) fetch_block(w[s][j][c], s, j, c);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    for (int s0 = 0;; s0 += NBUF) {
#pragma unroll
        for (int u = 0; u < NBUF; ++u) {
            const int s = s0 + u;
            // the activations of stage s have arrived (what was requested behind them may be in flight), and every wavefront has read stage s - 1
            __builtin_amdgcn_sched_barrier(0);
            asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(CF::BEHIND) : "memory");
            __builtin_amdgcn_sched_barrier(0);
            fetch_rows(s + R - 1);
            __builtin_amdgcn_sched_barrier(0);
            const v4u_t* at = tall_lds + (s % R) * CF::STAGE + kg * (J * 128) + piece;
#pragma unroll
            for (int j = 0; j < J; ++j) {
                bf16x8_t a[2][RT];
#pragma unroll
                for (int r = 0; r < RT; ++r)
#pragma unroll
                    for (int p = 0; p < 2; ++p) a[p][r] = __builtin_bit_cast(bf16x8_t, at[(r * SK * 2 + 2 * j + p) * 64]);
#pragma unroll
                for (int c = 0; c < CT; ++c) {
#pragma unroll
                    for (int p = 0; p < 2; ++p)
#pragma unroll
                        for (int r = 0; r < RT; ++r) acc[p][r][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[u][j][c], a[p][r], acc[p][r][c], 0, 0, 0);
                    fetch_block(w[u][j][c], s + NBUF, j, c);
                }
            }
            if (s + 1 >= nst) goto summed;                            // (uniform; leaving is the only branch, so the waits inside stay exact)
        }
    }
summed:
    wait_vmem();                                                      // (the last requests: zeros to a ring that the exchange reuses)
    // the wavefronts of a column group share its column tiles out: tile c is finished by wavefront c % KW of them
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    f32x4_t* const ex = reinterpret_cast<f32x4_t*>(tall_lds) + cg * CT * (KW - 1) * RT * 64 + lane;
#pragma unroll
    for (int c = 0; c < CT; ++c)
        if (c % KW != kg) {
#pragma unroll
            for (int r = 0; r < RT; ++r) ex[((c * (KW - 1) + kg - (kg > c % KW)) * RT + r) * 64] = acc[0][r][c] + acc[1][r][c];
        }
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
    for (int c = 0; c < CT; ++c) {
        if (c % KW != kg || ct0 + c >= ntiles) continue;              // (uniform)
#pragma unroll
        for (int r = 0; r < RT; ++r) {
            f32x4_t v = acc[0][r][c] + acc[1][r][c];
#pragma unroll
            for (int k = 0; k < KW - 1; ++k) v += ex[((c * (KW - 1) + k) * RT + r) * 64];
            // this lane: columns 4 (lane / 16) .. + 3 of the tile, one row
            const int row = r * 16 + (lane & 15);
            if constexpr (EPI == WIDE_SILU) {
                f32x4_t up;
#pragma unroll
                for (int e = 0; e < 4; ++e) up[e] = __shfl_xor(v[e], 32, 64);
                if (lane < 32 && row < M) {
                    float y[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) y[e] = v[e] / (1.0f + expf(-v[e])) * up[e];
                    store_afrag4(frag, kblks_out, row, 8 * (ct0 + c) + 4 * (lane >> 4), y[0], y[1], y[2], y[3]);
                }
            } else if (row < M) *reinterpret_cast<f32x4_t*>(Y + (size_t)row * ldy + (ct0 + c) * 16 + 4 * (lane >> 4)) = v;
        }
    }
}

}  // namespace hivis
