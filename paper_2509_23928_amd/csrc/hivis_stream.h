// Weight-streaming GEMM phases of bf16 models on row fragments (passes of up to 16 rows, one launch per phase).
//
// The activation rows of a pass travel between its kernels as MFMA operands: every kernel that produces rows multiplies them by the
// gain of the RMSNorm that follows, splits them into a bf16 high and a bf16 low part and stores both as row fragments; the sums of
// squares that the norm needs go out per 16 columns.  A GEMM workgroup then requests fragments and weights with plain loads and
// multiplies; 1/rms is applied to the sums.  (Staging fp32 rows instead, every workgroup of every launch converted every row and
// moved it through LDS before its first product: two further dependent steps at the start of each launch, a thousand vector
// instructions per wavefront, and registers that the weights in flight need.)  HBM bound.  Kernel traces, before -> now: 7B widths, 6 rows:
// q|k|v 20.4 -> 20.0 us, O 11.3 -> 9.3, gate|up 32.0 -> 31.1, down 20.1 -> 18.8, attention (which now writes fragments) 13.4 -> 11.6; LM head 49.3 ->
// 46.2; 2048 wide, 12 rows: q|k|v 10.2 -> 7.8, O 9.5 -> 6.0, gate|up 14.4 -> 11.0, down 18.0 -> 10.8.  A plain stream of the same bytes takes 16.4, 6.4,
// 27.2, 14.7 and 38.5 us.
//
// Row fragments of M rows of K values: K block kb (32 values), part p (0 high, 1 low), row r, piece g (8 values)
//   frag[((kb * 2 + p) * M + r) * 4 + g]        16 bytes each
// so that a K block is M * 128 contiguous bytes, whatever M is, and a part of it M * 64 (with a row's parts side by side every load of the
// 16-row form touched half of twice as many cache lines: 12 rows, 2048 wide, down 16.2 -> 14.1 us, O 7.4 -> 6.6).
// Not for more than 16 rows: every workgroup reads all fragments, 717 MB through the L2s for the down projection of 61 rows, 53 us where the
// K-sliced GEMM (gemm_wide_kernel) and its row kernel take 29.
#pragma once
#include "hivis_fused.h"

namespace hivis {

__device__ __forceinline__ float buffer_f32(__amdgpu_buffer_rsrc_t r, int byte) { return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, byte, 0, 0)); }
__device__ __forceinline__ float buffer_bf16(__amdgpu_buffer_rsrc_t r, int byte) { return bf16_to_f32((bf16_t)__builtin_amdgcn_raw_buffer_load_b16(r, byte, 0, 0)); }
constexpr int STREAM_MAX_D = 8192;             // row widths served (registers for a row's sums of squares, and for a row)

// the lane's operand row: 8-row form: row 2 (i / 4) + i % 2, high part for i & 2 == 0; 16-row form: row i, both parts
// (of the n rows from r0 on, in fragments of M rows)
template <typename WT> __device__ __forceinline__ int frag_lane_offset(int lane, int M, int r0, int n);
template <> __device__ __forceinline__ int frag_lane_offset<bf16_t>(int lane, int M, int r0, int n) {
    const int i = lane & 15, row = 2 * (i >> 2) + (i & 1);
    return row < n ? ((((i >> 1) & 1) * M + r0 + row) * 4 + (lane >> 4)) * 16 : OUT_OF_RANGE;
}
template <> __device__ __forceinline__ int frag_lane_offset<bf16w_t>(int lane, int, int r0, int n) {
    const int row = lane & 15;
    return row < n ? ((r0 + row) * 4 + (lane >> 4)) * 16 : OUT_OF_RANGE;
}
// fragments of K blocks [kb0, kb0 + nkb)
template <int U>
__device__ __forceinline__ void issue_rows(bf16x8_t (&a)[U], const uint4* __restrict__ A, int M, int lane_off, int kb0, int nkb) {
    const __amdgpu_buffer_rsrc_t r = buffer_of(A + (size_t)kb0 * M * 8, nkb * M * 128);
#pragma unroll
    for (int j = 0; j < U; ++j) a[j] = __builtin_bit_cast(bf16x8_t, __builtin_amdgcn_raw_buffer_load_b128(r, lane_off + j * M * 128, 0, 0));
}
template <int U>
__device__ __forceinline__ void issue_rows(HiLoFrag (&a)[U], const uint4* __restrict__ A, int M, int lane_off, int kb0, int nkb) {
    const __amdgpu_buffer_rsrc_t r = buffer_of(A + (size_t)kb0 * M * 8, nkb * M * 128);
#pragma unroll
    for (int j = 0; j < U; ++j) {
        a[j].hi = __builtin_bit_cast(bf16x8_t, __builtin_amdgcn_raw_buffer_load_b128(r, lane_off + j * M * 128, 0, 0));
        a[j].lo = __builtin_bit_cast(bf16x8_t, __builtin_amdgcn_raw_buffer_load_b128(r, lane_off + (2 * j + 1) * M * 64, 0, 0));
    }
}

// U K blocks per unit (and wavefront), D units in flight.  AB passes' fragments are held; the loop body covers PU passes, so that
// every buffer index is a constant and nothing in it is conditional: the compiler then counts its waits instead of draining the
// queue.  K of more than 2048: 128 KB of weights in flight per workgroup (16-row form: units of half the size, as the fragments take twice
// the registers, and twice as many).  SHORT, K up to 2048: a wavefront has at most eight blocks of a tile, two units of four; blocks beyond
// K cost a load's issue slots all the same (16 cycles of the CU's one address pipeline), and half of the longer units would be such.
template <typename WT, int G, bool SHORT> struct StreamCfg {
    static constexpr bool W16 = std::is_same<WT, bf16w_t>::value;
    static constexpr int U = W16 || SHORT ? 4 : 8, D = W16 && !SHORT ? 4 : 2;
    static constexpr int AB = G == 1 ? D : 2;
    static constexpr int PU = G == 1 ? D : (2 * G % D == 0 ? 2 : 4);
    static constexpr int NHI = G <= 4 ? 2 : 1;       // (16-row form: two accumulators for the high parts where a group's tiles are few)
    static_assert(PU % AB == 0 && (PU * G) % D == 0, "buffer indices repeat with the loop body");
};
// (LM head of a draft step, 1024 wide, 8000 columns and those of w1: long units 11.8 us, short ones 8.2, staged fp32 rows 8.8)
constexpr int STREAM_SHORT_K = 2048;
// distance of two rows' sums of squares of n parts (whole 16-byte pieces)
__host__ __device__ constexpr int ssq_stride(int n) { return (n + 3) & ~3; }
__host__ __device__ constexpr size_t stream_lds_floats(int G, int RPL) { return (size_t)FUSED_NW * G * 64 * RPL + 16 + 16; }

// sum over the 16 lanes of a row of lanes, in every one of them
__device__ __forceinline__ float row16_sum(float v) {
    v = quad_sum(v);
    v += dpp_move<DPP_ROW_ROR4, 0xF>(v, v);
    v += dpp_move<DPP_ROW_ROR8, 0xF>(v, v);
    return v;
}

// K blocks of a wavefront in one pass: the passes (a multiple of PU) share K evenly, the last one what is left of it
struct StreamUnits {
    int kblks, bw;
    __device__ __forceinline__ int blocks(int p) const { return max(0, min(bw, (kblks - p * FUSED_NW * bw + FUSED_NW - 1) / FUSED_NW)); }
    __device__ __forceinline__ int first(int p, int wave) const { return p * FUSED_NW * bw + wave * blocks(p); }
    __device__ __forceinline__ int count(int p, int wave) const { return max(0, min(blocks(p), kblks - first(p, wave))); }
};

// One GEMM phase: workgroup b owns a contiguous range of 16-column tiles (XCD by XCD, as in gemm_phase) and all of K, in groups of up
// to G tiles.
template <typename WT, int EPI, int G, bool SHORT, bool KEEP>
__device__ __forceinline__ void stream_gemm(const Phase& ph, const PassParams& pp, float* __restrict__ lds) {
#define HIVIS_MARK(k) if (pp.prof2 && blockIdx.x == 0 && threadIdx.x == 0) pp.prof2[k] = wall_clock64();
    typedef StreamCfg<WT, G, SHORT> CF;
    typedef typename KVType<WT>::type KT;
    constexpr int RPL = WTraits<WT>::RPL, ROWS = WTraits<WT>::ROWS, U = CF::U, D = CF::D, AB = CF::AB, PU = CF::PU, NW = FUSED_NW, NT = FUSED_NT;
    constexpr bool PAIRS = EPI == FEPI_QKV || EPI == FEPI_SILU;                  // an epilogue slot covers two columns
    constexpr int CPT = PAIRS ? 8 : 16;                                          // slots per tile and row
    constexpr int NSLOT = G * CPT * ROWS, SLOTS = (NSLOT + NT - 1) / NT;
    HIVIS_MARK(0)
    float* red = lds;                                   // [NW][G][64][RPL]
    float* inv_rms = lds + (size_t)NW * G * 64 * RPL;   // [16]
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int K = ph.K, N = ph.N, kblks = K / 32, ntiles = N / 16;
    int vb = (gridDim.x % 8 == 0) ? (int)((blockIdx.x % 8) * (gridDim.x / 8) + blockIdx.x / 8) : (int)blockIdx.x, nwg = gridDim.x;
    // Two workgroups per tile (the 8-row form given more rows, see launch_phases): rows [r0, r0 + M) of Mt, neighbours on one XCD
    const int Mt = pp.M;
    int r0 = 0, M = Mt;
    if constexpr (std::is_same<WT, bf16_t>::value && G == 1 && !PAIRS) {
        if (Mt > ROWS) { M = (Mt + 1) / 2; if (vb & 1) { r0 = M; M = Mt - M; } vb >>= 1; nwg >>= 1; }
    }
    const int t_begin = __builtin_amdgcn_readfirstlane((int)((unsigned)vb * (unsigned)ntiles / (unsigned)nwg));
    const int t_end = __builtin_amdgcn_readfirstlane((int)((unsigned)(vb + 1) * (unsigned)ntiles / (unsigned)nwg));
    const int npass = (kblks + NW * U * PU - 1) / (NW * U * PU) * PU;
    const StreamUnits un = {kblks, (kblks + NW * npass - 1) / (NW * npass)};
    const int lane_off = frag_lane_offset<WT>(lane, Mt, r0, M);

    // the slot of this thread: tile of the group, row, column(s)
    int s_g[SLOTS], s_row[SLOTS], s_c[SLOTS];
#pragma unroll
    for (int sl = 0; sl < SLOTS; ++sl) {
        const int idx = threadIdx.x + sl * NT;
        s_c[sl] = idx % CPT; s_row[sl] = (idx / CPT) % ROWS; s_g[sl] = idx / (CPT * ROWS);
    }
    // the token of the thread's row (the same for all its slots): given, or the greedy one of the LM-head phase before this one, reduced
    // here by the 16 lanes of the row (lowest index wins ties); the workgroups of tile 0 also store it
    int tok = 0;
    static_assert((EPI != FEPI_ADDVEC && EPI != FEPI_LOGITS) || NT % (CPT * ROWS) == 0, "a thread serves one row");
    if constexpr (EPI == FEPI_ADDVEC) {
        const int r = r0 + min(s_row[0], M - 1);
        if (ph.tok) tok = __hip_atomic_load(&ph.tok[seq_of(pp, r) * ph.tok_sseq + row_in_seq(pp, r) * ph.tok_srow], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        else {
            float bv = -INFINITY; int bi = 0x7FFFFFFF;
#pragma unroll 4
            for (int i0 = 0; i0 < ph.ncand; i0 += 16) {
                const int at = r * ph.ncand + min(i0 + (lane & 15), ph.ncand - 1);
                const float v = ph.pm[at]; const int i = ph.pi[at];
                if (v > bv || (v == bv && i < bi)) { bv = v; bi = i; }
            }
#pragma unroll
            for (int o = 8; o > 0; o >>= 1) {
                const float ov = __shfl_xor(bv, o, 64); const int oi = __shfl_xor(bi, o, 64);
                if (ov > bv || (ov == bv && oi < bi)) { bv = ov; bi = oi; }
            }
            tok = bi;
            if (vb == 0 && s_c[0] == 0 && s_g[0] == 0 && s_row[0] < M) {
                if (pp.bad && (unsigned)bi >= (unsigned)pp.V) st_wt(pp.bad, 1);
                st_wt(&ph.tok_out[(r / pp.m) * ph.o_sseq + (r % pp.m) * ph.o_srow], clamp_token(bi, pp.V));
            }
        }
    }
    // residual rows / rotary table entries / biases / gains of the slots of the group that starts at tile tg_
    float e_a[SLOTS], e_b[SLOTS], e_c[SLOTS];
    auto epi_request = [&](int tg_) {
#pragma unroll
        for (int sl = 0; sl < SLOTS; ++sl) {
            const int row = r0 + min(s_row[sl], M - 1);
            if constexpr (EPI == FEPI_ADD_TO || EPI == FEPI_ADDVEC) {
                const int col = min((tg_ + s_g[sl]) * 16 + s_c[sl], N - 1);
                e_b[sl] = buffer_bf16(buffer_of(ph.fgain, ph.fgain ? N * 2 : 0), col * 2);
                if constexpr (EPI == FEPI_ADD_TO) e_a[sl] = ph.R[(size_t)row * ph.ldr + col];
                else e_c[sl] = bf16_to_f32(((const bf16_t*)ph.vec)[(size_t)ph.vec_idx * N + col]);
            } else if constexpr (EPI == FEPI_QKV) {
                const int col = min((tg_ + s_g[sl]) * 16 + 2 * s_c[sl], N - 2);
                const int seq = seq_of(pp, row);
                const int delta = ph.pos_delta ? ph.pos_delta[row] : ph.offset + row_in_seq(pp, row);
                const int pos = min((ph.att.nbase > 0 ? ph.att.base_val[seq] : ph.base[seq]) + delta, ph.maxL - 1);
                const float2 cs = *reinterpret_cast<const float2*>(ph.rope + ((size_t)pos * (pp.hd / 2) + ((col % pp.hd) >> 1)) * 2);
                e_a[sl] = cs.x; e_b[sl] = cs.y;
            }
        }
    };
    // ---- what the end of the phase needs, requested first: loads return in order
    epi_request(t_begin);
    // (PRO_RMS) the rows' sums of squares: wavefront w takes rows w (and w + 8); whole pieces of four, then the last three
    constexpr bool RMS = PAIRS;
    constexpr int RPW = RMS ? ROWS / NW : 0, SQ = STREAM_MAX_D / 16 / 256;
    float4 sq[RMS ? RPW : 1][SQ]; float sq1[RMS ? RPW : 1];
#pragma unroll
    for (int q = 0; q < RPW; ++q) {
        const int row = wave + q * NW, n4 = row < M ? ph.nssq & ~3 : 0, n = row < M ? ph.nssq : 0;
        const float* src = ph.ssq + (size_t)row * ssq_stride(ph.nssq);
#pragma unroll
        for (int e = 0; e < SQ; ++e) sq[q][e] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(buffer_of(src, n4 * 4), (lane + 64 * e) * 16, 0, 0));
        sq1[q] = buffer_f32(buffer_of(src, n * 4), lane < 3 ? (n4 + lane) * 4 : OUT_OF_RANGE);
    }
    // ---- first units: the fragments of AB passes and D units of weights in turn.  (Both take the same time in the CU's address
    // pipeline, 2 us for a workgroup's first 256 KB; with all weights in front the first products waited for all of it.)
    typename AFrag<WT>::type a[AB][U];
    uint4 w[D][U];
    // (a pass nobody needs, a tile beyond the range: no blocks)
#define HIVIS_ROWS(buf_, pass_, on_) issue_rows(a[buf_], ph.Af, Mt, lane_off, un.first(pass_, wave), (on_) ? un.count(pass_, wave) : 0)
#define HIVIS_UNIT(buf_, tile_, pass_) issue_unit<WT, KEEP>(w[buf_], ph.W, kblks, tile_, un.first(pass_, wave), (tile_) < t_end ? un.count(pass_, wave) : 0, lane)
    __builtin_amdgcn_sched_barrier(0);
    HIVIS_MARK(1)
#pragma unroll
    for (int s = 0; s < (D > AB ? D : AB); ++s) {
        if (s < AB) HIVIS_ROWS(s, s, true);
        if (s < D) HIVIS_UNIT(s, t_begin + s % G, s / G);
    }
    __builtin_amdgcn_sched_barrier(0);
    HIVIS_MARK(2)
    // the fusion FC's embedding half, from the table (its token was requested before everything else)
    if constexpr (EPI == FEPI_ADDVEC) {
#pragma unroll
        for (int sl = 0; sl < SLOTS; ++sl) e_a[sl] = ph.add_rows[(size_t)clamp_token(tok, pp.V) * N + min((t_begin + s_g[sl]) * 16 + s_c[sl], N - 1)];
    }
    // 1/rms of the rows
    if constexpr (RMS) {
#pragma unroll
        for (int q = 0; q < RPW; ++q) {
            float t = sq1[q];
#pragma unroll
            for (int e = 0; e < SQ; ++e) t += (sq[q][e].x + sq[q][e].y) + (sq[q][e].z + sq[q][e].w);
            t = wave_sum(t);
            if (lane == 0) inv_rms[wave + q * NW] = 1.0f / sqrtf(t / (float)K + pp.eps);
        }
    }

    float best_v = -INFINITY; int best_i = 0x7FFFFFFF;      // greedy-token candidate (LOGITS): a thread always serves one row
    for (int tg = t_begin; tg < t_end; tg += G) {
        const int ng = min(G, t_end - tg);
        typename AccT<WT, CF::NHI>::type acc[G];
#pragma unroll
        for (int g = 0; g < G; ++g) acc_zero(acc[g]);
        for (int p = 0; p < npass; p += PU) {
            const bool last = p + PU >= npass;             // the units requested now and used after this trip belong to the next group
            const int tg_n = last ? tg + G : tg, p_n = last ? 0 : p + PU;
#pragma unroll
            for (int s = 0; s < PU * G; ++s) {
                const int pl = s / G, g = s % G, s2 = s + D;
                mfma_unit(acc[g], a[pl % AB], w[s % D]);
                if (g == G - 1) {
                    if (pl + AB < PU) HIVIS_ROWS(pl % AB, p + pl + AB, true);
                    else HIVIS_ROWS(pl % AB, p_n + pl + AB - PU, tg_n < t_end);
                }
                if (s2 < PU * G) HIVIS_UNIT(s % D, tg + s2 % G, p + s2 / G);
                else HIVIS_UNIT(s % D, tg_n + (s2 - PU * G) % G, p_n + (s2 - PU * G) / G);
            }
        }
        if (tg == t_begin) { HIVIS_MARK(3) }
        // ---- the wavefronts' sums meet in LDS
        if (tg > t_begin) lds_barrier();                   // (the last group's have been read)
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const auto& x = acc[g];
            float* dst = red + ((size_t)(wave * G + g) * 64 + lane) * RPL;
            if constexpr (RPL == 2) {
                *reinterpret_cast<float2*>(dst) = make_float2(x[0] + x[2], x[1] + x[3]);
            } else {
                float y[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) y[e] = (CF::NHI == 2 ? x.hi[0][e] + x.hi[CF::NHI - 1][e] : x.hi[0][e]) + x.lo[e];
                *reinterpret_cast<float4*>(dst) = make_float4(y[0], y[1], y[2], y[3]);
            }
        }
        lds_barrier();
        if (tg == t_begin) { HIVIS_MARK(4) }
        auto sum = [&](int g, int row, int c) {
            const float* src = red + ((size_t)g * 64 + c + 16 * (row / RPL)) * RPL + row % RPL;
            float s = 0.f;
#pragma unroll
            for (int w_ = 0; w_ < NW; ++w_) s += src[(size_t)w_ * G * 64 * RPL];
            return RMS ? s * inv_rms[row] : s;
        };
        // ---- epilogue
#pragma unroll
        for (int sl = 0; sl < SLOTS; ++sl) {
            const int g = s_g[sl], row = s_row[sl], tile = tg + g;
            if (g >= ng || row >= M) continue;             // (uniform over the slots of one tile and row)
            if constexpr (EPI == FEPI_ADD_TO || EPI == FEPI_ADDVEC) {
                const int c = s_c[sl], col = tile * 16 + c;
                const int rw = r0 + row;
                const float v = sum(g, row, c);
                const float y = EPI == FEPI_ADD_TO ? e_a[sl] + v : v + e_c[sl] + e_a[sl];
                if (ph.Y) st_wt(&ph.Y[(size_t)rw * ph.ldy + col], y);
                if (ph.F) {
                    const float z = ph.fgain ? y * e_b[sl] : y, z1 = dpp_move<DPP_QUAD_XOR1, 0xF>(z, z);
                    if ((c & 1) == 0) st_row_pair(ph.F, Mt, rw, col, z, z1);
                }
                if (ph.ssq_out) {
                    const float s = row16_sum(y * y);
                    if (c == 0) st_wt(&ph.ssq_out[(size_t)rw * ssq_stride(ntiles) + tile], s);
                }
            } else if constexpr (EPI == FEPI_SILU) {
                const int c = s_c[sl], col = tile * 8 + c;
                const float v = sum(g, row, c), up = sum(g, row, c + 8);
                const float y = v / (1.0f + expf(-v)) * up, y1 = dpp_move<DPP_QUAD_XOR1, 0xF>(y, y);
                if ((c & 1) == 0) st_row_pair(ph.F, M, row, col, y, y1);
            } else if constexpr (EPI == FEPI_QKV) {
                // a rotary pair of q or k, or two elements of v
                const int col = tile * 16 + 2 * s_c[sl], qd = pp.Hq * pp.hd, kd = pp.Hkv * pp.hd, hd = pp.hd, seq = seq_of(pp, row);
                const int slot = min((ph.att.nbase > 0 ? ph.att.base_val[seq] : ph.base[seq]) + ph.offset + row_in_seq(pp, row), ph.maxL - 1);
                float x1 = sum(g, row, 2 * s_c[sl]), x2 = sum(g, row, 2 * s_c[sl] + 1);
                if (ph.bias) { x1 += ph.bias[col]; x2 += ph.bias[col + 1]; }
                if (col < qd + kd) {
                    float y1, y2;
                    rotate_pair(x1, x2, e_a[sl], e_b[sl], y1, y2);
                    if (col < qd) st_wt_pair(&ph.Y[(size_t)row * ph.ldy + col], y1, y2);
                    else {
                        const int c2 = col - qd;
                        st_wt_kv_pair((KT*)ph.kc + (((size_t)seq * pp.Hkv + c2 / hd) * ph.maxL + slot) * hd * KVWidth<KT>::W, hd, c2 % hd, y1, y2);
                    }
                } else {
                    const int c2 = col - qd - kd;
                    st_wt_kv_pair((KT*)ph.vc + (((size_t)seq * pp.Hkv + c2 / hd) * ph.maxL + slot) * hd * KVWidth<KT>::W, hd, c2 % hd, x1, x2);
                }
            } else {
                const int col = tile * 16 + s_c[sl];
                const float v = sum(g, row, s_c[sl]);
                if (col < pp.V) {
                    st_wt(&ph.Y[(size_t)row * ph.ldy + col], v);
                    if (v > best_v || (v == best_v && col < best_i)) { best_v = v; best_i = col; }
                } else {
                    st_wt(&ph.Y2[(size_t)row * ph.ldy2 + (col - pp.V)], v + bf16_to_f32(((const bf16_t*)ph.vec)[(size_t)ph.vec_idx * (N - pp.V) + (col - pp.V)]));
                }
            }
        }
        if (tg + G < t_end) {
            epi_request(tg + G);
            if constexpr (EPI == FEPI_ADDVEC) {
#pragma unroll
                for (int sl = 0; sl < SLOTS; ++sl) e_a[sl] = ph.add_rows[(size_t)clamp_token(tok, pp.V) * N + min((tg + G + s_g[sl]) * 16 + s_c[sl], N - 1)];
            }
        }
    }
#undef HIVIS_ROWS
#undef HIVIS_UNIT
    HIVIS_MARK(5)
    if constexpr (EPI == FEPI_LOGITS) {
        // the workgroup's candidate per row: 16 lanes hold one row's columns, then the groups of lanes of a row meet in LDS
#pragma unroll
        for (int o = 8; o > 0; o >>= 1) {
            const float ov = __shfl_xor(best_v, o, 64); const int oi = __shfl_xor(best_i, o, 64);
            if (ov > best_v || (ov == best_v && oi < best_i)) { best_v = ov; best_i = oi; }
        }
        constexpr int NG = NT / 16 / ROWS;                 // lane groups per row
        lds_barrier();
        float* cv = red; int* ci = reinterpret_cast<int*>(red + NT / 16);
        if ((lane & 15) == 0) { cv[threadIdx.x / 16] = best_v; ci[threadIdx.x / 16] = best_i; }
        lds_barrier();
        const int r = threadIdx.x;
        if (r < ROWS && r < M) {
            float bv = cv[r]; int bi = ci[r];
#pragma unroll
            for (int q = 1; q < NG; ++q) {
                const float v = cv[q * ROWS + r]; const int i = ci[q * ROWS + r];
                if (v > bv || (v == bv && i < bi)) { bv = v; bi = i; }
            }
            st_wt(&ph.pm[(size_t)r * gridDim.x + blockIdx.x], bv); st_wt(&ph.pi[(size_t)r * gridDim.x + blockIdx.x], bi);
        }
        if (ph.cnt) lm_head_elect(ph, pp, reinterpret_cast<int*>(inv_rms));
    }
    HIVIS_MARK(6)
#undef HIVIS_MARK
}

// (KEEP: see issue_unit)
template <typename WT, int EPI, int G, bool SHORT, bool KEEP = false>
__global__ __launch_bounds__(FUSED_NT) void stream_kernel(Phase ph, PassParams pp) {
    extern __shared__ __align__(16) float lds[];
    kernarg_warm<sizeof(Phase) + sizeof(PassParams)>();
    prof_enter(pp.prof3, blockIdx.x);
    stream_gemm<WT, EPI, G, SHORT, KEEP>(ph, pp, lds);
    prof_leave(pp.prof3, blockIdx.x);
}

// Final norm of a verify pass: rows A * gain / rms as fp32 rows Y (the features) and as row fragments F.  One workgroup per row.
__global__ __launch_bounds__(FUSED_NT) void stream_norm_kernel(Phase ph, PassParams pp) {
#pragma clang fp contract(off)       // (the fragments are those of the fp32 rows, not of the unrounded products)
    __shared__ float part[FUSED_NW];
    constexpr int N4 = STREAM_MAX_D / (4 * FUSED_NT);
    const int row = blockIdx.x;
    const float* src = ph.A + (size_t)row * ph.lda;
    float4 x[N4], gn[N4];
    float ss = 0.f;
#pragma unroll
    for (int e = 0; e < N4; ++e) {
        const int c = min(4 * ((int)threadIdx.x + e * FUSED_NT), pp.d - 4);
        x[e] = *reinterpret_cast<const float4*>(src + c);
        gn[e] = load4_f32((const bf16_t*)ph.gain + c);
    }
#pragma unroll
    for (int e = 0; e < N4; ++e)
        if (4 * ((int)threadIdx.x + e * FUSED_NT) < pp.d) ss += x[e].x * x[e].x + x[e].y * x[e].y + x[e].z * x[e].z + x[e].w * x[e].w;
    ss = wave_sum(ss);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = ss;
    lds_barrier();
    float tot = 0.f;
#pragma unroll
    for (int w = 0; w < FUSED_NW; ++w) tot += part[w];
    const float inv = 1.0f / sqrtf(tot / (float)pp.d + pp.eps);
#pragma unroll
    for (int e = 0; e < N4; ++e) {
        const int c = 4 * ((int)threadIdx.x + e * FUSED_NT);
        if (c < pp.d) {
            const float y[4] = {x[e].x * gn[e].x * inv, x[e].y * gn[e].y * inv, x[e].z * gn[e].z * inv, x[e].w * gn[e].w * inv};
            float* o = ph.Y + (size_t)row * ph.ldy + c;
#pragma unroll
            for (int j = 0; j < 4; ++j) st_wt(o + j, y[j]);
            st_row_quad(ph.F, pp.M, row, c, y[0], y[1], y[2], y[3]);
        }
    }
}

// fp32 rows x (row stride ldx) -> rows row0 .. of `rows` as row fragments, times a gain (optional), and one sum of squares per row (optional).
__global__ __launch_bounds__(FUSED_NT) void stream_rows_kernel(const float* __restrict__ x, int ldx, int d, const bf16_t* __restrict__ gain,
                                                               uint4* __restrict__ frag, int row0, int rows, float* __restrict__ ssq) {
    __shared__ float part[FUSED_NW];
    const int row = row0 + blockIdx.x;
    float ss = 0.f;
    for (int c = 4 * threadIdx.x; c < d; c += 4 * FUSED_NT) {
        const float4 v = *reinterpret_cast<const float4*>(x + (size_t)blockIdx.x * ldx + c);
        const float4 g = gain ? load4_f32(gain + c) : make_float4(1.f, 1.f, 1.f, 1.f);
        ss += v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
        st_row_quad(frag, rows, row, c, v.x * g.x, v.y * g.y, v.z * g.z, v.w * g.w);
    }
    if (ssq == nullptr) return;
    ss = wave_sum(ss);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = ss;
    lds_barrier();
    if (threadIdx.x == 0) {
        float t = 0.f;
        for (int w = 0; w < FUSED_NW; ++w) t += part[w];
        st_wt(&ssq[row * ssq_stride(1)], t);
    }
}

// Embedding rows of a verify pass: fp32 rows (the residual stream), fragments times the first norm's gain, one sum of squares per row
__global__ __launch_bounds__(FUSED_NT) void stream_prep_kernel(Phase ph, PassParams pp) {
    __shared__ float part[FUSED_NW];
    const int row = blockIdx.x;
    int32_t tok = ph.ids[(row / pp.m) * ph.id_sseq + (row % pp.m) * ph.id_srow];
    tok = min(max(tok, 0), pp.V - 1);
    const bf16_t* src = (const bf16_t*)ph.gain + (size_t)tok * pp.d;
    float ss = 0.f;
    for (int c = 4 * threadIdx.x; c < pp.d; c += 4 * FUSED_NT) {
        const float4 x = load4_f32(src + c), gn = load4_f32((const bf16_t*)ph.fgain + c);
        ss += x.x * x.x + x.y * x.y + x.z * x.z + x.w * x.w;
        float* y = ph.Y + (size_t)row * ph.ldy + c;
        st_wt(y, x.x); st_wt(y + 1, x.y); st_wt(y + 2, x.z); st_wt(y + 3, x.w);
        st_row_quad(ph.F, pp.M, row, c, x.x * gn.x, x.y * gn.y, x.z * gn.z, x.w * gn.w);
    }
    ss = wave_sum(ss);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = ss;
    lds_barrier();
    if (threadIdx.x == 0) {
        float s = 0.f;
        for (int w = 0; w < FUSED_NW; ++w) s += part[w];
        st_wt(&ph.ssq_out[row * ssq_stride(1)], s);
    }
}

}  // namespace hivis
