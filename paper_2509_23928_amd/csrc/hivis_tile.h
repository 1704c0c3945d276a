// GEMM phases of fp32 models whose K fits one pass and whose tiles do not outnumber the workgroups (at most 1024 values per row, one tile per
// workgroup): models of a few MB, whose launches are latency, not bandwidth.
//
// A launch of these matrices costs what its chain of dependent steps costs: arguments, one round trip to memory, products, reduction, stores.
// gemm_phase stages rows through LDS for eight wavefronts with eight K blocks each, so that at K = 256 two of them did all the work,
// requests the operands of its epilogue behind the products and reduces in two steps.  Here the wavefronts share K evenly (U blocks
// each at most), a lane loads its operand pieces straight from the fp32 rows, everything that the launch needs is requested at its head, and
// the threads of the epilogue add the wavefronts' sums themselves.
// 256 wide, 5 rows, kernel traces, gemm_phase -> now: O 5.4 -> 3.0 us, down (K = 688) 5.4 -> 3.9, gate|up 6.1 -> 3.4, q|k|v 7.0 -> 3.8 and with table rows
// 7.6 -> 4.7, LM head 7.8 -> 3.8 and with the election of the greedy tokens 9.7 -> 5.6, fusion FC 7.0 -> 3.6; an empty launch takes 2.4.
#pragma once
#include "hivis_fused.h"

namespace hivis {

constexpr int TILE_MAX_BLOCKS = 8 * FUSED_NW;       // K blocks of 16 values

template <int EPI, int U>
__device__ __forceinline__ void tile_gemm(const Phase& ph, const PassParams& pp) {
#define HIVIS_MARK(k) if (pp.prof2 && blockIdx.x == 0 && threadIdx.x == 0) pp.prof2[k] = wall_clock64();
    HIVIS_MARK(0)
    constexpr int NW = FUSED_NW;
    constexpr bool TAB = EPI == FEPI_QKV_TAB, QKV = EPI == FEPI_QKV || TAB, RMS = QKV || EPI == FEPI_SILU;       // (RMS: the rows' norm is applied here)
    __shared__ __align__(16) float red[NW * 64 * 4];
    __shared__ float ssq[NW * 16];
    __shared__ int flag[1];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int M = pp.M, K = ph.K, N = ph.N, kblks = K / 16, tile = blockIdx.x;
    const int per = (kblks + NW - 1) / NW, kb0 = min(wave * per, kblks), nkb = min(kblks - kb0, per);        // this wavefront's K blocks
    const int row = min(lane & 15, M - 1), g = lane >> 4;                            // operand row (rows beyond M repeat the last) and piece
    // the thread's slot of the epilogue: one column of one row (the first 16 M threads)
    const int er = threadIdx.x >> 4, ec = threadIdx.x & 15, erow = min(er, M - 1), col = tile * 16 + ec;
    int eseq = 0, epos = 0;
    if constexpr (QKV) {
        eseq = seq_of(pp, erow);
        epos = min((ph.att.nbase > 0 ? ph.att.base_val[eseq] : ph.base[eseq]) + ph.offset + row_in_seq(pp, erow), ph.maxL - 1);
    }
    // ---- everything the launch needs; blocks beyond the wavefront's are replaced by one of the matrix and not multiplied
    float4 x[U], gn[U], t[U];
    uint4 w[U];
    int k[U];
#pragma unroll
    for (int j = 0; j < U; ++j) {
        const int kb = min(kb0 + j, kblks - 1);
        k[j] = kb * 16 + 4 * g;
        x[j] = *reinterpret_cast<const float4*>(ph.A + (size_t)row * ph.lda + k[j]);
        w[j] = ph.W[((size_t)tile * kblks + kb) * 64 + lane];
        if constexpr (RMS) gn[j] = *reinterpret_cast<const float4*>((const float*)ph.gain + k[j]);
    }
    float e_a = 0.f, e_b = 0.f;                                                      // operands of the slot
    if constexpr (EPI == FEPI_ADD_TO) e_a = ph.R[(size_t)erow * ph.ldr + col];
    if constexpr (EPI == FEPI_ADDVEC) e_b = ((const float*)ph.vec)[(size_t)ph.vec_idx * N + col];
    if constexpr (QKV) {
        const float2 cs = *reinterpret_cast<const float2*>(ph.rope + ((size_t)epos * (pp.hd / 2) + ((col % pp.hd) >> 1)) * 2);
        e_a = cs.x; e_b = cs.y;
    }
    // ---- tokens of the rows: given, or the greedy ones of the LM-head phase before this one, reduced by every wavefront (16 lanes a row, four
    // rows at a time; lowest index wins ties); workgroup 0 also stores them
    if constexpr (TAB || EPI == FEPI_ADDVEC) {
        int tok_x = 0, tok_e = 0;
        if (ph.tok) {
            auto given = [&](int r) { return __hip_atomic_load(&ph.tok[(r / pp.m) * ph.tok_sseq + (r % pp.m) * ph.tok_srow], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
            if constexpr (TAB) tok_x = given(row); else tok_e = given(erow);
        } else {
            for (int r0 = 0; r0 < M; r0 += 4) {
                const int r = min(r0 + g, M - 1);
                float bv = -INFINITY; int bi = 0x7FFFFFFF;
                auto better = [&](float v, int i) { const bool take = (v > bv) | ((v == bv) & (i < bi)); bv = take ? v : bv; bi = take ? i : bi; };
                for (int i0 = 0; i0 < ph.ncand; i0 += 16 * 5) {                      // (five per lane and trip: the 80 of 1024 columns and w1's 256)
                    float v[5]; int i[5];
#pragma unroll
                    for (int e = 0; e < 5; ++e) {
                        const int at = r * ph.ncand + min(i0 + 16 * e + (lane & 15), ph.ncand - 1);
                        v[e] = ph.pm[at]; i[e] = ph.pi[at];
                    }
#pragma unroll
                    for (int e = 0; e < 5; ++e) better(v[e], i[e]);
                }
#pragma unroll
                for (int o = 8; o > 0; o >>= 1) better(__shfl_xor(bv, o, 64), __shfl_xor(bi, o, 64));
                if (tile == 0 && wave == 0 && (lane & 15) == 0 && r0 + g < M) {
                    if (pp.bad && (unsigned)bi >= (unsigned)pp.V) st_wt(pp.bad, 1);
                    st_wt(&ph.tok_out[(r / pp.m) * ph.o_sseq + (r % pp.m) * ph.o_srow], clamp_token(bi, pp.V));
                }
                const int bx = __shfl(bi, 16 * (row & 3), 64), be = __shfl(bi, 16 * (erow & 3), 64);
                if (row >> 2 == r0 >> 2) tok_x = bx;
                if (erow >> 2 == r0 >> 2) tok_e = be;
            }
        }
        if constexpr (TAB) {
            // the activation rows are A + the tokens' table rows; workgroup 0 leaves them for the O projection
#pragma unroll
            for (int j = 0; j < U; ++j) t[j] = *reinterpret_cast<const float4*>(ph.add_rows + (size_t)clamp_token(tok_x, pp.V) * K + k[j]);
#pragma unroll
            for (int j = 0; j < U; ++j) {
                x[j].x += t[j].x; x[j].y += t[j].y; x[j].z += t[j].z; x[j].w += t[j].w;
                if (tile == 0 && j < nkb && (lane & 15) < M) {
                    float* o = ph.wb + (size_t)row * K + k[j];
                    st_wt2(o, x[j].x, x[j].y); st_wt2(o + 2, x[j].z, x[j].w);
                }
            }
        } else e_a = ph.add_rows[(size_t)clamp_token(tok_e, pp.V) * N + col];
    }
    HIVIS_MARK(1)
    // ---- products
    f32x4_t acc = f32x4_t{0.f, 0.f, 0.f, 0.f};
    float ss = 0.f;
#pragma unroll
    for (int j = 0; j < U; ++j) {
        if (j < nkb) {                                                               // (uniform)
            float4 a = x[j];
            if constexpr (RMS) {
                ss += a.x * a.x + a.y * a.y + a.z * a.z + a.w * a.w;
                a.x *= gn[j].x; a.y *= gn[j].y; a.z *= gn[j].z; a.w *= gn[j].w;
            }
            mfma_block(acc, a, w[j]);
        }
    }
    *reinterpret_cast<f32x4_t*>(red + (wave * 64 + lane) * 4) = acc;
    if constexpr (RMS) {
        ss += __shfl_xor(ss, 16, 64);
        ss += __shfl_xor(ss, 32, 64);
        if (lane < 16) ssq[wave * 16 + lane] = ss;
    }
    HIVIS_MARK(3)
    lds_barrier();
    // ---- epilogue: 16 lanes per row
    if (er < M) {
        float v = 0.f;
#pragma unroll
        for (int w_ = 0; w_ < NW; ++w_) v += red[(w_ * 64 + ec + 16 * (er >> 2)) * 4 + (er & 3)];
        if constexpr (RMS) {
            float s = 0.f;
#pragma unroll
            for (int w_ = 0; w_ < NW; ++w_) s += ssq[w_ * 16 + er];
            v *= 1.0f / sqrtf(s / (float)K + pp.eps);
        }
        if constexpr (EPI == FEPI_ADD_TO) st_wt(&ph.Y[(size_t)er * ph.ldy + col], e_a + v);
        else if constexpr (EPI == FEPI_ADDVEC) st_wt(&ph.Y[(size_t)er * ph.ldy + col], v + e_b + e_a);
        else if constexpr (EPI == FEPI_SILU) {
            const float up = __shfl_xor(v, 8, 64);
            if (ec < 8) st_wt(&ph.Y[(size_t)er * ph.ldy + tile * 8 + ec], v / (1.0f + expf(-v)) * up);
        } else if constexpr (QKV) {
            // an even column handles the pair (col, col + 1): a rotary pair of q or k, or two elements of v
            const int qd = pp.Hq * pp.hd, kd = pp.Hkv * pp.hd, hd = pp.hd;
            if (ph.bias) v += ph.bias[col];
            const float x2 = __shfl_xor(v, 1, 64);
            if ((ec & 1) == 0) {
                float y1 = v, y2 = x2;
                if (col < qd + kd) rotate_pair(v, x2, e_a, e_b, y1, y2);
                if (col < qd) st_wt_pair(&ph.Y[(size_t)er * ph.ldy + col], y1, y2);
                else {
                    const int c2 = col < qd + kd ? col - qd : col - qd - kd;
                    st_wt_kv_pair((float*)(col < qd + kd ? ph.kc : ph.vc) + (((size_t)eseq * pp.Hkv + c2 / hd) * ph.maxL + epos) * hd, hd, c2 % hd, y1, y2);
                }
            }
        } else {
            float best_v = -INFINITY; int best_i = 0x7FFFFFFF;
            if (col < pp.V) {
                st_wt(&ph.Y[(size_t)er * ph.ldy + col], v);
                if (v > best_v || (v == best_v && col < best_i)) { best_v = v; best_i = col; }
            } else st_wt(&ph.Y2[(size_t)er * ph.ldy2 + (col - pp.V)], v + ((const float*)ph.vec)[(size_t)ph.vec_idx * (N - pp.V) + (col - pp.V)]);
#pragma unroll
            for (int o = 8; o > 0; o >>= 1) {
                const float ov = __shfl_xor(best_v, o, 64); const int oi = __shfl_xor(best_i, o, 64);
                if (ov > best_v || (ov == best_v && oi < best_i)) { best_v = ov; best_i = oi; }
            }
            if (ec == 0) { st_wt(&ph.pm[(size_t)er * gridDim.x + tile], best_v); st_wt(&ph.pi[(size_t)er * gridDim.x + tile], best_i); }
        }
    }
    if constexpr (EPI == FEPI_LOGITS) { if (ph.cnt) lm_head_elect(ph, pp, flag); }
    HIVIS_MARK(6)
#undef HIVIS_MARK
}

template <int EPI, int U>
__global__ __launch_bounds__(FUSED_NT) void tile_kernel(Phase ph, PassParams pp) {
    kernarg_warm<sizeof(Phase) + sizeof(PassParams)>();
    prof_enter(pp.prof3, blockIdx.x);
    tile_gemm<EPI, U>(ph, pp);
    prof_leave(pp.prof3, blockIdx.x);
}

}  // namespace hivis
