// Sizes of the whole-prompt prefill buffers (bf16 models), which of them holds what, the plans of the GEMMs that fill them, and the work
// items of the phase programs' attention.
// Host arithmetic only, no HIP: the library sizes and checks with it, and a test compiles it alone.
#pragma once
#include <algorithm>
#include <cmath>
#include <cstddef>

namespace hivis {

constexpr int MAX_ROWS = 64;        // rows per pass that the activation buffers hold (tree verify: root + 63 candidates)
constexpr int CHAIN_MAX_ROWS = 32;  // chain verify rows B*(K+1); prefill chunk; rows per launch of the skinny GEMM

// values in the activation fragments of M rows of K (whole tiles of 16 rows)
inline size_t frag_values(int M, int K) { return (size_t)((M + 15) / 16 * 16) * K; }

struct PrefillSizes {
    int rows;                       // the longest prompt, or as many sequences at a time as fit 4096 rows; whole row tiles
    size_t frag, frag2;             // values the two fragment buffers hold: of d / 2 d / q_dim wide rows, and of the MLP's inner rows
};
inline PrefillSizes prefill_sizes(int d, int qd, int F, int batch, int max_vis, int max_text) {
    const int one = max_vis + max_text;
    PrefillSizes s{};
    s.rows = (std::max(one, std::min(batch * one, 4096)) + 15) & ~15;
    s.frag = (size_t)s.rows * std::max(2 * d, qd);
    s.frag2 = (size_t)s.rows * F;
    return s;
}

// The fragment buffer (1 or 2) that takes M rows of K, 0 if neither does.  (Rows of the MLP's inner width outgrow the first one:
// 61 rows of 11008 values need more than 80 rows of 8192.)
inline int frag_buffer(const PrefillSizes& s, int M, int K) {
    const size_t n = frag_values(M, K);
    return n <= s.frag ? 1 : n <= s.frag2 ? 2 : 0;
}

// Column tiles per wavefront and K slices of a tall GEMM: the pair with the least estimated time.  One workgroup per CU; a round of them takes 0.14 us
// per K block (the rows' reads, the barrier) plus 0.048 per K block and column tile, and 4 to start and finish.  What all CUs together
// switch comes on top (the card's power limit): 0.008 us per K block and column tile, 3 tiles more for the rows, times the share of a round that the tiles fill.
// Slices cost their partial sums, written once and read once.  Fitted to all forms and slices of 15 products (widths 2048..5120, K to 18944) at 18 row
// counts from 70 to 4000, for the choice: what it picks is 0.1 % over the best of them on average, 6 % at most.  (An estimate in proportion to
// the column tiles, 0.066 us each, took narrow tiles for large products: 3008 rows of 4096 on 22016 columns 798 us with 6, 767 with 8;
// 4096 columns of 11008 377 with 7, 369 with 8 in two slices; 0.7 % over the best on average, 18 % at most.)  only: 6..8, that many column tiles (0: any).
constexpr int TALL_ROWS = 128;
struct TallPlan { int cw, ksplit; double us; };
inline TallPlan tall_plan(int num_cu, int M, int kblks, int ntiles, bool may_split, int only = 0) {
    TallPlan best{8, 1, 1e30};
    const int nrow = (M + TALL_ROWS - 1) / TALL_ROWS;
    for (int cw = only ? only : 8; cw >= (only ? only : 6); --cw)
        for (int S = 1; S <= (may_split ? 8 : 1); ++S) {
            const int kper = (kblks + S - 1) / S;
            if (S > 1 && ((S - 1) * kper >= kblks || kper < 8)) continue;        // no empty slice, no tiny ones
            const double tiles = (double)nrow * ((ntiles + 2 * cw - 1) / (2 * cw)) * S;
            const double rounds = std::ceil(tiles / num_cu);
            double us = rounds * (kper * (0.14 + 0.048 * cw) + 4.0) + tiles / num_cu * kper * 0.008 * (cw + 3);
            if (S > 1) us += 2.0 * S * M * ntiles * 16 * 4.0 / 4.0e6;
            if (us < best.us - 1e-9) best = {cw, S, us};
        }
    return best;
}

// The q|k|v and the gate|up product end in the GEMM itself unless K slices win back more than the row kernel costs
// (ROW_KERNEL_US: its launch and ramp; its traffic is in the slices' estimate).  At most 64 rows: gate|up likewise, q|k|v never.
// (Gate|up of ten models 256 to 8192 wide at 17..61 rows: in the GEMM 0.5 to 8.5 us faster than slices and row kernel, 5.0 against 7.1 us for 1408 columns of 256 at 17 rows, 17.1 and 19.0 for
// 11264 of 2048 and 39.3 and 41.7 for 22016 of 4096 at 61, 140 and 144 for 57344 of 8192 at 17; the rule takes the GEMM for all of them.)
constexpr double ROW_KERNEL_US = 8.0;
template <typename Plan> bool tall_fused(const Plan& whole, const Plan& sliced) { return whole.us <= sliced.us + ROW_KERNEL_US; }

// GEMMs of at most 64 rows: column tiles of a workgroup ((8 / kw) * ct: kw wavefronts share ct column tiles, see gemm_wide_kernel) and K slices (of
// kper K blocks each), the pair with the least estimated time.  One workgroup per CU; more of them than CUs only as one slice.  A workgroup
// takes 0.0277 us per K block and row tile plus 0.0231 per K block and column tile when the CU is the limit; all of them together stream
// 7.7 MB of weights per us and 24 of activations (read once per column block), the less of both the fewer CUs work; writing a
// slice costs its bytes at 2 MB per us, reading it again in the consumer at 3.5.  Fitted to 286 launches (15 products of the 7B and 13B widths at 31, 32, 61 and 64
// rows, all forms and slices): 4.7 % off on average; what it picks is at most 4 % slower than the best of them, but for the down projection of 18944 rows
// at 64 rows (8 %).  Elsewhere (42 products of widths 256 to 8192 at 17..61 rows, all forms and slices) the pick is within 7 % of the best (launches under 5 us: as far as two runs
// of one differ), but for products whose workgroups begin a power of two of 512 KB or more of weights apart, which the estimate does not see: LM head of 2048 x 32000 16..19 % (17 rows 29.5 us,
// 24.8 with 10 column tiles), of 4096 x 32000 up to 9 %, O of 8192 14..19 % (29.7, 24.8), down of 8192 x 2048 3..11 %.  The kernel before this one (128 columns, up to 16
// slices) took 31.7 us for the first and 29.9 for O; of all these products it was faster only on matrices of up to 2 MB, by up to 0.4 us.
constexpr int WIDE_STAGE = 4;       // K blocks that a workgroup takes at a time
struct WideForm { int kw, ct; };
constexpr WideForm WIDE_FORMS[] = {{4, 2}, {4, 3}, {2, 2}, {4, 5}, {2, 3}, {2, 4}, {2, 5}};       // 4, 6, 8, 10, 12, 16, 20 column tiles
constexpr int WIDE_NFORMS = sizeof(WIDE_FORMS) / sizeof(WIDE_FORMS[0]);
constexpr int wide_forms(int M) { return M <= 32 ? WIDE_NFORMS : WIDE_NFORMS - 1; }                // (the widest: up to 32 rows, its sums fill the registers)
// the most slices of a product: the room for them (splitk_floats) holds 3 * num_cu * 128 columns; none empty, none of less than 4 K blocks
inline int wide_slices(int num_cu, int kblks, int ntiles) {
    int S = std::max(1, std::min(16, 3 * num_cu / ((ntiles + 7) / 8)));
    while (S > 1 && ((S - 1) * ((kblks + S - 1) / S) >= kblks || (kblks + S - 1) / S < 4)) --S;
    return S;
}
struct WidePlan { int form, tiles, ksplit, kper; double us; };
inline WidePlan wide_plan(int num_cu, int M, int kblks, int ntiles, bool may_split) {
    WidePlan best{0, 4, 1, kblks, 1e30};
    const int rt = M <= 32 ? 2 : 4, most = may_split ? wide_slices(num_cu, kblks, ntiles) : 1;
    for (int f = 0; f < wide_forms(M); ++f)
        for (int S = 1; S <= most; ++S) {
            const int tiles = 8 / WIDE_FORMS[f].kw * WIDE_FORMS[f].ct, kper = ((kblks + WIDE_STAGE - 1) / WIDE_STAGE + S - 1) / S * WIDE_STAGE;
            const int wgs = (ntiles + tiles - 1) / tiles * S;
            if (S > 1 && ((S - 1) * kper >= kblks || wgs > num_cu)) continue;
            const int rounds = (wgs + num_cu - 1) / num_cu;
            const double fill = (double)wgs / (rounds * num_cu), sums = 4.0e-6 * S * M * ntiles * 16;
            const double cu = rounds * kper * (0.0277 * rt + 0.0231 * tiles);
            const double all = (1.024e-3 * kblks * ntiles / 7.7 + 2.0e-3 * wgs * kper * rt / 24.0) / std::pow(fill, 0.31);
            const double us = 2.6 + std::max(cu, all) + 3.0 * (rounds - 1) + sums * (1 / 2.0 + 1 / 3.5);
            if (us < best.us - 1e-9) best = {f, tiles, S, kper, us};
        }
    return best;
}

// Floats that hold the K slices of every product of a context: the most that a pass of up to 64 rows needs (slices x column
// blocks <= 3 per CU), and that a prefill of up to `rows` rows needs.  A plan depends on the row count through whole row blocks, and
// inside a block the more rows, the fewer slices: the slices of a block's first row count, times its last, bound all of it.
inline size_t splitk_floats(int num_cu, int d, int qd, int kd, int F, int rows) {
    size_t need = (size_t)MAX_ROWS * 3 * num_cu * 128;
    const int K[6] = {d, qd, d, F, d, 2 * d}, N[6] = {qd + 2 * kd, d, 2 * F, d, d, d};      // q|k|v, O, gate|up, down, fusion FC
    for (int r0 = MAX_ROWS + 1; r0 <= rows; r0 = (r0 - 1) / TALL_ROWS * TALL_ROWS + TALL_ROWS + 1) {
        const int r1 = std::min(rows, (r0 - 1) / TALL_ROWS * TALL_ROWS + TALL_ROWS);
        for (int i = 0; i < 6; ++i) {
            const TallPlan sliced = tall_plan(num_cu, r0, K[i] / 32, N[i] / 16, true);
            if (sliced.ksplit == 1) continue;
            if ((i == 0 || i == 2) && tall_fused(tall_plan(num_cu, r0, K[i] / 32, N[i] / 16, false), sliced)) continue;
            need = std::max(need, (size_t)sliced.ksplit * r1 * N[i]);
        }
    }
    return need;
}

// Attention of a phase program: work items of up to FUSED_RMAX (query head, row) pairs of one key head and sequence, each with its keys cut
// into up to ATTN_MAX_SPLITS ranges.  alone: every head and row an item of its own.
constexpr int FUSED_RMAX = 8;
constexpr int ATTN_MAX_SPLITS = 16;
struct AttnCut { int mi, gh, n_hblk, n_rblk, items; };      // rows and heads per item, blocks of each, items
inline AttnCut attn_cut(int nseq, int m, int hq, int hkv, bool alone) {
    AttnCut a{};
    const int group = hq / hkv;
    if (alone) { a.mi = 1; a.gh = 1; }
    else if (m >= FUSED_RMAX) { a.mi = FUSED_RMAX; a.gh = 1; }
    else { a.mi = m; a.gh = std::max(1, std::min(group, FUSED_RMAX / m)); }
    a.n_hblk = (group + a.gh - 1) / a.gh; a.n_rblk = (m + a.mi - 1) / a.mi;
    a.items = nseq * hkv * a.n_hblk * a.n_rblk;
    return a;
}
// key splits of a launch over `keys` cached rows, of at most `most`
inline int attn_splits(int keys, int most, int keys_per_split) { return std::max(1, std::min(most, (keys + keys_per_split - 1) / keys_per_split)); }
// The same for half-precision caches, whose kernel takes 128 keys at a time (attn_split_kernel): as few blocks per workgroup as `most` splits allow, and no more
// splits than that needs.  A block more costs 2 us, a split more 0.1: 32 heads over 650 keys in 4 splits of two blocks 11.0 us, in 6 of one 10.6; one head group over
// 130..190 keys in one split 7.7, in two 7.2; but 28 heads over 1130 keys (8 splits at most: two blocks) in 5 splits 13.4, in 6 13.5, in 8 13.8.
constexpr int ATTN_BLOCK_KEYS = 128;
inline int attn_block_splits(int keys, int most) {
    const int per = (keys + ATTN_BLOCK_KEYS * most - 1) / (ATTN_BLOCK_KEYS * most) * ATTN_BLOCK_KEYS;
    return std::max(1, std::min(most, (keys + per - 1) / per));
}
inline int attn_blocks(int keys, int splits) { return ((keys + splits - 1) / splits + ATTN_BLOCK_KEYS - 1) / ATTN_BLOCK_KEYS; }       // of a workgroup
// Whether the workgroups of such a launch walk so many blocks that the form without a barrier per block is faster (attn_tiles_kernel): its wavefronts run on by
// themselves, but merge eight softmaxes at the end.  rm: (head,row) pairs an item may hold.  us, block form -> tiles: a prompt's last 128 of 3000 rows, 32 heads (256 items of 24
// blocks) 74 -> 66, two such prompts (512 items) 138 -> 104, 32 heads of 64 of four (1024 items) 142 -> 88; 128 rows over 400 keys the same in 4 blocks, over 200 keys 0.84 times as long in the block
// form.  Eight rows or fewer: 40 heads of eight sequences over 4000 keys (320 items) 266 -> 254, below a workgroup per CU within 3 % either way.  More items than CUs pay for
// every block that a CU's one workgroup waits at, and two workgroups of the tiles form of 64-wide heads fit a CU.
inline bool attn_walks(int num_cu, int hd, int items, int rm, int blocks) {
    if (items > num_cu) return blocks >= (hd == 64 ? 2 : 4);
    return rm > FUSED_RMAX && blocks >= (hd == 64 ? 3 : 6);
}
// Whether the rows of an fp32 pass over `keys` cached rows of each of nseq sequences are items of their own.  The vector ALU works on an
// item's rows one after the other, so that sharing an item costs a row about what 230 keys of 64 values cost.  Alone, rows leave fewer CUs
// to split the keys over, and the items of a key head, dealt to all eight XCDs, fetch its cached rows up to eight times (a megabyte costs
// what 8 keys do).  Measured over 14 head counts (4/4 to 64/4, 64 and 128 wide), 1..8 sequences, 1..16 rows and 100..3000 keys; us per verify pass
// of four layers and 5 rows, shared -> alone: 4/4 heads of 64 over 100 keys 171 -> 150; 8/8 over 3000 keys 197 -> 184; 32/32 of 128 over 2000 keys
// 301 -> 415, which the rule leaves shared.  Of 1296 such points it takes none that loses more than 0.3 us a layer, and 97 % of what the others gain.
inline bool attn_alone(int nseq, int m, int hq, int hkv, int hd, int keys, int splits_alone, int splits_shared) {
    const AttnCut s = attn_cut(nseq, m, hq, hkv, false);
    const double alone = (keys + splits_alone - 1) / splits_alone, shared = (keys + splits_shared - 1) / splits_shared;
    const double mb = 8.0e-6 * nseq * hkv * keys * hd * std::min(8, m * (hq / hkv));
    return (alone - shared) * hd / 64 + 8 * mb <= 230 * s.mi * s.gh;
}
// partials (each FUSED_RMAX rows of head_dim + 2 floats) that there is room for: what fills `grid` workgroups
inline size_t attn_partials(int grid, int items) { return (size_t)items * std::min(ATTN_MAX_SPLITS, std::max(1, grid / items)); }

}  // namespace hivis
