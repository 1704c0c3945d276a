// Sizes of the whole-prompt prefill buffers (bf16 models) and which of them holds what.  Host arithmetic only, no HIP: the
// library sizes and checks with it, and a test compiles it alone.
#pragma once
#include <algorithm>
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

}  // namespace hivis
