"""Host arithmetic of the buffers of bf16 models.  The prefill buffers are also the operand buffers of the 11..64-row passes:
whatever a pass packs has to fit the buffer it is sent to, down to the smallest context that takes such a pass (64 rows of room).
And the room for K slices covers every row count, so that it grows at most once.  Work items of the phase programs' attention."""
import ctypes
import itertools

import pytest

from host_header import load

SOURCE = """
#include "hivis_sizes.h"
using namespace hivis;
extern "C" int rows(int d, int qd, int F, int B, int vis, int text) { return prefill_sizes(d, qd, F, B, vis, text).rows; }
// rows beyond the end of the buffer that M rows of K are sent to (0: they fit), -1: no buffer takes them
extern "C" long over(int d, int qd, int F, int B, int vis, int text, int M, int K) {
    const PrefillSizes s = prefill_sizes(d, qd, F, B, vis, text);
    const int which = frag_buffer(s, M, K);
    if (!which) return -1;
    const size_t room = which == 1 ? s.frag : s.frag2, need = frag_values(M, K);
    return need <= room ? 0 : (long)((need - room + K - 1) / K);
}
// most floats of K slices over all row counts of a prefill pass, as the passes choose them, beyond what splitk_floats says
extern "C" long slices_over(int cu, int d, int qd, int kd, int F, int rows) {
    const size_t room = splitk_floats(cu, d, qd, kd, F, rows);
    const int K[6] = {d, qd, d, F, d, 2 * d}, N[6] = {qd + 2 * kd, d, 2 * F, d, d, d};
    long over = 0;
    for (int M = 65; M <= rows; ++M)
        for (int i = 0; i < 6; ++i) {
            const TallPlan sliced = tall_plan(cu, M, K[i] / 32, N[i] / 16, true), whole = tall_plan(cu, M, K[i] / 32, N[i] / 16, false);
            if (sliced.ksplit == 1 || ((i == 0 || i == 2) && tall_fused(whole, sliced))) continue;
            over = std::max(over, (long)sliced.ksplit * M * N[i] - (long)room);
        }
    return over;
}
extern "C" long wide_over(int cu, int K, int N) {
    long over = 0;
    for (int M = 1; M <= 64; ++M) {
        const int S = wide_slices(cu, K / 32, N / 16);
        if (S > 1) over = std::max(over, (long)S * M * N - (long)splitk_floats(cu, 64, 64, 64, 64, 64));
    }
    return over;
}
extern "C" void cut(int nseq, int m, int hq, int hkv, int alone, int* out) {
    const AttnCut a = attn_cut(nseq, m, hq, hkv, alone);
    out[0] = a.mi; out[1] = a.gh; out[2] = a.n_hblk; out[3] = a.n_rblk; out[4] = a.items;
}
// whether a pass of an fp32 model on 256 CUs takes items of one row
extern "C" int alone(int nseq, int m, int hq, int hkv, int hd, int keys) {
    const AttnCut s = attn_cut(nseq, m, hq, hkv, false), a = attn_cut(nseq, m, hq, hkv, true);
    if (a.items > 256) return 0;
    auto splits = [&](int items) { return attn_splits(keys, std::min(ATTN_MAX_SPLITS, std::max(1, 256 / ((items + 7) / 8 * 8))), 192); };
    return attn_alone(nseq, m, hq, hkv, hd, keys, splits(a.items), splits(s.items));
}
extern "C" long partials(int grid, int items) { return attn_partials(grid, items); }
"""

#           d, q_dim, F
WIDTHS = [(4096, 4096, 11008), (5120, 5120, 13824), (3584, 3584, 18944), (2048, 2048, 5632), (256, 256, 1024), (256, 768, 4096),
          (8320, 8320, 28672), (64, 1024, 96), (4096, 4096, 32)]


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return load(SOURCE, tmp_path_factory.mktemp("sizes"))


@pytest.mark.parametrize("widths", WIDTHS, ids=str)
def test_packed_rows_fit(lib, widths):
    d, qd, F = widths
    for room, B in itertools.product([64, 65, 80, 81, 96, 112, 160, 168, 400], [1, 2, 7]):
        one = -(-room // B) if B > 1 else room
        vis, text = one // 2, one - one // 2
        PR = lib.rows(d, qd, F, B, vis, text)
        assert PR % 16 == 0 and PR >= one
        if PR < 64:
            continue
        for M in range(1, 65):                      # decode, verify and re-feed passes
            for K in {d, 2 * d, qd, F}:
                assert lib.over(d, qd, F, B, vis, text, M, K) == 0, (PR, M, K)
        for K in {d, 2 * d, qd, F}:                 # a prefill pass over all the rows there are
            assert lib.over(d, qd, F, B, vis, text, PR, K) == 0, (PR, K)


def test_refuses_what_fits_nowhere(lib):
    assert lib.over(256, 256, 1024, 1, 32, 32, 65, 1024) == -1


@pytest.mark.parametrize("widths", WIDTHS, ids=str)
@pytest.mark.parametrize("cu", [256, 64])
def test_room_for_every_slice(lib, widths, cu):
    d, qd, F = widths
    for kd in {64, qd}:
        for rows in (64, 129, 640, 3008, 4096):
            assert lib.slices_over(cu, d, qd, kd, F, rows) <= 0, (kd, rows)
    for K, N in itertools.product({d, 2 * d, qd, F}, {d, 2 * F, 3 * qd, 32000, 152064, 528}):
        assert lib.wide_over(cu, K, N) <= 0, (K, N)


def test_attention_items(lib):
    """Every (sequence, key head, query head, row) in one item of at most eight pairs; room for the partials of a grid of workgroups."""
    for nseq, m, (hq, hkv), alone in itertools.product([1, 2, 4, 9], [1, 2, 5, 8, 9, 16], [(4, 4), (32, 4), (28, 4), (32, 8), (6, 3)], [0, 1]):
        out = (ctypes.c_int * 5)()
        lib.cut(nseq, m, hq, hkv, alone, out)
        mi, gh, nh, nr, items = out
        assert mi * gh <= (1 if alone else 8) and (nh - 1) * gh < hq // hkv <= nh * gh and (nr - 1) * mi < m <= nr * mi
        assert items == nseq * hkv * nh * nr
        for grid in (64, 256):
            assert items <= lib.partials(grid, items) <= max(items, grid)


@pytest.mark.parametrize("alone,shape", [
    (1, (1, 5, 4, 4, 64, 100)), (1, (1, 5, 8, 8, 64, 3000)), (1, (1, 8, 32, 8, 128, 450)), (1, (1, 1, 32, 4, 128, 3000)), (1, (1, 16, 16, 16, 64, 700)),
    (1, (1, 5, 32, 8, 64, 700)), (1, (1, 8, 28, 4, 128, 700)),
    (0, (1, 5, 32, 32, 128, 2000)), (0, (1, 5, 28, 4, 128, 2000)), (0, (4, 4, 16, 16, 64, 700)), (0, (2, 1, 32, 8, 128, 3000)), (0, (1, 5, 32, 32, 64, 2000)),
], ids=str)
def test_rows_alone_where_they_were_faster(lib, alone, shape):
    """sequences, rows, query and key heads, head_dim, cached rows: measured faster as items of one row, or slower"""
    assert lib.alone(*shape) == alone
