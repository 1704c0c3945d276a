"""The prefill buffers are also the operand buffers of the 11..64-row passes: whatever a pass packs has to fit the buffer it
is sent to, down to the smallest context that takes such a pass (64 rows of room)."""
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
