"""The rotation of a q or k pair (one routine for all kernels) rounds once: it returns the float32 nearest to the exact value."""
import ctypes

import numpy as np

from host_header import load

SOURCE = """
#include "hivis_rotary.h"
extern "C" void rotate(const float* x1, const float* x2, const float* c, const float* s, float* y1, float* y2, int n) {
    for (int i = 0; i < n; ++i) hivis::rotate_pair(x1[i], x2[i], c[i], s[i], y1[i], y2[i]);
}
"""


def test_rounds_once(tmp_path):
    lib = load(SOURCE, tmp_path)
    rng = np.random.default_rng(0)
    n = 20000
    x1, x2, a = (rng.standard_normal(n) for _ in range(3))
    x1, x2, c, s = x1.astype(np.float32), x2.astype(np.float32), np.cos(a * 50).astype(np.float32), np.sin(a * 50).astype(np.float32)
    x2[::2] = x1[::2] * c[::2] / s[::2]                    # the first component nearly cancels
    y = np.zeros((2, n), np.float32)
    ptr = [v.ctypes.data_as(ctypes.POINTER(ctypes.c_float)) for v in (x1, x2, c, s, y[0], y[1])]
    lib.rotate(*ptr, n)
    L = np.longdouble
    exact = np.stack([L(x1) * L(c) - L(x2) * L(s), L(x2) * L(c) + L(x1) * L(s)])
    # half a unit in the last place, and the double sum's own rounding, which cancellation can make as large
    bound = np.spacing(np.abs(exact).astype(np.float32)) / 2 + 2.0 ** -53 * np.abs(L(x1) * L(c))
    assert np.all(np.abs(y - exact) <= bound * 1.001)
