// The rotation every kernel applies to a pair of q or k.  No HIP needed: a test compiles it with the host's compiler.
#pragma once
#ifdef __HIPCC__
#define HIVIS_ANY __host__ __device__ __forceinline__
#else
#define HIVIS_ANY inline
#endif

namespace hivis {

// (y1, y2) = (x1 c - x2 s, x2 c + x1 s).  Products and sums in double, rounded once: in float the two products of a component
// that nearly cancel leave their own rounding errors behind.
HIVIS_ANY void rotate_pair(float x1, float x2, double c, double s, float& y1, float& y2) {
    y1 = (float)((double)x1 * c - (double)x2 * s);
    y2 = (float)((double)x2 * c + (double)x1 * s);
}

}  // namespace hivis
