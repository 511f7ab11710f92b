// Ray and sample arithmetic shared by the projector and its transpose.
//
// Both use the same rays and the same samples.  A sample on a cell's face
// has the same weights from both of its cells, so each may decide by its own
// rounding to which one a sample within rounding of a face belongs, as long
// as it gives every sample to exactly one.
//
// Sample coordinates are computed in double precision whatever the data
// type: a sample about 1000 mm from the source needs its direction to
// ~1e-9 relative to land within 1e-5 voxel of its true position, beyond
// float's 24-bit mantissa.  Double FMA, floor and convert run at the same
// vector rate as non-packed float on gfx950.
#pragma once

#include "cbct_internal.hpp"

namespace cbct {

// Index-space origin Q and per-sample increment D of the ray through
// pixel (i, j) of view vc (see ViewConst).
__device__ __forceinline__ void ray_setup(const ViewConst &vc, const DetConst &dc, int i, int j,
                                          double Q[3], double D[3]) {
#pragma clang fp contract(off)
    const double u = __builtin_fma((double)i, dc.aud, dc.u0d);
    const double v = __builtin_fma((double)j, dc.avd, dc.v0d);
    const double l2 = __builtin_fma(u, u, __builtin_fma(v, v, dc.sdd2d));
    const double inv = 1.0 / __builtin_sqrt(l2);
    D[0] = __builtin_fma(u, vc.Ud[0], vc.Wd[0]) * inv;
    D[1] = __builtin_fma(u, vc.Ud[1], vc.Wd[1]) * inv;
    D[2] = (v * vc.Vzd) * inv;
    Q[0] = vc.Qd[0];
    Q[1] = vc.Qd[1];
    Q[2] = vc.Qd[2];
}

// ---------------------------------------------------------------------------
// Sample cells and trilinear weights.
//
// Float data (the production path): the samples of a ray are grouped in
// segments of SEG consecutive indices n (a global lattice, n_s = n & ~(SEG-1),
// independent of where the ray enters the grid).  The segment origin
// q(n_s) = Q + n_s D is evaluated in double and split into an integer cell
// I and a float fraction f in [0, 1]; inside the segment
//     l = fma(m, D_f, f),   m = n - n_s in [0, SEG),  D_f = (float)D,
// cell = I + floor(l), weight = l - floor(l).  With the default step
// (|D_a| <= 1/2) |l| stays below SEG/2 + 1 = 129, so float keeps the
// position to ~1.5e-5 voxel (one rounding of l plus the rounding of D_f
// over 256 steps), and the double work is paid once per segment.
//
// Double data (derivative checks): q = fma(n, D, Q) in double per sample.
constexpr int SEG = 256;

struct SegOrigin {
    int I[3];
    float f[3];
};

__device__ __forceinline__ SegOrigin seg_origin(const double Q[3], const double D[3], int ns) {
#pragma clang fp contract(off)
    SegOrigin o;
    const double nd = (double)ns;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const double q = __builtin_fma(nd, D[a], Q[a]);
        const double fl = __builtin_floor(q);
        o.I[a] = (int)fl;
        o.f[a] = (float)(q - fl);
    }
    return o;
}

// Cell offset (relative to the segment's integer origin) and weight along
// one axis for in-segment index m.
__device__ __forceinline__ void seg_axis(float m, float Df, float f, int &dc, float &w) {
#pragma clang fp contract(off)
    const float l = __builtin_fmaf(m, Df, f);
    const float fl = __builtin_floorf(l);
    dc = (int)fl;
    w = l - fl;
}

__device__ __forceinline__ void to_float3(const double D[3], float Df[3]) {
    Df[0] = (float)D[0];
    Df[1] = (float)D[1];
    Df[2] = (float)D[2];
}

// Voxel-index coordinate of sample n along one axis.
__device__ __forceinline__ double sample_coord(double n, double D, double Q) {
    return __builtin_fma(n, D, Q);
}

// Interval [lo, hi] (real-valued, unrounded) of sample indices whose
// coordinate along one axis lies in [a, b); returns false if none can.
__device__ __forceinline__ bool axis_interval(double Q, double D, double a, double b, double &lo,
                                              double &hi) {
    if (D > 0.0) {
        const double inv = 1.0 / D;
        lo = (a - Q) * inv;
        hi = (b - Q) * inv;
        return true;
    }
    if (D < 0.0) {
        const double inv = 1.0 / D;
        lo = (b - Q) * inv;
        hi = (a - Q) * inv;
        return true;
    }
    lo = -1e30;
    hi = 1e30;
    return Q >= a && Q < b;
}

// Clamp a real sample index into a range safe for int conversion.
__device__ __forceinline__ int clamp_to_int(double x) {
    x = x < -4.0 ? -4.0 : x;
    x = x > (double)(1 << 24) ? (double)(1 << 24) : x;
    return (int)x;
}

}  // namespace cbct
