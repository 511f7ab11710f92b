// Transpose of the projector, P^T, in gather form without atomics.
//
// The paper computes the gradient of E2 per voxel by a gather (Eq. (2)) to
// avoid the write conflicts of the scattering matrix transpose.  Here the
// gather is the EXACT transpose of the discrete projector, organised by
// interpolation cell rather than by voxel:
//
//   * a cell c = (cx, cy, cz), c_a in [-1, N_a - 1], is the box between
//     voxel centres c and c + 1; every sample lies in exactly one cell;
//   * preparation (geometry only, once per plan or workspace): the ray
//     increment of every pixel of every view, and every brick's footprint
//     on the detector and map from cells to pixels per view;
//   * pass 1 (one lane per cell, a workgroup per brick of 16x16x1 cells or of
//     about as many; of few bricks, several per brick with a share of the
//     views each):
//     for every view the workgroup stages the rays of its brick's footprint
//     in LDS (unless the source is very near, see choose_cells); each lane
//     then visits the pixels whose rays can cross its cell and adds each
//     ray's samples in the cell, r * (trilinear corner weight), to eight
//     moments in registers, the samples of one crossing in closed form (see
//     crossing_sums), in float and double alike;
//   * pass 2 (one lane per voxel): sum the matching corner of the eight
//     cells that share the voxel, optionally fused with Step 1 of
//     Algorithm A1, g = f - tau * P^T r.
//
// Each (ray, cell) crossing is visited once, not once per trilinear tap,
// every sum has a fixed order, and no lane writes memory another lane
// writes.
#include <algorithm>
#include <type_traits>

#include "ray.hpp"

namespace cbct {

namespace {

constexpr int CB_X = 16, CB_Y = 16, CB_Z = 1;  // cells per workgroup: one z layer (see brick_shape)
constexpr int TABLE = 560;                     // rays staged at a time (at most 40 B each, 80 in double)
constexpr int COLUMNS = 256;                   // and pixel columns (k_cells by columns; 16 B)
constexpr int PARTS = 6;                       // views staged at a time, at most
constexpr int G_BX = 64, G_BY = 4;            // pass-2 block

// Row pitch (in elements) of the cell corner-sum array: nx + 1 cells
// rounded up to 32, so that every brick row of cells (16 consecutive x
// cells, starting at a multiple of 16) is a whole, aligned 64-byte segment
// for float and the rows of a plane start on 128-byte boundaries.
__host__ __device__ __forceinline__ long long cell_pitch(int nx) {
    return ((long long)nx + 1 + 31) & ~31LL;
}

// Ray table entry per pixel and view (prepared once): the ray increment D
// in double.  Components below TINY_D are stored as TINY_D: such a ray then
// crosses the faces of that axis far outside every sample, on the right
// sides, and its samples' positions are unchanged to the last bit.  24 bytes.
constexpr double TINY_D = 1e-20;

struct PixelRay {
    double D[3];
};

__device__ __forceinline__ float rcp(float x) { return __builtin_amdgcn_rcpf(x); }
// to half an ulp and 2^-100, in seven instructions for a division's eleven
__device__ __forceinline__ double rcp(double x) {
    double r = __builtin_amdgcn_rcp(x);
#pragma unroll
    for (int q = 0; q < 3; ++q) r = __builtin_fma(__builtin_fma(-x, r, 1.0), r, r);
    return r;
}

template <typename T> __device__ __forceinline__ T fma_t(T a, T b, T c);
template <> __device__ __forceinline__ float fma_t(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
template <> __device__ __forceinline__ double fma_t(double a, double b, double c) { return __builtin_fma(a, b, c); }
__device__ __forceinline__ float min_t(float a, float b) { return fminf(a, b); }
__device__ __forceinline__ double min_t(double a, double b) { return fmin(a, b); }
__device__ __forceinline__ float max_t(float a, float b) { return fmaxf(a, b); }
__device__ __forceinline__ double max_t(double a, double b) { return fmax(a, b); }
// a limited to [0, hi]
__device__ __forceinline__ float clamp_t(float a, float hi) { return __builtin_amdgcn_fmed3f(a, 0.0f, hi); }
__device__ __forceinline__ double clamp_t(double a, double hi) { return fmin(fmax(a, 0.0), hi); }
__device__ __forceinline__ float ceil_t(float a) { return __builtin_ceilf(a); }
__device__ __forceinline__ double ceil_t(double a) { return __builtin_ceil(a); }

// Geometry-only preparation, once per plan and workspace:
//   k_rays:        the increment D (double) of the ray through every pixel of
//                  every view;
//   k_brick_views: for every brick and view, the pixels whose rays can reach
//                  the brick and where its cells project, and the views of a
//                  brick that are staged together.
__global__ __launch_bounds__(256) void k_rays(const ViewConst *__restrict__ views, DetConst dc,
                                              int nu, int nv, PixelRay *__restrict__ rays) {
    const int i = blockIdx.x * 64 + (threadIdx.x & 63);
    const int j = blockIdx.y * 4 + (threadIdx.x >> 6);
    const int k = blockIdx.z;
    if (i >= nu || j >= nv) return;
    double Q[3], D[3];
    ray_setup(views[k], dc, i, j, Q, D);
    PixelRay e;
#pragma unroll
    for (int a = 0; a < 3; ++a) e.D[a] = fabs(D[a]) < TINY_D ? TINY_D : D[a];
    rays[((long long)k * nv + j) * nu + i] = e;
}

// How the rays through pixel columns i0 .. i1 of a view run in x and y, a sum
// of these.  1: x increases along them, 2: y does.  4: for both axes they all
// run the same way, and not too near zero to tell.  8: their main axis, along
// which each advances, in cells, at least a third as fast as along the other,
// is y, else x.  Only rays more than 50 degrees apart in one brick (in
// cells), which the source is then very near to, have none (see by_columns).
__host__ __device__ __forceinline__ int ray_directions(const ViewConst &vc, const DetConst &dc,
                                                       int i0, int i1) {
    const float ua = dc.u0 + (float)i0 * dc.au, ub = dc.u0 + (float)i1 * dc.au;
    const float tol = 1e-4f * (fabsf(vc.W[0]) + fabsf(vc.W[1]));
    float da[2], db[2];
    int dir = 4;
#pragma unroll
    for (int a = 0; a < 2; ++a) {
        da[a] = vc.W[a] + ua * vc.U[a];
        db[a] = vc.W[a] + ub * vc.U[a];
        if (da[a] > 0.0f) dir |= 1 << a;
        if (!(fminf(da[a], db[a]) > tol || fmaxf(da[a], db[a]) < -tol)) dir &= ~4;
    }
    auto leads = [&](int a) {  // at both ends, so between: the ratio is monotone in u
        return da[a] * db[a] > 0.0f && 3.0f * fabsf(da[a]) >= fabsf(da[1 - a]) &&
               3.0f * fabsf(db[a]) >= fabsf(db[1 - a]);
    };
    if (leads(1) &&
        (!leads(0) || fminf(fabsf(da[1]), fabsf(db[1])) > fminf(fabsf(da[0]), fabsf(db[0]))))
        dir |= 8;
    return dir;
}

// A brick in one view (prepared once), 64 bytes.
//
// Its footprint: pixels (i0, j0) .. (i0 + w - 1, j0 + h - 1), the rays that
// can reach it (w = h = 0 if none), and their directions (ray_directions).
//
// For each of its cells (px, py), relative to (i0, j0): the pixels whose rays
// can cross the cell lie in columns c .. c + W - 1 and rows r .. r + H - 1,
//     c = ceil(a0 + ax px + ay py),   r = ceil(b0 + bx px + by py).
// That is the cell's projection with its centre's perspective map replaced
// by the tangent map at the brick's centre, widened by the bound of what
// that leaves out, of the cells' different sizes in the view and of 0.01
// pixel: a few hundredths of a pixel for a brick of 16 cells.
//
// Views are staged in batches of consecutive views whose footprints fit the
// table together and whose rays, for k_cells by rays, have the same
// directions: batch_n views and batch_rays rays when a batch begins with this
// view (batch_n = 0: the footprint alone exceeds the table and is staged in
// parts), base this view's first table entry in its batch.  For k_cells by
// columns both hold the pixel columns too, in the upper 16 bits.
struct BrickView {
    int i0, j0, w, h;
    int W, H, dirs, base;
    float a0, ax, ay, b0, bx, by;
    int batch_n, batch_rays;
};
static_assert(sizeof(BrickView) == 64, "one 64-byte scalar load");

__host__ __device__ inline BrickView brick_view(const ViewConst &vc, const DetConst &dc, double hx,
                                                double hy, double hz, int nu, int nv,
                                                const int c0[3], const int c1[3]) {
    const double cs = vc.csd, sn = vc.snd;
    // brick centre and half extents (mm) from the source; n across the view, d its depth
    const double ex = 0.5 * (c1[0] - c0[0]) * hx, ey = 0.5 * (c1[1] - c0[1]) * hy;
    const double wx = (0.5 * (c0[0] + c1[0]) - vc.Qd[0]) * hx;
    const double wy = (0.5 * (c0[1] + c1[1]) - vc.Qd[1]) * hy;
    const double d = wy * cs - wx * sn, r = 1.0 / d, u = (wx * cs + wy * sn) * r;
    const double gx = cs + u * sn, gy = sn - u * cs;  // d u = (gx dx + gy dy) / depth
    const double D = ex * fabs(sn) + ey * fabs(cs);   // depth is within d -+ D
    const double G = ex * fabs(gx) + ey * fabs(gy);
    const double rmax = 1.0 / (d - D), rmin = 1.0 / (d + D);
    const double U = G * rmax;                        // u is within u -+ U
    const double za = (c0[2] - vc.Qd[2]) * hz, zb = (c1[2] - vc.Qd[2]) * hz;
    const double su = dc.sddd / dc.aud, sv = dc.sddd / dc.avd;
    const double ci = -dc.u0d / dc.aud, cj = -dc.v0d / dc.avd;
    BrickView o;
    // footprint, widened by 0.01 pixel and clamped to the detector
    const double fi0 = ceil((u - U) * su + ci - 0.01), fi1 = floor((u + U) * su + ci + 0.01);
    const double fj0 = ceil(fmin(za * rmin, za * rmax) * sv + cj - 0.01);
    const double fj1 = floor(fmax(zb * rmin, zb * rmax) * sv + cj + 0.01);
    o.i0 = (int)fmin(fmax(fi0, 0.0), nu - 1.0);
    o.j0 = (int)fmin(fmax(fj0, 0.0), nv - 1.0);
    o.w = (int)fmin(fi1, nu - 1.0) - o.i0 + 1;
    o.h = (int)fmin(fj1, nv - 1.0) - o.j0 + 1;
    if (!(fi0 <= nu - 1.0 && fj0 <= nv - 1.0 && fi1 >= fi0 && fj1 >= fj0) || o.w <= 0 || o.h <= 0)
        o.w = o.h = 0;
    o.dirs = o.w > 0 ? ray_directions(vc, dc, o.i0, o.i0 + o.w - 1) : 0;
    // cells: half width in u, the tangent map's error, and the same in v/sdd
    const double hw = (0.5 * hx * (fabs(gx) + U * fabs(sn)) + 0.5 * hy * (fabs(gy) + U * fabs(cs))) * rmax;
    const double eu = G * D * r * rmax;
    const double P = (hw + eu) * su + 0.01;
    const double zm = 0.5 * (za + zb);
    const double m = 0.5 * (hx * fabs(sn) + hy * fabs(cs));
    const double Pv = (0.5 * (zb - za) * rmax + fabs(zm) * (m * rmax * rmax + D * D * r * r * rmax)) * sv + 0.01;
    const double dx = (c0[0] + 0.5 - 0.5 * (c0[0] + c1[0])) * hx;  // cell (0, 0) from the centre
    const double dy = (c0[1] + 0.5 - 0.5 * (c0[1] + c1[1])) * hy;
    o.a0 = (float)(u * su + ci + su * r * (gx * dx + gy * dy) - P - o.i0);
    o.ax = (float)(su * r * gx * hx);
    o.ay = (float)(su * r * gy * hy);
    o.b0 = (float)(zm * sv * (r - r * r * (dy * cs - dx * sn)) + cj - Pv - o.j0);
    o.bx = (float)(zm * sv * r * r * hx * sn);
    o.by = (float)(-zm * sv * r * r * hy * cs);
    o.W = (int)fmin(floor(2.0 * P) + 1.0, 1e8);  // may exceed w
    o.H = (int)fmin(floor(2.0 * Pv) + 1.0, 1e8);
    o.base = 0;
    o.batch_n = 0;
    o.batch_rays = 0;
    return o;
}

// One wavefront per brick, one view per lane, 64 views at a time (batches end
// there, and at multiples of chunk); the wavefront then walks its lanes' footprints to form the batches,
// in scalar registers.
__global__ __launch_bounds__(64) void k_brick_views(const ViewConst *__restrict__ views,
                                                    DetConst dc, GridConst gc, double hx,
                                                    double hy, double hz, int nu, int nv,
                                                    int2 shape, int nbx, int nby, int nviews,
                                                    int chunk, bool by_columns,
                                                    BrickView *__restrict__ out) {
    const int b = blockIdx.x, lane = threadIdx.x;
    const int c0[3] = {(b % nbx) * shape.x - 1, ((b / nbx) % nby) * shape.y - 1,
                       b / (nbx * nby) - 1};
    const int c1[3] = {min(c0[0] + shape.x, gc.nx), min(c0[1] + shape.y, gc.ny), c0[2] + 1};
    for (int k0 = 0; k0 < nviews; k0 += 64) {
        const int k = min(k0 + lane, nviews - 1);
        BrickView o = brick_view(views[k], dc, hx, hy, hz, nu, nv, c0, c1);
        // a footprint beyond the table stands alone (batch_n = 0)
        const long long pixels = (long long)o.w * o.h;
        const bool alone = pixels > TABLE || (by_columns && o.w > COLUMNS);
        const int size = alone ? -1 : (int)pixels | (by_columns ? o.w << 16 : 0);
        const int dir = o.dirs & 4 ? o.dirs & 7 : 0;
        int head = 0, n = 0, rays = 0, cols = 0, dirs = 0;
        auto close = [&](int next) {
            if (lane == head && n > 0) {
                o.batch_n = n;
                o.batch_rays = rays | cols << 16;
                if (!by_columns) o.dirs = dirs;
            }
            head = next;
            n = rays = cols = dirs = 0;
        };
        const int count = min(64, nviews - k0);
        for (int q = 0; q < count; ++q) {
            const int sq = __builtin_amdgcn_readlane(size, q);
            const int dq = __builtin_amdgcn_readlane(dir, q);
            if (sq < 0) {
                close(q + 1);
                continue;
            }
            const int rq = sq & 0xffff, cq = sq >> 16;
            if (n == PARTS || rays + rq > TABLE || cols + cq > COLUMNS ||
                (!by_columns && rays > 0 && rq > 0 && dq != dirs) || (k0 + q) % chunk == 0)
                close(q);
            if (rays == 0) dirs = dq;
            if (lane == q) o.base = rays | cols << 16;
            rays += rq;
            cols += cq;
            ++n;
        }
        close(count);
        if (k0 + lane < nviews) out[(long long)b * nviews + k0 + lane] = o;
    }
}

// ---------------------------------------------------------------------------
// Pass 1.
//
// A ray relative to a brick: n counts the ray's samples from the first one
// in the brick, N of them lie in it, and q_a(n) = f_a + n D_a is sample n's
// coordinate in cells from the brick's first cell.  inv = 1/D, so
// fma(c, inv, -f inv) is the (real) n at which the ray crosses face c.  For
// z, of which a brick has one layer, the centred weight is
// fma(n, D_z, f_z - 1/2) itself.
template <typename T> using vec4 = T __attribute__((ext_vector_type(4)));
template <typename T> using vec2 = T __attribute__((ext_vector_type(2)));

template <typename T> struct BrickRay {
    T inv[3], D[3], f[3], N;
};

// As it is staged for k_cells by rays.
template <typename T> struct StagedRay {
    vec4<T> a;  // inv_x, -f_x inv_x, inv_y, -f_y inv_y
    vec4<T> b;  // D_x, D_y, D_z, f_z - 1/2
    vec2<T> c;  // N, residual
};

// The ray with increment D as the brick's cells use it.
//
// Which samples lie in the brick is decided by the ray's face crossings
// T(c) = (c - q) / D_f counted from sample n_mid (q the float coordinate of
// that sample, the same for every brick): neighbouring bricks form the same
// float for the face they share, so every sample is in exactly one brick,
// and inside a brick in exactly one cell (crossing_sums), whatever the
// rounding.  A sample within rounding of a face (6e-5 of a step at 512
// voxels) may get the cell beside the exact one; its weights, formed from its
// position in that cell, then are off by twice its distance from the face at
// the face's voxels and by minus that distance at their neighbours on both
// sides: second differences, to which smooth data are blind.
template <typename T>
__device__ __forceinline__ BrickRay<T> brick_ray(const double D[3], const double Qd[3], int nmid,
                                                 const int c0[3], const int c1[3]) {
    BrickRay<T> e;
    double qm[3];
    T lo = T(-8388608), hi = T(8388608);  // 2^23: beyond every sample
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        qm[a] = __builtin_fma((double)nmid, D[a], Qd[a]);
        const T q = (T)qm[a];
        e.D[a] = (T)D[a];
        e.inv[a] = rcp(e.D[a]);
        const T t0 = ((T)c0[a] - q) * e.inv[a], t1 = ((T)c1[a] - q) * e.inv[a];
        lo = max_t(lo, min_t(t0, t1));
        hi = min_t(hi, max_t(t0, t1));
    }
    lo = min_t(ceil_t(lo), T(8388608));
    hi = ceil_t(hi);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        // in double the sample's own coordinate, rounded once
        const double q = sizeof(T) == 8 ? __builtin_fma(nmid + (double)lo, D[a], Qd[a])
                                        : __builtin_fma((double)lo, D[a], qm[a]);
        e.f[a] = (T)(q - (double)c0[a]);
    }
    e.N = max_t(hi - lo, T(0));
    return e;
}

template <typename T>
__device__ __forceinline__ StagedRay<T> stage_ray(const BrickRay<T> &e, T rv) {
    StagedRay<T> o;
    o.a = vec4<T>{e.inv[0], -e.f[0] * e.inv[0], e.inv[1], -e.f[1] * e.inv[1]};
    o.b = vec4<T>{e.D[0], e.D[1], e.D[2], e.f[2] - T(0.5)};
    o.c = vec2<T>{e.N, rv};
    return o;
}

// A lane's cell in its brick: face coordinates for the crossings (the
// brick's own faces moved outward: there N decides), and the constants
// c = (face 0) - (the cell's lower face) - 1/2 of the weights.  Face 0 is
// the one the ray enters through when the directions of the rays are known
// (ORDERED), else the lower one.
template <typename T> struct CellFaces {
    T x0, x1, y0, y1;
    T cx, cy;
};

// a * b, and zero where b is zero, whatever a: one instruction in float.
__device__ __forceinline__ float mul_zero(float a, float b) {
    float p;
    asm("v_mul_legacy_f32 %0, %1, %2" : "=v"(p) : "v"(a), "v"(b));
    return p;
}
__device__ __forceinline__ double mul_zero(double a, double b) { return b == 0.0 ? 0.0 : a * b; }

// The moments' sums below, of A and B and the samples' mean position.
template <typename T>
__device__ __forceinline__ void add_crossing(T m[8], T A, T B, T x, T y, T z, T Dx, T Dy, T Dz) {
    const T bx = B * Dx, by = B * Dy;
    const T bxy = bx * Dy, bxz = bx * Dz, byz = by * Dz;
    const T px = A * x, py = A * y;
    const T pxy = fma_t(px, y, bxy);
    m[0] += A;
    m[1] += px;
    m[2] += py;
    m[3] = fma_t(A, z, m[3]);
    m[4] += pxy;
    m[5] = fma_t(px, z, m[5]) + bxz;
    m[6] = fma_t(py, z, m[6]) + byz;
    m[7] = fma_t(pxy, z, fma_t(bxz, y, fma_t(byz, x, m[7])));
}

// Add the ray's samples in the cell to the moments m = sum r (1, x, y, z,
// xy, xz, yz, xyz), x, y, z the weights minus 1/2.
//
// The samples of the crossing are n0 .. n1 - 1, k of them, equally spaced
// along a line: with their mean position (x, y, z), increments D and
// B = r k (k^2 - 1) / 12 = r sum (n - mean)^2, the third central moments
// vanish by symmetry and
//     sum r       = r k,             sum r x   = r k x,
//     sum r x y   = r k x y + B Dx Dy,
//     sum r x y z = r k x y z + B (Dx Dy z + Dx Dz y + Dy Dz x)
// exactly.  No loop over the samples, so lanes whose rays have different
// numbers of them in their cells do not wait for one another.
//
// A = r k by mul_zero: a residual that is not finite then adds nothing to
// the cells its ray does not cross.
template <bool ORDERED, typename T>
__device__ __forceinline__ void crossing_sums(T m[8], const vec4<T> ra, const vec4<T> rb,
                                              const vec2<T> rc, const CellFaces<T> &cf) {
    const T tx0 = fma_t(cf.x0, ra.x, ra.y), tx1 = fma_t(cf.x1, ra.x, ra.y);
    const T ty0 = fma_t(cf.y0, ra.z, ra.w), ty1 = fma_t(cf.y1, ra.z, ra.w);
    const T n0 = ceil_t(
        ORDERED ? max_t(max_t(tx0, ty0), T(0))
                : max_t(max_t(min_t(tx0, tx1), min_t(ty0, ty1)), T(0)));
    const T n1 = ceil_t(
        ORDERED ? min_t(min_t(tx1, ty1), rc.x)
                : min_t(min_t(max_t(tx0, tx1), max_t(ty0, ty1)), rc.x));
    const T k = max_t(n1 - n0, T(0));
    const T n = fma_t(T(0.5), n0 + n1, T(-0.5));
    const T x = fma_t(n - tx0, rb.x, cf.cx);
    const T y = fma_t(n - ty0, rb.y, cf.cy);
    const T z = fma_t(n, rb.z, rb.w);
    const T A = mul_zero(rc.y, k);
    const T B = A * fma_t(k * k, T(1) / T(12), T(-1) / T(12));
    add_crossing(m, A, B, x, y, z, rb.x, rb.y, rb.z);
}

// The same for a cell c .. c + 1 by itself, from the ray's increment: its face
// crossings are brick_ray's of those faces.
template <typename T>
__device__ __forceinline__ void cell_sums(T m[8], const double D[3], T rv, const double Qd[3],
                                          double nmid, const int c[3]) {
    double qm[3];
    T lo = T(-8388608), hi = T(8388608);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        qm[a] = __builtin_fma(nmid, D[a], Qd[a]);
        const T q = (T)qm[a], inv = rcp((T)D[a]);
        const T t0 = ((T)c[a] - q) * inv, t1 = ((T)(c[a] + 1) - q) * inv;
        lo = max_t(lo, min_t(t0, t1));
        hi = min_t(hi, max_t(t0, t1));
    }
    const T n0 = min_t(ceil_t(lo), T(8388608)), k = max_t(ceil_t(hi) - n0, T(0));
    const double n = (double)n0 + 0.5 * ((double)k - 1.0);
    auto at = [&](int a) {
        const double q = sizeof(T) == 8 ? __builtin_fma(nmid + n, D[a], Qd[a])
                                        : __builtin_fma(n, D[a], qm[a]);
        return (T)(q - ((double)c[a] + 0.5));
    };
    const T x = at(0), y = at(1), z = at(2);
    const T A = mul_zero(rv, k);
    const T B = A * fma_t(k * k, T(1) / T(12), T(-1) / T(12));
    add_crossing(m, A, B, x, y, z, (T)D[0], (T)D[1], (T)D[2]);
}

// The same by pixel columns.  The rays of a column of pixels lie in one plane
// with the z axis' direction: seen along z they are one line, y = g x + h (x
// the main axis here; where it is y, x and y change places).  Where that line
// enters and leaves a cell in x, and y, are found once for the column, and
// its rays need the moments in x and z alone, sum r (1, x, x^2, z, x z,
// x^2 z): 31 VALU instructions a ray instead of 42, and 26 a column.
//     column: g, h, 1/g, -h/g
//     ray a:  1/D_x, -f_x/D_x, D_x, f_x     ray b: D_z, f_z - 1/2, N, residual
template <typename T> struct ColumnSums {
    T s0, s1, s2, z0, z1, z2;
    T w;  // half of what D_x D_z adds to x^2 z
};

template <typename T>
__device__ __forceinline__ void column_ray(ColumnSums<T> &c, const vec4<T> ra, const vec4<T> rb,
                                           T in, T out, T centre) {
    const T n0 = ceil_t(max_t(fma_t(in, ra.x, ra.y), T(0)));
    const T n1 = ceil_t(clamp_t(fma_t(out, ra.x, ra.y), rb.z));
    const T k = max_t(n1 - n0, T(0));
    const T n = fma_t(T(0.5), n0 + n1, T(-0.5));
    const T x = fma_t(n, ra.z, ra.w) - centre;
    const T z = fma_t(n, rb.x, rb.y);
    const T A = mul_zero(rb.w, k);
    const T B = A * fma_t(k * k, T(1) / T(12), T(-1) / T(12));
    const T Bx = B * ra.z, Bxz = Bx * rb.x, Ax = A * x;
    const T q = fma_t(Ax, x, Bx * ra.z);
    c.s0 += A;
    c.s1 += Ax;
    c.s2 += q;
    c.z0 = fma_t(A, z, c.z0);
    c.z1 = fma_t(Ax, z, c.z1) + Bxz;
    c.z2 = fma_t(q, z, c.z2);
    c.w = fma_t(x, Bxz, c.w);
}

// The column's part of the moments; y = y0 + g x from the cell's centre.
template <bool Y_MAIN, typename T>
__device__ __forceinline__ void add_column(T m[8], const ColumnSums<T> &c, T y0, T g) {
    constexpr int X = Y_MAIN ? 2 : 1, Y = 3 - X, XZ = Y_MAIN ? 6 : 5, YZ = 11 - XZ;
    m[0] += c.s0;
    m[X] += c.s1;
    m[Y] = fma_t(y0, c.s0, fma_t(g, c.s1, m[Y]));
    m[4] = fma_t(y0, c.s1, fma_t(g, c.s2, m[4]));
    m[3] += c.z0;
    m[XZ] += c.z1;
    m[YZ] = fma_t(y0, c.z0, fma_t(g, c.z1, m[YZ]));
    m[7] = fma_t(y0, c.z1, fma_t(g, fma_t(T(2), c.w, c.z2), m[7]));
}

// Corner sums (index ox + 2 oy + 4 oz): corner weights are the products of
// 1/2 -+ x, 1/2 -+ y and 1/2 -+ z.
template <typename T>
__device__ __forceinline__ void moments_to_corners(const T m[8], T c[8]) {
#pragma unroll
    for (int o = 0; o < 8; ++o) {
        const T sx = o & 1 ? 1 : -1, sy = o & 2 ? 1 : -1, sz = o & 4 ? 1 : -1;
        c[o] = T(0.125) * m[0] + T(0.25) * (sx * m[1] + sy * m[2] + sz * m[3]) +
               T(0.5) * (sx * sy * m[4] + sx * sz * m[5] + sy * sz * m[6]) + sx * sy * sz * m[7];
    }
}

// The cells c0 .. c1 - 1 of a brick.  Bricks x-fastest, then y, then z; each
// XCD takes one contiguous range, so the bricks resident on an XCD at a time
// are neighbours whose footprints (ray table rows) overlap in its L2.
__device__ __forceinline__ void brick_cells(int brick, int2 shape, const GridConst &gc, int c0[3],
                                            int c1[3]) {
    const int nbx = (gc.nx + shape.x) / shape.x, nby = (gc.ny + shape.y) / shape.y;
    c0[0] = (brick % nbx) * shape.x - 1;
    c0[1] = ((brick / nbx) % nby) * shape.y - 1;
    c0[2] = brick / (nbx * nby) - 1;
    c1[0] = min(c0[0] + shape.x, gc.nx);
    c1[1] = min(c0[1] + shape.y, gc.ny);
    c1[2] = c0[2] + 1;
}

// A lane's cell in its brick.  A wavefront of a 16 x 16 brick covers 8 x 8
// cells, every 16 consecutive lanes 4 x 4 of them: the rays such lanes read
// together are then few and near each other in the table, whatever the view's
// direction.  Other bricks take their cells row by row (lanes beyond the last
// row idle).
__device__ __forceinline__ void lane_cell(int tid, int2 shape, int &lx, int &ly) {
    const bool square = shape.x == 16 && shape.y == 16;
    lx = square ? (tid & 3) | ((tid >> 2) & 4) | ((tid >> 3) & 8) : tid % shape.x;
    ly = square ? ((tid >> 2) & 3) | ((tid >> 3) & 4) | ((tid >> 4) & 8) : tid / shape.x;
}

// The corner sums of cell (cx, cy, cz) into the workgroup's chunk of `cells`, or
// added to what is there.
template <typename T>
__device__ __forceinline__ void store_corners(const T m[8], const GridConst &gc, int cx, int cy,
                                              int cz, T step, bool add, T *__restrict__ cells) {
    const long long cp = cell_pitch(gc.nx);
    const long long ncell = cp * (gc.ny + 1) * (gc.nz + 1);
    const long long lin =
        (long long)(cx + 1) + cp * ((cy + 1) + (long long)(gc.ny + 1) * (cz + 1));
    T out[8];
    moments_to_corners(m, out);
    cells += 8 * ncell * blockIdx.y;
    cells += lin;
    if (add) {
#pragma unroll
        for (int o = 0; o < 8; ++o) cells[o * ncell] += out[o] * step;
    } else {
#pragma unroll
        for (int o = 0; o < 8; ++o) cells[o * ncell] = out[o] * step;
    }
}

// Workgroups of 256 lanes, one per brick (see brick_shape) and chunk of views
// (see cut_of).
//
// Bound by VALU issue: a visit of a (ray, cell) pair is 42 VALU and 3 LDS
// instructions (40 bytes a lane; by columns 31 and 2, 32 bytes), of which fused multiply-adds take about
// 2.8 cycles of a SIMD and min, max, ceil, compare, select and integer
// instructions about 4.2 (measured with chains of each).  So what is not
// arithmetic of the moments is kept out of the visits: no counters in the
// lanes (blocks of W x H pixels), no test per sample, no order of the two
// faces where the rays' directions are known; and out of the views: where
// a cell projects is two affine maps, prepared.  Against the previous
// kernel, which tested candidate samples one by one (117 VALU a sample with
// the lanes' different counts): head transpose (512 x 512 x 70, 40 views)
// 17.63 -> 8.34 ms, 256 x 256 x 64 / 60 views 3.87 -> 1.52, 128^3 / 60 views
// 2.00 -> 0.87, 64^3 / 16 views 0.150 -> 0.081; 2.5 cycles an instruction.
// By columns, where a cell spans three pixel rows or more, the head's goes
// on to 7.7 ms (see by_columns).
// Table of 560 rays: seven groups fill the LDS (22.4 KB) as the 65 to 71 VGPRs
// allow; 480 rays 1.5% slower, 650 (six groups) 2%.  Up to six views a
// batch: 1 to 2% over four.
//
// Double data (derivative checks) took every candidate sample of every pixel
// from the ray table; with the staged rays and the closed form a transpose
// of 32^3 from 60 views takes 76 us instead of 213
// (163 with one chunk of views).  It goes by rays always: a column's line, the
// same for all its rays, carries the rounding of one ray's increment, some
// hundred cells from the source, into all of them, and the transpose was up
// to 15% further from 80-bit sums than with each ray's own; 3 to 12% faster.
template <typename T, bool COL>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(COL && sizeof(T) == 4 ? 7 : 2, 8))) void k_cells(
    const ViewConst *__restrict__ views, GridConst gc, int2 shape, int nu, int nv, int nviews,
    int chunk, const PixelRay *__restrict__ rays, const BrickView *__restrict__ bviews,
    const T *__restrict__ r, T *__restrict__ cells, T step, bool add, bool alike) {
    __shared__ vec4<T> tab[2 * TABLE];
    __shared__ vec2<T> tabc[COL ? 1 : TABLE];
    __shared__ vec4<T> tabl[COL ? COLUMNS : 1];
    __shared__ int4 slots[PARTS];   // first entry, width, first pixel of the batch's views
    __shared__ int2 cslots[PARTS];  // and first column, whether y is the main axis
    static_assert(CB_Z == 1, "a brick is one z layer of cells");
    const int tid = threadIdx.x;
    const int brick = xcd_tile(blockIdx.x, gridDim.x);
    const BrickView *bv = bviews + (long long)brick * nviews;
    int c0[3], c1[3], lx, ly;
    brick_cells(brick, shape, gc, c0, c1);
    lane_cell(tid, shape, lx, ly);
    T m[8];
#pragma unroll
    for (int o = 0; o < 8; ++o) m[o] = T(0);

    // The lane's cell (px, py) in the brick and its faces.  They pass through
    // an empty asm statement, here and where rays are staged: their
    // conversions, formed where they are used, then take no registers across
    // the loops.
    auto cell_faces = [&](int dirs, int &px, int &py) {
        px = lx;
        py = ly;
        asm volatile("" : "+v"(px), "+v"(py));
        const float fx = (float)px, fy = (float)py;
        // the brick's own faces moved outward
        const float fx0 = px == 0 ? -0.25f : fx, fy0 = py == 0 ? -0.25f : fy;
        const float fx1 = fx + (c0[0] + px + 1 == c1[0] ? 1.25f : 1.0f);
        const float fy1 = fy + (c0[1] + py + 1 == c1[1] ? 1.25f : 1.0f);
        CellFaces<T> cf;
        cf.x0 = dirs == 0 || (dirs & 1) ? fx0 : fx1;
        cf.x1 = dirs == 0 || (dirs & 1) ? fx1 : fx0;
        cf.y0 = dirs == 0 || (dirs & 2) ? fy0 : fy1;
        cf.y1 = dirs == 0 || (dirs & 2) ? fy1 : fy0;
        cf.cx = cf.x0 - fx - T(0.5);
        cf.cy = cf.y0 - fy - T(0.5);
        return cf;
    };
    const int kend = min(nviews, (int)(blockIdx.y + 1) * chunk);
    for (int k = blockIdx.y * chunk; k < kend;) {
        // the batch, or the parts of a view too large for the table: bands of
        // rows, or pieces of a row
        int n = bv[k].batch_n, total = bv[k].batch_rays & 0xffff;
        int columns = bv[k].batch_rays >> 16;
        // (batches formed for columns mix directions)
        const int dirs = alike && bv[k].dirs & 4 ? bv[k].dirs : 0;
        int cols = 1, pw = 0, ph = 0, parts = 1;
        if (n == 0) {
            constexpr int WIDEST = COL ? COLUMNS : TABLE;
            n = 1;
            cols = (bv[k].w + WIDEST - 1) / WIDEST;
            pw = (bv[k].w + cols - 1) / cols;
            ph = min(TABLE / pw, bv[k].h);
            parts = cols * ((bv[k].h + ph - 1) / ph);
        }
        for (int part = 0; part < parts; ++part) {
            int oi = 0, oj = 0, w = bv[k].w, h = bv[k].h;  // the part within the view
            if (parts > 1) {
                oi = (part % cols) * pw;
                oj = (part / cols) * ph;
                w = max(min(pw, w - oi), 0);
                h = min(ph, h - oj);
                total = w * h;
                columns = w;
            }
            if (tid < PARTS) {
                int4 s = make_int4(0x7fffffff, 1, 0, 0);
                int2 c = make_int2(0x7fffffff, 0);
                if (tid < n) {
                    const BrickView &b = bv[k + tid];
                    s = make_int4(b.base & 0xffff, parts > 1 ? w : b.w, b.i0 + oi,
                                  b.j0 + oj);
                    c = make_int2(b.base >> 16, b.dirs & 8);
                }
                slots[tid] = s;
                if constexpr (COL) cslots[tid] = c;
            }
            __syncthreads();  // readers of the table are done, the slots are there
            for (int t = tid; t < total; t += 256) {
                int f0[3] = {c0[0], c0[1], c0[2]}, f1[3] = {c1[0], c1[1], c1[2]};
                asm volatile("" : "+s"(f0[0]), "+s"(f0[1]), "+s"(f0[2]), "+s"(f1[0]),
                                  "+s"(f1[1]), "+s"(f1[2]));
                int v = 0;
#pragma unroll
                for (int q = 1; q < PARTS; ++q) v += t >= slots[q].x;
                const int4 sl = slots[v];
                // row of the view's entry e by a float reciprocal: exact
                // below 2^13, since (e + 1/2)/w stays >= 1/(2 w) from an
                // integer
                const int e = t - sl.x;
                const int row = (int)(((float)e + 0.5f) * rcp((float)sl.y));
                const int col = e - row * sl.y;
                const long long pix =
                    ((long long)(k + v) * nv + (sl.w + row)) * nu + (sl.z + col);
                const PixelRay g = rays[pix];
                const ViewConst &vc = views[k + v];
                const double Qd[3] = {vc.Qd[0], vc.Qd[1], vc.Qd[2]};
                const BrickRay<T> ray = brick_ray<T>(g.D, Qd, vc.nmid, f0, f1);
                if constexpr (COL) {
                    const bool ym = cslots[v].y != 0;
                    const T inv = ym ? ray.inv[1] : ray.inv[0], f = ym ? ray.f[1] : ray.f[0];
                    tab[t] = vec4<T>{inv, -f * inv, ym ? ray.D[1] : ray.D[0], f};
                    tab[t + TABLE] = vec4<T>{ray.D[2], ray.f[2] - T(0.5), ray.N, r[pix]};
                } else {
                    const StagedRay<T> e = stage_ray(ray, r[pix]);
                    tab[t] = e.a;
                    tab[t + TABLE] = e.b;
                    tabc[t] = e.c;
                }
            }
            for (int t = tid; COL && t < columns; t += 256) {
                int v = 0;
#pragma unroll
                for (int q = 1; q < PARTS; ++q) v += t >= cslots[q].x;
                const int4 sl = slots[v];
                const int2 cs = cslots[v];
                const PixelRay g =
                    rays[((long long)(k + v) * nv + sl.w) * nu + (sl.z + t - cs.x)];
                const ViewConst &vc = views[k + v];
                const bool ym = cs.y != 0;
                const double qx = vc.Qd[0] - c0[0], qy = vc.Qd[1] - c0[1];
                const double gd = ym ? g.D[0] / g.D[1] : g.D[1] / g.D[0];
                const double hd = ym ? qx - gd * qy : qy - gd * qx;
                const double id = 1.0 / gd;
                tabl[t] = vec4<T>{(T)gd, (T)hd, (T)id, (T)(-hd * id)};
            }
            __syncthreads();
            int px, py;
            const CellFaces<T> cf = cell_faces(COL ? 0 : dirs, px, py);
            const float fx = (float)px, fy = (float)py;
            auto visit = [&](auto ordered) {
                constexpr bool ORD = decltype(ordered)::value;
                for (int v = 0; v < n; ++v) {
                    const BrickView b = bv[k + v];
                    const int bw = parts > 1 ? w : b.w, bh = parts > 1 ? h : b.h;
                    if (bw == 0) continue;
                    // Every lane visits a block of W x H pixels that holds its
                    // cell's, moved inside the part: a ray that does not cross
                    // a cell adds nothing to it, and loops without per-lane
                    // counters are shorter.
                    const int W = min(b.W, bw), H = min(b.H, bh);
                    const int ci = (int)__builtin_ceilf(b.a0 + b.ax * fx + b.ay * fy) - oi;
                    const int cj = (int)__builtin_ceilf(b.b0 + b.bx * fx + b.by * fy) - oj;
                    if (parts > 1 && !__builtin_amdgcn_ballot_w64(ci + b.W > 0 && ci < bw &&
                                                                  cj + b.H > 0 && cj < bh))
                        continue;
                    const int e =
                        (b.base & 0xffff) + max(min(cj, bh - H), 0) * bw + max(min(ci, bw - W), 0);
                    const vec4<T> *p = tab + e;
                    const vec2<T> *pc = tabc + e;
                    for (int y = 0; y < H; ++y, p += bw, pc += bw) {
                        int x = 0;
                        for (; x + 1 < W; x += 2) {
                            crossing_sums<ORD>(m, p[x], p[x + TABLE], pc[x], cf);
                            crossing_sums<ORD>(m, p[x + 1], p[x + 1 + TABLE], pc[x + 1], cf);
                        }
                        if (x < W) crossing_sums<ORD>(m, p[x], p[x + TABLE], pc[x], cf);
                    }
                }
            };
            auto visit_columns = [&](const BrickView &b, int bw, int bh, auto y_main) {
                constexpr bool YM = decltype(y_main)::value;
                const int W = min(b.W, bw), H = min(b.H, bh);
                const int ci = (int)__builtin_ceilf(b.a0 + b.ax * fx + b.ay * fy) - oi;
                const int cj = (int)__builtin_ceilf(b.b0 + b.bx * fx + b.by * fy) - oj;
                if (parts > 1 && !__builtin_amdgcn_ballot_w64(ci + b.W > 0 && ci < bw &&
                                                              cj + b.H > 0 && cj < bh))
                    return;
                const int ec = max(min(ci, bw - W), 0), er = max(min(cj, bh - H), 0);
                const vec4<T> *p = tab + (b.base & 0xffff) + er * bw + ec;
                const vec4<T> *pl = tabl + (b.base >> 16) + ec;
                const bool up = b.dirs & (YM ? 2 : 1);
                const T x0 = YM ? cf.y0 : cf.x0, x1 = YM ? cf.y1 : cf.x1;
                const T y0 = YM ? cf.x0 : cf.y0, y1 = YM ? cf.x1 : cf.y1;
                const T cx = (YM ? fy : fx) + T(0.5), cy = (YM ? fx : fy) + T(0.5);
                for (int x = 0; x < W; ++x) {
                    const vec4<T> l = pl[x];
                    const T t0 = fma_t(y0, l.z, l.w), t1 = fma_t(y1, l.z, l.w);
                    const T lo = max_t(x0, min_t(t0, t1)), hi = min_t(x1, max_t(t0, t1));
                    const T in = up ? lo : hi, out = up ? hi : lo;
                    ColumnSums<T> c = {};
                    const vec4<T> *q = p + x;
                    int y = 0;
                    for (; y + 1 < H; y += 2, q += 2 * bw) {
                        column_ray(c, q[0], q[TABLE], in, out, cx);
                        column_ray(c, q[bw], q[bw + TABLE], in, out, cx);
                    }
                    if (y < H) column_ray(c, q[0], q[TABLE], in, out, cx);
                    add_column<YM>(m, c, fma_t(cx, l.x, l.y) - cy, l.x);
                }
            };
            if constexpr (COL) {
                for (int v = 0; v < n; ++v) {
                    const BrickView b = bv[k + v];
                    const int bw = parts > 1 ? w : b.w, bh = parts > 1 ? h : b.h;
                    if (bw == 0) continue;
                    if (b.dirs & 8)
                        visit_columns(b, bw, bh, std::true_type());
                    else
                        visit_columns(b, bw, bh, std::false_type());
                }
            } else if (dirs) {
                visit(std::true_type());
            } else {
                visit(std::false_type());
            }
        }
        k += n;
    }
    if (c0[0] + lx < c1[0] && c0[1] + ly < c1[1])
        store_corners(m, gc, c0[0] + lx, c0[1] + ly, c0[2], step, add, cells);
}

// The same where the source is so near that a brick's blocks of pixels are far
// more than its cells need (see choose_cells): each lane takes the pixels of
// its own cell, their rays from the ray table.  A visit is about 75 VALU
// instructions, a third of them in double, and two loads, and wavefronts wait
// for no others.
template <typename T>
__global__ __launch_bounds__(256) void k_cells_near(
    const ViewConst *__restrict__ views, DetConst dc, GridConst gc, int2 shape, int nu, int nv,
    int nviews, int chunk, const PixelRay *__restrict__ rays, const T *__restrict__ r,
    T *__restrict__ cells, T step, bool add) {
    int c0[3], c1[3], lx, ly;
    brick_cells(xcd_tile(blockIdx.x, gridDim.x), shape, gc, c0, c1);
    lane_cell(threadIdx.x, shape, lx, ly);
    const int c[3] = {c0[0] + lx, c0[1] + ly, c0[2]};
    if (c[0] >= c1[0] || c[1] >= c1[1]) return;
    T m[8];
#pragma unroll
    for (int o = 0; o < 8; ++o) m[o] = T(0);
    const float su = (float)(dc.sddd / dc.aud), sv = (float)(dc.sddd / dc.avd * gc.hz);
    const float ci = (float)(-dc.u0d / dc.aud), cj = (float)(-dc.v0d / dc.avd);
    const int kend = min(nviews, (int)(blockIdx.y + 1) * chunk);
    for (int k = blockIdx.y * chunk; k < kend; ++k) {
        const ViewConst &vc = views[k];
        // the bounds of the cell's projection, from its corners' (at most
        // 4e-7 of an index off), and 0.01 pixel more
        const double n = __builtin_fma((double)c[0], vc.en[0],
                                       __builtin_fma((double)c[1], vc.en[1], vc.en[2]));
        const double d = __builtin_fma((double)c[0], vc.ew[0],
                                       __builtin_fma((double)c[1], vc.ew[1], vc.ew[2]));
        float umin = 3e38f, umax = -3e38f, rmin = 3e38f, rmax = 0.0f;
#pragma unroll
        for (int o = 0; o < 4; ++o) {
            const float id = rcp((float)(d + (o & 1 ? vc.ew[0] : 0.0) + (o & 2 ? vc.ew[1] : 0.0)));
            const float u =
                (float)(n + (o & 1 ? vc.en[0] : 0.0) + (o & 2 ? vc.en[1] : 0.0)) * id * su;
            umin = fminf(umin, u);
            umax = fmaxf(umax, u);
            rmin = fminf(rmin, id);
            rmax = fmaxf(rmax, id);
        }
        const float va = (float)(c[2] - vc.Qd[2]) * sv, vb = (float)(c[2] + 1 - vc.Qd[2]) * sv;
        const float vmin = fminf(va * rmin, va * rmax), vmax = fmaxf(vb * rmin, vb * rmax);
        const float mu = 0.01f + 4e-7f * fmaxf(fabsf(umin), fabsf(umax));
        const float mv = 0.01f + 4e-7f * fmaxf(fabsf(vmin), fabsf(vmax));
        const int i0 = max((int)__builtin_ceilf(umin - mu + ci), 0);
        const int j0 = max((int)__builtin_ceilf(vmin - mv + cj), 0);
        const int i1 = min((int)__builtin_floorf(umax + mu + ci), nu - 1);
        const int j1 = min((int)__builtin_floorf(vmax + mv + cj), nv - 1);
        const double Qd[3] = {vc.Qd[0], vc.Qd[1], vc.Qd[2]};
        const double nmid = vc.nmid;
        const long long view = (long long)k * nu * nv;
        int i = i0, j = j0;
        auto next = [&] {
            const long long at = view + (long long)j * nu + i;
            if (++i > i1) {
                i = i0;
                ++j;
            }
            return at;
        };
        // two rays at a time: a few cells next to the source have most of a
        // view's rays, and their lanes' chains are what the chip waits for
        int q = i0 <= i1 && j0 <= j1 ? (i1 - i0 + 1) * (j1 - j0 + 1) : 0;
        for (; q > 1; q -= 2) {
            const long long a = next(), b = next();
            const PixelRay ga = rays[a], gb = rays[b];
            const T ra = r[a], rb = r[b];
            cell_sums(m, ga.D, ra, Qd, nmid, c);
            cell_sums(m, gb.D, rb, Qd, nmid, c);
        }
        if (q > 0) {
            const long long a = next();
            cell_sums(m, rays[a].D, r[a], Qd, nmid, c);
        }
    }
    store_corners(m, gc, c[0], c[1], c[2], step, add, cells);
}

// Pass 2: out = sum of corner o of cell (v - o) over o in {0,1}^3 and over the
// chunks of views, then out = f - tau * out when f is given.
template <typename T>
__global__ __launch_bounds__(256) void k_gather(GridConst gc, int chunks,
                                                const T *__restrict__ cells,
                                                const T *__restrict__ f, T tau,
                                                T *__restrict__ out) {
    const int ix = blockIdx.x * G_BX + threadIdx.x;
    const int iy = blockIdx.y * G_BY + threadIdx.y;
    const int iz = blockIdx.z;
    if (ix >= gc.nx || iy >= gc.ny) return;
    const long long cxn = cell_pitch(gc.nx), cxyn = cxn * (gc.ny + 1);
    const long long ncell = cxyn * (gc.nz + 1);
    // cell (ix - ox, iy - oy, iz - oz) is stored at (ix - ox + 1, ...)
    const long long base = (long long)(ix + 1) + cxn * (iy + 1) + cxyn * (iz + 1);
    T s = T(0);
    for (int c = 0; c < chunks; ++c, cells += 8 * ncell)
#pragma unroll
        for (int o = 0; o < 8; ++o) {
            const int ox = o & 1, oy = (o >> 1) & 1, oz = o >> 2;
            // voxel v is corner o of cell v - o (corners of cell c are c + o)
            s += cells[o * ncell + base - ox - oy * cxn - oz * cxyn];
        }
    const long long v = (long long)ix + (long long)gc.nx * (iy + (long long)gc.ny * iz);
    out[v] = f ? f[v] - tau * s : s;
}

// The paper's Eq. (2) gradient, voxel-driven: a lane sums, for ZC voxels of a
// column, over the views L^3/(L0 l^2) times the bilinear interpolant of the
// residual at the voxel's imager point (zero beyond the outermost pixel
// centres), and scales by hx hy hz / (au av) (the transpose's scale).  The
// imager point in double (1/d from a float reciprocal refined by one double
// Newton step), the distance l and the interpolation in float, weights and
// sum in double.  L^3/(L0 l^2) is evaluated as L0^2 l / d^3 (L/l = L0/d along
// the ray, d the depth of the voxel along the central ray).
//
// Everything of a view but the row coordinate and l is the same along a
// column.  Where all the wavefront's imager points have their four taps on
// the detector, their tests go too.  Bound by VALU issue, the double
// arithmetic above all, and by the gathers: about 33 instructions a voxel
// and view with four voxels a lane, 26 / 4 of them for the view, and two
// loads.  Head (512 x 512 x 70, 40 views) 1640 us with one voxel a lane and
// tested taps, 825 with four, 786 with six and what all lanes share in scalar
// registers (96 vector registers; eight voxels take 116 and 4% longer).  The
// row's fraction read from the low word of a double 2^20 above it took 724,
// but is then cut at 2^-32 of a row: further from the exact values than before
// in 22 of 40 geometries, by up to 0.2% of their error.  A view's loads are
// issued before its sums by a barrier to the scheduler: left to itself it
// orders them so or not, 780 or 875 us, by what changes elsewhere.  With one
// voxel a lane, where few wavefronts wait for a view's latencies, a view has no
// branch and its taps no tests, and the two pixels of a row are one load: 64^3
// from 16 views 14.5 -> 10.5 us (14.8 with the first kernel), 14 x 14 x 25 from
// 21 views 15.0 -> 10.3 (14.1), 64^3 from 20 views with the source at 1.3 radii
// 14.0 -> 12.2 (18.6; a load for each pixel 16.2).
constexpr int Q_BX = 64, Q_BY = 4;

// sqrt(x) for x > 0: the hardware's reciprocal root and a correction, which
// gives the correctly rounded value (checked for every mantissa of both
// parities of the exponent, at five exponents).
__device__ __forceinline__ float sqrt_pos(float x) {
    const float r = __builtin_amdgcn_rsqf(x);
    const float y = x * r;
    return __builtin_fmaf(__builtin_fmaf(-y, y, x), 0.5f * r, y);
}

// The same double in every lane, in scalar registers.
__device__ __forceinline__ double uniform(double v) {
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)b);
    const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(b >> 32));
    return __builtin_bit_cast(double, (unsigned long long)hi << 32 | lo);
}

// What a view is to a column of voxels (i, j): the fractional pixel indices fi,
// and fj + q dj in plane q of the column, w0 = weight / l and the square of l's
// part in the xy plane.
struct Eq2View {
    double fi, fj, dj, w0, lxy2;
};

__device__ __forceinline__ Eq2View eq2_view(const ViewConst &vc, const DetConst &dc, int i, int j,
                                            double kz, double su, double svh, double ci,
                                            double cj) {
    // source-to-voxel vector (mm): n along e_u, d along e_w (depth)
    const double n = __builtin_fma((double)i, vc.en[0], __builtin_fma((double)j, vc.en[1], vc.en[2]));
    const double d = __builtin_fma((double)i, vc.ew[0], __builtin_fma((double)j, vc.ew[1], vc.ew[2]));
    // 1/d from the float reciprocal and one Newton step in double: the
    // relative error squares, from ~2e-7 to ~4e-14
    const double id0 = (double)__builtin_amdgcn_rcpf((float)d);
    const double id = id0 * __builtin_fma(-d, id0, 2.0);
    Eq2View v;
    v.fi = __builtin_fma(n * id, su, ci);
    v.dj = id * svh;
    v.fj = __builtin_fma(kz, v.dj, cj);
    v.w0 = dc.sdd2d * (id * id * id);
    v.lxy2 = __builtin_fma(n, n, d * d);
    return v;
}

template <int ZC>
__global__ __launch_bounds__(256) void k_eq2(const ViewConst *__restrict__ views, DetConst dc,
                                             GridConst gc, double hx, double hy, double hz,
                                             int nu, int nv, int nviews,
                                             const float *__restrict__ r,
                                             const float *__restrict__ f, double scale,
                                             double tau, float *__restrict__ out) {
    const int i = blockIdx.x * Q_BX + threadIdx.x;
    const int j = blockIdx.y * Q_BY + threadIdx.y;
    const int k0 = blockIdx.z * ZC;
    if (i >= gc.nx || j >= gc.ny) return;
    // what all lanes share, in scalar registers where vector ones are short
    // (two voxels a lane lose 3% by it)
    auto same = [](double v) { return ZC > 2 ? uniform(v) : v; };
    const double su = same(dc.sddd / dc.aud), svh = same(dc.sddd / dc.avd * hz);
    // index of u = 0, v = 0
    const double ci = same(-dc.u0d / dc.aud), cj = same(-dc.v0d / dc.avd);
    const double kz = same((double)k0 - views[0].Qd[2]);  // the same in every view
    double sum[ZC], wz2[ZC];
#pragma unroll
    for (int q = 0; q < ZC; ++q) {
        sum[q] = 0.0;
        wz2[q] = same((kz + q) * hz * ((kz + q) * hz));
    }
    // 32-bit byte offsets within a view, 24-bit factors, rows below 2^20
    const bool narrow = (long long)nu * nv < (1LL << 30) && nu < (1 << 22) && nv < (1 << 20);
    auto weight = [&](const Eq2View &v, int q) {
        return v.w0 * (double)sqrt_pos((float)(wz2[q] + v.lxy2));
    };
    int t0 = 0;
    if (ZC == 1 && nu > 1 && (long long)nu * nv < (1LL << 28) && nu < (1 << 21) && nv < (1 << 20)) {
        // Few wavefronts: a view takes its chain of latencies, shorter without
        // branches and with the next view's beside it.  A view is a buffer that
        // reads zero beyond its ends.
#pragma unroll 2
        for (int t = 0; t < nviews; ++t) {
            const Eq2View v = eq2_view(views[t], dc, i, j, kz, su, svh, ci, cj);
            const double i0d = __builtin_floor(v.fi), j0d = __builtin_floor(v.fj);
            const float a = (float)(v.fi - i0d), b = (float)(v.fj - j0d);
            const int i0 = (int)fmax(fmin(i0d, (double)nu), -2.0);
            const int j0 = (int)fmax(fmin(j0d, (double)nv), -2.0);
            // the pair of a row's pixels that holds those of the two that are there
            const int ip = max(min(i0, nu - 2), 0);
            const unsigned nu4 = 4u * (unsigned)nu;
            const unsigned o = (unsigned)__mul24(j0, 4 * nu) + 4u * (unsigned)ip;
            const __amdgpu_buffer_rsrc_t rt = __builtin_amdgcn_make_buffer_rsrc(
                (void *)(r + (long long)t * nu * nv), (short)0, 4 * nu * nv, 0x00020000);
            using pair = unsigned __attribute__((ext_vector_type(2)));
            const pair p0 = __builtin_amdgcn_raw_buffer_load_b64(rt, o, 0, 0);
            const pair p1 = __builtin_amdgcn_raw_buffer_load_b64(rt, o + nu4, 0, 0);
            const bool left = i0 < 0, right = i0 > nu - 2;
            const bool in0 = i0 >= 0 && i0 < nu, in1 = i0 >= -1 && i0 < nu - 1;
            auto first = [&](pair p) {
                return in0 ? __builtin_bit_cast(float, right ? p[1] : p[0]) : 0.0f;
            };
            auto second = [&](pair p) {
                return in1 ? __builtin_bit_cast(float, left ? p[0] : p[1]) : 0.0f;
            };
            const float r00 = first(p0), r10 = second(p0), r01 = first(p1), r11 = second(p1);
            const float v0 = r00 + a * (r10 - r00), v1 = r01 + a * (r11 - r01);
            sum[0] = __builtin_fma(weight(v, 0), (double)(v0 + b * (v1 - v0)), sum[0]);
        }
        t0 = nviews;
    }
    for (int t = t0; t < nviews; ++t) {
        const Eq2View v = eq2_view(views[t], dc, i, j, kz, su, svh, ci, cj);
        const double fj1 = __builtin_fma((double)(ZC - 1), v.dj, v.fj);
        const double i0d = __builtin_floor(v.fi);
        const float a = (float)(v.fi - i0d);
        const float *rt = r + (long long)t * nu * nv;
        const bool inside = narrow && v.fi >= 0.0 && v.fi < nu - 1.0 && fmin(v.fj, fj1) >= 0.0 &&
                            fmax(v.fj, fj1) < nv - 1.0;
        if (!__builtin_amdgcn_ballot_w64(!inside)) {
            const float *rt1 = rt + nu;
            const unsigned nu4 = 4u * (unsigned)nu;
            const unsigned i4 = 4u * (unsigned)(int)i0d;
            float r00[ZC], r10[ZC], r01[ZC], r11[ZC], b[ZC];
#pragma unroll
            for (int q = 0; q < ZC; ++q) {
                const double fj = __builtin_fma((double)q, v.dj, v.fj);
                const unsigned o = __umul24((unsigned)(int)fj, nu4) + i4;
                b[q] = (float)__builtin_amdgcn_fract(fj);
                const float *p = (const float *)((const char *)rt + o);
                const float *p1 = (const float *)((const char *)rt1 + o);
                r00[q] = p[0], r10[q] = p[1], r01[q] = p1[0], r11[q] = p1[1];
            }
            // all loads go out before the first is waited for
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int q = 0; q < ZC; ++q) {
                const float v0 = r00[q] + a * (r10[q] - r00[q]);
                const float v1 = r01[q] + a * (r11[q] - r01[q]);
                sum[q] = __builtin_fma(weight(v, q), (double)(v0 + b[q] * (v1 - v0)), sum[q]);
            }
            continue;
        }
        const int i0 = (int)fmax(fmin(i0d, (double)nu), -2.0);
        const bool in0 = i0 >= 0 && i0 < nu, in1 = i0 + 1 >= 0 && i0 + 1 < nu;
#pragma unroll
        for (int q = 0; q < ZC; ++q) {
            const double fj = __builtin_fma((double)q, v.dj, v.fj);
            const double j0d = __builtin_floor(fj);
            const float b = (float)(fj - j0d);
            const int j0 = (int)fmax(fmin(j0d, (double)nv), -2.0);
            const bool jn0 = j0 >= 0 && j0 < nv, jn1 = j0 + 1 >= 0 && j0 + 1 < nv;
            const float r00 = (in0 && jn0) ? rt[(long long)j0 * nu + i0] : 0.0f;
            const float r10 = (in1 && jn0) ? rt[(long long)j0 * nu + i0 + 1] : 0.0f;
            const float r01 = (in0 && jn1) ? rt[(long long)(j0 + 1) * nu + i0] : 0.0f;
            const float r11 = (in1 && jn1) ? rt[(long long)(j0 + 1) * nu + i0 + 1] : 0.0f;
            const float v0 = r00 + a * (r10 - r00), v1 = r01 + a * (r11 - r01);
            sum[q] = __builtin_fma(weight(v, q), (double)(v0 + b * (v1 - v0)), sum[q]);
        }
    }
#pragma unroll
    for (int q = 0; q < ZC; ++q) {
        if (k0 + q >= gc.nz) break;
        const long long v = (long long)i + (long long)gc.nx * (j + (long long)gc.ny * (k0 + q));
        const double s = scale * sum[q];
        out[v] = f ? (float)((double)f[v] - tau * s) : (float)s;
    }
}

}  // namespace

namespace {

// Cells of a brick in x and y: 16 x 16, or of the near-square shapes of at
// most 256 the one that covers the grid's nx + 1 by ny + 1 cells with the
// fewest bricks.  A grid of 2^k voxels has one cell more than whole 16 x 16
// bricks, and a last row and column of nearly empty ones: 18 bricks of
// 22 x 11 instead of 25 cover 65 x 65 cells, 70 of 13 x 19 instead of 81
// 129 x 129.  Transposes 16 x 16 / so (us): 64^3 / 16 views 67 / 58, 96^3 / 16
// 132 / 121, 128^3 / 60 893 / 821.  Rows of other bricks do not line up with
// the wavefronts: with 3% fewer bricks, at 256 x 256 x 64 and 256^3, the time
// is the same to 1% more, so 16 x 16 stays where others save less than 5%.
int2 brick_shape(const cbct_geom &g) {
    auto bricks = [&](int2 s) {
        return (long long)((g.nx + s.x) / s.x) * ((g.ny + s.y) / s.y);
    };
    const int2 square = make_int2(CB_X, CB_Y);
    int2 best = square;
    for (int x = 11; x <= 23; ++x) {
        const int2 s = make_int2(x, CB_X * CB_Y / x);
        const long long a = bricks(s), b = bricks(best);
        if (a < b || (a == b && abs(s.x - s.y) < abs(best.x - best.y))) best = s;
    }
    return 20 * bricks(best) <= 19 * bricks(square) ? best : square;
}

// Whether the cell pass goes by pixel columns: where a cell spans three rows of
// them or more at the grid's centre, so that a column's own arithmetic is
// small against its rays'.  256 x 256 x 48, 40 views, by rays / by columns
// (us): 2 rows 677 / 728, 2.5 774 / 796, 3 906 / 896, 3.5 1017 / 976, 4
// 1114 / 1052, 5 1278 / 1167; 512 x 512 x 70 (4.8 rows) 8790 / 7740.
constexpr double COLUMN_ROWS = 3.0;

//
// A view's rays through a brick then need a main axis (see ray_directions).
// They have one if their directions in cells lie within an interval of angles
// that reaches less than from atan(1/3) to atan(3); with cells of sides 1 and
// a, that is from atan(1/(3a)) to atan(3/a), at the narrowest.  A brick's rays
// spread over at most its diagonal over the nearest depth, times the length of
// (1, u/sdd); half the angle is left unused.
bool by_columns(const cbct_geom &g) {
    if (!(g.hz * g.sdd >= COLUMN_ROWS * g.sad * g.av)) return false;
    const int2 shape = brick_shape(g);
    const double D = hypot(shape.x * g.hx, shape.y * g.hy);
    const double depth = g.sad - hypot(0.5 * (g.nx + 1) * g.hx + fabs(g.x_off),
                                       0.5 * (g.ny + 1) * g.hy + fabs(g.y_off));
    const double fan = (0.5 * g.nu * g.au + fabs(g.u_off)) / g.sdd + D / depth;
    const double a = std::max(g.hx, g.hy) / std::min(g.hx, g.hy);
    return 2.0 * D / depth * hypot(1.0, fan) < atan(3.0 / a) - atan(1.0 / (3.0 * a));
}

// Views a workgroup of the cell pass takes.  A small grid has fewer bricks
// than the chip has room for (about 1800 workgroups), and each works its way
// through the views' loads and barriers alone; its views are then cut into
// up to eight chunks, with cell sums of their own, as long as no more than
// SPLIT_GROUPS workgroups result and each keeps enough views to fill its
// batches: the more, the better the bricks fill the chip by themselves.
// Transposes (us) with 1 chunk / up to 3072 workgroups / up to 6144: 32^3 / 60
// views 115 / 50 / 50, 48^3 / 16 47 / 38 / 39.  With 1 / 2 chunks, and as
// chunks of 4 views, float: 1170 bricks (64^3), 16 views 59 / 57, 59 (and 2%
// for 4 with finer pixels); 1340 (66^3), 16 66 / 61, 65; 1470 (128 x 128 x 20),
// 16 54 / 54, 60; 2072 (109 x 115 x 36), 16 177 / 166, 24 260 / 240; 2268 (80^3),
// 8 57 / -, 60, 16 88 / 87; 2324 (82^3), 16 95 / 94, 24 135 / 129; 2784 (86^3), 16
// 108 / 113, 24 155 / 159, 40 242 / 246; double: 2072, 16 359 / 349; 2268, 8 95 /
// -, 103, 16 155 / 160; 2324, 24 257 / 243; 2784, 16 206 / 234.
constexpr int SPLIT_GROUPS = 6144, SPLIT_MAX = 8;

int least_views(long long bricks) { return bricks < 1300 ? 4 : bricks < 2500 ? 8 : 16; }

// How the cell pass cuts a grid and its views.
struct Cut {
    int2 shape;       // cells of a brick
    dim3 bricks;
    int slab;           // views of a launch
    int chunk, chunks;  // views of a workgroup; chunks of a launch's views
};

// Bricks' views are kept for all views where they take no more than TABLE_BYTES.
// Beyond that they take a quarter, or TABLE_BYTES where that is more: a launch
// then goes through a slab of the views, prepared anew for each call, and adds
// its cell sums to the slabs' before.  512^3 voxels from 720 views: 8.6 GB
// instead of 25.7, in a call or a solve.  Preparing and adding take
// a tenth of the transpose's time (320^3, 480 views in four slabs 89.4 -> 98.8
// ms), so tables that the card easily holds are kept.
constexpr long long TABLE_BYTES = 8LL << 30;

Cut cut_of(const cbct_geom &g) {
    Cut c;
    c.shape = brick_shape(g);
    c.bricks = dim3((g.nx + c.shape.x) / c.shape.x, (g.ny + c.shape.y) / c.shape.y, g.nz + 1);
    const long long bricks = (long long)c.bricks.x * c.bricks.y * c.bricks.z;
    const long long view = (long long)sizeof(BrickView) * bricks;
    const long long most = std::max(TABLE_BYTES / view, (g.n_views + 3LL) / 4);
    const int slabs = (int)((g.n_views + most - 1) / most);
    c.slab = (g.n_views + slabs - 1) / slabs;
    const int want = (int)std::min((long long)SPLIT_MAX, SPLIT_GROUPS / bricks);
    const int n = std::max(1, std::min(want, c.slab / least_views(bricks)));
    c.chunk = (c.slab + n - 1) / n;
    c.chunks = (c.slab + c.chunk - 1) / c.chunk;
    return c;
}

size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

size_t table_bytes(const Cut &c) {
    return sizeof(BrickView) * (size_t)c.bricks.x * c.bricks.y * c.bricks.z * c.slab;
}

size_t ray_bytes(const cbct_geom &g) {
    return align256(sizeof(PixelRay) * (size_t)g.n_views * g.nu * g.nv);
}

size_t sums_bytes(const cbct_geom &g, const Cut &c, size_t elem) {
    return align256(elem * 8 * c.chunks * (size_t)cell_pitch(g.nx) * (g.ny + 1) * (g.nz + 1));
}

hipError_t launch_brick_views(const cbct_plan &p, const Cut &c, int k, int views, BrickView *out,
                              hipStream_t s) {
    const dim3 b = c.bricks;
    hipLaunchKernelGGL(k_brick_views, dim3(b.x * b.y * b.z), dim3(64), 0, s, p.d_views + k, p.det,
                       p.grid, p.g.hx, p.g.hy, p.g.hz, p.g.nu, p.g.nv, c.shape, (int)b.x, (int)b.y,
                       views, c.chunk, by_columns(p.g), out);
    return hipGetLastError();
}

}  // namespace

// The cell sums, and after them a slab's bricks' views.
size_t bp_cells_bytes(const cbct_geom &g, size_t elem) {
    const Cut c = cut_of(g);
    return sums_bytes(g, c, elem) + (c.slab < g.n_views ? align256(table_bytes(c)) : 0);
}

// The ray table, and after it the bricks' views if all are kept.
size_t bp_geom_bytes(const cbct_geom &g) {
    const Cut c = cut_of(g);
    return ray_bytes(g) + (c.slab < g.n_views ? 0 : table_bytes(c));
}

size_t bp_workspace_bytes(const cbct_geom &g, size_t elem) {
    return bp_cells_bytes(g, elem) + bp_geom_bytes(g);
}

void *bp_geom_in(void *ws, const cbct_geom &g, size_t elem) {
    return (char *)ws + bp_cells_bytes(g, elem);
}

void cell_pass_config(int32_t out[4]) {
    out[0] = CB_X;
    out[1] = CB_Y;
    out[2] = CB_Z;
    out[3] = TABLE;
}

hipError_t launch_bp_prepare(const cbct_plan &p, void *geom, hipStream_t s) {
    const Cut c = cut_of(p.g);
    char *base = (char *)geom;
    hipLaunchKernelGGL(k_rays, dim3((p.g.nu + 63) / 64, (p.g.nv + 3) / 4, p.g.n_views), dim3(256),
                       0, s, p.d_views, p.det, p.g.nu, p.g.nv, (PixelRay *)base);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || c.slab < p.g.n_views) return e;
    return launch_brick_views(p, c, 0, p.g.n_views, (BrickView *)(base + ray_bytes(p.g)), s);
}

// What decides is how many pixels the lanes of a brick visit, on average, and
// how many its cells have: a sample of bricks and views, the same for a
// geometry each time.  A visit's cost is the unit; a staged ray, a share of
// the brick's 256 lanes, and a view's own costs are fitted to measurements.
// Near the source a brick's blocks of pixels grow with the distances and
// sizes of its cells; where its footprint exceeds the table, whole parts are
// visited for the few of a wavefront's cells that lie in them.  Measured over
// 170 geometries, the source 1.15 to 10 radii of the grid from the axis: the
// choice is the slower one by more than 7% in two of them (float, 18% at most)
// and in four (double, 33%), and against the kernel before k_cells, which
// tested candidate samples, none loses more than 2% but one, 100 x 100 x 50 in
// double with steps of two voxels (250 -> 282 us).  Transposes by that
// kernel / k_cells / this choice (us; float, double): 40 x 40 x 20 beside the
// source 267 / 422 / 103, 266 / 647 / 118; 160 x 160 x 80 beside it 1776 /
// 14963 / 1031, 2034 / 23747 / 1357; 64^3 at 1.3 radii 401 / 2007 / 226, 483 /
// 3799 / 311, at 3 radii 150 / 92 / 99, 194 / 175 / 138; 64 x 64 x 20 with
// pixels of a fifteenth of a voxel 2199 / 1858 / 1092, 2348 / 2672 / 1388.
void choose_cells(cbct_plan &p) {
    const cbct_geom &g = p.g;
    const Cut c = cut_of(g);
    const int n[4] = {(int)c.bricks.x, (int)c.bricks.y, (int)c.bricks.z, g.n_views};
    const int most[4] = {5, 5, 3, 4};
    int m[4], total = 1;
    for (int a = 0; a < 4; ++a) total *= m[a] = std::min(n[a], most[a]);
    const double column = by_columns(g) ? 0.75 : 1.0;  // a visit by columns
    double visits = 0.0, staged = 0.0, own = 0.0, views = 0.0;
    for (int q = 0; q < total; ++q) {
        int at[4];
        for (int a = 0, e = q; a < 4; e /= m[a++])
            at[a] = (int)((2LL * (e % m[a]) + 1) * n[a] / (2 * m[a]));
        const int c0[3] = {at[0] * c.shape.x - 1, at[1] * c.shape.y - 1, at[2] - 1};
        const int c1[3] = {std::min(c0[0] + c.shape.x, g.nx), std::min(c0[1] + c.shape.y, g.ny),
                           c0[2] + 1};
        const ViewConst &vc = p.h_views[at[3]];
        const BrickView b = brick_view(vc, p.det, g.hx, g.hy, g.hz, g.nu, g.nv, c0, c1);
        if (b.w == 0) continue;
        double rows = std::min(b.H, b.h);
        if ((long long)b.w * b.h > TABLE)  // those of a wavefront's cells, rounded out to parts
            rows = std::min(rows + 7.0 * (fabs(b.bx) + fabs(b.by)) + std::max(TABLE / b.w, 1),
                            (double)b.h);
        visits += std::min(b.W, b.w) * rows;
        staged += (double)b.w * b.h / 256.0;
        // the extents of a cell at the brick's centre
        const double x = 0.5 * (c0[0] + c1[0]), y = 0.5 * (c0[1] + c1[1]);
        const double z = fabs(c0[2] + 0.5 - vc.Qd[2]);
        const double r = 1.0 / (vc.ew[0] * x + vc.ew[1] * y + vc.ew[2]);
        const double u = (vc.en[0] * x + vc.en[1] * y + vc.en[2]) * r;
        const double W =
            (fabs(vc.en[0] - u * vc.ew[0]) + fabs(vc.en[1] - u * vc.ew[1])) * r * g.sdd / g.au;
        const double H =
            (1.0 + z * (fabs(vc.ew[0]) + fabs(vc.ew[1])) * r) * g.hz * r * g.sdd / g.av;
        own += (W + 1.0) * (H + 1.0);
        views += 1.0;
    }
    p.near32 = column * visits + staged > 1.35 * (own + views);
    p.near64 = visits + 3.0 * staged + 4.0 * views > 1.75 * own;
}

template <typename T>
hipError_t launch_backproject_cells(const cbct_plan &p, const T *r, void *cells,
                                    const void *geom, hipStream_t s) {
    const Cut c = cut_of(p.g);
    const dim3 grid(c.bricks.x * c.bricks.y * c.bricks.z, c.chunks);
    const bool near = sizeof(T) == 4 ? p.near32 : p.near64, kept = c.slab == p.g.n_views;
    BrickView *bv = kept ? (BrickView *)((char *)geom + ray_bytes(p.g))
                         : (BrickView *)((char *)cells + sums_bytes(p.g, c, sizeof(T)));
    for (int k = 0; k < p.g.n_views; k += c.slab) {
        const int views = std::min(c.slab, p.g.n_views - k);
        const long long first = (long long)k * p.g.nu * p.g.nv;
        const PixelRay *rays = (const PixelRay *)geom + first;
        if (near) {
            hipLaunchKernelGGL(k_cells_near<T>, grid, dim3(256), 0, s, p.d_views + k, p.det,
                               p.grid, c.shape, p.g.nu, p.g.nv, views, c.chunk, rays, r + first,
                               (T *)cells, (T)p.g.step, k > 0);
        } else {
            if (!kept) {
                const hipError_t e = launch_brick_views(p, c, k, views, bv, s);
                if (e != hipSuccess) return e;
            }
            auto kernel = k_cells<T, false>;
            if constexpr (sizeof(T) == 4) {
                if (by_columns(p.g)) kernel = k_cells<T, true>;
            }
            hipLaunchKernelGGL(kernel, grid, dim3(256), 0, s, p.d_views + k, p.grid, c.shape,
                               p.g.nu, p.g.nv, views, c.chunk, rays, bv, r + first, (T *)cells,
                               (T)p.g.step, k > 0, !by_columns(p.g));
        }
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <typename T>
hipError_t launch_gather_cells(const cbct_plan &p, const void *ws, const T *f, double tau,
                               T *out, hipStream_t s) {
    dim3 grid((p.g.nx + G_BX - 1) / G_BX, (p.g.ny + G_BY - 1) / G_BY, p.g.nz);
    hipLaunchKernelGGL(k_gather<T>, grid, dim3(G_BX, G_BY), 0, s, p.grid,
                       cut_of(p.g).chunks, (const T *)ws, f, (T)tau, out);
    return hipGetLastError();
}

hipError_t launch_eq2(const cbct_plan &p, const float *r, const float *f, double tau,
                      float *out, hipStream_t s) {
    const double scale = p.g.hx * p.g.hy * p.g.hz / (p.g.au * p.g.av);
    auto launch = [&](auto kernel, int zc) {
        dim3 grid((p.g.nx + Q_BX - 1) / Q_BX, (p.g.ny + Q_BY - 1) / Q_BY,
                  (p.g.nz + zc - 1) / zc);
        hipLaunchKernelGGL(kernel, grid, dim3(Q_BX, Q_BY), 0, s, p.d_views, p.det, p.grid,
                           p.g.hx, p.g.hy, p.g.hz, p.g.nu, p.g.nv, p.g.n_views, r, f, scale, tau,
                           out);
    };
    // Voxels a lane: more share a view's arithmetic, fewer leave more
    // wavefronts.  Measured, us with 1 / 2 / 4: 4096 wavefronts of single voxels
    // (64^3) 10 / 16 / 23, 13k (80^3) 27 / 27, 29k (157 x 141 x 67) 91 / 76 /
    // 91, 33k (128^3) 216 / 150 / 161, 66k (256 x 256 x 64) 407 / 309 / 289, 287k (head)
    // 1293 / 891 / 825; with 4 / 6: 66k 270 / 288, 160k 209 / 214, 246k 315 /
    // 306, 287k 757 / 726.
    const long long waves = ((p.g.nx + Q_BX - 1LL) / Q_BX) * ((p.g.ny + Q_BY - 1LL) / Q_BY) * Q_BY *
                            p.g.nz;
    if (waves >= 196608)
        launch(k_eq2<6>, 6);
    else if (waves >= 49152)
        launch(k_eq2<4>, 4);
    else if (waves >= 8192)
        launch(k_eq2<2>, 2);
    else
        launch(k_eq2<1>, 1);
    return hipGetLastError();
}

template hipError_t launch_backproject_cells<float>(const cbct_plan &, const float *, void *,
                                                    const void *, hipStream_t);
template hipError_t launch_backproject_cells<double>(const cbct_plan &, const double *, void *,
                                                     const void *, hipStream_t);
template hipError_t launch_gather_cells<float>(const cbct_plan &, const void *, const float *,
                                               double, float *, hipStream_t);
template hipError_t launch_gather_cells<double>(const cbct_plan &, const void *,
                                                const double *, double, double *, hipStream_t);

}  // namespace cbct
