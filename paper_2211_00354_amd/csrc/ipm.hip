// Inverse polygon mapping (Section 2.3; first order, as used in Section 2.4).
// Adjacent grid rays are the corners of image-plane cells of area dx dy; cell
// (i, j) with corners y(i,j), y(i+1,j), y(i+1,j+1), y(i,j+1) maps to a
// quadrilateral Q in the source plane, and its area is shared exactly among
// the pixels Q overlaps in proportion to the overlap areas: pixel P receives
// dx dy |Q n P| / |Q|; divided by the pixel area that is the magnification
// sum S_i / S_pixel.  A critical cell (its image's edges cross: the cell
// straddles a critical curve) is treated as if it were not critical: the
// region its edges enclose, the two triangles ("lobes") either side of the
// crossing point, takes the cell's area by overlap.  Only an image of zero
// area goes to its corners, a quarter of the cell to each corner's pixel
// (the zeroth-order, inverse-ray-shooting rule).
//
// Geometry in pixel units p = (y - ymin) S, S = npix/side.  Overlaps come
// from Green's theorem as a sum of edge terms (see poly_pixel_overlap), which
// needs no clipped polygon.  Contributions are summed as fixed-point integers
// (units of 2^-40 of a pixel's magnification) with 64-bit atomics, so the map
// does not depend on the order of the additions; a final pass adds them to
// the caller's FP64 map.
//
// Two kernels share the cells of a pass:
//   * k_ipm, a thread per cell: a cell inside one pixel (the common case)
//     adds the whole cell; a cell whose bounding box spans at most
//     kPairMax pixels is apportioned pixel by pixel, its (cell, pixel) pairs
//     shared out evenly over the workgroup; a wider cell (next to a star its
//     image can stretch over much of the map) is queued;
//   * k_ipm_wide, a wave per 16 queued cells: their images (the quadrilateral,
//     or a folded cell's two lobes) are rasterised edge by edge, so the work is
//     proportional to their perimeters in pixels: an edge adds its Green term to
//     the few pixels it crosses in each row and a constant to the row's
//     pixels right of it through a row-difference accumulator that the final
//     pass prefix-sums along the row.
#include "device_common.h"

namespace lensfmm {

namespace {

constexpr int kThreads = 256;
constexpr double kFix = 1099511627776.0;  // 2^40
// widest bounding box (in pixels) apportioned by the per-cell pair path: a pair
// costs four edge terms, a rasterised cell its perimeter.  16384^2 rays at mu
// = 50 into 2000^2 pixels, k_ipm + k_ipm_wide: 64 pixels 10.6 + 5.6 ms, 32
// 9.2 + 6.6, 16 8.3 + 7.2, 4 6.9 + 11.3 (in turn on one card; on another, whose
// statistics are kept, 9.2 + 8.6 with 16).
constexpr int32_t kPairMax = 16;

__device__ __forceinline__ double orient2(double ax, double ay, double bx, double by, double cx,
                                          double cy) {
  return (bx - ax) * (cy - ay) - (by - ay) * (cx - ax);
}

// Strictly opposite signs (a zero is neither).
__device__ __forceinline__ bool opposite(double u, double v) {
  return (u > 0 && v < 0) || (u < 0 && v > 0);
}

__device__ __forceinline__ double clamp01(double x) { return fmin(fmax(x, 0.0), 1.0); }

// Signed contribution of edge a -> b to the area of (polygon n unit square):
// the line integral of clamp01(x) dy over the edge's part with 0 <= y <= 1.
// On that part x(y) = lx + (y - ly) k is linear, so clamp01(x(y)) is linear
// between the heights where x crosses 0 and 1 and the trapezoid rule on those
// pieces is exact.  k = dx/dy and kinv = dy/dx (0 for a vertical edge) depend
// only on the edge's direction, not on the pixel or on where the edge ends.
__device__ __forceinline__ double edge_term(double ax, double ay, double bx, double by, double k,
                                            double kinv) {
  if (ay == by) return 0.0;
  const bool up = by > ay;
  const double lx = up ? ax : bx, ly = up ? ay : by, hy = up ? by : ay;
  const double y0 = fmax(ly, 0.0), y1 = fmin(hy, 1.0);
  if (!(y0 < y1)) return 0.0;
  // breakpoints (heights where x = 0 and x = 1); a vertical edge has kinv =
  // 0, so both fall at ly <= y0 and are ignored, as they should be
  const double ya = fma(-lx, kinv, ly), yb = ya + kinv;
  const double lo = fmin(ya, yb), hi = fmax(ya, yb);
  double s0 = (lo > y0 && lo < y1) ? lo : y1;
  double s1 = (hi > y0 && hi < y1) ? hi : y1;
  if (s0 == y1) s0 = s1, s1 = y1;
  const double x0 = clamp01(fma(y0 - ly, k, lx));
  const double xa = clamp01(fma(s0 - ly, k, lx));
  const double xb = clamp01(fma(s1 - ly, k, lx));
  const double x1 = clamp01(fma(y1 - ly, k, lx));
  const double v = 0.5 * fma(x0 + xa, s0 - y0, fma(xa + xb, s1 - s0, (xb + x1) * (y1 - s1)));
  return up ? v : -v;
}

// Edge a -> b against the unit square at (u, v).
__device__ __forceinline__ double edge_at(const double (&a)[2], const double (&b)[2], double k,
                                          double kinv, double u, double v) {
  return edge_term(a[0] - u, a[1] - v, b[0] - u, b[1] - v, k, kinv);
}

// Slopes k = dx/dy (0 for a horizontal edge) and kinv = dy/dx (0 for a
// vertical one) of the edge a -> b, through the refined hardware reciprocal
// (within an ulp or two of the quotient, a fraction of the cost of an IEEE
// division).
__device__ __forceinline__ void edge_slope(const double (&a)[2], const double (&b)[2], double &k,
                                           double &kinv) {
  const double dx = b[0] - a[0], dy = b[1] - a[1];
  k = dy != 0.0 ? dx * rcp_f64(dy) : 0.0;
  kinv = dx != 0.0 ? dy * rcp_f64(dx) : 0.0;
}

// The image of a cell as the polygons that carry its area.
//   kind 0: the quadrilateral q itself (convex or not; Green's theorem holds
//           for any simple polygon);
//   kind 1: edges 0-1 and 2-3 cross at X: lobes (X, q1, q2) and (q0, X, q3);
//   kind 2: edges 1-2 and 3-0 cross at X: lobes (X, q2, q3) and (q1, X, q0).
// area = |Q| or |T1| + |T2| (pixel units).
struct Cell {
  double q[4][2];
  double X[2];
  int kind;
  double area;
};

__device__ __forceinline__ double tri_area(const double (&a)[2], const double (&b)[2],
                                           const double (&c)[2]) {
  return fabs(0.5 * orient2(a[0], a[1], b[0], b[1], c[0], c[1]));
}

__device__ __forceinline__ void classify(Cell &c) {
  // Twice the signed areas of four corner triangles, on differences of
  // corners (a small image far from the map origin keeps its digits):
  // A = o(q0,q1,q2), B = o(q0,q1,q3), C = o(q2,q3,q0), D = o(q2,q3,q1),
  // o(a,b,c) = (b - a) x (c - a), unchanged by a cyclic shift of a, b, c.
  // Segments 0-1 and 2-3 cross iff A, B and C, D have opposite signs;
  // segments 1-2 and 3-0 iff D, A and B, C do; and A + C is twice the
  // signed area of q (its triangles q0 q1 q2 and q0 q2 q3).
  const double(&q)[4][2] = c.q;
  const double e01x = q[1][0] - q[0][0], e01y = q[1][1] - q[0][1];
  const double e23x = q[3][0] - q[2][0], e23y = q[3][1] - q[2][1];
  const double A = e01x * (q[2][1] - q[0][1]) - e01y * (q[2][0] - q[0][0]);
  const double B = e01x * (q[3][1] - q[0][1]) - e01y * (q[3][0] - q[0][0]);
  const double C = e23x * (q[0][1] - q[2][1]) - e23y * (q[0][0] - q[2][0]);
  const double D = e23x * (q[1][1] - q[2][1]) - e23y * (q[1][0] - q[2][0]);
  const bool c01 = opposite(A, B) && opposite(C, D);
  const bool c12 = !c01 && opposite(D, A) && opposite(B, C);
  if (c01 || c12) {
    const int ia = c01 ? 0 : 1;
    const double(&a)[2] = c.q[ia];
    const double(&b)[2] = c.q[ia + 1];
    const double(&cc)[2] = c.q[ia + 2];
    const double(&d)[2] = c.q[(ia + 3) & 3];
    const double den = (b[0] - a[0]) * (d[1] - cc[1]) - (b[1] - a[1]) * (d[0] - cc[0]);
    const double t = ((cc[0] - a[0]) * (d[1] - cc[1]) - (cc[1] - a[1]) * (d[0] - cc[0])) / den;
    c.X[0] = a[0] + t * (b[0] - a[0]);
    c.X[1] = a[1] + t * (b[1] - a[1]);
    c.kind = c01 ? 1 : 2;
    c.area = tri_area(c.X, b, cc) + tri_area(a, c.X, d);
  } else {
    c.X[0] = c.X[1] = 0.0;
    c.kind = 0;
    c.area = fabs(0.5 * (A + C));
  }
}

// Area of the cell's image inside the unit square at (u, v); k/kinv are the
// slopes of the four edges q[e] -> q[e+1] (sub-edges of a lobe run along
// them in the same direction).
__device__ double cell_pixel_overlap(const double (&q)[4][2], const double (&X)[2], int kind,
                                     const double (&k)[4], const double (&kinv)[4], double u,
                                     double v) {
  if (kind == 0) {
    double s = 0.0;
#pragma unroll
    for (int e = 0; e < 4; ++e) s += edge_at(q[e], q[(e + 1) & 3], k[e], kinv[e], u, v);
    return fabs(s);
  }
  if (kind == 1) {
    const double t1 = edge_at(X, q[1], k[0], kinv[0], u, v) + edge_at(q[1], q[2], k[1], kinv[1], u, v) +
                      edge_at(q[2], X, k[2], kinv[2], u, v);
    const double t2 = edge_at(q[0], X, k[0], kinv[0], u, v) + edge_at(X, q[3], k[2], kinv[2], u, v) +
                      edge_at(q[3], q[0], k[3], kinv[3], u, v);
    return fabs(t1) + fabs(t2);
  }
  const double t1 = edge_at(X, q[2], k[1], kinv[1], u, v) + edge_at(q[2], q[3], k[2], kinv[2], u, v) +
                    edge_at(q[3], X, k[3], kinv[3], u, v);
  const double t2 = edge_at(q[1], X, k[1], kinv[1], u, v) + edge_at(X, q[0], k[3], kinv[3], u, v) +
                    edge_at(q[0], q[1], k[0], kinv[0], u, v);
  return fabs(t1) + fabs(t2);
}

// Area of the part of the simple quadrilateral q with x < xs (across_x) or
// y < ys, for a cell whose image spans two pixels that share that line.  By
// Green's theorem the area of q n {w < 0}, w = x - xs, is |the line integral
// of min(w, 0) dy| around q (with w = y - ys and x in the place of y for the
// other split).  min(w, 0) is linear along an edge except where the edge
// crosses w = 0, at t = wa / (wa - wb) of its length, so the trapezoid rule
// on the one or two pieces is exact.
__device__ __forceinline__ double split_area(const double (&q)[4][2], bool across_x, double xs,
                                             double ys) {
  double s = 0.0;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const double(&a)[2] = q[e];
    const double(&b)[2] = q[(e + 1) & 3];
    const double wa = across_x ? a[0] - xs : a[1] - ys, wb = across_x ? b[0] - xs : b[1] - ys;
    const double dz = across_x ? b[1] - a[1] : b[0] - a[0];
    const double ma = fmin(wa, 0.0), mb = fmin(wb, 0.0);
    double m = ma + mb;
    if ((wa < 0.0) != (wb < 0.0)) {
      const double t = wa * rcp_f64(wa - wb);
      m = ma * t + mb * (1.0 - t);
    }
    s += m * dz;
  }
  return fabs(0.5 * s);
}

// Orientation of a convex q (+1 counter-clockwise, -1 clockwise), or 0 if q
// is not convex.
__device__ __forceinline__ int convex_orientation(const double (&q)[4][2]) {
  int pos = 0, neg = 0;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int e1 = (e + 1) & 3, e2 = (e + 2) & 3;
    const double c = orient2(q[e][0], q[e][1], q[e1][0], q[e1][1], q[e2][0], q[e2][1]);
    pos += c > 0.0;
    neg += c < 0.0;
  }
  return neg == 0 ? 1 : (pos == 0 ? -1 : 0);
}

// True if the pixel [u,u+1] x [v,v+1] lies (by more than a rounding margin)
// outside one of the edge lines of the convex q of orientation o, so that
// their overlap is empty: the largest value over the pixel of the edge's
// signed distance function is its value at the centre plus (|dx| + |dy|)/2.
__device__ __forceinline__ bool convex_misses(const double (&q)[4][2], int o, double u, double v) {
  const double uc = u + 0.5, vc = v + 0.5;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int e1 = (e + 1) & 3;
    const double dx = q[e1][0] - q[e][0], dy = q[e1][1] - q[e][1];
    const double f = (double)o * (dx * (vc - q[e][1]) - dy * (uc - q[e][0]));
    if (f + (0.5 + 1e-9) * (fabs(dx) + fabs(dy)) < 0.0) return true;
  }
  return false;
}

__device__ __forceinline__ int64_t pixel_of(const double (&p)[2], int32_t npix) {
  if (!(p[0] >= 0.0) || !(p[1] >= 0.0)) return -1;
  const double f1 = floor(p[0]), f2 = floor(p[1]);
  if (f1 >= (double)npix || f2 >= (double)npix) return -1;
  return (int64_t)f2 * npix + (int64_t)f1;
}

struct IpmArgs {
  const double *y;      // rows [ybase, ...) of the mapped grid, nx rays per row
  int64_t nx, ybase, j0, j1;  // cells of rows [j0, j1), all nx - 1 columns
  double cell_px, y1min, y2min, S;
  int32_t npix;
  unsigned long long *acc;   // [npix][npix]
  unsigned long long *diff;  // row differences of wide cells, tiled (diff_index)
  int64_t diff_cols;         // its tiles per row of tiles
  uint32_t *queue;           // wide cells: index (j - j0) (nx - 1) + i
  uint32_t *qcount;
};

// Corners of cell (i, j) (pixel units); false if any is not finite.
__device__ __forceinline__ bool load_quad(const IpmArgs &a, int64_t i, int64_t j,
                                          double (&q)[4][2]) {
  const int64_t r0 = (j - a.ybase) * a.nx + i, r1 = r0 + a.nx;
  const int64_t id[4] = {r0, r0 + 1, r1 + 1, r1};
  double z = 0.0;  // stays 0 unless a value is infinite or NaN
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    q[k][0] = (a.y[2 * id[k]] - a.y1min) * a.S;
    q[k][1] = (a.y[2 * id[k] + 1] - a.y2min) * a.S;
    z = fma(q[k][0], 0.0, z);
    z = fma(q[k][1], 0.0, z);
  }
  return z == 0.0;
}

// Pixel bounding box of q clamped to the map; false if it misses the map
// (the box is then of no use).  The corners are clamped to the map before
// the conversion, so it is a 32-bit one.
__device__ __forceinline__ bool quad_bbox(const double (&q)[4][2], int32_t npix, int32_t &u0,
                                          int32_t &v0, int32_t &u1, int32_t &v1, bool &inside) {
  double lo0 = q[0][0], hi0 = q[0][0], lo1 = q[0][1], hi1 = q[0][1];
#pragma unroll
  for (int k = 1; k < 4; ++k) {
    lo0 = fmin(lo0, q[k][0]);
    hi0 = fmax(hi0, q[k][0]);
    lo1 = fmin(lo1, q[k][1]);
    hi1 = fmax(hi1, q[k][1]);
  }
  const double top = (double)npix, last = top - 1.0;
  u0 = (int32_t)floor(fmin(fmax(lo0, 0.0), last));
  v0 = (int32_t)floor(fmin(fmax(lo1, 0.0), last));
  u1 = (int32_t)floor(fmin(fmax(hi0, 0.0), last));
  v1 = (int32_t)floor(fmin(fmax(hi1, 0.0), last));
  inside = lo0 >= 0.0 && lo1 >= 0.0 && hi0 < top && hi1 < top;
  return !(hi0 < 0.0 || hi1 < 0.0 || lo0 >= top || lo1 >= top);
}

__device__ __forceinline__ unsigned long long to_fix(double x) {
  return (unsigned long long)llrint(x * kFix);
}

// Workgroup-local sums of pixel contributions: an LDS hash table of 64-byte
// segments of the map (8 pixels), flushed to the map once per workgroup, so
// the many cells of a patch that land in the same pixels (all of them, away
// from stars; those around a star's caustic, near one) cost few global
// atomics.  The chip takes 23.7e9 atomic requests a second whatever their
// addresses or scope, but a request carries every lane of an instruction that
// falls in one 64-byte segment (188e9 lane operations a second with 8 lanes
// to a segment): a segment's pixels lie side by side in the table, so the
// flush sends one request for all of them.  Two probes, then the global map:
// patches near a star touch more pixels than the table holds, and long probe
// chains there (a wave waits for its slowest lane) cost more than the atomics
// they save.
constexpr int kSegBits = 7, kSegs = 1 << kSegBits;
constexpr int kTable = 8 * kSegs;
constexpr int kPatch = 32;  // a workgroup takes kPatch x kPatch cells

__device__ __forceinline__ void table_add(int32_t *tseg, unsigned long long *tval,
                                          unsigned long long *__restrict__ acc, int32_t key,
                                          unsigned long long v) {
  const int32_t seg = key >> 3;
  const uint32_t h = ((uint32_t)seg * 2654435761u) >> (32 - kSegBits);
  for (int probe = 0; probe < 2; ++probe) {
    const int slot = (int)((h + (uint32_t)probe) & (kSegs - 1));
    int32_t k = tseg[slot];
    if (k == -1) {
      const int32_t old = atomicCAS(&tseg[slot], -1, seg);
      k = old == -1 ? seg : old;
    }
    if (k == seg) {
      atomicAdd(&tval[8 * slot + (key & 7)], v);
      return;
    }
  }
  atomicAdd(&acc[key], v);  // crowded table
}

__device__ __forceinline__ int32_t block_excl_scan(int32_t x, int32_t *wsum, int32_t *total) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  int32_t inc = x;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int32_t v = __shfl_up(inc, d);
    if (lane >= d) inc += v;
  }
  if (lane == 63) wsum[w] = inc;
  __syncthreads();
  int32_t off = 0, tot = 0;
#pragma unroll
  for (int q = 0; q < kThreads / 64; ++q) {
    if (q < w) off += wsum[q];
    tot += wsum[q];
  }
  *total = tot;
  return off + inc - x;
}

// One workgroup per kPatch x kPatch patch of cells, taken 256 cells at a
// time, one thread per cell.  The (cell, pixel) pairs of the batch's
// multi-pixel cells are numbered by a scan and shared out evenly over the
// workgroup's threads, so a few cells near a star do not hold a whole wave.
// Four waves per SIMD (at most 128 VGPRs), as many as its LDS allows.
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(4))) void k_ipm(
    IpmArgs a) {
  __shared__ int32_t tseg[kSegs];
  __shared__ unsigned long long tval[kTable];
  __shared__ double sq[kThreads][10];       // multi-pixel cells of the batch: corners, X,
  __shared__ double sinv[kThreads];         // 1 / area,
  __shared__ int32_t sshape[kThreads];      // kind | (convex orientation + 1) << 2,
  __shared__ int32_t sbox[kThreads][3];     // u0, v0, columns of the bounding box
  __shared__ int32_t sfirst[kThreads + 1];  // first pair index of each cell
  __shared__ int32_t wsum[kThreads / 64];
  const int t = threadIdx.x;
  for (int e = t; e < kTable; e += kThreads) {
    if ((e & 7) == 0) tseg[e >> 3] = -1;
    tval[e] = 0ull;
  }
  __syncthreads();
  const int64_t ncx = a.nx - 1;
  const int64_t npx_x = (ncx + kPatch - 1) / kPatch;
  const int64_t pi = blockIdx.x % npx_x, pj = blockIdx.x / npx_x;
  const int32_t npix = a.npix;
  const unsigned long long q_cell = to_fix(a.cell_px);
  const unsigned long long q_quarter = to_fix(0.25 * a.cell_px);
  for (int base = 0; base < kPatch * kPatch; base += kThreads) {
    const int k = base + t;
    const int64_t i = pi * kPatch + (k % kPatch), j = a.j0 + pj * kPatch + (k / kPatch);
    int32_t npairs = 0;
    Cell c;
    int32_t u0, v0, u1, v1;
    bool inside;
    // up to two pixels take their shares at once (a cell in one pixel, or
    // across one pixel edge)
    unsigned long long s0 = 0ull, s1 = 0ull;
    if (i < ncx && j < a.j1 && load_quad(a, i, j, c.q) &&
        quad_bbox(c.q, npix, u0, v0, u1, v1, inside)) {
      classify(c);
      const int64_t npx = (int64_t)(u1 - u0 + 1) * (v1 - v0 + 1);
      if (!(c.area > 0.0)) {
        // no shape: a quarter of the cell to each corner's pixel
#pragma unroll
        for (int cc = 0; cc < 4; ++cc) {
          const int64_t pk = pixel_of(c.q[cc], npix);
          if (pk >= 0) table_add(tseg, tval, a.acc, (int32_t)pk, q_quarter);
        }
      } else if (npx == 1 && inside) {
        s0 = q_cell;  // wholly inside
      } else if (npx == 2 && inside && c.kind == 0) {
        // across one pixel edge: the first pixel's overlap by Green's
        // theorem, the second takes the rest of the cell (in fixed point,
        // so the cell's total is exact)
        const double ov = split_area(c.q, u1 != u0, (double)(u0 + 1), (double)(v0 + 1));
        const double f = fmin(fmax(ov / c.area, 0.0), 1.0);
        s0 = to_fix(a.cell_px * f);
        s1 = q_cell >= s0 ? q_cell - s0 : 0ull;
      } else if (npx > kPairMax) {
        const uint32_t slot = atomicAdd(a.qcount, 1u);
        a.queue[slot] = (uint32_t)((j - a.j0) * ncx + i);
      } else {
        npairs = (int32_t)npx;
#pragma unroll
        for (int cc = 0; cc < 4; ++cc) {
          sq[t][2 * cc] = c.q[cc][0];
          sq[t][2 * cc + 1] = c.q[cc][1];
        }
        sq[t][8] = c.X[0];
        sq[t][9] = c.X[1];
        sinv[t] = 1.0 / c.area;
        sshape[t] = c.kind | ((c.kind == 0 ? convex_orientation(c.q) + 1 : 1) << 2);
        sbox[t][0] = u0;
        sbox[t][1] = v0;
        sbox[t][2] = u1 - u0 + 1;
      }
    }
    if (s0) table_add(tseg, tval, a.acc, v0 * npix + u0, s0);
    if (s1) table_add(tseg, tval, a.acc, v1 * npix + u1, s1);
    int32_t total;
    const int32_t first = block_excl_scan(npairs, wsum, &total);
    sfirst[t] = first;
    if (t == kThreads - 1) sfirst[kThreads] = first + npairs;
    __syncthreads();
    // each thread takes a contiguous range of the batch's pairs, so its
    // owner cell changes rarely: found once by search, then walked forward,
    // with the cell's corners and edge slopes kept in registers meanwhile
    const int32_t chunk = (total + kThreads - 1) / kThreads;
    int32_t w = t * chunk;
    const int32_t wend = min(total, w + chunk);
    if (w < wend) {
      int lo = 0, hi = kThreads - 1;
      while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (sfirst[mid] <= w) lo = mid; else hi = mid - 1;
      }
      int cur = -1;
      double cq[4][2], X[2], k[4], kinv[4], inv = 0.0;
      int kind = 0, o = 0;
      int32_t bu = 0, bv = 0, bw = 1;
      for (; w < wend; ++w) {
        // sfirst[lo] <= w < sfirst[lo + 1] (cells without pairs are skipped)
        while (w >= sfirst[lo + 1]) ++lo;
        if (lo != cur) {
          cur = lo;
#pragma unroll
          for (int cc = 0; cc < 4; ++cc) {
            cq[cc][0] = sq[lo][2 * cc];
            cq[cc][1] = sq[lo][2 * cc + 1];
          }
          X[0] = sq[lo][8];
          X[1] = sq[lo][9];
#pragma unroll
          for (int e = 0; e < 4; ++e) edge_slope(cq[e], cq[(e + 1) & 3], k[e], kinv[e]);
          inv = sinv[lo];
          kind = sshape[lo] & 3;
          o = (sshape[lo] >> 2) - 1;
          bu = sbox[lo][0];
          bv = sbox[lo][1];
          bw = sbox[lo][2];
        }
        const int32_t local = w - sfirst[lo];
        const int32_t u = bu + local % bw, v = bv + local / bw;
        if (kind == 0 && o != 0 && convex_misses(cq, o, (double)u, (double)v)) continue;
        const double ov = cell_pixel_overlap(cq, X, kind, k, kinv, (double)u, (double)v);
        if (ov > 0.0) table_add(tseg, tval, a.acc, v * npix + u, to_fix(a.cell_px * (ov * inv)));
      }
    }
    __syncthreads();  // the batch's shared cells are consumed
  }
  for (int e = t; e < kTable; e += kThreads) {
    const unsigned long long v = tval[e];
    if (v != 0ull) atomicAdd(&a.acc[(int64_t)tseg[e >> 3] * 8 + (e & 7)], v);
  }
}

// Wide cells are apportioned edge by edge.  By Green's theorem the overlap
// of a polygon with pixel (u, v) is the sum over its edges of
// T_e(u) = +-int clamp01(x(y) - u) dy over the edge's part in the strip
// [v, v+1] (edge_term), signed by the polygon's orientation.  Along a map row
// T_e(u) is the constant C_e = +-(height of that part) for every pixel left
// of the edge, 0 for every pixel right of it, and needs the integral only
// for the pixels the edge passes through.  Since the C_e of a closed polygon
// sum to zero in every strip,
//     sum_e T_e(u) = sum_e ( -C_e [u >= ulo_e] + P_e(u) [ulo_e <= u <= uhi_e] ),
// with [ulo_e, uhi_e] the pixels the edge crosses in that row and P_e = T_e
// there: each (edge, row) adds -C_e + P_e(ulo) at ulo_e, P_e(u) - P_e(u-1) at
// the next pixels and -P_e(uhi) after the last to the row-difference
// accumulator, which the final pass prefix-sums along the row.  C_e is formed
// in fixed point as G(y_end) - G(y_start) with G(y) = fix((y - v) w), so the
// constants of a closed polygon cancel exactly in integers and pixels outside
// it receive exactly nothing.  Work is proportional to the image's perimeter
// in pixels, not its area.
//
// The edge between two wide cells, neither of them folded, belongs to both:
// it is rasterised once with both weights (each in its own fixed point), by
// the cell left of it or below it.

// An edge's part in the strip [v, v+1]: heights yb < yt, the x extent
// [xl, xh] there and (signed) start/end heights in the edge's direction.
__device__ __forceinline__ bool edge_strip(double ax, double ay, double bx, double by, double k,
                                           double v, double &xl, double &xh, double &ys,
                                           double &ye) {
  const double ey0 = fmin(ay, by), ey1 = fmax(ay, by);
  const double yb = fmax(ey0, v), yt = fmin(ey1, v + 1.0);
  if (!(yb < yt)) return false;
  const double xb = yb == ay ? ax : (yb == by ? bx : ax + (yb - ay) * k);
  const double xt = yt == ay ? ax : (yt == by ? bx : ax + (yt - ay) * k);
  xl = fmin(xb, xt);
  xh = fmax(xb, xt);
  const bool up = by > ay;
  ys = up ? yb : yt;
  ye = up ? yt : yb;
  return true;
}

// One polygon edge a -> b: signed weight w0 of the cell it was taken from, w1
// of the cell on its other side (0: none), whose polygon runs along it the
// other way.
struct EdgeJob {
  double ax, ay, bx, by, k, kinv, w0, w1;
  int32_t r0, c0;
};
constexpr int kBatch = 16;              // cells per wave and batch
constexpr int kMaxJobs = 6 * kBatch;    // two triangles per folded cell

// Both cells' fixed-point shares of a signed term t of the edge.
__device__ __forceinline__ unsigned long long edge_fix(const EdgeJob &e, double t) {
  return to_fix(t * e.w0) - to_fix(t * e.w1);
}
// ... and of the edge's height in row v, from ys to ye.
__device__ __forceinline__ unsigned long long edge_const(const EdgeJob &e, double ys, double ye,
                                                         double v) {
  return edge_fix(e, ye - v) - edge_fix(e, ys - v);
}

// The row differences lie in 64-byte tiles of 4 rows by 2 columns: one atomic
// request carries every lane of an instruction in one tile, in whatever lanes
// they are, and a steep edge's rows lie above each other (a request per ~2
// rows, where rows of 8 columns take one or two per row).
__device__ __forceinline__ int64_t diff_index(int32_t v, int32_t u, int64_t cols) {
  return (((int64_t)(v >> 2) * cols + (u >> 1)) << 3) + ((v & 3) << 1) + (u & 1);
}

// Row v of a steep edge (at least as many rows as columns in the map), by
// four neighbouring lanes (sub = 0..3), an entry of the difference row each.
__device__ __forceinline__ void row_item(const EdgeJob &e, int32_t v, int sub, const IpmArgs &a) {
  const int32_t npix = a.npix;
  double xl = 0, xh = 0, ys = 0, ye = 0;
  if (!edge_strip(e.ax, e.ay, e.bx, e.by, e.k, (double)v, xl, xh, ys, ye)) return;
  const double ulo = floor(xl);
  if (!(ulo < (double)npix)) return;
  const int32_t ua = ulo < 0.0 ? 0 : (int32_t)ulo;
  const double uhi = fmin(ceil(xh) - 1.0, (double)(npix - 1));
  const int32_t ub = uhi < (double)ua ? ua - 1 : (int32_t)uhi;
  unsigned long long carry = 0ull;
  for (int32_t u0 = ua; u0 <= ub + 1; u0 += 4) {  // the same for the four lanes
    const int32_t u = u0 + sub;
    unsigned long long P = 0ull;
    if (u <= ub) P = edge_fix(e, edge_term(e.ax - u, e.ay - v, e.bx - u, e.by - v, e.k, e.kinv));
    const unsigned long long left = __shfl_up(P, 1, 4);
    unsigned long long d = P - (sub == 0 ? carry : left);
    carry = __shfl(P, 3, 4);
    if (u == ua) d -= edge_const(e, ys, ye, (double)v);
    if (u <= ub + 1 && d != 0ull) atomicAdd(&a.diff[diff_index(v, u, a.diff_cols)], d);
  }
}

// Row v of a flat edge: its constant only (its pixels are column_item's).
__device__ __forceinline__ void flat_row_item(const EdgeJob &e, int32_t v, const IpmArgs &a) {
  double xl, xh, ys, ye;
  if (!edge_strip(e.ax, e.ay, e.bx, e.by, e.k, (double)v, xl, xh, ys, ye)) return;
  const double ulo = floor(xl);
  if (!(ulo < (double)a.npix)) return;
  const unsigned long long c = edge_const(e, ys, ye, (double)v);
  const int32_t d = ulo < 0.0 ? 0 : (int32_t)ulo;
  if (c != 0ull) atomicAdd(&a.diff[diff_index(v, d, a.diff_cols)], 0ull - c);
}

// Column u of a flat edge (rows [r0, r0 + nr) of the map): the pixels it
// crosses there.
__device__ __forceinline__ void column_item(const EdgeJob &e, int32_t nr, int32_t u, const IpmArgs &a) {
  const int32_t npix = a.npix;
  const double ex0 = fmin(e.ax, e.bx), ex1 = fmax(e.ax, e.bx);
  const double x0 = fmax(ex0, (double)u), x1 = fmin(ex1, (double)u + 1.0);
  if (!(x0 <= x1)) return;
  const double y0 = x0 == e.ax ? e.ay : (x0 == e.bx ? e.by : e.ay + (x0 - e.ax) * e.kinv);
  const double y1 = x1 == e.ax ? e.ay : (x1 == e.bx ? e.by : e.ay + (x1 - e.ax) * e.kinv);
  // rows this column's part may touch, one row of margin either way; a row
  // takes the pixel only if its own strip test puts u among the crossed ones
  const double vlo = fmax(floor(fmin(y0, y1)) - 1.0, (double)e.r0);
  const double vhi = fmin(ceil(fmax(y0, y1)), (double)(e.r0 + nr - 1));
  for (int32_t v = (int32_t)vlo; (double)v <= vhi; ++v) {
    double xl, xh, ys, ye;
    if (!edge_strip(e.ax, e.ay, e.bx, e.by, e.k, (double)v, xl, xh, ys, ye)) continue;
    if ((double)u < floor(xl) || (double)u > ceil(xh) - 1.0) continue;
    const unsigned long long P = edge_fix(e, edge_term(e.ax - u, e.ay - v, e.bx - u, e.by - v, e.k, e.kinv));
    if (P != 0ull) atomicAdd(&a.acc[(int64_t)v * npix + u], P);
  }
}

// Twice the signed area of polygon P (n vertices): its edge terms carry the
// orientation, so the weight does.
template <int N>
__device__ __forceinline__ double signed_weight(const double (&P)[N][2], double w) {
  double s = 0.0;
#pragma unroll
  for (int e = 0; e < N; ++e) {
    const int e1 = e + 1 == N ? 0 : e + 1;
    s += (P[e][0] - P[0][0]) * (P[e1][1] - P[0][1]) - (P[e1][0] - P[0][0]) * (P[e][1] - P[0][1]);
  }
  return s < 0.0 ? -w : w;
}

// The weight of an unfolded wide cell (as k_ipm queues them) of the pass, or
// 0 for any other.
__device__ __forceinline__ double wide_weight(const IpmArgs &a, int64_t i, int64_t j) {
  if (i < 0 || i >= a.nx - 1 || j < a.j0 || j >= a.j1) return 0.0;
  Cell c;
  if (!load_quad(a, i, j, c.q)) return 0.0;
  classify(c);
  if (c.kind != 0 || !(c.area > 0.0)) return 0.0;
  int32_t u0, v0, u1, v1;
  bool inside;
  if (!quad_bbox(c.q, a.npix, u0, v0, u1, v1, inside)) return 0.0;
  if ((int64_t)(u1 - u0 + 1) * (v1 - v0 + 1) <= kPairMax) return 0.0;
  return signed_weight(c.q, a.cell_px / c.area);
}

__device__ __forceinline__ int32_t wave_excl_scan(int32_t x, int lane, int32_t &total) {
  int32_t inc = x;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int32_t y = __shfl_up(inc, d);
    if (lane >= d) inc += y;
  }
  total = __shfl(inc, 63);
  return inc - x;
}

// (The high-magnification map above: 5.6 ms for the cells beyond 64 pixels,
// 18.1 with a wave per cell, an atomic per pixel and difference, and every
// edge twice: it ran at the chip's 23.7e9 atomic requests a second.)
//
// Up to sixteen queued cells per wave and batch: four lanes of each classify it,
// one edge to a lane (with the neighbour across it), and write the edges to be
// rasterised -- the quadrilateral's, or a folded cell's two lobes' -- to a
// table in LDS; the wave's lanes then take the table's items in turn: the rows
// of steep edges, four lanes each, the columns of flat ones, and their rows.
// Waves pull batches in a fixed stride and exit past the queue's end.  A cell can
// be a thousand pixels wide, so a queue of few batches is shared out: up to sixteen
// waves form the same table and take a share of its items each (256^2 rays into
// 4000^2 pixels, 50 stars: 1300 us a call with a wave per batch, 380 so; a wave per
// cell and every edge twice 525).
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(4))) void k_ipm_wide(
    IpmArgs a) {
  __shared__ EdgeJob jobs_all[kThreads / 64][kMaxJobs];
  // first item of each job, by kind: steep rows, flat columns, flat rows
  __shared__ int32_t first_all[kThreads / 64][3][kMaxJobs + 1];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  EdgeJob *jobs = jobs_all[wv];
  int32_t(*first)[kMaxJobs + 1] = first_all[wv];
  const uint32_t nq = *a.qcount;
  const int64_t ncx = a.nx - 1;
  const uint32_t waves = gridDim.x * (kThreads / 64);
  const int e = lane & 3, sub = lane & 3;
  // a short queue: several waves to a batch, an equal share of its items each
  const uint32_t parts = min(16u, max(1u, waves / max(1u, (nq + kBatch - 1) / kBatch))), teams = waves / parts;
  const uint32_t batch = min((uint32_t)kBatch, (nq + teams - 1) / teams);
  const uint32_t wave = blockIdx.x * (kThreads / 64) + wv, team = wave / parts;
  const int32_t part = (int32_t)(wave % parts);
  const uint64_t step = (uint64_t)teams * batch;
  uint64_t base = team < teams ? (uint64_t)team * batch : nq;
  for (; base < nq; base += step) {
    const bool on = (uint32_t)(lane >> 2) < batch && base + (lane >> 2) < nq;
    const uint32_t id = a.queue[on ? base + (lane >> 2) : base];
    const int64_t i = (int64_t)(id % (uint64_t)ncx), j = a.j0 + (int64_t)(id / (uint64_t)ncx);
    Cell c;
    load_quad(a, i, j, c.q);  // finite: it was queued
    classify(c);
    const double w = a.cell_px / c.area;
    // up to two edges of this lane: A (edge e of the quadrilateral, or of the
    // first lobe), B (edge e of the second lobe)
    double A[4], B[4], wa = 0.0, wa1 = 0.0, wb = 0.0;
    auto pick = [](int k, const double (&p0)[2], const double (&p1)[2], const double (&p2)[2],
                   const double (&p3)[2], double &x, double &y) {
      x = k == 0 ? p0[0] : (k == 1 ? p1[0] : (k == 2 ? p2[0] : p3[0]));
      y = k == 0 ? p0[1] : (k == 1 ? p1[1] : (k == 2 ? p2[1] : p3[1]));
    };
    B[0] = B[1] = B[2] = B[3] = 0.0;
    bool has_a = on, has_b = false;
    if (c.kind == 0) {
      pick(e, c.q[0], c.q[1], c.q[2], c.q[3], A[0], A[1]);
      pick((e + 1) & 3, c.q[0], c.q[1], c.q[2], c.q[3], A[2], A[3]);
      wa = signed_weight(c.q, w);
      // the cell across: below, right, above, left
      wa1 = wide_weight(a, i + (e == 1) - (e == 3), j + (e == 2) - (e == 0));
      if (wa1 != 0.0 && (e == 0 || e == 3)) has_a = false;  // the neighbour's
    } else {
      const bool k1 = c.kind == 1;
      double T[3][2], U[3][2];
#pragma unroll
      for (int x = 0; x < 2; ++x) {
        T[0][x] = c.X[x], T[1][x] = k1 ? c.q[1][x] : c.q[2][x], T[2][x] = k1 ? c.q[2][x] : c.q[3][x];
        U[0][x] = k1 ? c.q[0][x] : c.q[1][x], U[1][x] = c.X[x], U[2][x] = k1 ? c.q[3][x] : c.q[0][x];
      }
      const int e1 = e == 2 ? 0 : e + 1;
      pick(e, T[0], T[1], T[2], T[2], A[0], A[1]);
      pick(e1, T[0], T[1], T[2], T[2], A[2], A[3]);
      pick(e, U[0], U[1], U[2], U[2], B[0], B[1]);
      pick(e1, U[0], U[1], U[2], U[2], B[2], B[3]);
      wa = signed_weight(T, w);
      wb = signed_weight(U, w);
      has_a = has_b = on && e < 3;
    }
    wave_sync();  // the previous batch's items have read the table
    int njobs = 0;
    int32_t totals[3] = {0, 0, 0};
    auto emit = [&](bool has, const double (&E)[4], double w0, double w1) {
      const double ax = E[0], ay = E[1], bx = E[2], by = E[3], top = (double)a.npix;
      const double ey0 = fmin(ay, by), ey1 = fmax(ay, by), ex0 = fmin(ax, bx), ex1 = fmax(ax, bx);
      // horizontal edges have no term; an edge wholly left of the map
      // (ex1 < 0) still shifts its rows
      has = has && ay != by && ey1 >= 0.0 && ey0 < top && ex0 < top;
      const int32_t r0 = (int32_t)fmin(fmax(floor(ey0), 0.0), top - 1.0);
      const int32_t r1 = (int32_t)fmax(fmin(floor(ey1), top - 1.0), 0.0);
      const int32_t c0 = (int32_t)fmin(fmax(floor(ex0), 0.0), top - 1.0);
      const int32_t c1 = (int32_t)fmax(fmin(floor(ex1), top - 1.0), -1.0);
      const int32_t nr = r1 - r0 + 1, nc = c1 >= c0 ? c1 - c0 + 1 : 0;
      const bool steep = nr >= nc;
      const uint64_t m = __ballot(has);
      const int slot = njobs + __popcll(m & ((1ull << lane) - 1));
      const int32_t n[3] = {has && steep ? nr : 0, has && !steep ? nc : 0, has && !steep ? nr : 0};
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        int32_t tot;
        const int32_t f = totals[q] + wave_excl_scan(n[q], lane, tot);
        if (has) first[q][slot] = f;
        totals[q] += tot;
      }
      if (has) {
        EdgeJob &jb = jobs[slot];
        jb.ax = ax, jb.ay = ay, jb.bx = bx, jb.by = by, jb.w0 = w0, jb.w1 = w1;
        const double pa[2] = {ax, ay}, pb[2] = {bx, by};
        edge_slope(pa, pb, jb.k, jb.kinv);
        jb.r0 = r0;
        jb.c0 = c0;
      }
      njobs += __popcll(m);
    };
    emit(has_a, A, wa, wa1);
    if (__any(has_b)) emit(has_b, B, wb, 0.0);
    if (lane < 3) first[lane][njobs] = lane == 0 ? totals[0] : (lane == 1 ? totals[1] : totals[2]);
    wave_sync();
    // a lane's items grow, so its job is found by walking on
    int jb = 0;
    for (int32_t t = (lane >> 2) + 16 * part; t < totals[0]; t += 16 * (int32_t)parts) {
      while (first[0][jb + 1] <= t) ++jb;
      row_item(jobs[jb], jobs[jb].r0 + (t - first[0][jb]), sub, a);
    }
    jb = 0;
    for (int32_t t = lane + 64 * part; t < totals[1]; t += 64 * (int32_t)parts) {
      while (first[1][jb + 1] <= t) ++jb;
      column_item(jobs[jb], first[2][jb + 1] - first[2][jb], jobs[jb].c0 + (t - first[1][jb]), a);
    }
    jb = 0;
    for (int32_t t = lane + 64 * part; t < totals[2]; t += 64 * (int32_t)parts) {
      while (first[2][jb + 1] <= t) ++jb;
      flat_row_item(jobs[jb], jobs[jb].r0 + (t - first[2][jb]), a);
    }
  }
}

// mu[v][u] += (acc[v][u] + sum_{u' <= u} diff[v][u']) 2^-40: a wave per map
// row, four to a workgroup (a row of tiles), the row's differences
// prefix-summed 256 at a time, four to a lane (integers, so the result does
// not depend on the order).
__global__ __launch_bounds__(kThreads) void k_ipm_finish(const unsigned long long *__restrict__ acc,
                                                         const unsigned long long *__restrict__ diff,
                                                         int64_t cols, int32_t npix,
                                                         double *__restrict__ mu) {
  const int32_t v = (int32_t)blockIdx.x * 4 + (int32_t)(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (v >= npix) return;
  unsigned long long carry = 0;
  for (int64_t base = 0; base < npix; base += 256) {
    const int64_t u0 = base + 4 * lane;
    unsigned long long x[4], sum = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      sum += u0 + q < npix ? diff[diff_index(v, (int32_t)(u0 + q), cols)] : 0ull;
      x[q] = sum;
    }
    unsigned long long inc = sum;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const unsigned long long y = __shfl_up(inc, d);
      if (lane >= d) inc += y;
    }
    const unsigned long long off = carry + inc - sum;
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (u0 + q < npix) {
        const int64_t idx = (int64_t)v * npix + u0 + q;
        mu[idx] += (double)(long long)(acc[idx] + off + x[q]) * (1.0 / kFix);
      }
    carry += __shfl(inc, 63);
  }
}

__global__ __launch_bounds__(kThreads) void k_zero_u64(unsigned long long *__restrict__ p, int64_t n) {
  for (int64_t k = (int64_t)blockIdx.x * kThreads + threadIdx.x; k < n;
       k += (int64_t)gridDim.x * kThreads)
    p[k] = 0ull;
}

unsigned grid_for(int64_t n) {
  const int64_t b = (n + kThreads - 1) / kThreads;
  return (unsigned)(b < 1 ? 1 : (b > 65536 ? 65536 : b));
}

// columns of 4 x 2 tiles of the difference rows (npix + 1 entries each)
int64_t diff_tile_cols(int32_t npix) { return ((int64_t)npix + 2) / 2; }

// workgroups of the wide-cell kernel
constexpr unsigned kWideBlocks = 1024;  // four waves per SIMD (its register limit)

}  // namespace

int64_t ipm_diff_len(int32_t npix) { return ((int64_t)npix + 3) / 4 * diff_tile_cols(npix) * 8; }

void launch_ipm_zero(unsigned long long *acc, int64_t n, hipStream_t stream) {
  hipLaunchKernelGGL(k_zero_u64, dim3(grid_for(n)), dim3(kThreads), 0, stream, acc, n);
  LENS_HIP(hipGetLastError());
}

void launch_ipm_cells(const IpmPass &p, hipStream_t stream) {
  const int64_t ncx = p.nx - 1, nrows = p.j1 - p.j0;
  if (ncx <= 0 || nrows <= 0) return;
  const int64_t patches = ((ncx + kPatch - 1) / kPatch) * ((nrows + kPatch - 1) / kPatch);
  if (patches > 0x7fffffff) fail(LENS_EUNSUPPORTED, "IPM pass too large");
  if (ncx * nrows > (int64_t)0xffffffffu) fail(LENS_EUNSUPPORTED, "IPM pass too large");
  IpmArgs a{p.y, p.nx, p.ybase, p.j0, p.j1, p.cell_px, p.y1min, p.y2min, p.S, p.npix,
            p.acc, p.diff, diff_tile_cols(p.npix), p.queue, p.qcount};
  launch_fill_u32(p.qcount, 1, 0u, stream);
  hipLaunchKernelGGL(k_ipm, dim3((unsigned)patches), dim3(kThreads), 0, stream, a);
  LENS_HIP(hipGetLastError());
  hipLaunchKernelGGL(k_ipm_wide, dim3(kWideBlocks), dim3(kThreads), 0, stream, a);
  LENS_HIP(hipGetLastError());
}

void launch_ipm_finish(const unsigned long long *acc, const unsigned long long *diff, int32_t npix,
                       double *mu, hipStream_t stream) {
  hipLaunchKernelGGL(k_ipm_finish, dim3((unsigned)((npix + 3) / 4)), dim3(kThreads), 0, stream, acc,
                     diff, diff_tile_cols(npix), npix, mu);
  LENS_HIP(hipGetLastError());
}

}  // namespace lensfmm
