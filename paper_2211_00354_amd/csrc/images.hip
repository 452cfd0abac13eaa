// Inverse lens equation, critical curves and multi-plane chaining, built on
// the deflection of a ray grid (Section 2.5 finds the images of a source
// behind a particle halo; Appendix A notes that the expansions give the
// derivatives of the field in closed form; the introduction's footnote
// extends the thin lens to a chain of planes).
//
// Images.  The grid rays are the corners of cells, each split along its
// (i, j)-(i+1, j+1) diagonal into two triangles.  A triangle whose mapped
// corners contain a source (inclusive barycentric test, so a source on a
// shared edge is seen by both sides) seeds a candidate at the preimage of the
// source under the triangle's linear map.  Candidates are then refined by
// Newton steps on y(x) = beta with the Jacobian
//     A = [[c1 - Re f', Im f'], [Im f', c2 + Re f']],   f' = -sum m/(z - z_i)^2,
// (alpha = conj f, f holomorphic), steps clamped in length and to the ray
// region.
//
// Critical curves.  det A at every grid ray, then marching squares on the
// cells: a cell edge whose end values differ in sign is cut where the linear
// interpolant vanishes; a cell cut on four edges is split by the sign of the
// mean of its corners.
#include "device_common.h"

namespace lensfmm {

namespace {

constexpr int kThreads = 256;

__device__ __forceinline__ double cross2(double ax, double ay, double bx, double by) {
  return ax * by - ay * bx;
}

__global__ __launch_bounds__(kThreads) void k_image_cells(ImageCellArgs a) {
  const int64_t ncx = a.nx - 1;
  const int64_t ncell = ncx * (a.j1 - a.j0);
  const int64_t k = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (k >= ncell) return;
  const int64_t i = k % ncx, j = a.j0 + k / ncx;
  const int64_t r0 = (j - a.ybase) * a.nx + i, r1 = r0 + a.nx;
  const int64_t id[4] = {r0, r0 + 1, r1 + 1, r1};
  // image-plane corners (grid rays) and their images
  const double X[4] = {grid_coord(a.grid.x0, a.grid.dx, i), grid_coord(a.grid.x0, a.grid.dx, i + 1),
                       grid_coord(a.grid.x0, a.grid.dx, i + 1), grid_coord(a.grid.x0, a.grid.dx, i)};
  const double Y[4] = {grid_coord(a.grid.y0, a.grid.dy, j), grid_coord(a.grid.y0, a.grid.dy, j),
                       grid_coord(a.grid.y0, a.grid.dy, j + 1), grid_coord(a.grid.y0, a.grid.dy, j + 1)};
  double q[4][2];
  bool finite = true;
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    q[c][0] = a.y[2 * id[c]];
    q[c][1] = a.y[2 * id[c] + 1];
    finite = finite && isfinite(q[c][0]) && isfinite(q[c][1]);
  }
  if (!finite) return;
  double lo0 = q[0][0], hi0 = q[0][0], lo1 = q[0][1], hi1 = q[0][1];
#pragma unroll
  for (int c = 1; c < 4; ++c) {
    lo0 = fmin(lo0, q[c][0]);
    hi0 = fmax(hi0, q[c][0]);
    lo1 = fmin(lo1, q[c][1]);
    hi1 = fmax(hi1, q[c][1]);
  }
  for (int32_t s = 0; s < a.n_src; ++s) {
    const double b0 = a.src[2 * s], b1 = a.src[2 * s + 1];
    if (b0 < lo0 || b0 > hi0 || b1 < lo1 || b1 > hi1) continue;
    // triangles (0, 1, 2) and (0, 2, 3)
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int cb = t == 0 ? 1 : 2, cc = t == 0 ? 2 : 3;
      const double ux = q[cb][0] - q[0][0], uy = q[cb][1] - q[0][1];
      const double vx = q[cc][0] - q[0][0], vy = q[cc][1] - q[0][1];
      const double px = b0 - q[0][0], py = b1 - q[0][1];
      const double d = cross2(ux, uy, vx, vy);
      if (!(d != 0.0)) continue;
      const double lb = cross2(px, py, vx, vy) / d, lc = cross2(ux, uy, px, py) / d;
      if (!(lb >= 0.0 && lc >= 0.0 && lb + lc <= 1.0)) continue;
      const unsigned long long slot = atomicAdd(a.count, 1ull);
      if ((int64_t)slot >= a.cap) continue;
      a.cand_x[2 * slot] = X[0] + lb * (X[cb] - X[0]) + lc * (X[cc] - X[0]);
      a.cand_x[2 * slot + 1] = Y[0] + lb * (Y[cb] - Y[0]) + lc * (Y[cc] - Y[0]);
      a.cand_s[slot] = s;
    }
  }
}

// One Newton step x <- x + A^-1 (beta - y) from the residual (r0, r1) of
// length res and f', its length clamped to max_step and x to the box; no step
// if !move.  Returns det A.
__device__ __forceinline__ double newton_step(const NewtonArgs &a, double r0, double r1, double res,
                                              double fr, double fi, bool move, double &x0, double &x1) {
  const double A11 = a.c1 - fr, A22 = a.c2 + fr, A12 = fi;
  const double det = A11 * A22 - A12 * A12;
  if (!move || !(res > 0.0) || !(det != 0.0) || !isfinite(det)) return det;
  double d0 = (A22 * r0 - A12 * r1) / det, d1 = (A11 * r1 - A12 * r0) / det;
  const double len = sqrt(d0 * d0 + d1 * d1);
  if (!(len <= a.max_step)) {
    const double f = isfinite(len) ? a.max_step / len : 0.0;
    d0 *= f;
    d1 *= f;
  }
  x0 = fmin(fmax(x0 + d0, a.box[0]), a.box[2]);
  x1 = fmin(fmax(x1 + d1, a.box[1]), a.box[3]);
  return det;
}

// One Newton step per candidate from y(x) and f'(x) (the direct sum's, or those
// of many candidates as explicit rays).  res
// receives |beta - y| at the x the step started from; *unconverged counts
// those above tol.
__global__ __launch_bounds__(kThreads) void k_newton(NewtonArgs a) {
  const int64_t k = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (k >= a.n) return;
  const int32_t s = a.cand_s[k];
  const double r0 = a.src[2 * s] - a.y[2 * k], r1 = a.src[2 * s + 1] - a.y[2 * k + 1];
  const double res = sqrt(r0 * r0 + r1 * r1);
  a.res[k] = res;
  if (!(res <= a.tol)) atomicAdd(a.unconverged, 1u);
  a.det[k] = newton_step(a, r0, r1, res, a.dfdz[2 * k], a.dfdz[2 * k + 1], a.step != 0, a.cand_x[2 * k],
                         a.cand_x[2 * k + 1]);
}

// Newton iterations of the candidates on the FMM, a wave per candidate: each
// iteration evaluates y and f' at x -- the lanes share the stars of the 3x3
// leaf neighbourhood, their sums added across the wave in FP64, and the local
// expansion and its derivative come from one Horner recurrence -- and steps as
// k_newton does.  One launch takes a.iters iterations and keeps every one's
// (x after the step, residual, det A) and the number of candidates above tol,
// so the caller can stop at the first iteration that leaves none.  (A launch
// per stage of each iteration -- sort the candidates by box, evaluate, step,
// read the count back -- took 110 us an iteration for ~1000 candidates; this
// kernel takes about 3.  Its lanes all sum the same expansion, so many candidates
// are better off with a lane each: see wave_candidates.)
template <bool MIXED>
__global__ __launch_bounds__(64) void k_newton_fmm(NewtonArgs a, EvalArgs e, NewtonHistory h) {
  const int lane = threadIdx.x;
  const int64_t k = blockIdx.x;
  const int32_t sid = a.cand_s[k];
  const double beta0 = a.src[2 * sid], beta1 = a.src[2 * sid + 1];
  double x0 = a.cand_x[2 * k], x1 = a.cand_x[2 * k + 1];
  const int64_t nL = int64_t(1) << e.g.L;
  const double s = ldexp(e.g.side, -e.g.L), inv_s = 1.0 / s;
  for (int it = 0; it < h.iters; ++it) {
    // the candidate's box, clamped to the window (as explicit rays are)
    int64_t ix = box_coord(x0, e.g.x0, s, nL) - e.win.bx0;
    int64_t iy = box_coord(x1, e.g.y0, s, nL) - e.win.by0;
    ix = ix < 0 ? 0 : (ix >= e.win.nbx ? e.win.nbx - 1 : ix);
    iy = iy < 0 ? 0 : (iy >= e.win.nby ? e.win.nby - 1 : iy);
    const int64_t gx = e.win.bx0 + ix, gy = e.win.by0 + iy;
    int32_t rs[3], pre[4];
    pre[0] = 0;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const int64_t row = gy - 1 + d;
      rs[d] = 0;
      int32_t re = 0;
      if (row >= 0 && row < nL) {
        rs[d] = e.leaf_start[row * nL + (gx > 0 ? gx - 1 : 0)];
        re = e.leaf_start[row * nL + (gx + 1 < nL ? gx + 1 : nL - 1) + 1];
      }
      pre[d + 1] = pre[d] + (re - rs[d]);
    }
    double a1 = 0.0, a2 = 0.0, dre = 0.0, dim = 0.0;
    for (int32_t t = lane; t < pre[3]; t += 64) {
      const int d = t >= pre[2] ? 2 : (t >= pre[1] ? 1 : 0);
      const int64_t i = (d == 2 ? rs[2] - pre[2] : (d == 1 ? rs[1] - pre[1] : rs[0])) + (int64_t)t;
      const double ex = x0 - e.sxy[2 * i], ey = x1 - e.sxy[2 * i + 1];
      if (MIXED) {
        constexpr float tiny = 0x1p-100f;
        const float dx = (float)ex, dy = (float)ey;
        const float r2 = fmaf(dx, dx, fmaf(dy, dy, tiny)), inv = rcp_f32(r2), w = e.sm32[i] * inv;
        const float u = r2 > tiny ? w * inv : 0.0f;
        a1 += (double)(w * dx);
        a2 += (double)(w * dy);
        dre += (double)(-u * ((dx - dy) * (dx + dy)));
        dim += (double)((u + u) * (dx * dy));
      } else {
        constexpr double tiny = 0x1p-664;
        const double r2 = fma(ex, ex, fma(ey, ey, tiny)), inv = rcp_f64(r2), w = e.sm[i] * inv;
        const double u = r2 > tiny ? w * inv : 0.0;
        a1 = fma(w, ex, a1);
        a2 = fma(w, ey, a2);
        dre = fma(-u, (ex - ey) * (ex + ey), dre);
        dim = fma(u + u, ex * ey, dim);
      }
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
      a1 += __shfl_xor(a1, d);
      a2 += __shfl_xor(a2, d);
      dre += __shfl_xor(dre, d);
      dim += __shfl_xor(dim, d);
    }
    // far field: f = sum b_l w^l and its derivative
    const double2 *lb = reinterpret_cast<const double2 *>(e.loc) + (iy * e.win.nbx + ix) * e.p;
    const cplx w = {(x0 - (e.g.x0 + ((double)gx + 0.5) * s)) * inv_s,
                    (x1 - (e.g.y0 + ((double)gy + 0.5) * s)) * inv_s};
    cplx f = {0.0, 0.0}, df = {0.0, 0.0};
#pragma unroll 4
    for (int l = e.p - 1; l >= 0; --l) {
      const double2 b = lb[l];
      df = cmad(df, w, f);
      f = cmad(f, w, cplx{b.x, b.y});
    }
    const double y0 = a.c1 * x0 - (f.re + a1), y1 = a.c2 * x1 - (a2 - f.im);
    const double fr = fma(df.re, inv_s, dre), fi = fma(df.im, inv_s, dim);
    const double r0 = beta0 - y0, r1 = beta1 - y1;
    const double res = sqrt(r0 * r0 + r1 * r1);
    const double det = newton_step(a, r0, r1, res, fr, fi, h.last_steps || it + 1 < h.iters, x0, x1);
    if (lane == 0) {
      const int64_t o = (int64_t)it * a.n + k;
      h.x[2 * o] = x0;
      h.x[2 * o + 1] = x1;
      h.res[o] = res;
      h.det[o] = det;
      if (!(res <= a.tol)) atomicAdd(&h.unconverged[it], 1u);
    }
  }
  if (lane == 0) {
    a.cand_x[2 * k] = x0;
    a.cand_x[2 * k + 1] = x1;
  }
}

// det A at the four corners of a cell: zero crossings on its edges.
__global__ __launch_bounds__(kThreads) void k_crit_cells(CritArgs a) {
  const int64_t ncx = a.nx - 1;
  const int64_t ncell = ncx * (a.j1 - a.j0);
  const int64_t k = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (k >= ncell) return;
  const int64_t i = k % ncx, j = a.j0 + k / ncx;
  const int64_t r0 = (j - a.ybase) * a.nx + i, r1 = r0 + a.nx;
  const int64_t id[4] = {r0, r0 + 1, r1 + 1, r1};
  const double X[4] = {grid_coord(a.grid.x0, a.grid.dx, i), grid_coord(a.grid.x0, a.grid.dx, i + 1),
                       grid_coord(a.grid.x0, a.grid.dx, i + 1), grid_coord(a.grid.x0, a.grid.dx, i)};
  const double Y[4] = {grid_coord(a.grid.y0, a.grid.dy, j), grid_coord(a.grid.y0, a.grid.dy, j),
                       grid_coord(a.grid.y0, a.grid.dy, j + 1), grid_coord(a.grid.y0, a.grid.dy, j + 1)};
  double d[4];
  int npos = 0;
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const double fr = a.dfdz[2 * id[c]], fi = a.dfdz[2 * id[c] + 1];
    d[c] = (a.c1 - fr) * (a.c2 + fr) - fi * fi;
    if (!isfinite(d[c])) return;
    npos += d[c] > 0.0;
  }
  if (npos == 0 || npos == 4) return;
  // crossing points on edges c -> c+1, in order round the cell
  double px[4], py[4];
  int ncut = 0;
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const int e = (c + 1) & 3;
    if ((d[c] > 0.0) == (d[e] > 0.0)) continue;
    const double t = d[c] / (d[c] - d[e]);
    px[ncut] = X[c] + t * (X[e] - X[c]);
    py[ncut] = Y[c] + t * (Y[e] - Y[c]);
    ++ncut;
  }
  int pairs[2][2] = {{0, 1}, {2, 3}};
  int nseg = 1;
  if (ncut == 4) {
    nseg = 2;
    // corners 0 and 2 share a sign, 1 and 3 the other; if the centre takes
    // corner 0's sign the curve separates corners 1 and 3 from it: the cut
    // on edge 0-1 joins the cut on edge 1-2, and 2-3 joins 3-0
    const bool centre_pos = 0.25 * (d[0] + d[1] + d[2] + d[3]) > 0.0;
    if (centre_pos == (d[0] > 0.0)) {
      pairs[0][0] = 0; pairs[0][1] = 1; pairs[1][0] = 2; pairs[1][1] = 3;
    } else {
      pairs[0][0] = 0; pairs[0][1] = 3; pairs[1][0] = 1; pairs[1][1] = 2;
    }
  } else if (ncut != 2) {
    return;
  }
  for (int sg = 0; sg < nseg; ++sg) {
    const unsigned long long slot = atomicAdd(a.count, 1ull);
    if ((int64_t)slot >= a.cap) continue;
    double4 v;
    v.x = px[pairs[sg][0]];
    v.y = py[pairs[sg][0]];
    v.z = px[pairs[sg][1]];
    v.w = py[pairs[sg][1]];
    reinterpret_cast<double4 *>(a.seg)[slot] = v;
  }
}

// Multi-plane: x_j = x_0 - sum_{i<j} beta_ij alpha_i (alpha_i = x_i - y_i of
// plane i), for grid or explicit x_0.
__global__ __launch_bounds__(kThreads) void k_mp_positions(MultiPlaneArgs a) {
  const int64_t k = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (k >= a.n) return;
  double x0, x1;
  if (a.grid_mode) {
    x0 = grid_coord(a.grid.x0, a.grid.dx, k % a.grid.nx);
    x1 = grid_coord(a.grid.y0, a.grid.dy, k / a.grid.nx);
  } else {
    x0 = a.rays[2 * k];
    x1 = a.rays[2 * k + 1];
  }
  for (int32_t i = 0; i < a.j; ++i) {
    const double b = a.beta[i];
    const double *al = a.alpha + (size_t)i * 2 * a.n;
    x0 -= b * al[2 * k];
    x1 -= b * al[2 * k + 1];
  }
  a.x_out[2 * k] = x0;
  a.x_out[2 * k + 1] = x1;
}

// alpha_j = x_j - y_j, kept for the later planes.
__global__ __launch_bounds__(kThreads) void k_mp_alpha(const double *__restrict__ x,
                                                       const double *__restrict__ y,
                                                       double *__restrict__ alpha, int64_t n2) {
  const int64_t k = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (k < n2) alpha[k] = x[k] - y[k];
}

unsigned blocks_for(int64_t n) { return (unsigned)((n + kThreads - 1) / kThreads); }

}  // namespace

void launch_image_cells(const ImageCellArgs &a, hipStream_t stream) {
  const int64_t ncell = (a.nx - 1) * (a.j1 - a.j0);
  if (ncell <= 0) return;
  if ((ncell + kThreads - 1) / kThreads > 0x7fffffff) fail(LENS_EUNSUPPORTED, "image pass too large");
  hipLaunchKernelGGL(k_image_cells, dim3(blocks_for(ncell)), dim3(kThreads), 0, stream, a);
  LENS_HIP(hipGetLastError());
}

void launch_newton(const NewtonArgs &a, hipStream_t stream) {
  if (a.n <= 0) return;
  hipLaunchKernelGGL(k_newton, dim3(blocks_for(a.n)), dim3(kThreads), 0, stream, a);
  LENS_HIP(hipGetLastError());
}

void launch_newton_fmm(const NewtonArgs &a, const EvalArgs &e, const NewtonHistory &h, int precision,
                       hipStream_t stream) {
  if (a.n <= 0) return;
  if (a.n > 0x7fffffff) fail(LENS_EUNSUPPORTED, "too many image candidates");
  if (precision == LENS_MIXED)
    hipLaunchKernelGGL(k_newton_fmm<true>, dim3((unsigned)a.n), dim3(64), 0, stream, a, e, h);
  else
    hipLaunchKernelGGL(k_newton_fmm<false>, dim3((unsigned)a.n), dim3(64), 0, stream, a, e, h);
  LENS_HIP(hipGetLastError());
}

void launch_crit_cells(const CritArgs &a, hipStream_t stream) {
  const int64_t ncell = (a.nx - 1) * (a.j1 - a.j0);
  if (ncell <= 0) return;
  if ((ncell + kThreads - 1) / kThreads > 0x7fffffff) fail(LENS_EUNSUPPORTED, "critical-curve pass too large");
  hipLaunchKernelGGL(k_crit_cells, dim3(blocks_for(ncell)), dim3(kThreads), 0, stream, a);
  LENS_HIP(hipGetLastError());
}

void launch_mp_positions(const MultiPlaneArgs &a, hipStream_t stream) {
  if (a.n <= 0) return;
  hipLaunchKernelGGL(k_mp_positions, dim3(blocks_for(a.n)), dim3(kThreads), 0, stream, a);
  LENS_HIP(hipGetLastError());
}

void launch_mp_alpha(const double *x, const double *y, double *alpha, int64_t n, hipStream_t stream) {
  if (n <= 0) return;
  hipLaunchKernelGGL(k_mp_alpha, dim3(blocks_for(2 * n)), dim3(kThreads), 0, stream, x, y, alpha,
                     2 * n);
  LENS_HIP(hipGetLastError());
}

}  // namespace lensfmm
