// Adjoint of the lens map with respect to the lenses (the gradient of a loss
// L(y) with respect to star positions and masses), derived from eq. 1 of
// Section 1.  With g_k = dL/dy1_k + i dL/dy2_k per ray and
//
//     h(z) = sum_k g_k / (z - z_k)          (a Cauchy sum: rays are the
//                                            sources, with complex charges)
//
// the gradients at star i are
//
//     dL/dm_i              = Re h(z_i)
//     dL/dx_i + i dL/dy_i  = m_i conj(h'(z_i)),   h'(z) = -sum_k g_k/(z - z_k)^2
//
// (from y = x - conj(sum m_i / (z - z_i)) and dL = Re sum_k conj(g_k) dy_k).
// The FMM evaluates h and h' with the same tree, expansions and downward pass
// as the forward problem, sources and targets exchanged: P2M over rays with
// complex charges, then at the stars the local expansion and its derivative
// (Horner) plus the near field over the rays of the 3x3 leaf neighbourhood.
// A ray exactly on a star is skipped, as in the forward map.
#include <algorithm>

#include "device_common.h"

namespace lensfmm {

namespace {

constexpr int kThreads = 256;
constexpr int32_t kFlushSources = 128;  // LENS_MIXED near-field partials per FP64 flush
constexpr int64_t kHeldLanes = 1 << 19;  // lanes of k_eval_adj the chip holds at once, about

// One source (position, complex charge) against the R targets of a lane:
// h += q/d, hp -= q/d^2 with d = z_target - z_source.  A coincident pair has
// d = 0 and adds exactly zero (the tiny term keeps 1/|d|^2 finite).
template <bool MIXED, int R, typename A>
__device__ __forceinline__ void adj_pair(const double (&tx)[R], const double (&ty)[R], double sx,
                                         double sy, double qr, double qi, A (&hr)[R], A (&hi)[R],
                                         A (&pr)[R], A (&pi)[R]) {
  using T = A;
  constexpr T tiny = MIXED ? (T)0x1p-66f : (T)0x1p-664;
  const T q_re = (T)qr, q_im = (T)qi;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const T dx = (T)(tx[r] - sx), dy = (T)(ty[r] - sy);
    const T r2 = fma(dx, dx, fma(dy, dy, tiny));
    const T w = MIXED ? (T)rcp_f32((float)r2) : (T)rcp_f64((double)r2);
    // 1/d = (dx - i dy) w
    const T ir = dx * w, ii = -dy * w;
    // q/d
    const T ar = fma(q_re, ir, -q_im * ii), ai = fma(q_re, ii, q_im * ir);
    hr[r] += ar;
    hi[r] += ai;
    // q/d^2 = (q/d)(1/d)
    pr[r] -= fma(ar, ir, -ai * ii);
    pi[r] -= fma(ar, ii, ai * ir);
  }
}

// h and h' at the targets, SPLIT lanes to a target and neighbouring targets
// (sorted by leaf box) in neighbouring lanes, each lane with its own box's
// sources: clustered lenses leave most boxes a few targets, so a wave to a box
// had most of its lanes idle (2e5 clustered stars, 1e6 rays: 318 us, now 80).
// What is left is the loads' latency, so a lane keeps four sources in flight
// behind the four that it works on (one instead: 94 us).  A lane
// walks the three contiguous source ranges of its 3x3 neighbourhood, in groups
// of kFlushSources sources; with SPLIT > 1 the lanes of a target take its groups
// in turn.  LENS_MIXED sums a group in FP32 and the groups in FP64, so a
// neighbourhood of thousands of rays does not accumulate thousands of FP32
// roundings.
template <bool MIXED, int SPLIT>
__global__ __launch_bounds__(kThreads) void k_eval_adj(
    EvalArgs a, int64_t nt, const double *__restrict__ loc, const double *__restrict__ sxy,
    const double *__restrict__ sq, const int32_t *__restrict__ leaf_start,
    const double *__restrict__ txy, const double *__restrict__ tm, const uint32_t *__restrict__ tperm,
    double *__restrict__ grad_xy, double *__restrict__ grad_m) {
  using acc_t = typename std::conditional<MIXED, float, double>::type;
  const int64_t gid = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  const int part = (int)(gid % SPLIT);
  const bool act = gid / SPLIT < nt;
  const int64_t t = act ? gid / SPLIT : nt - 1;
  const int64_t nL = int64_t(1) << a.g.L;
  const double s = ldexp(a.g.side, -a.g.L);
  const double inv_s = 1.0 / s;
  const int p = a.p;
  const double tx[1] = {txy[2 * t]}, ty[1] = {txy[2 * t + 1]};
  // the target's box, in the window (as the targets' sort places them)
  int64_t ix = box_coord(tx[0], a.g.x0, s, nL) - a.win.bx0;
  int64_t iy = box_coord(ty[0], a.g.y0, s, nL) - a.win.by0;
  ix = ix < 0 ? 0 : (ix >= a.win.nbx ? a.win.nbx - 1 : ix);
  iy = iy < 0 ? 0 : (iy >= a.win.nby ? a.win.nby - 1 : iy);
  const int64_t gx = a.win.bx0 + ix, gy = a.win.by0 + iy;
  // source ranges of the three rows, and their running totals
  int32_t rs[3], pre[4];
  pre[0] = 0;
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const int64_t row = gy - 1 + d;
    rs[d] = 0;
    int32_t re = 0;
    if (act && row >= 0 && row < nL) {
      rs[d] = leaf_start[row * nL + (gx > 0 ? gx - 1 : 0)];
      re = leaf_start[row * nL + (gx + 1 < nL ? gx + 1 : nL - 1) + 1];
    }
    pre[d + 1] = pre[d] + (re - rs[d]);
  }
  const int32_t n = pre[3];
  const double2 *sz = reinterpret_cast<const double2 *>(sxy), *sg = reinterpret_cast<const double2 *>(sq);
  double Sr = 0.0, Si = 0.0, Tr = 0.0, Ti = 0.0;
  acc_t hr[1] = {0}, hi[1] = {0}, pr[1] = {0}, pi[1] = {0};
  for (int32_t g = part; (int64_t)g * kFlushSources < n; g += SPLIT) {
    // (unsigned: a place may pass 2^31 by a step)
    uint32_t k = (uint32_t)g * kFlushSources;
    const uint32_t end = min((uint32_t)n, k + kFlushSources);
    // the next four sources' loads are issued before the current four pairs
    double2 nz[4], nq[4];
    auto fetch = [&](uint32_t q0) {
#pragma unroll
      for (uint32_t j = 0; j < 4; ++j) {
        const int32_t q = (int32_t)min(q0 + j, end - 1);
        const int32_t i = q >= pre[2] ? rs[2] + (q - pre[2]) : (q >= pre[1] ? rs[1] + (q - pre[1]) : rs[0] + q);
        nz[j] = sz[i];
        nq[j] = sg[i];
      }
    };
    fetch(k);
    for (; k < end; k += 4) {
      double2 z[4], q[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) z[j] = nz[j], q[j] = nq[j];
      fetch(k + 4);
#pragma unroll
      for (uint32_t j = 0; j < 4; ++j)
        if (k + j < end) adj_pair<MIXED, 1>(tx, ty, z[j].x, z[j].y, q[j].x, q[j].y, hr, hi, pr, pi);
    }
    if (MIXED) {
      Sr += (double)hr[0];
      Si += (double)hi[0];
      Tr += (double)pr[0];
      Ti += (double)pi[0];
      hr[0] = hi[0] = pr[0] = pi[0] = 0;
    }
  }
  if (!MIXED) Sr = hr[0], Si = hi[0], Tr = pr[0], Ti = pi[0];
#pragma unroll
  for (int d = SPLIT / 2; d >= 1; d >>= 1) {
    Sr += __shfl_xor(Sr, d);
    Tr += __shfl_xor(Tr, d);
    Ti += __shfl_xor(Ti, d);
  }
  (void)Si;  // Im h enters no gradient
  // far field: h = sum b_l w^l and dh/dw by one Horner recurrence
  const double2 *lb = reinterpret_cast<const double2 *>(loc) + (iy * a.win.nbx + ix) * p;
  const cplx w = {(tx[0] - (a.g.x0 + ((double)gx + 0.5) * s)) * inv_s,
                  (ty[0] - (a.g.y0 + ((double)gy + 0.5) * s)) * inv_s};
  cplx f = {0.0, 0.0}, df = {0.0, 0.0};
#pragma unroll 4
  for (int l = p - 1; l >= 0; --l) {
    const double2 b = lb[l];
    df = cmad(df, w, f);
    f = cmad(f, w, cplx{b.x, b.y});
  }
  if (!act || part != 0) return;
  const uint32_t o = tperm[t];
  const double m = tm[t];
  grad_m[o] = f.re + Sr;
  grad_xy[2 * (int64_t)o] = m * (df.re * inv_s + Tr);
  grad_xy[2 * (int64_t)o + 1] = -(m * (df.im * inv_s + Ti));
}

// Direct FP64 gradient: every star against every ray, rays streamed through
// LDS as (x, y, Re g, Im g) tiles.  The comparator of the adjoint FMM.
constexpr int kAdjTile = 512;

template <int R>
__global__ __launch_bounds__(kThreads) void k_direct_adj(int64_t n_stars,
                                                         const double *__restrict__ star_xy,
                                                         const double *__restrict__ star_m,
                                                         int64_t n_rays,
                                                         const double *__restrict__ rays_xy,
                                                         const double *__restrict__ grad_y,
                                                         double *__restrict__ grad_xy,
                                                         double *__restrict__ grad_m) {
  __shared__ double rx[kAdjTile], ry[kAdjTile], gr[kAdjTile], gi[kAdjTile];
  const int tid = threadIdx.x;
  double tx[R], ty[R], hr[R], hi[R], pr[R], pi[R];
  int64_t sid[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    sid[r] = (int64_t)blockIdx.x * kThreads * R + (int64_t)r * kThreads + tid;
    const int64_t k = sid[r] < n_stars ? sid[r] : 0;
    tx[r] = n_stars ? star_xy[2 * k] : 0.0;
    ty[r] = n_stars ? star_xy[2 * k + 1] : 0.0;
    hr[r] = hi[r] = pr[r] = pi[r] = 0.0;
  }
  for (int64_t base = 0; base < n_rays; base += kAdjTile) {
    const int cnt = (int)(n_rays - base < kAdjTile ? n_rays - base : kAdjTile);
    __syncthreads();
    for (int t = tid; t < cnt; t += kThreads) {
      rx[t] = rays_xy[2 * (base + t)];
      ry[t] = rays_xy[2 * (base + t) + 1];
      gr[t] = grad_y[2 * (base + t)];
      gi[t] = grad_y[2 * (base + t) + 1];
    }
    __syncthreads();
    for (int k = 0; k < cnt; ++k)
      adj_pair<false, R>(tx, ty, rx[k], ry[k], gr[k], gi[k], hr, hi, pr, pi);
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
    if (sid[r] >= n_stars) continue;
    const double m = star_m[sid[r]];
    grad_m[sid[r]] = hr[r];
    grad_xy[2 * sid[r]] = m * pr[r];
    grad_xy[2 * sid[r] + 1] = -(m * pi[r]);
  }
}

__global__ __launch_bounds__(kThreads) void k_grid_rays(lens_grid g, double *__restrict__ out) {
  const int64_t k = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (k >= g.nx * g.ny) return;
  out[2 * k] = grid_coord(g.x0, g.dx, k % g.nx);
  out[2 * k + 1] = grid_coord(g.y0, g.dy, k / g.nx);
}

template <bool MIXED, int SPLIT>
void adj_launch(const EvalArgs &a, const AdjArgs &d, hipStream_t stream) {
  const int64_t blocks = (d.nt * SPLIT + kThreads - 1) / kThreads;
  hipLaunchKernelGGL((k_eval_adj<MIXED, SPLIT>), dim3((unsigned)blocks), dim3(kThreads), 0, stream, a,
                     d.nt, a.loc, a.sxy, d.sq, a.leaf_start, d.txy, d.tm, d.tperm, d.grad_xy, d.grad_m);
}

template <bool MIXED>
void adj_dispatch(const EvalArgs &a, const AdjArgs &d, hipStream_t stream) {
  // Lanes to a target: more where each still finds whole groups of the mean
  // neighbourhood's sources, or where the chip holds all lanes at once and an
  // uneven distribution's longest chain is all that counts.  Whole backward
  // pass, mixed: 1e5 stars on 1e6 rays within a tenth of their radius 6.7 ms
  // with one lane, 1.1 with sixteen (a wave to a box: 4.3); half of the rays
  // within 1/60 of it 47 and 14 ms with four; even rays pay 259 against 286 us.
  // A launch takes fewer than 2^32 threads.
  const double groups = 9.0 * d.per_box / kFlushSources;
  const auto fits = [&](int64_t split) { return d.nt * split <= (int64_t(1) << 32) - kThreads; };
  if ((groups >= 16.0 || d.nt <= kHeldLanes / 16) && fits(16))
    adj_launch<MIXED, 16>(a, d, stream);
  else if ((groups >= 4.0 || d.nt <= kHeldLanes / 4) && fits(4))
    adj_launch<MIXED, 4>(a, d, stream);
  else
    adj_launch<MIXED, 1>(a, d, stream);
}

}  // namespace

void launch_eval_adj(const EvalArgs &a, const AdjArgs &d, int precision, hipStream_t stream) {
  if (a.win.count() == 0 || d.nt == 0) return;
  if (precision == LENS_MIXED)
    adj_dispatch<true>(a, d, stream);
  else
    adj_dispatch<false>(a, d, stream);
  LENS_HIP(hipGetLastError());
}

void launch_direct_adj(int64_t n_stars, const double *star_xy, const double *star_m, int64_t n_rays,
                       const double *rays_xy, const double *grad_y, double *grad_xy,
                       double *grad_m, hipStream_t stream) {
  if (n_stars == 0) return;
  constexpr int R = 2;
  const int64_t nblk = (n_stars + kThreads * R - 1) / (kThreads * R);
  hipLaunchKernelGGL((k_direct_adj<R>), dim3((unsigned)nblk), dim3(kThreads), 0, stream, n_stars,
                     star_xy, star_m, n_rays, rays_xy, grad_y, grad_xy, grad_m);
  LENS_HIP(hipGetLastError());
}

void launch_grid_rays(const lens_grid &g, double *out, hipStream_t stream) {
  const int64_t n = g.nx * g.ny;
  if (n == 0) return;
  hipLaunchKernelGGL(k_grid_rays, dim3((unsigned)((n + kThreads - 1) / kThreads)), dim3(kThreads), 0,
                     stream, g, out);
  LENS_HIP(hipGetLastError());
}

}  // namespace lensfmm
