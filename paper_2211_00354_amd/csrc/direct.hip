// Plain FP64 direct sum of the lens equation (Section 1, eq. 1): every ray
// against every star, O(N_* x N_x).  This is the method the FMM replaces and
// the FP64 comparator it is measured against.
//
// A thread holds a ray; the stars are the same for every lane of a wave, so
// they are read with scalar loads and used as scalar operands of the vector
// instructions, ~14 issue slots a pair (0.36 ps; 0.41 with the stars
// broadcast from LDS tiles to two rays a thread).  Where the rays make too few
// waves to fill the chip, a workgroup's four waves take a quarter of the stars
// each for the same rays and add their sums in LDS.  A wave that has its rays to
// itself sums the same quarters one after another and adds them in the same
// order, so that a ray's bits depend neither on the number of rays of a launch
// nor on the passes that a call is cut into.  Pairs with |x - x_i| = 0
// contribute exactly zero.
#include "device_common.h"

namespace lensfmm {

namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;
constexpr int32_t kFewStars = 32;  // not shared out: a chain no longer than a launch's own time

// DERIV also sums f'(z) = -sum m / (z - z_i)^2 (see the evaluation kernel).
// SLICES: the stars are shared out over the workgroup's waves.
template <bool MAP, bool GRID, bool DERIV, bool SLICES>
__global__ __launch_bounds__(kThreads) void k_direct(DirectArgs a, const double *__restrict__ sxy,
                                                     const double *__restrict__ sm) {
  constexpr int V = DERIV ? 4 : 2;
  constexpr int RPB = SLICES ? 64 : kThreads;  // rays per workgroup
  __shared__ double part[SLICES ? (kWaves - 1) * V * 64 : 1];
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int64_t local = (int64_t)blockIdx.x * RPB + (SLICES ? lane : (int)threadIdx.x);
  const bool act = local < a.n_rays;
  const int64_t k = a.ray_offset + (act ? local : 0);
  double rx, ry, ax = 0.0, ay = 0.0, dre = 0.0, dim = 0.0;
  if (GRID) {
    rx = grid_coord(a.grid.x0, a.grid.dx, k % a.grid.nx);
    ry = grid_coord(a.grid.y0, a.grid.dy, k / a.grid.nx);
  } else {
    rx = a.rxy[2 * k];
    ry = a.rxy[2 * k + 1];
  }
  auto star = [&](double sx, double sy, double m) {
    // a coincident pair has dx = dy = 0: the tiny term keeps its weight
    // finite, so it adds exactly zero (no other pair closer than ~1e-92
    // is affected)
    const double dx = rx - sx;
    const double dy = ry - sy;
    const double r2 = fma(dx, dx, fma(dy, dy, 0x1p-664));
    const double inv = rcp_f64(r2);
    const double w = m * inv;
    ax = fma(w, dx, ax);
    ay = fma(w, dy, ay);
    if (DERIV) {
      const double t = r2 > 0x1p-664 ? w * inv : 0.0;
      dre = fma(-t, (dx - dy) * (dx + dy), dre);
      dim = fma(t + t, dx * dy, dim);
    }
  };
  // star counts fit 31 bits
  const int32_t n = (int32_t)a.n_stars;
  // sums over quarter w of the stars (of a few: all of them, or none); whole
  // steps of four but for the last one's
  auto first = [&](int w) -> int32_t {
    if (w == 0 || w == kWaves) return w == 0 ? 0 : n;
    return n < kFewStars ? n : (int32_t)((int64_t)n * w / kWaves) & ~3;
  };
  auto quarter = [&](int w) {
    const int32_t i = first(w);
    const double *xy = sxy + 2 * (int64_t)i, *mass = sm + i;
    ax = ay = dre = dim = 0.0;
    int32_t left = first(w + 1) - i;
    // four stars per step: their scalar loads issue together
    for (; left >= 4; left -= 4, xy += 8, mass += 4) {
      double sx[4], sy[4], m[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        sx[q] = xy[2 * q];
        sy[q] = xy[2 * q + 1];
        m[q] = mass[q];
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) star(sx[q], sy[q], m[q]);
    }
    for (; left > 0; --left, xy += 2, ++mass) star(xy[0], xy[1], mass[0]);
  };
  if constexpr (SLICES) {
    quarter(wv);
    double *o = part + (wv > 0 ? wv - 1 : 0) * V * 64 + lane;
    if (wv > 0) {
      o[0] = ax;
      o[64] = ay;
      if (DERIV) {
        o[128] = dre;
        o[192] = dim;
      }
    }
    __syncthreads();
    if (wv > 0) return;
#pragma unroll
    for (int w = 0; w < kWaves - 1; ++w, o += V * 64) {
      ax += o[0];
      ay += o[64];
      if (DERIV) {
        dre += o[128];
        dim += o[192];
      }
    }
  } else {
    quarter(0);
    if (n >= kFewStars) {
      double sax = ax, say = ay, sre = dre, sim = dim;
#pragma unroll 1
      for (int w = 1; w < kWaves; ++w) {
        quarter(w);
        sax += ax;
        say += ay;
        sre += dre;
        sim += dim;
      }
      ax = sax;
      ay = say;
      dre = sre;
      dim = sim;
    }
  }
  if (!act) return;
  const double y1 = a.c1 * rx - ax;
  const double y2 = a.c2 * ry - ay;
  if (MAP) {
    const double t1 = (y1 - a.y1min) * a.S;
    const double t2 = (y2 - a.y2min) * a.S;
    if (t1 >= 0.0 && t2 >= 0.0) {
      const double f1 = floor(t1), f2 = floor(t2);
      if (f1 < (double)a.npix && f2 < (double)a.npix)
        atomicAdd(&a.counts[(int64_t)f2 * a.npix + (int64_t)f1], 1);
    }
  } else {
    a.y_out[2 * k] = y1;
    a.y_out[2 * k + 1] = y2;
    if (DERIV) {
      a.dfdz_out[2 * k] = dre;
      a.dfdz_out[2 * k + 1] = dim;
    }
  }
}

template <bool SLICES>
void direct_launch(const DirectArgs &a, hipStream_t stream) {
  constexpr int64_t RPB = SLICES ? 64 : kThreads;
  const dim3 grid((unsigned)((a.n_rays + RPB - 1) / RPB)), block(kThreads);
  const bool map = a.counts != nullptr;
  const bool deriv = !map && a.dfdz_out != nullptr;
#define LENS_DIRECT_LAUNCH(MAP, GRID, DERIV) \
  hipLaunchKernelGGL((k_direct<MAP, GRID, DERIV, SLICES>), grid, block, 0, stream, a, a.sxy, a.sm)
  if (a.grid_mode) {
    if (map) LENS_DIRECT_LAUNCH(true, true, false);
    else if (deriv) LENS_DIRECT_LAUNCH(false, true, true);
    else LENS_DIRECT_LAUNCH(false, true, false);
  } else {
    if (map) LENS_DIRECT_LAUNCH(true, false, false);
    else if (deriv) LENS_DIRECT_LAUNCH(false, false, true);
    else LENS_DIRECT_LAUNCH(false, false, false);
  }
#undef LENS_DIRECT_LAUNCH
}

// Rays that fill the chip (8192 waves: two workgroups a SIMD) with a wave's
// rays each to itself; fewer share the stars out over four waves (1000 stars,
// whole call: 512^2 rays 104 us against 121, 256^2 31 against 56, 64^2 15
// against 57).
constexpr int64_t kFewRays = 64 * 8192;
// A launch takes fewer than 2^32 threads.
constexpr int64_t kMaxRays = int64_t(1) << 31;

}  // namespace

void launch_direct(const DirectArgs &a, hipStream_t stream) {
  if (a.n_rays == 0) return;
  DirectArgs part = a;
  for (int64_t at = 0; at < a.n_rays; at += kMaxRays) {
    part.ray_offset = a.ray_offset + at;
    part.n_rays = a.n_rays - at < kMaxRays ? a.n_rays - at : kMaxRays;
    if (part.n_rays <= kFewRays)
      direct_launch<true>(part, stream);
    else
      direct_launch<false>(part, stream);
    LENS_HIP(hipGetLastError());
  }
}

}  // namespace lensfmm
