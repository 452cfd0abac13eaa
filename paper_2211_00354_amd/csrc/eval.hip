// Evaluation at the rays (Appendix A, steps 6 and 7) fused with the smooth
// field (Section 2.4, step 3) and, for maps, inverse-ray-shooting binning
// (Section 2.3).
//
// Grid rays: work unit = one chunk of up to 64*R rays of one leaf box of the target
// window, handled by one wave (a 64-thread workgroup):
//   * the stars of the box's 3x3 neighbourhood (three contiguous row ranges
//     of the sorted star array) and the box's local expansion are the same
//     for every lane, so they are read with wave-uniform scalar loads into
//     SGPRs and used directly as VALU operands -- every star is fetched once
//     per wave and shared by all 64*R rays;
//   * near field: alpha_near = sum m (x - x_i)/|x - x_i|^2 over those stars;
//     LENS_MIXED takes ray and star coordinates relative to the box centre
//     (FP64, rounded to FP32) and does the pair arithmetic in FP32;
//   * far field: f(z) = sum_l b~_l w^l, w = (z - c)/s, in FP64, by Horner or,
//     four mirror images to a lane, by sums that the four share;
//     alpha_far = conj(f);
//   * y = (1-kappa_s-gamma, 1-kappa_s+gamma) * x - alpha in FP64, written as
//     [n][2] or binned into the map: counts are summed in an LDS table
//     and added to the map by segments of pixels.
// Units are spread over a bounded grid; consecutive units (neighbouring
// boxes, which share stars) go to the same XCD so that they share its L2.
#include <algorithm>

#include "device_common.h"

namespace lensfmm {

namespace {

constexpr int kWave = 64;
constexpr int kXcd = 8;
constexpr int32_t kFlushStars = 128;  // LENS_MIXED near-field partials per FP64 flush
constexpr int kThreads = 256;  // explicit rays, helper kernels
constexpr int64_t kManyLanes = 1 << 18;  // half the lanes of k_eval_rays that the chip holds


// One star against the R rays of a lane.  The pair difference x - x_i is
// formed in FP64 from absolute coordinates (the star's are wave-uniform
// scalars), so it is exact to ~1e-16 of the coordinates however close the
// pair; LENS_MIXED rounds it once to FP32 and does the rest of the pair
// arithmetic in FP32, so every pair carries only a few FP32 roundings
// relative to its own size.  A coincident pair (dx = dy = 0) contributes
// exactly zero: the tiny term keeps its weight finite (for |m| below ~1e8 in
// FP32, ~1e108 in FP64) and it multiplies dx = dy = 0, so no branch or
// select is needed; it changes no pair farther apart than ~1e-13 (FP32).
//
// DERIV also accumulates f'(z) = -sum m / (z - z_i)^2: with dz = dx + i dy,
// 1/dz^2 = (dx^2 - dy^2 - 2i dx dy) / r^4, so f' gains -t (dx - dy)(dx + dy)
// (real) and 2 t dx dy (imaginary), t = m / r^4; a coincident pair has
// r2 = tiny exactly and gets t = 0.
template <bool MIXED, bool DERIV, int R, typename A, typename M>
__device__ __forceinline__ void pair_update(const double (&rx)[R], const double (&ry)[R], double sx,
                                            double sy, M mm, A (&ax)[R], A (&ay)[R],
                                            A (&dre)[R], A (&dim)[R]) {
  if constexpr (MIXED) {
    const float m = mm;  // the mass, rounded to FP32 when the stars were sorted
    constexpr float tiny = 0x1p-100f;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const float dx = (float)(rx[r] - sx);
      const float dy = (float)(ry[r] - sy);
      const float r2 = fmaf(dx, dx, fmaf(dy, dy, tiny));
      const float inv = rcp_f32(r2);
      const float w = m * inv;
      ax[r] = fmaf(w, dx, ax[r]);
      ay[r] = fmaf(w, dy, ay[r]);
      if constexpr (DERIV) {
        const float t = r2 > tiny ? w * inv : 0.0f;
        dre[r] = fmaf(-t, (dx - dy) * (dx + dy), dre[r]);
        dim[r] = fmaf(t + t, dx * dy, dim[r]);
      }
    }
  } else {
    constexpr double tiny = 0x1p-664;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const double dx = rx[r] - sx;
      const double dy = ry[r] - sy;
      const double r2 = fma(dx, dx, fma(dy, dy, tiny));
      const double inv = rcp_f64(r2);
      const double w = mm * inv;
      ax[r] = fma(w, dx, ax[r]);
      ay[r] = fma(w, dy, ay[r]);
      if constexpr (DERIV) {
        const double t = r2 > tiny ? w * inv : 0.0;
        dre[r] = fma(-t, (dx - dy) * (dx + dy), dre[r]);
        dim[r] = fma(t + t, dx * dy, dim[r]);
      }
    }
  }
}

// Map counts are first summed in a small per-wave table in LDS: kMapSegs rows of
// half a 64-byte segment of the map (8 pixels) each, two 16-bit counts to a word
// (open addressing by segment with four linear probes; a ray whose segment finds
// all probed rows taken goes straight to the global map).  At a unit's end, or
// when a pass leaves the table half full, they are added to the map by rows,
// eight lanes to one.  The map's atomics bound such calls where a box's image
// is wide: the memory side takes 23.7 requests per ns, and the lanes of an
// instruction within one segment make one.
constexpr int kSegBits = 3, kSegPixels = 1 << kSegBits;
constexpr int kMapSegBits = 7, kMapSegs = 1 << kMapSegBits;
constexpr int kMapPasses = 64;  // passes of at most 256 rays whose counts fit in 16 bits

struct MapTable {
  int32_t seg[kMapSegs];  // key / kSegPixels, or -1
  uint32_t val[kMapSegs * kSegPixels / 2];
  uint8_t used[kMapSegs];  // the rows in use, listed for the flush
};

__device__ __forceinline__ void map_table_clear(MapTable &t, int lane) {
  for (int e = lane; e < kMapSegs; e += kWave) t.seg[e] = -1;
  for (int e = lane; e < kMapSegs * kSegPixels / 2; e += kWave) t.val[e] = 0;
}

__device__ __forceinline__ void map_table_add(MapTable &t, int32_t key, int32_t *__restrict__ counts) {
  const int32_t seg = key >> kSegBits;
  uint32_t slot = ((uint32_t)seg * 2654435761u) >> (32 - kMapSegBits);
#pragma unroll
  for (int probe = 0; probe < 4; ++probe) {
    // a read first: the lanes share it, while their exchanges would queue
    int32_t have = *(volatile int32_t *)&t.seg[slot];
    if (have == -1) have = atomicCAS(&t.seg[slot], -1, seg);
    if (have == -1 || have == seg) {
      const uint32_t px = slot * kSegPixels + (key & (kSegPixels - 1));
      atomicAdd(&t.val[px >> 1], px & 1 ? 0x10000u : 1u);
      return;
    }
    slot = (slot + 1) & (kMapSegs - 1);
  }
  atomicAdd(&counts[key], 1);
}

// adds the counts to the map and clears them if more than `above` rows are used
__device__ __forceinline__ bool map_table_flush(MapTable &t, int above, int32_t *__restrict__ counts, int lane) {
  wave_sync();
  int n = 0;
  bool have[kMapSegs / kWave];
  uint64_t mask[kMapSegs / kWave];
#pragma unroll
  for (int q = 0; q < kMapSegs / kWave; ++q) {
    have[q] = t.seg[q * kWave + lane] >= 0;
    mask[q] = __ballot(have[q]);
    n += __popcll(mask[q]);
  }
  if (n <= above) return false;
  int base = 0;
#pragma unroll
  for (int q = 0; q < kMapSegs / kWave; ++q) {
    if (have[q]) t.used[base + __popcll(mask[q] & ((uint64_t(1) << lane) - 1))] = (uint8_t)(q * kWave + lane);
    base += __popcll(mask[q]);
  }
  wave_sync();
  for (int i = lane >> kSegBits; i < n; i += kWave >> kSegBits) {
    const int row = t.used[i], px = lane & (kSegPixels - 1), word = (row * kSegPixels + px) >> 1;
    const uint32_t two = t.val[word];
    const int32_t seg = t.seg[row];
    wave_sync();  // read by all, then cleared
    if (!(px & 1)) t.val[word] = 0;
    if (px == 0) t.seg[row] = -1;
    const uint32_t v = px & 1 ? two >> 16 : two & 0xffffu;
    if (v) atomicAdd(&counts[(seg << kSegBits) + px], (int32_t)v);
  }
  wave_sync();
  return true;
}

// QUAD: a lane's four rays are mirror images of each other in the centre lines
// of the box's rays (the expansion b is first moved to that centre, unless the two
// agree, in LENS_MIXED but for rounding), at w, -conj w, conj w and -w.  With
// z = w^2, f(w) = E(z) + w O(z) from the even and the odd coefficients, and
// P(z) = (c_0 - |z|^2 B_2) + z B_1 with the real recurrence
// B_k = c_k + 2 Re(z) B_k+1 - |z|^2 B_k+2 serves conj z as well: 4 p FMAs for the
// four rays where a Horner sum for each takes 16 p.  |z| <= 1/2, so the
// recurrence damps its roundings.  The pair sums gain too: the four rays have
// two columns and two rows, so a star costs them four differences, not eight.
// 1e6 stars, 8192^2 rays, p = 12: 343 to 256 million VALU instructions, 700 to
// 550 us.
constexpr double kSameCentre = 0x1p-50;  // LENS_MIXED

struct InverseInts {
  double v[LENS_MAX_ORDER + 1];
  constexpr InverseInts() : v{} {
    for (int i = 1; i <= LENS_MAX_ORDER; ++i) v[i] = 1.0 / i;
  }
};
__constant__ const InverseInts kInverse = InverseInts();

// b_k <- sum_m C(k+m, m) d^m b_k+m, a lane to a k; m runs while the largest
// C(p-1, m) |d|^m counts
__device__ __forceinline__ void shift_local(double2 *b, int p, cplx d, int lane) {
  const double size = fabs(d.re) + fabs(d.im);
  cplx t = {1.0, 0.0};
  double left = 1.0;
  double2 sum = lane < p ? b[lane] : make_double2(0.0, 0.0);
  for (int m = 1; m < p; ++m) {
    left *= size * (double)(p - m) * kInverse.v[m];
    if (left < 0x1p-60) break;
    const double up = (double)(lane + m) * kInverse.v[m];
    t = cplx{(t.re * d.re - t.im * d.im) * up, (t.re * d.im + t.im * d.re) * up};
    if (lane + m < p) {
      const double2 c = b[lane + m];
      sum.x += t.re * c.x - t.im * c.y;
      sum.y += t.re * c.y + t.im * c.x;
    }
  }
  wave_sync();
  if (lane < p) b[lane] = sum;
  wave_sync();
}

// P at z and conj z from B_1 and B_2 (n1, n2): (c0 + q n2) + z n1, q = -|z|^2
struct Conj {
  cplx at, cj;
};
__device__ __forceinline__ Conj quad_values(cplx z, double q, double2 c0, cplx n1, cplx n2) {
  const cplx m = {fma(z.re, n1.re, fma(q, n2.re, c0.x)), fma(z.re, n1.im, fma(q, n2.im, c0.y))};
  return {{fma(-z.im, n1.im, m.re), fma(z.im, n1.re, m.im)}, {fma(z.im, n1.im, m.re), fma(-z.im, n1.re, m.im)}};
}
__device__ __forceinline__ cplx quad_step(double r, double q, double2 c, cplx n1, cplx n2) {
  return {fma(r, n1.re, fma(q, n2.re, c.x)), fma(r, n1.im, fma(q, n2.im, c.y))};
}

// f (DERIV: and df/dw) at w, -conj w, conj w, -w; b[p] is 0.  The derivative
// needs P'(z) = B_1 + 2 i Im(z) Q(z), Q's coefficients being B_2, B_3, ...: the
// same recurrence once more.
template <bool DERIV>
__device__ __forceinline__ void quad_local(const double2 *b, int p, cplx w, cplx (&f)[4], cplx (&g)[4]) {
  const cplx z = {fma(w.re, w.re, -w.im * w.im), 2.0 * w.re * w.im};
  const double r = 2.0 * z.re, q = -fma(z.re, z.re, z.im * z.im);
  cplx e1 = {0.0, 0.0}, e2 = {0.0, 0.0}, o1 = {0.0, 0.0}, o2 = {0.0, 0.0};
  cplx c1 = {0.0, 0.0}, c2 = {0.0, 0.0}, d1 = {0.0, 0.0}, d2 = {0.0, 0.0};
#pragma unroll 2
  for (int k = (p - 1) >> 1; k >= 1; --k) {
    const cplx e = quad_step(r, q, b[2 * k], e1, e2), o = quad_step(r, q, b[2 * k + 1], o1, o2);
    if (DERIV && k >= 3) {
      const cplx c = quad_step(r, q, make_double2(e.re, e.im), c1, c2);
      const cplx d = quad_step(r, q, make_double2(o.re, o.im), d1, d2);
      c2 = c1;
      c1 = c;
      d2 = d1;
      d1 = d;
    }
    e2 = e1;
    e1 = e;
    o2 = o1;
    o1 = o;
  }
  const Conj E = quad_values(z, q, b[0], e1, e2), O = quad_values(z, q, b[1], o1, o2);
  const cplx wo = {fma(w.re, O.at.re, -w.im * O.at.im), fma(w.re, O.at.im, w.im * O.at.re)};
  const cplx wc = {fma(w.re, O.cj.re, w.im * O.cj.im), fma(w.re, O.cj.im, -w.im * O.cj.re)};
  f[0] = cplx{E.at.re + wo.re, E.at.im + wo.im};
  f[1] = cplx{E.cj.re - wc.re, E.cj.im - wc.im};
  f[2] = cplx{E.cj.re + wc.re, E.cj.im + wc.im};
  f[3] = cplx{E.at.re - wo.re, E.at.im - wo.im};
  if constexpr (DERIV) {
    // f' = (O + 2 z O') +- 2 w E'
    const Conj C = quad_values(z, q, make_double2(e2.re, e2.im), c1, c2);
    const Conj D = quad_values(z, q, make_double2(o2.re, o2.im), d1, d2);
    const double t = 2.0 * z.im;
    const cplx ea = {fma(-t, C.at.im, e1.re), fma(t, C.at.re, e1.im)};
    const cplx ec = {fma(t, C.cj.im, e1.re), fma(-t, C.cj.re, e1.im)};
    const cplx oa = {fma(-t, D.at.im, o1.re), fma(t, D.at.re, o1.im)};
    const cplx oc = {fma(t, D.cj.im, o1.re), fma(-t, D.cj.re, o1.im)};
    const cplx sa = {fma(r, oa.re, fma(-t, oa.im, O.at.re)), fma(r, oa.im, fma(t, oa.re, O.at.im))};
    const cplx sc = {fma(r, oc.re, fma(t, oc.im, O.cj.re)), fma(r, oc.im, fma(-t, oc.re, O.cj.im))};
    const double u = 2.0 * w.re, v = 2.0 * w.im;
    const cplx ua = {fma(u, ea.re, -v * ea.im), fma(u, ea.im, v * ea.re)};
    const cplx uc = {fma(u, ec.re, v * ec.im), fma(u, ec.im, -v * ec.re)};
    g[0] = cplx{sa.re + ua.re, sa.im + ua.im};
    g[1] = cplx{sc.re - uc.re, sc.im - uc.im};
    g[2] = cplx{sc.re + uc.re, sc.im + uc.im};
    g[3] = cplx{sa.re - ua.re, sa.im - ua.im};
  }
}

// The mixed kernels are compiled for five waves per SIMD (at most 96 VGPRs;
// the R = 4 instances spill a few bytes of per-lane scratch outside the pair
// loop), which measured faster than four waves without spills.
template <int PMAX, bool MIXED, bool MAP, int R, bool DERIV, bool QUAD>
__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(MIXED && !DERIV ? 5 : 1))) void k_eval(EvalArgs a, const double *__restrict__ loc,
                                                const double *__restrict__ sxy,
                                                const double *__restrict__ sm,
                                                const float *__restrict__ sm32,
                                                const int32_t *__restrict__ leaf_start,
                                                const int32_t *__restrict__ col_start,
                                                const int32_t *__restrict__ row_start,
                                                double *__restrict__ y_out,
                                                int32_t *__restrict__ counts) {
  // the box's local expansion, read by every lane (LDS broadcast)
  __shared__ double2 lds_loc[PMAX + 1];
  // LENS_MIXED: FP64 sums of the lanes' FP32 near-field partials, flushed
  // every kFlushStars stars (alpha; f' with DERIV)
  __shared__ double2 lds_acc[MIXED ? kWave * R * (DERIV ? 2 : 1) : 1];
  __shared__ typename std::conditional<MAP, MapTable, int>::type table;
  const int lane = threadIdx.x;
  if constexpr (MAP) map_table_clear(table, lane);
  // unit counts fit in 31 bits (checked at launch)
  const uint32_t CH = (uint32_t)(QUAD ? a.quad_chunks : a.chunks_per_box);
  const uint32_t nbx = (uint32_t)a.win.nbx;
  const uint32_t nunits = (uint32_t)(a.win.count() * CH);
  // XCD-aware virtual block id: blocks dispatched to one XCD (blockIdx % 8)
  // take a contiguous range of units in each sweep of the grid.
  const uint32_t G = gridDim.x;
  const uint32_t per_xcd = G / kXcd;
  const uint32_t vb = (G % kXcd == 0) ? (blockIdx.x % kXcd) * per_xcd + blockIdx.x / kXcd : blockIdx.x;
  const int64_t nL = int64_t(1) << a.g.L;
  const double s = ldexp(a.g.side, -a.g.L);
  const double inv_s = 1.0 / s;
  const int p = a.p;
  // a wave's R slots are R tiles of TX x TY rays (TX * TY = 64)
  const int tsh = QUAD ? a.quad_shift : a.tile_shift;
  const int TX = 1 << tsh, TY = kWave >> tsh;
  const int lx = lane & (TX - 1), ly = lane >> tsh;

  for (uint32_t u = vb; u < nunits; u += G) {
    const uint32_t b = CH == 1 ? u : u / CH;
    const uint32_t c0 = u - b * CH;
    const uint32_t byw = b / nbx, bxw = b - byw * nbx;
    const int64_t gx = a.win.bx0 + bxw, gy = a.win.by0 + byw;

    // the box's rays are columns [i0, i0+W) x rows [j0, j0+H); they (QUAD: the
    // quarter at the low corner) are cut into nt = TW x TH tiles, tpc
    // consecutive tiles per unit.  QUAD: all rows of the box in the grid, of
    // which those of the band [j_begin, j_end) are evaluated, so that a ray's
    // bits don't depend on the bands that a call is cut into.
    const int32_t i0 = col_start[bxw], W = col_start[bxw + 1] - i0;
    const int32_t j0 = row_start[byw], H = row_start[byw + 1] - j0;
    const int32_t Wt = QUAD ? (W + 1) >> 1 : W;
    int32_t qa = 0, Ht = QUAD ? (H + 1) >> 1 : H;  // the rows [qa, Ht) hold tiles
    bool cut = false;
    if (QUAD) {
      const int32_t ja = (int32_t)max(a.j_begin - j0, (int64_t)0), jb = (int32_t)min(a.j_end - j0, (int64_t)H);
      cut = ja > 0 || jb < H;
      if (cut) {  // the band's rows [ja, jb) of the quarter, and their images
        const int32_t half = Ht;
        const int32_t lo1 = ja, hi1 = min(jb, half), lo2 = max(H - jb, 0), hi2 = min(H - ja, half);
        qa = min(lo1 < hi1 ? lo1 : half, lo2 < hi2 ? lo2 : half);
        Ht = max(lo1 < hi1 ? hi1 : 0, lo2 < hi2 ? hi2 : 0);
      }
    }
    const int32_t TW = (Wt + TX - 1) >> tsh;
    const int32_t nt = Ht > qa ? TW * ((Ht - qa + TY - 1) / TY) : 0;
    const int32_t tpc = (nt + (int32_t)CH - 1) / (int32_t)CH;
    if (nt == 0 || (int64_t)c0 * tpc >= nt) continue;  // uniform

    int32_t rs[3], re[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const int64_t row = gy - 1 + d;
      rs[d] = 0;
      re[d] = 0;
      if (row >= 0 && row < nL) {
        const int64_t cx0 = gx > 0 ? gx - 1 : 0;
        const int64_t cx1 = gx + 1 < nL ? gx + 1 : nL - 1;
        rs[d] = leaf_start[row * nL + cx0];
        re[d] = leaf_start[row * nL + cx1 + 1];
      }
    }
    const double cx = a.g.x0 + ((double)gx + 0.5) * s;
    const double cy = a.g.y0 + ((double)gy + 0.5) * s;
    wave_sync();  // the previous unit's reads of lds_loc are done
    if (lane < p) lds_loc[lane] = reinterpret_cast<const double2 *>(loc + 2 * (int64_t)b * p)[lane];
    if (QUAD && lane == p) lds_loc[p] = make_double2(0.0, 0.0);
    wave_sync();
    if constexpr (QUAD) {
      // the expansion about the centre of the box's rays
      const double ccx = 0.5 * (grid_coord(a.grid.x0, a.grid.dx, i0) + grid_coord(a.grid.x0, a.grid.dx, i0 + W - 1));
      const double ccy = 0.5 * (grid_coord(a.grid.y0, a.grid.dy, j0) + grid_coord(a.grid.y0, a.grid.dy, j0 + H - 1));
      constexpr double same = MIXED ? kSameCentre : 0.0;
      if (fabs(ccx - cx) > same * fabs(cx) || fabs(ccy - cy) > same * fabs(cy))
        shift_local(lds_loc, p, cplx{(ccx - cx) * inv_s, (ccy - cy) * inv_s}, lane);
    }

    // passes of R tiles, or of one tile and its three mirror images
    const int32_t pend = min(nt, (int32_t)c0 * tpc + tpc);
    int held = 0;  // passes whose counts the table holds
    for (int32_t pos = (int32_t)c0 * tpc; pos < pend; pos += QUAD ? 1 : R) {
      // slot r's column and row in the box (an inactive slot takes tile place
      // 0, 0); QUAD: r & 1 mirrors the column, r & 2 the row, and the middle
      // column or row of an odd box is its own image
      auto place = [&](int r, int32_t &ci, int32_t &cj) -> bool {
        const int32_t t = QUAD ? pos : pos + r;  // wave-uniform tile index
        const int32_t ty = t / TW, tx = t - ty * TW;
        ci = tx * TX + lx;
        cj = qa + ty * TY + ly;
        bool on = t < pend && ci < Wt && cj < Ht;
        ci = on ? ci : 0;
        cj = on ? cj : 0;
        if (QUAD && (r & 1)) {
          on = on && 2 * ci + 1 != W;
          ci = W - 1 - ci;
        }
        if (QUAD && (r & 2)) {
          on = on && 2 * cj + 1 != H;
          cj = H - 1 - cj;
        }
        return QUAD ? on && j0 + cj >= a.j_begin && j0 + cj < a.j_end : on;
      };
      if (QUAD && cut) {  // nothing of this tile in the band (uniform)
        bool any = false;
#pragma unroll
        for (int r = 0; r < R; ++r) {
          int32_t ci, cj;
          any = place(r, ci, cj) || any;
        }
        if (!__any(any)) continue;
      }
      double rx[R], ry[R];
      using acc_t = typename std::conditional<MIXED, float, double>::type;
      acc_t ax[R], ay[R], dre[R], dim[R];
      int64_t oidx[R];
      bool act[R];
#pragma unroll
      for (int r = 0; r < R; ++r) {
        // its output index is formed after the pair loop
        int32_t ci, cj;
        (void)place(r, ci, cj);
        rx[r] = grid_coord(a.grid.x0, a.grid.dx, i0 + ci);
        ry[r] = grid_coord(a.grid.y0, a.grid.dy, j0 + cj);
        ax[r] = 0;
        ay[r] = 0;
        dre[r] = 0;
        dim[r] = 0;
      }

      // LENS_MIXED reads the masses' FP32 copies (no conversion per star)
      using mass_t = typename std::conditional<MIXED, float, double>::type;
      auto mass = [&](int32_t i) -> mass_t {
        if constexpr (MIXED) return sm32[i]; else return sm[i];
      };
      auto star = [&](double x, double y, mass_t m) {
        pair_update<MIXED, DERIV, R>(rx, ry, x, y, m, ax, ay, dre, dim);
      };
      // LENS_MIXED: every kFlushStars stars the FP32 partial sums move into
      // FP64 ones in LDS (a wave-uniform count), so a ray with thousands
      // of near stars (a cluster's core) does not accumulate thousands of
      // FP32 roundings; a box of fewer stars never flushes
      int32_t since = 0;
      bool flushed = false;
      auto flush = [&]() {
        if constexpr (MIXED) {
#pragma unroll
          for (int r = 0; r < R; ++r) {
            double2 &acc = lds_acc[r * kWave + lane];
            const double2 old = flushed ? acc : make_double2(0.0, 0.0);
            acc = make_double2(old.x + (double)ax[r], old.y + (double)ay[r]);
            ax[r] = 0;
            ay[r] = 0;
            if (DERIV) {
              double2 &acd = lds_acc[(R + r) * kWave + lane];
              const double2 od = flushed ? acd : make_double2(0.0, 0.0);
              acd = make_double2(od.x + (double)dre[r], od.y + (double)dim[r]);
              dre[r] = 0;
              dim[r] = 0;
            }
          }
          flushed = true;
          since = 0;
        }
      };
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        int32_t i = rs[d];
        // four stars per step: their scalar loads issue together
        for (; i + 4 <= re[d]; i += 4) {
          double sx[4], sy[4];
          mass_t mm[4];
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            sx[q] = sxy[2 * (int64_t)(i + q)];
            sy[q] = sxy[2 * (int64_t)(i + q) + 1];
            mm[q] = mass(i + q);
          }
#pragma unroll
          for (int q = 0; q < 4; ++q) star(sx[q], sy[q], mm[q]);
          if (MIXED) {
            since += 4;
            if (since >= kFlushStars) flush();
          }
        }
        for (; i < re[d]; ++i) star(sxy[2 * (int64_t)i], sxy[2 * (int64_t)i + 1], mass(i));
      }

      // ray offsets from the box centre (FP64) for the far field; grid rays'
      // output indices and activity recomputed from the lane's tile position
      // (integers) rather than kept live through the pair loop
      double dxr[R], dyr[R];
#pragma unroll
      for (int r = 0; r < R; ++r) {
        dxr[r] = rx[r] - cx;
        dyr[r] = ry[r] - cy;
      }
#pragma unroll
      for (int r = 0; r < R; ++r) {
        int32_t ci, cj;
        act[r] = place(r, ci, cj);
        oidx[r] = (int64_t)(j0 + cj) * a.grid.nx + (i0 + ci);
      }
      cplx f[R], gd[R];
      if constexpr (QUAD) {
        // half the distances to the images: w of slot 0; slots 1..3 are
        // -conj(w), conj(w), -w
        quad_local<DERIV>(lds_loc, p, cplx{0.5 * (rx[0] - rx[1]) * inv_s, 0.5 * (ry[0] - ry[2]) * inv_s}, f, gd);
      } else {
      // far field: Horner over the R rays from the top coefficient down, one
      // LDS read per coefficient
      // (DERIV: the derivative sum g = sum l b_l w^(l-1) in the same sweep,
      // g <- g w + f before f <- f w + b_l; f' = g / s)
      cplx w[R];
      {
        const double2 top = lds_loc[p - 1];
#pragma unroll
        for (int r = 0; r < R; ++r) {
          w[r] = cplx{dxr[r] * inv_s, dyr[r] * inv_s};
          f[r] = cplx{top.x, top.y};
          gd[r] = cplx{0.0, 0.0};
        }
      }
      // a runtime trip count (the order-guarded unrolled form keeps one
      // spilled branch mask per level)
#pragma unroll 2
      for (int l = p - 2; l >= 0; --l) {
        const double2 c = lds_loc[l];
#pragma unroll
        for (int r = 0; r < R; ++r) {
          if (DERIV) gd[r] = cmad(gd[r], w[r], f[r]);
          f[r] = cmad(f[r], w[r], cplx{c.x, c.y});
        }
      }

      }
      int32_t key[R];
#pragma unroll
      for (int r = 0; r < R; ++r) {
        // the FP64 near-field sum: the FP32 partial plus, where a flush
        // happened, the flushed ones
        double nx = (double)ax[r], ny = (double)ay[r];
        if (MIXED && flushed) {
          const double2 acc = lds_acc[r * kWave + lane];
          nx += acc.x;
          ny += acc.y;
        }
        const double al1 = f[r].re + nx;
        const double al2 = ny - f[r].im;
        const double y1 = a.c1 * rx[r] - al1;
        const double y2 = a.c2 * ry[r] - al2;
        if (MAP) {
          key[r] = -1;
          const double t1 = (y1 - a.y1min) * a.S;
          const double t2 = (y2 - a.y2min) * a.S;
          if (act[r] && t1 >= 0.0 && t2 >= 0.0) {
            const double f1 = floor(t1), f2 = floor(t2);
            if (f1 < (double)a.npix && f2 < (double)a.npix)
              key[r] = (int32_t)f2 * a.npix + (int32_t)f1;
          }
        } else if (act[r]) {
          *reinterpret_cast<double2 *>(y_out + 2 * oidx[r]) = make_double2(y1, y2);
          if (DERIV) {
            double nre = (double)dre[r], nim = (double)dim[r];
            if (MIXED && flushed) {
              const double2 acd = lds_acc[(R + r) * kWave + lane];
              nre += acd.x;
              nim += acd.y;
            }
            *reinterpret_cast<double2 *>(a.dfdz_out + 2 * oidx[r]) =
                make_double2(fma(gd[r].re, inv_s, nre), fma(gd[r].im, inv_s, nim));
          }
        }
      }
      if constexpr (MAP) {
#pragma unroll
        for (int r = 0; r < R; ++r)
          if (key[r] >= 0) map_table_add(table, key[r], counts);
        ++held;
        if (pos + (QUAD ? 1 : R) < pend && map_table_flush(table, held < kMapPasses ? kMapSegs / 2 : 0, counts, lane))
          held = 0;
      }
    }
    if constexpr (MAP) (void)map_table_flush(table, 0, counts, lane);
  }
}

// Explicit rays, SPLIT lanes to a ray and neighbouring rays (sorted by leaf box)
// in neighbouring lanes, each with its own box's locals and stars, so that no lane
// is idle where boxes hold few rays, and none waits where some hold many.  Bound
// by the stars' loads, of which a lane keeps four in flight behind the four that
// it works on.  The stars of a ray's neighbourhood are summed in groups, each by
// one lane, and the groups' sums are added in FP64 in their order, so that a ray's
// bits do not depend on SPLIT.  A group ends where k_eval moves its FP32 sums:
// with the 32nd whole step of four stars (steps do not reach over a row's end), in
// FP64 with the 64th.  Whole calls, mixed, a wave to a box before, now: 1e3 stars
// and 1e6 rays 1249, 153 us; 1e4 and 1e5 119, 119; 1e5 and 1e6 225, 200; 1e6 and
// 1e5 406, 290; 1e3 stars and 1e3 rays, one chain's latency, 72, 76 (as much as
// the sort's box starts, which only the other form needed, took).
template <bool MIXED, bool DERIV, int SPLIT>
__global__ __launch_bounds__(kThreads) void k_eval_rays(EvalArgs a, int64_t n, const double2 *__restrict__ loc,
                                                        const double2 *__restrict__ sz,
                                                        const double *__restrict__ sm,
                                                        const float *__restrict__ sm32,
                                                        const int32_t *__restrict__ leaf_start,
                                                        const double2 *__restrict__ rxy,
                                                        const uint32_t *__restrict__ rperm,
                                                        double2 *__restrict__ y_out) {
  using acc_t = typename std::conditional<MIXED, float, double>::type;
  constexpr int32_t kSteps = (MIXED ? kFlushStars : 2 * kFlushStars) / 4;
  const int64_t gid = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  const int part = (int)(gid % SPLIT);
  const bool act = gid / SPLIT < n;
  const int64_t t = act ? gid / SPLIT : n - 1;
  const int64_t nL = int64_t(1) << a.g.L;
  const double s = ldexp(a.g.side, -a.g.L);
  const double inv_s = 1.0 / s;
  const double2 z = rxy[t];
  // the ray's box, in the window (as the rays' sort places them)
  int64_t ix = box_coord(z.x, a.g.x0, s, nL) - a.win.bx0;
  int64_t iy = box_coord(z.y, a.g.y0, s, nL) - a.win.by0;
  ix = ix < 0 ? 0 : (ix >= a.win.nbx ? a.win.nbx - 1 : ix);
  iy = iy < 0 ? 0 : (iy >= a.win.nby ? a.win.nby - 1 : iy);
  const int64_t gx = a.win.bx0 + ix, gy = a.win.by0 + iy;
  // star ranges of the three rows, and their running totals
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
  const int32_t ns = pre[3];
  // whole steps up to the end of each row, and the last group
  const int32_t w1 = pre[1] >> 2, w2 = w1 + ((pre[2] - pre[1]) >> 2), w3 = w2 + ((ns - pre[2]) >> 2);
  const int32_t last = w3 / kSteps;
  // group g's first star (a place in the three rows together)
  auto first = [&](int32_t g) -> uint32_t {
    const int32_t w = g * kSteps;  // the whole steps before it
    if (w == 0) return 0u;
    return 4u * (uint32_t)w + (w > w2 ? pre[2] - 4 * w2 : (w > w1 ? pre[1] - 4 * w1 : 0));
  };
  const double rx[1] = {z.x}, ry[1] = {z.y};
  double Sx = 0.0, Sy = 0.0, Tr = 0.0, Ti = 0.0;
  for (int32_t g0 = 0; g0 <= last; g0 += SPLIT) {
    const int32_t g = g0 + part;
    acc_t ax[1] = {0}, ay[1] = {0}, dre[1] = {0}, dim[1] = {0};
    uint32_t k = g <= last ? first(g) : 0u;
    const uint32_t end = g < last ? first(g + 1) : (g == last ? (uint32_t)ns : 0u);
    double2 nz[4];
    acc_t nm[4];
    auto fetch = [&](uint32_t q0) {
#pragma unroll
      for (uint32_t j = 0; j < 4; ++j) {
        const int32_t q = (int32_t)min(q0 + j, end - 1);
        const int32_t i = q >= pre[2] ? rs[2] + (q - pre[2]) : (q >= pre[1] ? rs[1] + (q - pre[1]) : rs[0] + q);
        nz[j] = sz[i];
        if constexpr (MIXED) nm[j] = sm32[i]; else nm[j] = sm[i];
      }
    };
    if (k < end) fetch(k);
    for (; k < end; k += 4) {
      double2 cz[4];
      acc_t cm[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) cz[j] = nz[j], cm[j] = nm[j];
      fetch(k + 4);
#pragma unroll
      for (uint32_t j = 0; j < 4; ++j)
        if (k + j < end) pair_update<MIXED, DERIV, 1>(rx, ry, cz[j].x, cz[j].y, cm[j], ax, ay, dre, dim);
    }
    if (SPLIT == 1 || last == 0) {  // (one group: lane 0's)
      Sx += (double)ax[0];
      Sy += (double)ay[0];
      if (DERIV) {
        Tr += (double)dre[0];
        Ti += (double)dim[0];
      }
    } else {  // the lanes of a ray go round together
#pragma unroll
      for (int q = 0; q < SPLIT; ++q) {
        Sx += (double)__shfl(ax[0], q, SPLIT);
        Sy += (double)__shfl(ay[0], q, SPLIT);
        if (DERIV) {
          Tr += (double)__shfl(dre[0], q, SPLIT);
          Ti += (double)__shfl(dim[0], q, SPLIT);
        }
      }
    }
  }
  // far field: Horner, with the derivative's sum in the same sweep
  const double2 *lb = loc + (iy * a.win.nbx + ix) * a.p;
  const cplx w = {(z.x - (a.g.x0 + ((double)gx + 0.5) * s)) * inv_s,
                  (z.y - (a.g.y0 + ((double)gy + 0.5) * s)) * inv_s};
  cplx f = {lb[a.p - 1].x, lb[a.p - 1].y}, gd = {0.0, 0.0};
#pragma unroll 4
  for (int l = a.p - 2; l >= 0; --l) {
    const double2 c = lb[l];
    if (DERIV) gd = cmad(gd, w, f);
    f = cmad(f, w, cplx{c.x, c.y});
  }
  if (!act || part != 0) return;
  const int64_t o = rperm[t];
  y_out[o] = make_double2(a.c1 * z.x - (f.re + Sx), a.c2 * z.y - (Sy - f.im));
  if (DERIV)
    reinterpret_cast<double2 *>(a.dfdz_out)[o] =
        make_double2(fma(gd.re, inv_s, Tr), fma(gd.im, inv_s, Ti));
}

// first ray column (row) of every box column (row) of the window: columns in
// blockIdx.y = 0, rows in blockIdx.y = 1 (one launch)
struct GridAxis {
  double x0, dx;       // grid origin and step along the axis
  int64_t lo_i, hi_i;  // ray index range searched
  double origin;       // root square origin along the axis
  int64_t b0, nb;      // first window box and window size along the axis
  int32_t *out;        // [nb + 1]
};

__global__ __launch_bounds__(kThreads) void k_grid_ranges(GridAxis ax, GridAxis ay, double s,
                                                          int64_t nL) {
  const GridAxis &a = blockIdx.y == 0 ? ax : ay;
  const int64_t c = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (c > a.nb) return;
  const int64_t B = a.b0 + c;
  int64_t lo = a.lo_i, hi = a.hi_i;
  while (lo < hi) {
    const int64_t mid = (lo + hi) >> 1;
    if (box_coord(grid_coord(a.x0, a.dx, mid), a.origin, s, nL) < B)
      lo = mid + 1;
    else
      hi = mid;
  }
  a.out[c] = (int32_t)lo;
}

constexpr int64_t kMaxEvalBlocks = 256 * 32 * 4;  // CUs x waves per CU x sweeps in flight

template <int PM, bool MIXED, bool MAP, int R, bool DERIV = false, bool QUAD = false>
void eval_launch_r(const EvalArgs &a, hipStream_t stream) {
  const int64_t units = a.win.count() * (QUAD ? a.quad_chunks : a.chunks_per_box);
  int64_t nblk = units < kMaxEvalBlocks ? units : kMaxEvalBlocks;
  if (nblk > kXcd) nblk = nblk / kXcd * kXcd;
  hipLaunchKernelGGL((k_eval<PM, MIXED, MAP, R, DERIV, QUAD>), dim3((unsigned)nblk), dim3(kWave), 0, stream,
                     a, a.loc, a.sxy, a.sm, a.sm32, a.leaf_start, a.col_start, a.row_start, a.y_out,
                     a.counts);
}

template <int PM, bool MIXED, bool MAP>
void eval_launch(const EvalArgs &a, hipStream_t stream) {
  if constexpr (!MAP) {
    // f' wanted: one instance of either form per order bucket, two rays per
    // lane where they are not mirror images
    if (a.dfdz_out) {
      if (a.quad_chunks)
        eval_launch_r<PM, MIXED, MAP, 4, true, true>(a, stream);
      else
        eval_launch_r<PM, MIXED, MAP, 2, true>(a, stream);
      return;
    }
  }
  if (a.quad_chunks) {
    eval_launch_r<PM, MIXED, MAP, 4, false, true>(a, stream);
    return;
  }
  switch (a.rays_per_lane) {
    case 1: eval_launch_r<PM, MIXED, MAP, 1>(a, stream); break;
    case 2: eval_launch_r<PM, MIXED, MAP, 2>(a, stream); break;
    case 3: eval_launch_r<PM, MIXED, MAP, 3>(a, stream); break;
    default: eval_launch_r<PM, MIXED, MAP, 4>(a, stream); break;
  }
}

template <int PM>
void eval_dispatch(const EvalArgs &a, int precision, hipStream_t stream) {
  const bool mixed = precision == LENS_MIXED, map = a.counts != nullptr;
  if (mixed) {
    if (map) eval_launch<PM, true, true>(a, stream);
    else eval_launch<PM, true, false>(a, stream);
  } else {
    if (map) eval_launch<PM, false, true>(a, stream);
    else eval_launch<PM, false, false>(a, stream);
  }
}

}  // namespace

// Rays per lane R and units per box CH for boxes of at most max_rays rays:
// the fewest lane slots 64*R*passes*CH, ties going to the larger R, with up
// to kPassesPerUnit passes of 64*R rays per unit.  A unit starts by loading
// its box's local expansion with a vector load, which waits for every
// earlier vector memory operation of the wave (the previous unit's stores or
// map atomics); several passes per unit spread that wait.
constexpr int64_t kPassesPerUnit = 8;

void eval_shape(int64_t max_rays, int *R, int64_t *CH) {
  int best_r = 1;
  int64_t best_ch = 1, best_slots = -1;
  for (int r = 1; r <= 4; ++r) {
    const int64_t passes = (max_rays + kWave * r - 1) / (kWave * r);
    const int64_t ch = (passes + kPassesPerUnit - 1) / kPassesPerUnit;
    const int64_t per = (passes + ch - 1) / ch;
    const int64_t slots = ch * per * kWave * r;
    if (best_slots < 0 || slots <= best_slots) {
      best_slots = slots;
      best_r = r;
      best_ch = ch < 1 ? 1 : ch;
    }
  }
  *R = best_r;
  *CH = best_ch;
}

// Tile shape for grid rays in boxes of at most W x H rays: TX = 2^shift
// columns by 64/TX rows, the fewest tiles per box, ties going to the
// squarest tile (rays of a square tile land close together in a map).
void grid_tile_shape(int64_t W, int64_t H, int *shift, int64_t *tiles) {
  int best = 3;
  int64_t best_t = -1;
  for (int sh : {3, 2, 4, 1, 5, 0, 6}) {
    const int64_t tx = int64_t(1) << sh, ty = kWave / tx;
    const int64_t t = ((W + tx - 1) / tx) * ((H + ty - 1) / ty);
    if (best_t < 0 || t < best_t) {
      best_t = t;
      best = sh;
    }
  }
  *shift = best;
  *tiles = best_t;
}

// Four mirror images to a lane where the slots of its units, filled or not, in a
// box of W x H rays are at most 1.15 times the ordinary form's (the units are shaped
// for at most Wmax x Hmax rays), unless the quarter makes two short units of 9 to 12
// passes.  Speed of the mirrored form over the ordinary one, p = 4 to 24, 1 to 20
// stars a box, 1024 to 16384 boxes (y in mixed precision | in FP64 | y and f' in
// either): ratio 1 (boxes of 16^2, 32^2, 63^2 rays) 1.0 to 1.3 | 1.0 to 1.15 | 0.9 to
// 1.2; 1.04 to 1.14 (49^2, 56^2, 100^2) 0.95 to 1.6 | 0.9 to 1.5 | 0.8 to 1.4; 1.33
// (24^2, 65^2) 0.94 to 1.36 | 0.83 to 1.2 | 0.83 to 1.2; 1.43 (33^2 to 36^2) 1.0 to
// 1.1 | 0.84 to 1.06 | 0.76 to 1.06; two short units (48^2) 0.94 to 1.06 | 0.86 to
// 0.94 | 0.7 to 0.9.
bool quad_shape(int64_t W, int64_t H, int64_t Wmax, int64_t Hmax, int64_t rows, int *shift, int64_t *CH) {
  auto up = [](int64_t a, int64_t b) { return (a + b - 1) / b; };
  auto tiles_of = [&](int64_t w, int64_t h) { return up(w, int64_t(1) << *shift) * up(h, kWave >> *shift); };
  int64_t most = 0, ch = 0;
  int R = 0;
  grid_tile_shape(Wmax, Hmax, shift, &most);
  eval_shape(most * kWave, &R, &ch);
  const int64_t ordinary = ch * up(up(tiles_of(W, H), ch), R) * R;
  grid_tile_shape((Wmax + 1) / 2, (Hmax + 1) / 2, shift, &most);
  const int64_t quarter = tiles_of((W + 1) / 2, (H + 1) / 2);
  ch = up(most, kPassesPerUnit);
  const int64_t mirrored = 4 * ch * up(quarter, ch);
  const bool use = 100 * mirrored <= 115 * ordinary && !(quarter > 8 && quarter <= 12);
  grid_tile_shape((Wmax + 1) / 2, std::min((Hmax + 1) / 2, rows), shift, &most);
  *CH = up(most, kPassesPerUnit);
  return use;
}

void launch_eval(const EvalArgs &a, int precision, hipStream_t stream) {
  if (a.win.count() == 0) return;
  if (precision == LENS_MIXED && !a.sm32)
    fail(LENS_EINVAL, "mixed-precision evaluation needs the plan's FP32 masses");
  LENS_PMAX_DISPATCH(a.p, eval_dispatch<PM>(a, precision, stream));
  LENS_HIP(hipGetLastError());
}

template <bool MIXED, int SPLIT>
void eval_rays(const EvalArgs &a, int64_t n, hipStream_t stream) {
  auto *kernel = a.dfdz_out ? k_eval_rays<MIXED, true, SPLIT> : k_eval_rays<MIXED, false, SPLIT>;
  hipLaunchKernelGGL(kernel, dim3((unsigned)((n * SPLIT + kThreads - 1) / kThreads)), dim3(kThreads), 0, stream,
                     a, n, reinterpret_cast<const double2 *>(a.loc), reinterpret_cast<const double2 *>(a.sxy),
                     a.sm, a.sm32, a.leaf_start, reinterpret_cast<const double2 *>(a.rxy), a.rperm,
                     reinterpret_cast<double2 *>(a.y_out));
}

// Lanes to a ray: as many as fill half of the chip with few rays, whose longest
// chain of stars is all that counts then (five clusters of 2e5 stars, mixed: 300
// rays 4.8 ms with one lane, 0.6 with sixteen; 30000 rays 4.8 ms with one, 1.3 with
// four, 0.9 with sixteen).  More rays would pay for the far field that a ray's lanes
// all sum: 30000 rays on 1e4 uniform stars in FP64 104 us with four lanes, 119 with
// sixteen; 1e5 rays on 1e5 stars 132 with one, 155 with four.  Few stars make no
// long chain, and a wave of fewer rays waits for more of their loads (1e3 rays on
// 1e3 stars in FP64 78 us with one lane, 84 with sixteen).
constexpr int64_t kManyStars = 2048;

template <bool MIXED>
void eval_rays_dispatch(const EvalArgs &a, int64_t n, int64_t n_stars, hipStream_t stream) {
  if (n_stars > kManyStars && n <= kManyLanes / 32)
    eval_rays<MIXED, 16>(a, n, stream);
  else if (n_stars > kManyStars && n <= kManyLanes / 4)
    eval_rays<MIXED, 4>(a, n, stream);
  else
    eval_rays<MIXED, 1>(a, n, stream);
}

void launch_eval_rays(const EvalArgs &a, int64_t n, int64_t n_stars, int precision, hipStream_t stream) {
  if (n == 0) return;
  if (precision == LENS_MIXED && !a.sm32)
    fail(LENS_EINVAL, "mixed-precision evaluation needs the plan's FP32 masses");
  if (precision == LENS_MIXED)
    eval_rays_dispatch<true>(a, n, n_stars, stream);
  else
    eval_rays_dispatch<false>(a, n, n_stars, stream);
  LENS_HIP(hipGetLastError());
}

void launch_grid_ranges(const lens_grid &grid, Geometry g, Window win, int64_t j_begin,
                        int64_t j_end, int32_t *col_start, int32_t *row_start,
                        hipStream_t stream) {
  const int64_t nL = int64_t(1) << g.L;
  const double s = ldexp(g.side, -g.L);
  const GridAxis ax{grid.x0, grid.dx, 0, grid.nx, g.x0, win.bx0, win.nbx, col_start};
  const GridAxis ay{grid.y0, grid.dy, j_begin, j_end, g.y0, win.by0, win.nby, row_start};
  const int64_t nmax = std::max(win.nbx, win.nby) + 1;
  hipLaunchKernelGGL(k_grid_ranges, dim3((unsigned)((nmax + kThreads - 1) / kThreads), 2),
                     dim3(kThreads), 0, stream, ax, ay, s, nL);
  LENS_HIP(hipGetLastError());
}

}  // namespace lensfmm
