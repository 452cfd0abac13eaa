// Upward pass (Appendix A, upward passes 1 and 2): P2M forms the order-p
// multipole of every leaf box from its sources (stars with real masses, or
// rays with complex charges for the adjoint); M2M shifts the four children's
// multipoles to their parent's centre toward the root.  Levels whose boxes
// hold a few sources on average, and the windowed fine levels, are formed
// straight from the stars (a star then enters several expansions), which
// replaces the largest M2M sweeps with passes over the stars; the coarser
// dense levels come from M2M, up to four levels per launch.  Everything runs
// in FP64.
//
// Coefficients are box-size rescaled: a~_k = sum_{i in box} m_i w_i^k,
// w_i = (z_i - c)/s, stored box-major as [box][p] complex (re, im).
#include <algorithm>
#include <type_traits>

#include "device_common.h"

namespace lensfmm {

namespace {

constexpr int kThreads = 256;
constexpr int kWave = 64;

typedef double d4v __attribute__((ext_vector_type(4)));

// Group-cooperative P2M of one box by GL neighbouring lanes of a wave (every
// lane of the group calls with the same box; `on` false: an empty box).  The
// box at `level` covers 2^(L-level) rows of leaf boxes, each a contiguous
// range of the sorted sources: they are taken GL rows at a time, their source
// counts scanned across the group so that its lanes share the sources evenly
// (lane t takes sources t, t + GL, ... of the concatenated rows), each lane
// accumulating all p coefficients with running powers m w^k into v (re, im
// interleaved), the next source's loads issued before the current powers.
template <int PMAX, int QDIM, int GL>
__device__ __forceinline__ void p2m_group_sum(const Geometry &g, int level, int64_t ix, int64_t iy,
                                              bool on, const double *__restrict__ sxy,
                                              const double *__restrict__ sq,
                                              const int32_t *__restrict__ leaf_start, int p,
                                              int32_t *row_first, int32_t *row_pre,
                                              double (&v)[2 * PMAX]) {
  const int lane = threadIdx.x & 63, gl = lane & (GL - 1), g0 = lane - gl;
  const double s = ldexp(g.side, -level);
  const double inv_s = 1.0 / s;
  const double cx = g.x0 + ((double)ix + 0.5) * s;
  const double cy = g.y0 + ((double)iy + 0.5) * s;
  const int sh = g.L - level;
  const int64_t nL = int64_t(1) << g.L;
  const int64_t span = int64_t(1) << sh;
#pragma unroll
  for (int k = 0; k < 2 * PMAX; ++k) v[k] = 0.0;
  for (int64_t rb = 0; rb < span; rb += GL) {  // the same count for every group
    int32_t first = 0, cnt = 0;
    if (on && rb + gl < span) {
      const int64_t row = (iy << sh) + rb + gl;
      first = leaf_start[row * nL + (ix << sh)];
      cnt = leaf_start[row * nL + (ix << sh) + span] - first;
    }
    int32_t inc = cnt;  // inclusive scan of the row counts across the group
#pragma unroll
    for (int d = 1; d < GL; d <<= 1) {
      const int32_t x = __shfl_up(inc, d, GL);
      if (gl >= d) inc += x;
    }
    const int32_t total = __shfl(inc, GL - 1, GL);
    wave_sync();  // the previous batch's reads are done
    row_first[lane] = first;
    row_pre[lane] = inc - cnt;
    wave_sync();
    auto source = [&](int32_t t) -> int64_t {
      // the last row whose prefix is <= t (rows past the batch have prefix
      // == total > t, so it is a real row)
      int lo = 0, hi = span > 1 ? GL - 1 : 0;
      while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (row_pre[g0 + mid] <= t) lo = mid; else hi = mid - 1;
      }
      return (int64_t)row_first[g0 + lo] + (t - row_pre[g0 + lo]);
    };
    double nx = 0.0, ny = 0.0, qr = 0.0, qi = 0.0;
    auto fetch = [&](int32_t t) {
      const int64_t i = source(t);
      nx = sxy[2 * i];
      ny = sxy[2 * i + 1];
      qr = sq[QDIM * i];
      if (QDIM == 2) qi = sq[2 * i + 1];
    };
    if (gl < total) fetch(gl);
    for (int32_t t = gl; t < total; t += GL) {
      const cplx w = {(nx - cx) * inv_s, (ny - cy) * inv_s};
      cplx pw = {qr, qi};
      if (t + GL < total) fetch(t + GL);
#pragma unroll
      for (int k = 0; k < PMAX; ++k)
        if (k < p) {
          v[2 * k] += pw.re;
          v[2 * k + 1] += pw.im;
          pw = cmul(pw, w);
        }
    }
  }
}

// Sums v over the D * 2 lanes whose indices differ in bits D, D/2, ..., 1,
// halving the values each lane keeps while their number is even (the lanes
// with the bit set keep the upper half): the lane ends with v[0, VEND) =
// elements [base, base + VEND) of the total, in a fixed order on every run.
// Returns whether this lane stores them (of lanes with equal results, one).
template <int V, int D, int N>
__device__ __forceinline__ bool group_reduce(double (&v)[N], int lane, int &base) {
  if constexpr (D == 0) {
    return true;
  } else if constexpr (V % 2 == 0) {
    constexpr int H = V / 2;
    const bool up = lane & D;
#pragma unroll
    for (int k = 0; k < H; ++k) {
      const double send = up ? v[k] : v[k + H], own = up ? v[k + H] : v[k];
      v[k] = own + __shfl_xor(send, D);
    }
    if (up) base += H;
    return group_reduce<H, D / 2>(v, lane, base);
  } else {
#pragma unroll
    for (int k = 0; k < V; ++k) v[k] += __shfl_xor(v[k], D);
    const bool mine = !(lane & D);
    return group_reduce<V, D / 2>(v, lane, base) && mine;
  }
}
constexpr int group_values(int v, int gl) {
  for (; gl > 1; gl >>= 1)
    if (v % 2 == 0) v /= 2;
  return v;
}

// Reduces the group's partial sums and stores box b's coefficients.
template <int PMAX, int GL>
__device__ __forceinline__ void p2m_group_store(double (&v)[2 * PMAX], bool on, int64_t b, int p,
                                                double *__restrict__ mp, float *__restrict__ mp32) {
  constexpr int VEND = group_values(2 * PMAX, GL);
  int base = 0;
  const bool mine = group_reduce<2 * PMAX, GL / 2>(v, (int)(threadIdx.x & 63), base);
  if (!on || !mine) return;
#pragma unroll
  for (int k = 0; k < VEND; ++k)
    if (base + k < 2 * p) {
      mp[b * 2 * p + base + k] = v[k];
      if (mp32) mp32[b * 2 * p + base + k] = (float)v[k];
    }
}

// The level below a P2M level, when it is already formed: its window (in its
// own box coordinates) and its [window][p] FP64 multipoles.  A crowded box
// whose four children are all in that window is formed from them by M2M
// (4 p(p-1)/2 shift updates) instead of from its stars.
struct ChildLevel {
  Window win;
  const double *mp;  // nullptr: no child level
};

__device__ __forceinline__ bool children_ready(const ChildLevel &c, int64_t ix, int64_t iy) {
  return c.mp != nullptr && 2 * ix >= c.win.bx0 && 2 * ix + 1 < c.win.bx0 + c.win.nbx &&
         2 * iy >= c.win.by0 && 2 * iy + 1 < c.win.by0 + c.win.nby;
}

// Coefficient l of a parent's rescaled multipole from its four children
// (M2M; one lane per coefficient): in child-size units child q's centre sits
// at d = (qa - 1/2) + i (qc - 1/2) from the parent's, and
//     a_l = 2^-l sum_q sum_{j<=l} C(l, j) d^j a_(l-j)(q),
// summed by Horner in d with the binomials of row l formed on the way
// (C(l, j-1) = C(l, j) j / (l - j + 1): integers below 2^53, so exact).
__device__ __forceinline__ cplx m2m_coeff(const ChildLevel &c, int64_t ix, int64_t iy, int p, int l) {
  cplx sum = {0.0, 0.0};
  for (int q = 0; q < 4; ++q) {
    const int qa = q & 1, qc = q >> 1;
    const double dr = qa - 0.5, di = qc - 0.5;
    const int64_t cb = (2 * iy + qc - c.win.by0) * c.win.nbx + (2 * ix + qa - c.win.bx0);
    const double2 *src = reinterpret_cast<const double2 *>(c.mp) + cb * p;
    double bin = 1.0;  // C(l, l)
    double2 v = src[0];
    cplx acc = {v.x, v.y};  // C(l, l) a_0
    for (int jj = l; jj >= 1; --jj) {
      // acc <- acc d + C(l, jj - 1) a_(l - jj + 1)
      bin = bin * (double)jj / (double)(l - jj + 1);
      v = src[l - jj + 1];
      const double re = fma(acc.re, dr, fma(-acc.im, di, bin * v.x));
      const double im = fma(acc.re, di, fma(acc.im, dr, bin * v.y));
      acc = cplx{re, im};
    }
    sum.re += acc.re;
    sum.im += acc.im;
  }
  return cplx{ldexp(sum.re, -l), ldexp(sum.im, -l)};
}

// A box holding more than kCrowdedBox sources is formed by M2M from its
// four children when the level below has them; one holding more than
// kWaveBox sources (and no formed children) is formed by the whole wave
// rather than by its own lane.
constexpr int64_t kCrowdedBox = 32;
constexpr int64_t kWaveBox = 256;

// The rescaled multipole of a box from its four formed children, in one
// lane: each child's coefficients are shifted to the parent's centre by the
// synthetic division (p(p-1)/2 updates
// a_j += d a_(j-1), d = (+-1/2, +-1/2) in child-size units) and the four
// are summed, then scaled by 2^-l.
template <int PMAX>
__device__ __forceinline__ void m2m_lane(const ChildLevel &c, int64_t ix, int64_t iy, int p,
                                         cplx (&acc)[PMAX]) {
#pragma unroll
  for (int k = 0; k < PMAX; ++k) acc[k] = cplx{0.0, 0.0};
  for (int q = 0; q < 4; ++q) {
    const int qa = q & 1, qc = q >> 1;
    const double dr = qa - 0.5, di = qc - 0.5;
    const int64_t cb = (2 * iy + qc - c.win.by0) * c.win.nbx + (2 * ix + qa - c.win.bx0);
    const double2 *src = reinterpret_cast<const double2 *>(c.mp) + cb * p;
    cplx a[PMAX];
#pragma unroll
    for (int k = 0; k < PMAX; ++k)
      if (k < p) {
        const double2 v = src[k];
        a[k] = cplx{v.x, v.y};
      }
#pragma unroll
    for (int k = 0; k + 1 < PMAX; ++k)
      if (k + 1 < p) {
#pragma unroll
        for (int j = PMAX - 1; j > k; --j)
          if (j < p) {
            a[j].re = fma(dr, a[j - 1].re, fma(-di, a[j - 1].im, a[j].re));
            a[j].im = fma(dr, a[j - 1].im, fma(di, a[j - 1].re, a[j].im));
          }
      }
#pragma unroll
    for (int k = 0; k < PMAX; ++k)
      if (k < p) {
        acc[k].re += a[k].re;
        acc[k].im += a[k].im;
      }
  }
#pragma unroll
  for (int k = 0; k < PMAX; ++k)
    if (k < p) acc[k] = cplx{ldexp(acc[k].re, -k), ldexp(acc[k].im, -k)};
}

// P2M for levels whose boxes hold few sources on average: one thread per box
// of `win` with all p coefficients in registers (running powers m w^k).
// Occupancy is heavy-tailed in clustered fields (a galaxy's centre, a
// cluster of lenses): a lane whose box holds more than kCrowdedBox sources
// forms it by M2M from its children when the level below has them all (in
// its own lane, so a wave of crowded boxes shifts them side by side), and a
// box of more than kWaveBox sources without them is left to the whole wave,
// which forms such boxes one after another -- or, with `defer`, to a second
// pass of k_p2m_group (a wave per box), this pass storing zeros for them.
// The kernel is bound by memory
// latency (a few sources per lane): a box of one or two leaf rows keeps its
// source ranges in registers and the next source's loads are issued before
// the current one's powers are summed.  The wave's 64 boxes are staged in
// LDS so that the [64][p] block is written with coalesced stores.
template <int PMAX, int QDIM>
__global__ __launch_bounds__(kWave) void k_p2m_box(Geometry g, int level, Window win,
                                                   const double *__restrict__ sxy,
                                                   const double *__restrict__ sq,
                                                   const int32_t *__restrict__ leaf_start, int p,
                                                   double *__restrict__ mp, float *__restrict__ mp32,
                                                   ChildLevel child, int defer) {
  constexpr int STR = 2 * PMAX + 1;
  __shared__ double stage[kWave * STR];
  __shared__ int32_t row_first[kWave], row_pre[kWave];
  const int lane = threadIdx.x;
  const int64_t nbox = win.count();
  const int64_t b0 = (int64_t)blockIdx.x * kWave;
  const int64_t b = b0 + lane;
  const int sh = g.L - level;
  const int64_t nL = int64_t(1) << g.L;
  const int64_t span = int64_t(1) << sh;
  const int64_t ix = b < nbox ? win.bx0 + b % win.nbx : 0;
  const int64_t iy = b < nbox ? win.by0 + b / win.nbx : 0;
  // source ranges of the box's (first two) leaf rows, and its source count
  int32_t a0 = 0, e0 = 0, a1 = 0, e1 = 0;
  int64_t count = 0;
  if (b < nbox) {
    const int64_t c0 = (iy << sh) * nL + (ix << sh);
    a0 = leaf_start[c0];
    e0 = leaf_start[c0 + span];
    if (span >= 2) {
      a1 = leaf_start[c0 + nL];
      e1 = leaf_start[c0 + nL + span];
    }
    count = (int64_t)(e0 - a0) + (e1 - a1);
    for (int64_t r = 2; r < span; ++r) {
      const int64_t row = (iy << sh) + r;
      count += leaf_start[row * nL + (ix << sh) + span] - leaf_start[row * nL + (ix << sh)];
    }
  }
  const bool by_m2m = count > kCrowdedBox && b < nbox && children_ready(child, ix, iy);
  const bool by_wave = count > kWaveBox && !by_m2m;
  cplx acc[PMAX];
#pragma unroll
  for (int k = 0; k < PMAX; ++k) acc[k] = cplx{0.0, 0.0};
  auto add_source = [&](double x, double y, cplx pw, const cplx &c, double inv_s) {
    const cplx w = {(x - c.re) * inv_s, (y - c.im) * inv_s};
#pragma unroll
    for (int k = 0; k < PMAX; ++k)
      if (k < p) {
        acc[k].re += pw.re;
        acc[k].im += pw.im;
        pw = cmul(pw, w);
      }
  };
  auto charge = [&](int64_t i) {
    return QDIM == 1 ? cplx{sq[i], 0.0} : cplx{sq[2 * i], sq[2 * i + 1]};
  };
  if (by_m2m) m2m_lane<PMAX>(child, ix, iy, p, acc);
  if (b < nbox && !by_m2m && !by_wave) {
    const double s = ldexp(g.side, -level);
    const double inv_s = 1.0 / s;
    const cplx c = {g.x0 + ((double)ix + 0.5) * s, g.y0 + ((double)iy + 0.5) * s};
    // the first two rows as one run of n0 + n1 sources, software-pipelined
    const int32_t n0 = e0 - a0, n = n0 + (e1 - a1);
    auto src = [&](int32_t t) { return (int64_t)(t < n0 ? a0 + t : a1 + (t - n0)); };
    double nx = 0.0, ny = 0.0;
    cplx nq = {0.0, 0.0};
    if (n > 0) {
      const int64_t i = src(0);
      nx = sxy[2 * i];
      ny = sxy[2 * i + 1];
      nq = charge(i);
    }
    for (int32_t t = 0; t < n; ++t) {
      const double x = nx, y = ny;
      const cplx q = nq;
      if (t + 1 < n) {
        const int64_t i = src(t + 1);
        nx = sxy[2 * i];
        ny = sxy[2 * i + 1];
        nq = charge(i);
      }
      add_source(x, y, q, c, inv_s);
    }
    for (int64_t r = 2; r < span; ++r) {
      const int64_t row = (iy << sh) + r;
      const int32_t i0 = leaf_start[row * nL + (ix << sh)];
      const int32_t i1 = leaf_start[row * nL + (ix << sh) + span];
      for (int32_t i = i0; i < i1; ++i) add_source(sxy[2 * (int64_t)i], sxy[2 * (int64_t)i + 1], charge(i), c, inv_s);
    }
  }
#pragma unroll
  for (int k = 0; k < PMAX; ++k)
    if (k < p) {
      stage[lane * STR + 2 * k] = acc[k].re;
      stage[lane * STR + 2 * k + 1] = acc[k].im;
    }
  __syncthreads();
  const int twop = 2 * p;
  const int64_t nb = nbox - b0 < kWave ? nbox - b0 : kWave;
  // the boxes left to the whole wave (bit = lane), unless a second pass
  // (k_p2m_group) forms them, a wave each, afterwards
  uint64_t todo = defer ? 0ull : __ballot(b < nbox && by_wave);
  for (int e = lane; e < nb * twop; e += kWave) {
    const int bl = e / twop, c = e - bl * twop;
    if ((todo >> bl) & 1) continue;
    const double v = stage[bl * STR + c];
    mp[b0 * twop + e] = v;
    if (mp32) mp32[b0 * twop + e] = (float)v;
  }
  if (todo) {  // one at a time, a wave-uniform loop
    double v[2 * PMAX];
    while (todo) {
      const int owner = __builtin_ctzll(todo);
      todo &= todo - 1;
      const int64_t ob = b0 + owner;
      p2m_group_sum<PMAX, QDIM, kWave>(g, level, win.bx0 + ob % win.nbx, win.by0 + ob / win.nbx, true,
                                       sxy, sq, leaf_start, p, row_first, row_pre, v);
      p2m_group_store<PMAX, kWave>(v, true, ob, p, mp, mp32);
    }
  }
}

// P2M with GL lanes per box (64 / GL boxes per wave): for levels whose boxes
// hold many sources, or are too few to fill the chip with a lane each.
// Occupancy is heavy-tailed in clustered fields: a box of more than 8 GL
// sources is formed by M2M from its children when the level below has them,
// and one of more than 64 GL without them, where GL < 64, by the whole wave
// after its other boxes.
// only_above >= 0: the second pass behind k_p2m_box, which left this kernel
// its boxes of more than only_above sources without formed children.
template <int PMAX, int QDIM, int GL>
__global__ __launch_bounds__(kWave) void k_p2m_group(Geometry g, int level, Window win,
                                                     const double *__restrict__ sxy,
                                                     const double *__restrict__ sq,
                                                     const int32_t *__restrict__ leaf_start, int p,
                                                     double *__restrict__ mp, float *__restrict__ mp32,
                                                     ChildLevel child, int64_t only_above) {
  __shared__ int32_t row_first[kWave], row_pre[kWave];
  const int lane = threadIdx.x, gl = lane & (GL - 1);
  const int64_t b = (int64_t)blockIdx.x * (kWave / GL) + lane / GL;
  bool on = b < win.count();
  const int64_t ix = on ? win.bx0 + b % win.nbx : 0, iy = on ? win.by0 + b / win.nbx : 0;
  const bool ready = on && children_ready(child, ix, iy);
  // the box's source count, its leaf rows spread over the group (where it
  // decides how the box is formed)
  int64_t cnt = 0;
  if (on && (GL < kWave || ready || only_above >= 0)) {
    const int sh = g.L - level;
    const int64_t nL = int64_t(1) << g.L;
    const int64_t span = int64_t(1) << sh;
    for (int64_t r = gl; r < span; r += GL) {
      const int64_t row = (iy << sh) + r;
      cnt += leaf_start[row * nL + (ix << sh) + span] - leaf_start[row * nL + (ix << sh)];
    }
  }
#pragma unroll
  for (int d = GL / 2; d >= 1; d >>= 1) cnt += __shfl_xor(cnt, d);
  if (only_above >= 0) {
    on = on && !ready && cnt > only_above;
    if (!__any(on)) return;  // wave-uniform
  }
  const bool by_m2m = on && ready && cnt > 8 * GL;
  const bool by_wave = GL < kWave && on && !by_m2m && cnt > 64 * GL;
  double v[2 * PMAX];
  p2m_group_sum<PMAX, QDIM, GL>(g, level, ix, iy, on && !by_m2m && !by_wave, sxy, sq, leaf_start, p,
                                row_first, row_pre, v);
  p2m_group_store<PMAX, GL>(v, on && !by_m2m && !by_wave, b, p, mp, mp32);
  if (by_m2m) {
    for (int l = gl; l < p; l += GL) {
      const cplx a = m2m_coeff(child, ix, iy, p, l);
      mp[b * 2 * p + 2 * l] = a.re;
      mp[b * 2 * p + 2 * l + 1] = a.im;
      if (mp32) {
        mp32[b * 2 * p + 2 * l] = (float)a.re;
        mp32[b * 2 * p + 2 * l + 1] = (float)a.im;
      }
    }
  }
  if constexpr (GL < kWave) {
    uint64_t todo = __ballot(by_wave && gl == 0);
    while (todo) {
      const int owner = __builtin_ctzll(todo);
      todo &= todo - 1;
      const int64_t ob = (int64_t)blockIdx.x * (kWave / GL) + owner / GL;
      p2m_group_sum<PMAX, QDIM, kWave>(g, level, win.bx0 + ob % win.nbx, win.by0 + ob / win.nbx, true,
                                       sxy, sq, leaf_start, p, row_first, row_pre, v);
      p2m_group_store<PMAX, kWave>(v, true, ob, p, mp, mp32);
    }
  }
}

// M2M for up to four consecutive levels in one launch, as FP64 MFMAs.  A
// workgroup owns a T x T tile of parent boxes at the finest level of the
// launch (T = min(8, boxes per side)); its parents are the rows of 16-row
// M-tiles, C[parents][2p] = sum_q A_q[children][2p] M_q over the four child
// quadrants q.  64 parents are four M-tiles, a wave each; their (T/2)^2
// parents and the coarser ones are one M-tile, its N-tiles of 16 outputs
// spread over the waves, with the children read back from LDS.  So a tile of
// 8 x 8 boxes yields its 4 x 4, 2 x 2 and 1 x 1 ancestors in the same launch.
// The products are short against a memory round trip, so the loads are
// ordered by hand: every child coefficient of the tile first, the next
// quadrant's operator while one multiplies, and the coarser stages' operator
// (the same for all of them) once (64 workgroups, p = 20: 18 us, against 41
// with a lane per child shifting it by synthetic division).
template <int KS>
__global__ __launch_bounds__(kThreads) void k_m2m_chain(M2MChain c, const double *__restrict__ frag) {
  constexpr int NT = (KS + 3) / 4, REC = 4 * KS + 1;
  __shared__ double bufA[64 * REC];  // stage 0 and 2 results
  __shared__ double bufB[16 * REC];  // stage 1 results
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, i = lane & 15, kq = lane >> 4;
  const int twop = 2 * c.p;
  const int64_t n = int64_t(1) << c.level;
  const int T = n < 8 ? (int)n : 8;
  const int64_t tiles = n / T;
  const int64_t tbx = blockIdx.x % tiles, tby = blockIdx.x / tiles;

  auto store = [&](int st, int mt, int nt, const d4v &acc) {
    const int Ts = T >> st, P = Ts * Ts, lts = 31 - __builtin_clz(Ts);
    const int64_t ns = n >> st;
    const int col = nt * 16 + i;
    double *keep = st == 1 ? bufB : bufA;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int par = mt * 16 + kq + 4 * r;
      if (par >= P || col >= twop) continue;
      const int64_t box = (tby * Ts + (par >> lts)) * ns + tbx * Ts + (par & (Ts - 1));
      c.out[st][box * twop + col] = acc[r];
      if (c.out32[st]) c.out32[st][box * twop + col] = (float)acc[r];
      if (st + 1 < c.nlev) keep[par * REC + col] = acc[r];
    }
  };
  // coefficients of the four children of parent `par` at stage 0.  The
  // K-steps of the product take the coefficients in the order 8 h + 2 kq,
  // 8 h + 2 kq + 1 (the operator's fragments are built to match), so that a
  // lane reads them in pairs of 16 bytes
  double av[4][KS];
  {
    const int P = T * T, par = (P == 64 ? wv * 16 : 0) + i, lts = 31 - __builtin_clz(T);
    const bool on = par < P;
    const int tx = on ? par & (T - 1) : 0, ty = on ? par >> lts : 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int64_t cb = (2 * (tby * T + ty) + (q >> 1)) * (2 * n) + 2 * (tbx * T + tx) + (q & 1);
      const double2 *src = reinterpret_cast<const double2 *>(c.child + cb * twop);
#pragma unroll
      for (int h = 0; h < KS / 2; ++h) {
        const double2 v = on && 4 * h + kq < c.p ? src[4 * h + kq] : make_double2(0.0, 0.0);
        av[q][2 * h] = v.x;
        av[q][2 * h + 1] = v.y;
      }
    }
  }
  int st = 0;
  if (T == 8) {
    // 64 parents, a wave per M-tile, N-tiles NH at a time
    constexpr int NH = KS <= 12 ? NT : 1;
    for (int n0 = 0; n0 < NT; n0 += NH) {
      d4v acc[NH];
      double b[2][KS * NH];
      auto load_b = [&](int q, double (&dst)[KS * NH]) {
        const double *bs = frag + ((size_t)q * KS * NT + n0) * 64 + lane;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
          for (int h = 0; h < NH; ++h) dst[ks * NH + h] = bs[(ks * NT + h) * 64];
      };
      load_b(0, b[0]);
#pragma unroll
      for (int h = 0; h < NH; ++h) acc[h] = d4v{0, 0, 0, 0};
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if (q < 3) load_b(q + 1, b[(q + 1) & 1]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
          for (int h = 0; h < NH; ++h)
            acc[h] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[q][ks], b[q & 1][ks * NH + h], acc[h], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int h = 0; h < NH; ++h) store(0, wv, n0 + h, acc[h]);
    }
    st = 1;
    if (c.nlev == 1) return;  // uniform
  }
  // at most 16 parents: one M-tile, wave wv takes N-tiles wv, wv + 4
  double b[4][KS];
  auto load_nt = [&](int nt) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) b[q][ks] = frag[((size_t)(q * KS + ks) * NT + nt) * 64 + lane];
    __builtin_amdgcn_sched_barrier(0);
  };
  if (wv < NT) load_nt(wv);
  for (; st < c.nlev; ++st) {
    __syncthreads();
    const int Ts = T >> st, P = Ts * Ts, lts = 31 - __builtin_clz(Ts);
    if (st > 0) {
      const bool on = i < P;
      const int tx = on ? i & (Ts - 1) : 0, ty = on ? i >> lts : 0;
      const double *kids = st == 2 ? bufB : bufA;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const double *src = kids + ((2 * ty + (q >> 1)) * (2 * Ts) + 2 * tx + (q & 1)) * REC;
#pragma unroll
        for (int h = 0; h < KS / 2; ++h) {
          const int k = 8 * h + 2 * kq;
          av[q][2 * h] = on && k < twop ? src[k] : 0.0;
          av[q][2 * h + 1] = on && k < twop ? src[k + 1] : 0.0;
        }
      }
    }
    for (int nt = wv; nt < NT; nt += kThreads / 64) {
      if (NT > 4 && (nt != wv || st > 0)) load_nt(nt);
      d4v acc = d4v{0, 0, 0, 0};
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
          acc = __builtin_amdgcn_mfma_f64_16x16x4f64(av[q][ks], b[q][ks], acc, 0, 0, 0);
      store(st, 0, nt, acc);
    }
  }
}

// Lanes per box (1, 4, 16 or 64) of a P2M level of `boxes` boxes holding
// `mean` sources each.  A lane per box is the fastest while the boxes fill the
// chip (2 waves per SIMD: 131072 lanes) with up to ~64 sources each; fewer
// boxes get as many lanes as fill it, but no more than they have sources
// (p = 17: 192 boxes of ~300 sources 7.7 us with 64 lanes, 154 with one; 256
// boxes of 8, p = 12, 10.9 with 4, 29 with one).  Fuller boxes get a lane per
// 16 sources (16384 boxes of 305: 84 us with 16 lanes, 156 with 64 and a
// butterfly over all coefficients), or per 4 in clustered fields, whose
// boxes differ so much that a wave's groups would wait for the fullest.
int p2m_lanes(int64_t boxes, double mean, bool clustered) {
  const double fill = 131072.0 / (double)boxes;
  const double want = mean > 64.0 ? std::max(mean / (clustered ? 4.0 : 16.0), std::min(mean, fill)) : std::min(mean, fill);
  return want >= 32.0 ? 64 : (want >= 8.0 ? 16 : (want >= 2.0 ? 4 : 1));
}

}  // namespace


void launch_p2m(Geometry g, int level, Window win, const double *sxy, const double *sq, int qdim,
                const int32_t *leaf_start, int p, double *mp, float *mp32, double win_sources,
                bool clustered, Window child_win, const double *child_mp, hipStream_t stream) {
  const ChildLevel child{child_win, child_mp};
  const int64_t boxes = win.count();
  if (boxes == 0) return;
  auto group = [&](auto gl_c, int64_t only_above) {
    constexpr int GL = decltype(gl_c)::value;
    const unsigned nb = (unsigned)((boxes * GL + kWave - 1) / kWave);
    if (qdim == 2)
      LENS_PMAX_DISPATCH(p, hipLaunchKernelGGL((k_p2m_group<PM, 2, GL>), dim3(nb), dim3(kWave), 0,
                                               stream, g, level, win, sxy, sq, leaf_start, p, mp, mp32,
                                               child, only_above));
    else
      LENS_PMAX_DISPATCH(p, hipLaunchKernelGGL((k_p2m_group<PM, 1, GL>), dim3(nb), dim3(kWave), 0,
                                               stream, g, level, win, sxy, sq, leaf_start, p, mp, mp32,
                                               child, only_above));
    LENS_HIP(hipGetLastError());
  };
  const double mean = win_sources / (double)boxes;
  const int gl = p2m_lanes(boxes, mean, clustered);
  if (gl == 64) return group(std::integral_constant<int, 64>{}, -1);
  if (gl == 16) return group(std::integral_constant<int, 16>{}, -1);
  if (gl == 4) return group(std::integral_constant<int, 4>{}, -1);
  // A thread per box.  In a clustered field whose leaf boxes hold a few
  // sources on average, those of more than kWaveBox sources get a wave each
  // in a second pass rather than their lane's wave one after another (above
  // the leaf level such boxes are formed from their children).
  const int defer = (clustered && mean > 2.0 && child_mp == nullptr) ? 1 : 0;
  const unsigned nb = (unsigned)((boxes + kWave - 1) / kWave);
  if (qdim == 2)
    LENS_PMAX_DISPATCH(p, hipLaunchKernelGGL((k_p2m_box<PM, 2>), dim3(nb), dim3(kWave), 0, stream,
                                             g, level, win, sxy, sq, leaf_start, p, mp, mp32,
                                             child, defer));
  else
    LENS_PMAX_DISPATCH(p, hipLaunchKernelGGL((k_p2m_box<PM, 1>), dim3(nb), dim3(kWave), 0, stream,
                                             g, level, win, sxy, sq, leaf_start, p, mp, mp32,
                                             child, defer));
  LENS_HIP(hipGetLastError());
  if (defer) group(std::integral_constant<int, 64>{}, kWaveBox);
}

int m2m_chain_levels(int level) {
  // T = min(8, 2^level) parents per tile side; T halves per fused level
  int T = level >= 3 ? 8 : (1 << level), k = 1;
  while (T > 1 && k < kMaxM2MChain) {
    T >>= 1;
    ++k;
  }
  return k;
}

void launch_m2m_chain(const M2MChain &c, const OpTables &t, hipStream_t stream) {
  if (c.nlev < 1 || c.nlev > m2m_chain_levels(c.level))
    fail(LENS_EINVAL, "M2M chain: bad level count");
  const int64_t n = int64_t(1) << c.level;
  const int64_t T = n < 8 ? n : 8;
  const unsigned blocks = (unsigned)((n / T) * (n / T));
  LENS_KS_DISPATCH(t.ks, hipLaunchKernelGGL((k_m2m_chain<KS>), dim3(blocks), dim3(kThreads), 0, stream,
                                            c, t.m2m_frag));
  LENS_HIP(hipGetLastError());
}

}  // namespace lensfmm
