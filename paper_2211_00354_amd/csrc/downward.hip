// Downward pass (Appendix A, downward passes 1 and 2), for each level
// l = 2..L over the target window (the boxes that hold rays):
//
//   M2L:  local(t)  = (1/s_l) sum_{tau in IL(t)} T_tau a~(t + tau)
//   L2L:  local(t) += L2L(local(parent(t)))        (l >= 3), FP64
//
// M2L of every level runs first (one batched launch per arithmetic type, as
// levels are independent there), then L2L sweeps the levels coarse to fine.
//
// IL(t) is the interaction list: the children of the parent's neighbours
// that are not neighbours of t.  For a target that is child (qx, qy) of its
// parent, tau = (c_src - c_tgt)/s ranges over [-2-qx, 3-qx] x [-2-qy, 3-qy]
// minus the 3x3 neighbourhood: 27 offsets out of 40 distinct ones, the same
// operators at every level on rescaled coefficients.  Source boxes outside the
// root are empty.
//
// M2L on MFMA (k_m2l_split, k_m2l_wide): a workgroup takes 8 x 8 tiles of
// target boxes; each wave takes the 16 targets of one quadrant class of a
// tile, to which the same 27 operators apply.  The source multipoles the tiles
// need (two more boxes on every side) are staged once in LDS (coalesced row
// loads of box-major coefficients).  For one offset the 16-target M-tile forms
// a real GEMM
//   C[16 targets][2p] += A[16][2p] B_tau[2p][2p]
// over interleaved (re, im) coefficients, done with 16x16x4 MFMAs: A rows are
// read from the LDS tile at the target + tau, B fragments come pre-swizzled
// in lane order from global memory (L1/L2 resident, shared by every wave).
// FP32 (fine levels of LENS_MIXED) uses v_mfma_f32_16x16x4f32, FP64 uses
// v_mfma_f64_16x16x4f64; B fragments of later offsets are loaded while the
// current one computes.  The result, scaled by 1/s, is stored as the FP64
// locals.
#include <type_traits>

#include "device_common.h"

namespace lensfmm {

namespace {

constexpr int kThreads = 256;

typedef float f4v __attribute__((ext_vector_type(4)));
typedef double d4v __attribute__((ext_vector_type(4)));

// ------------------------------------------------------------------- L2L

// L2L down up to three levels in one launch, as FP64 MFMAs: a workgroup owns
// one box of the chain's top level (its locals final) and its 4 + 16 + 64
// descendants.  At depth j the 4^(j-1) parents (the previous depth's result,
// kept in LDS) are the rows of one 16-row M-tile, and each of the four waves
// forms the children of one quadrant, C[parents][2p] = A[parents][2p] L_q,
// adds their M2L locals and stores them.  A box outside its level's window is
// skipped; its children lie outside theirs, and the rows of a product do not
// mix.  The kernel is bound by latency: the operators and the M2L locals of
// every depth are loaded before the first product, so one memory round trip is
// paid per launch (16 top boxes, p = 20: 9.5 us, against 34 with a thread per
// box that shifts it by synthetic division).
template <int KS>
__global__ __launch_bounds__(kThreads) void k_l2l_chain(L2LChain c, const double *__restrict__ frag) {
  constexpr int NT = (KS + 3) / 4, REC = 4 * KS + 1;
  constexpr bool KEEP = KS <= 12;  // operators in registers for every depth
  __shared__ double buf1[4 * REC], buf2[16 * REC];
  const int quad = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, i = lane & 15, kq = lane >> 4;
  const int qx = quad & 1, qy = quad >> 1;
  const int twop = 2 * c.p;
  const int64_t rb = blockIdx.x;
  const int64_t RX = c.win[0].bx0 + rb % c.win[0].nbx, RY = c.win[0].by0 + rb / c.win[0].nbx;

  // the child (in this wave's quadrant) of parent `row` at depth j, or nullptr
  auto child = [&](int j, int row) -> double * {
    const int sp = 1 << (j - 1);
    if (row >= sp * sp) return nullptr;
    const Window &w = c.win[j];
    const int64_t X = (RX << j) + 2 * (row & (sp - 1)) + qx - w.bx0;
    const int64_t Y = (RY << j) + 2 * (row >> (j - 1)) + qy - w.by0;
    if (X < 0 || Y < 0 || X >= w.nbx || Y >= w.nby) return nullptr;
    return c.loc[j] + (Y * w.nbx + X) * twop;
  };
  const double *bsrc = frag + (size_t)quad * KS * NT * 64 + lane;
  double bk[KEEP ? KS * NT : 1];
  if (KEEP) {
#pragma unroll
    for (int q = 0; q < KS * NT; ++q) bk[q] = bsrc[q * 64];
  }
  double old[6][NT];  // depth 1 and 2: register 0; depth 3: registers 0..3
  auto fetch = [&](int j, int r, double (&o)[NT]) {
    const double *d = j <= c.nlev ? child(j, kq + 4 * r) : nullptr;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      const int n = nt * 16 + i;
      o[nt] = d && n < twop ? d[n] : 0.0;
    }
  };
  fetch(1, 0, old[0]);
  fetch(2, 0, old[1]);
#pragma unroll
  for (int r = 0; r < 4; ++r) fetch(3, r, old[2 + r]);

  const double *root = c.loc[0] + rb * twop;
  auto depth = [&](auto J, const double *par, double *keep) {
    constexpr int j = decltype(J)::value, rows = j == 3 ? 16 : (j == 2 ? 4 : 1);
    d4v acc[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) acc[nt] = d4v{0, 0, 0, 0};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const int k = 4 * ks + kq;
      double av = 0.0;
      if (i < rows && k < twop) {
        if constexpr (j == 1) av = root[k]; else av = par[i * REC + k];
      }
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        const double bv = KEEP ? bk[ks * NT + nt] : bsrc[(ks * NT + nt) * 64];
        acc[nt] = __builtin_amdgcn_mfma_f64_16x16x4f64(av, bv, acc[nt], 0, 0, 0);
      }
    }
#pragma unroll
    for (int r = 0; r < (j == 3 ? 4 : 1); ++r) {
      const int row = kq + 4 * r;
      double *d = child(j, row);
      if (!d) continue;
      // row (py, px) of the parents: child (2 py + qy, 2 px + qx) of the next depth
      constexpr int sp = 1 << (j - 1);
      const int idx = (2 * (row >> (j - 1)) + qy) * (2 * sp) + 2 * (row & (sp - 1)) + qx;
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        const int n = nt * 16 + i;
        if (n >= twop) continue;
        const double v = old[j == 3 ? 2 + r : j - 1][nt] + acc[nt][r];
        d[n] = v;
        if (j < 3) keep[idx * REC + n] = v;
      }
    }
  };
  depth(std::integral_constant<int, 1>{}, nullptr, buf1);
  if (c.nlev < 2) return;  // uniform
  __syncthreads();
  depth(std::integral_constant<int, 2>{}, buf1, buf2);
  if (c.nlev < 3) return;
  __syncthreads();
  depth(std::integral_constant<int, 3>{}, buf2, nullptr);
}

// --------------------------------------------------------- M2L on MFMA

template <typename T>
struct Mfma;
template <>
struct Mfma<float> {
  using acc = f4v;
  __device__ static acc op(float a, float b, acc c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
};
template <>
struct Mfma<double> {
  using acc = d4v;
  __device__ static acc op(double a, double b, acc c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  __device__ static int row(int lane, int r) { return (lane >> 4) + 4 * r; }
};

// Interaction list of a quadrant class as 27 (tau_x, tau_y) offsets.
struct IList {
  int8_t t[4][27][2];
};
constexpr IList make_ilist() {
  IList il{};
  for (int q = 0; q < 4; ++q) {
    const int qx = q & 1, qy = q >> 1;
    int j = 0;
    for (int ty = -2 - qy; ty <= 3 - qy; ++ty)
      for (int tx = -2 - qx; tx <= 3 - qx; ++tx) {
        if (tx >= -1 && tx <= 1 && ty >= -1 && ty <= 1) continue;
        il.t[q][j][0] = (int8_t)tx;
        il.t[q][j][1] = (int8_t)ty;
        ++j;
      }
  }
  return il;
}
__constant__ IList kIL = make_ilist();

// Stages the source multipoles of the SX x SY boxes from (tx0 - 2, ty0 - 2) in
// LDS, records of 4 KS + 1 values, zero outside the stored window swin (which
// holds every source of the level's targets): all of a thread's loads are
// issued before its LDS stores.  16-byte loads where 2p is a multiple of 4
// (every box record is then 16-byte aligned).
template <typename T, int KS, int SX, int SY, int NTH>
__device__ __forceinline__ void stage_sources(const M2LLevel &a, const T *__restrict__ mp, int twop,
                                              int64_t tx0, int64_t ty0, T *lds) {
  constexpr int REC = 4 * KS + 1;
  if ((twop & 3) == 0) {
    constexpr int NE4 = SX * SY * KS, NIT4 = (NE4 + NTH - 1) / NTH;
    const int k4n = twop >> 2;
    using V4 = typename std::conditional<std::is_same<T, float>::value, float4, double4>::type;
    V4 v[NIT4];
#pragma unroll
    for (int it = 0; it < NIT4; ++it) {
      const int e = it * NTH + threadIdx.x;
      const int k4 = e % KS, bl = e / KS;
      const int bx = bl % SX, by = bl / SX;
      const int64_t gx = tx0 - 2 + bx - a.swin.bx0, gy = ty0 - 2 + by - a.swin.by0;
      v[it] = V4{0, 0, 0, 0};
      if (e < NE4 && k4 < k4n && gx >= 0 && gy >= 0 && gx < a.swin.nbx && gy < a.swin.nby)
        v[it] = reinterpret_cast<const V4 *>(mp + (gy * a.swin.nbx + gx) * twop)[k4];
    }
#pragma unroll
    for (int it = 0; it < NIT4; ++it) {
      const int e = it * NTH + threadIdx.x;
      if (e < NE4) {
        T *d = lds + (e / KS) * REC + 4 * (e % KS);
        d[0] = v[it].x;
        d[1] = v[it].y;
        d[2] = v[it].z;
        d[3] = v[it].w;
      }
    }
  } else {
    constexpr int KP = 4 * KS;
    constexpr int NE = SX * SY * KP, NIT = (NE + NTH - 1) / NTH;
    T v[NIT];
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
      const int e = it * NTH + threadIdx.x;
      const int k = e % KP, bl = e / KP;
      const int bx = bl % SX, by = bl / SX;
      const int64_t gx = tx0 - 2 + bx - a.swin.bx0, gy = ty0 - 2 + by - a.swin.by0;
      v[it] = 0;
      if (e < NE && k < twop && gx >= 0 && gy >= 0 && gx < a.swin.nbx && gy < a.swin.nby)
        v[it] = mp[(gy * a.swin.nbx + gx) * twop + k];
    }
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
      const int e = it * NTH + threadIdx.x;
      if (e < NE) lds[(e / KP) * REC + e % KP] = v[it];
    }
  }
}

// Orders p > 32 in FP64 over many tiles: 8 x 8 targets per workgroup, the 4
// waves own the quadrant classes (16 targets each, one M-tile), and a wave
// forms all NT N-tiles of 16 outputs (2p <= 4 KS of them): 200 accumulator
// and operator registers per lane, but every source read from LDS feeds NT
// MFMAs (256^2 targets, p = 40: 491 us against 558 for k_m2l_split's best).
// One launch serves several levels (M2L of different levels is independent):
// blockIdx.x indexes the concatenated tile lists.
template <int KS, bool FUSE>
__global__ __launch_bounds__(kThreads) void k_m2l_wide(M2LBatch bt, const double *__restrict__ bfrag,
                                                       const double *__restrict__ l2l_frag) {
  constexpr int TILE = 8, S = TILE + 4;  // source tile side
  constexpr int H = TILE / 2;            // targets per quadrant class per side
  constexpr int NT = (KS + 3) / 4;       // N-tiles: 2p <= 4 KS outputs
  constexpr int REC = 4 * KS + 1;        // LDS record stride (odd: spreads banks)
  extern __shared__ __align__(16) unsigned char lds_raw[];
  double *lds = reinterpret_cast<double *>(lds_raw);

  int li = 0;
  while (li + 1 < bt.count && (int64_t)blockIdx.x >= bt.tile_begin[li + 1]) ++li;
  const M2LLevel &a = bt.lv[li];
  const double *__restrict__ mp = static_cast<const double *>(a.mp);
  const int p = bt.p, twop = 2 * p;
  const int64_t ex0 = a.win.bx0 & ~int64_t(1), ey0 = a.win.by0 & ~int64_t(1);
  const int64_t ntx = (a.win.bx0 + a.win.nbx - ex0 + TILE - 1) / TILE;
  const int64_t tile = (int64_t)blockIdx.x - bt.tile_begin[li];
  const int64_t tx0 = ex0 + TILE * (tile % ntx);
  const int64_t ty0 = ey0 + TILE * (tile / ntx);

  stage_sources<double, KS, S, S, kThreads>(a, mp, twop, tx0, ty0, lds);
  __syncthreads();

  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int qx = wave & 1, qy = wave >> 1;
  using M = Mfma<double>;
  d4v acc[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) acc[nt] = d4v{0, 0, 0, 0};

  // A operand: lane holds row i = lane % 16 of the M-tile, column lane / 16
  const int i = lane & 15, kq = lane >> 4;
  const int base = ((2 * (i / H) + qy + 2) * S + (2 * (i % H) + qx + 2)) * REC + kq;

  // B fragments of the current offset, and of the next one in flight
  constexpr int NB = KS * NT;
  double bcur[NB], bnxt[NB];
  auto load_b = [&](int j, double (&dst)[NB]) {
    const int tx = kIL.t[wave][j][0], ty = kIL.t[wave][j][1];
    const double *src = bfrag + (size_t)((ty + 3) * 7 + (tx + 3)) * NB * 64 + lane;
#pragma unroll
    for (int q = 0; q < NB; ++q) dst[q] = src[q * 64];
  };
  load_b(0, bcur);
  for (int j = 0; j < 27; ++j) {
    load_b(j + 1 < 27 ? j + 1 : j, bnxt);
    const int tx = kIL.t[wave][j][0], ty = kIL.t[wave][j][1];
    const int toff = (ty * S + tx) * REC;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const double av = lds[base + toff + 4 * ks];
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) acc[nt] = M::op(av, bcur[ks * NT + nt], acc[nt]);
    }
#pragma unroll
    for (int q = 0; q < NB; ++q) bcur[q] = bnxt[q];
  }

  const double inv_s = 1.0 / a.s;
  auto target_xy = [&](int t, int64_t &gx, int64_t &gy) {
    gx = tx0 + 2 * (t % H) + qx;
    gy = ty0 + 2 * (t / H) + qy;
    return gx >= a.win.bx0 && gy >= a.win.by0 && gx < a.win.bx0 + a.win.nbx &&
           gy < a.win.by0 + a.win.nby;
  };
  // L2L: A = the targets' parent locals, B = L2L fragments of this wave's
  // quadrant; accumulated apart from the M2L part
  d4v acc2[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) acc2[nt] = d4v{0, 0, 0, 0};
  if constexpr (FUSE) {
    int64_t gx, gy, pidx = -1;
    if (target_xy(i, gx, gy))
      pidx = ((gy >> 1) - a.pwin.by0) * a.pwin.nbx + ((gx >> 1) - a.pwin.bx0);
    const double *lf = l2l_frag + (size_t)wave * KS * NT * 64 + lane;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const int k = 4 * ks + kq;
      const double av = (pidx >= 0 && k < twop) ? a.ploc[pidx * twop + k] : 0.0;
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) acc2[nt] = M::op(av, lf[(ks * NT + nt) * 64], acc2[nt]);
    }
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    int64_t gx, gy;
    if (!target_xy(M::row(lane, r), gx, gy)) continue;
    double *out = a.loc + ((gy - a.win.by0) * a.win.nbx + (gx - a.win.bx0)) * twop;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      const int n = nt * 16 + (lane & 15);
      if (n < twop) out[n] = FUSE ? fma(acc[nt][r], inv_s, acc2[nt][r]) : acc[nt][r] * inv_s;
    }
  }
}

// Every other order.  A workgroup takes MX 8 x 8 tiles of targets side by side
// (an M-tile of 16 each per wave) and NB of the NT N-tiles of 16 outputs, a
// wave per (quadrant, N-tile); the operators of the next two offsets are in
// flight while one computes.  A wave's time is its serial chain of 27 KS MX
// MFMAs plus the operators' latency, so for few tiles the finest split
// (MX = NB = 1) is the fastest: 64^2 targets take 10.4 us at p = 12 in FP32
// and 18.7 at p = 20 in FP64, where a wave that formed all outputs of 16 x 16
// (FP32) or 8 x 8 (FP64) targets took 38.4 and 55.8.  With many tiles the
// MFMA rate and the operators' traffic count: MX = 2 halves that traffic and
// NB = NT shares the staged sources (512^2 targets: 121 us at p = 12 in FP32,
// 460 at p = 20 in FP64, against 124 and 603).  Each output is the same
// sequence of MFMA additions in every form, so the forms agree bit for bit.
template <typename T, int KS, bool FUSE, int MX, int NB>
__global__ __launch_bounds__(kThreads * NB) void k_m2l_split(M2LBatch bt, const T *__restrict__ bfrag,
                                                        const double *__restrict__ l2l_frag) {
  constexpr int SX = 8 * MX + 4, SY = 12;  // source boxes staged
  constexpr int NT = (KS + 3) / 4;
  constexpr int REC = 4 * KS + 1;
  constexpr int PD = 3;                    // offsets in flight (27 = 9 PD)
  constexpr int NTH = kThreads * NB;
  constexpr int NG = (NT + NB - 1) / NB;
  extern __shared__ __align__(16) unsigned char lds_raw[];
  T *lds = reinterpret_cast<T *>(lds_raw);

  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t bid = blockIdx.x / NG;
  const int nt = (int)(blockIdx.x - bid * NG) * NB + (wv >> 2);
  int li = 0;
  while (li + 1 < bt.count && bid >= bt.tile_begin[li + 1]) ++li;
  const M2LLevel &a = bt.lv[li];
  const T *__restrict__ mp = static_cast<const T *>(a.mp);
  const int p = bt.p, twop = 2 * p;
  const int64_t ex0 = a.win.bx0 & ~int64_t(1), ey0 = a.win.by0 & ~int64_t(1);
  const int64_t ntx = (a.win.bx0 + a.win.nbx - ex0 + 8 * MX - 1) / (8 * MX);
  const int64_t tile = bid - bt.tile_begin[li];
  const int64_t tx0 = ex0 + 8 * MX * (tile % ntx);
  const int64_t ty0 = ey0 + 8 * (tile / ntx);

  const int quad = wv & 3;
  const int lane = threadIdx.x & 63;
  const int qx = quad & 1, qy = quad >> 1;
  const int i = lane & 15, kq = lane >> 4;

  // the quadrant's offsets (lane j holds the j-th), and the first operators
  const int own = lane < 27 ? lane : 0;
  const int off_x = kIL.t[quad][own][0], off_y = kIL.t[quad][own][1];
  const int boff = ((off_y + 3) * 7 + (off_x + 3)) * (KS * NT * 64);
  const int toff = (off_y * SX + off_x) * REC;
  const T *__restrict__ bsrc = bfrag + nt * 64 + lane;
  T b[PD][KS];
  auto load_b = [&](int j, T (&dst)[KS]) {
    const T *src = bsrc + __builtin_amdgcn_readlane(boff, j);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) dst[ks] = src[ks * NT * 64];
  };
#pragma unroll
  for (int d = 0; d < PD; ++d) load_b(d, b[d]);

  stage_sources<T, KS, SX, SY, NTH>(a, mp, twop, tx0, ty0, lds);

  // target t of M-tile mt
  auto target_xy = [&](int mt, int t, int64_t &gx, int64_t &gy) {
    gx = tx0 + 8 * mt + 2 * (t & 3) + qx;
    gy = ty0 + 2 * (t >> 2) + qy;
    return gx >= a.win.bx0 && gy >= a.win.by0 && gx < a.win.bx0 + a.win.nbx &&
           gy < a.win.by0 + a.win.nby;
  };
  using M = Mfma<T>;
  using M64 = Mfma<double>;

  // L2L of the parents' locals on FP64 MFMA, accumulated apart from the M2L
  d4v acc2[MX];
#pragma unroll
  for (int mt = 0; mt < MX; ++mt) acc2[mt] = d4v{0, 0, 0, 0};
  if constexpr (FUSE) {
    int64_t pidx[MX];
#pragma unroll
    for (int mt = 0; mt < MX; ++mt) {
      int64_t gx, gy;
      pidx[mt] = -1;
      if (target_xy(mt, i, gx, gy))
        pidx[mt] = ((gy >> 1) - a.pwin.by0) * a.pwin.nbx + ((gx >> 1) - a.pwin.bx0);
    }
    const double *lf = l2l_frag + ((size_t)quad * KS * NT + nt) * 64 + lane;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const int k = 4 * ks + kq;
      const double b2 = lf[(size_t)ks * NT * 64];
#pragma unroll
      for (int mt = 0; mt < MX; ++mt) {
        const double av = (pidx[mt] >= 0 && k < twop) ? a.ploc[pidx[mt] * twop + k] : 0.0;
        acc2[mt] = M64::op(av, b2, acc2[mt]);
      }
    }
  }
  __syncthreads();

  typename M::acc acc[MX];
#pragma unroll
  for (int mt = 0; mt < MX; ++mt) acc[mt] = typename M::acc{0, 0, 0, 0};
  const int base = ((2 * (i >> 2) + qy + 2) * SX + (2 * (i & 3) + qx + 2)) * REC + kq;
  for (int j0 = 0; j0 < 27; j0 += PD) {
#pragma unroll
    for (int d = 0; d < PD; ++d) {
      const T *as = lds + base + __builtin_amdgcn_readlane(toff, j0 + d);
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int mt = 0; mt < MX; ++mt)
          acc[mt] = M::op(as[8 * REC * mt + 4 * ks], b[d][ks], acc[mt]);
      if (j0 + PD < 27) load_b(j0 + PD + d, b[d]);
    }
  }

  const double inv_s = 1.0 / a.s;
  const int n = nt * 16 + i;
#pragma unroll
  for (int mt = 0; mt < MX; ++mt) {
    // result in the FP64 layout (lane l, register r: row l/16 + 4 r); FP32
    // has row 4 (l/16) + r, so row l/16 + 4 r is register l/16 of lane
    // 16 r + l%16
    double res[4];
    if constexpr (std::is_same<T, float>::value) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        float v = 0.0f;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const float x = __shfl(acc[mt][q], r * 16 + i, 64);
          v = kq == q ? x : v;
        }
        res[r] = (double)v;
      }
    } else {
#pragma unroll
      for (int r = 0; r < 4; ++r) res[r] = acc[mt][r];
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      int64_t gx, gy;
      if (n >= twop || !target_xy(mt, kq + 4 * r, gx, gy)) continue;
      a.loc[((gy - a.win.by0) * a.win.nbx + (gx - a.win.bx0)) * twop + n] =
          FUSE ? fma(res[r], inv_s, acc2[mt][r]) : res[r] * inv_s;
    }
  }
}

// Tile lists of every level for tiles of w x 8 targets; returns their number.
int64_t list_tiles(M2LBatch &b, int w) {
  int64_t acc = 0;
  for (int i = 0; i < b.count; ++i) {
    const Window &win = b.lv[i].win;
    const int64_t ex0 = win.bx0 & ~int64_t(1), ey0 = win.by0 & ~int64_t(1);
    b.tile_begin[i] = acc;
    acc += ((win.bx0 + win.nbx - ex0 + w - 1) / w) * ((win.by0 + win.nby - ey0 + 7) / 8);
  }
  b.tile_begin[b.count] = acc;
  return acc;
}

template <typename T, int KS, bool FUSE, int MX, int NB>
void split_batch(M2LBatch &b, const T *bfrag, const double *l2l_frag, hipStream_t stream) {
  constexpr int NG = ((KS + 3) / 4 + NB - 1) / NB;
  static_assert(NG * NB == (KS + 3) / 4, "workgroups hold NB whole N-tiles");
  const size_t lds = (size_t)(8 * MX + 4) * 12 * (4 * KS + 1) * sizeof(T);
  const int64_t tiles = list_tiles(b, 8 * MX);
  hipLaunchKernelGGL((k_m2l_split<T, KS, FUSE, MX, NB>), dim3((unsigned)(tiles * NG)),
                     dim3(kThreads * NB), lds, stream, b, bfrag, l2l_frag);
}

// The form of the M2L kernel by the number of 8 x 8 tiles (measured on square
// windows, both sides of each line in us):
//   * up to kFewTiles (2.5 per CU) the finest split: 192^2 targets (576
//     tiles) 29.6 against 34.5 (p = 12, FP32) and 87.1 against 117 (p = 20,
//     FP64); beyond, two tiles and every N-tile per workgroup: 256^2 targets
//     35.3 against 44.8 and 120 against 141;
//   * 16 K-steps in FP64: one tile per workgroup (two leave one workgroup
//     per CU and its registers spill: 512^2 targets 1192 against 1528);
//   * 20 K-steps (five N-tiles, which do not fit one workgroup): in FP32 two
//     tiles from 64 tiles on (96^2 targets 58 against 62), in FP64 k_m2l_wide
//     from 144 on (128^2 targets 135 against 175; 96^2: 124 against 107).
constexpr int64_t kFewTiles = 640;

template <typename T, int KS, bool FUSE>
void mfma_dispatch_tiles(M2LBatch &b, const T *bfrag, const double *l2l_frag, hipStream_t stream) {
  constexpr int NT = (KS + 3) / 4;
  constexpr bool f64 = std::is_same<T, double>::value;
  const int64_t tiles = list_tiles(b, 8);
  if (tiles == 0) return;
  if constexpr (KS == 20) {
    if (tiles <= (f64 ? 144 : 64)) {
      split_batch<T, KS, FUSE, 1, 1>(b, bfrag, l2l_frag, stream);
    } else if constexpr (f64) {
      const size_t lds = (size_t)12 * 12 * (4 * KS + 1) * sizeof(T);
      hipLaunchKernelGGL((k_m2l_wide<KS, FUSE>), dim3((unsigned)tiles), dim3(kThreads), lds, stream,
                         b, bfrag, l2l_frag);
    } else {
      split_batch<T, KS, FUSE, 2, 1>(b, bfrag, l2l_frag, stream);
    }
  } else {
    if (tiles <= kFewTiles)
      split_batch<T, KS, FUSE, 1, 1>(b, bfrag, l2l_frag, stream);
    else
      split_batch<T, KS, FUSE, f64 && KS == 16 ? 1 : 2, NT>(b, bfrag, l2l_frag, stream);
  }
}

// (a workgroup's source tile takes at most 155520 of the chip's 163840 bytes of LDS)
template <typename T, bool FUSE>
void mfma_dispatch(M2LBatch &b, const T *bfrag, const double *l2l_frag, int ks, hipStream_t stream) {
  LENS_KS_DISPATCH(ks, (mfma_dispatch_tiles<T, KS, FUSE>(b, bfrag, l2l_frag, stream)));
  LENS_HIP(hipGetLastError());
}

}  // namespace

void launch_l2l_chain(const L2LChain &c, const OpTables &t, hipStream_t stream) {
  if (c.nlev < 1 || c.nlev > kMaxL2LChain) fail(LENS_EINVAL, "L2L chain: bad level count");
  const int64_t n = c.win[0].count();
  if (n == 0) return;
  LENS_KS_DISPATCH(t.ks, hipLaunchKernelGGL((k_l2l_chain<KS>), dim3((unsigned)n), dim3(kThreads), 0,
                                            stream, c, t.l2l_frag));
  LENS_HIP(hipGetLastError());
}

void launch_m2l_batch(M2LBatch &b, const OpTables &t, bool fp32, hipStream_t stream) {
  if (b.count == 0) return;
  if (fp32)
    mfma_dispatch<float, false>(b, t.bfrag32, nullptr, t.ks, stream);
  else
    mfma_dispatch<double, false>(b, t.bfrag64, nullptr, t.ks, stream);
}

void launch_m2l_l2l(M2LBatch &b, const OpTables &t, bool fp32, hipStream_t stream) {
  if (b.count != 1 || !b.lv[0].ploc) fail(LENS_EINVAL, "M2L + L2L: one level with its parents' locals");
  if (b.lv[0].win.count() == 0) return;
  if (fp32)
    mfma_dispatch<float, true>(b, t.bfrag32, t.l2l_frag, t.ks, stream);
  else
    mfma_dispatch<double, true>(b, t.bfrag64, t.l2l_frag, t.ks, stream);
}

}  // namespace lensfmm
