// Quadtree construction (Appendix A, initialisation step): bounding boxes,
// leaf-box keys, a stable LSD radix sort of (key, index) pairs, gathers and
// per-box start offsets.  Keys are row-major leaf-box indices iy * 2^L + ix,
// so the 3 boxes of one row of a 3x3 neighbourhood are contiguous in the
// sorted order.  The sort is stable and every reduction runs in a fixed
// order, so the tree (and everything computed from it) is bitwise
// reproducible run to run.
#include <cfloat>

#include "device_common.h"

namespace lensfmm {

namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;

// ------------------------------------------------------------ bounding box

// v = {x1min, x2min, x1max, x2max} of the grid-strided points of xy[0, n).
__device__ inline void bbox_accumulate(const double *__restrict__ xy, int64_t n, double v[4]) {
  for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * kThreads) {
    const double a = xy[2 * i], b = xy[2 * i + 1];
    v[0] = fmin(v[0], a);
    v[1] = fmin(v[1], b);
    v[2] = fmax(v[2], a);
    v[3] = fmax(v[3], b);
  }
}

// v = min/max over the parts [0, nparts) of partial boxes laid out [part][4].
__device__ inline void bbox_merge_parts(const double *__restrict__ pp, int nparts, double v[4]) {
  for (int i = threadIdx.x; i < nparts; i += kThreads) {
    v[0] = fmin(v[0], pp[4 * i + 0]);
    v[1] = fmin(v[1], pp[4 * i + 1]);
    v[2] = fmax(v[2], pp[4 * i + 2]);
    v[3] = fmax(v[3], pp[4 * i + 3]);
  }
}

// Reduces every thread's box v over the workgroup (a fixed tree order) and
// writes the result to out[0..3].
__device__ inline void bbox_block_store(const double v[4], double *__restrict__ out) {
  __shared__ double red[4][kThreads];
  for (int c = 0; c < 4; ++c) red[c][threadIdx.x] = v[c];
  __syncthreads();
  for (int o = kThreads / 2; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) {
      red[0][threadIdx.x] = fmin(red[0][threadIdx.x], red[0][threadIdx.x + o]);
      red[1][threadIdx.x] = fmin(red[1][threadIdx.x], red[1][threadIdx.x + o]);
      red[2][threadIdx.x] = fmax(red[2][threadIdx.x], red[2][threadIdx.x + o]);
      red[3][threadIdx.x] = fmax(red[3][threadIdx.x], red[3][threadIdx.x + o]);
    }
    __syncthreads();
  }
  if (threadIdx.x < 4) out[threadIdx.x] = red[threadIdx.x][0];
}

// Per-workgroup bounding box of xy[0, n) (partial[part][4]) and, with
// has_box, the number of points inside the closed rectangle {b0, b1, b2, b3}
// (pcount[part]): one read of the points for both.
// Sum of one value per thread over the workgroup (the result in every thread).
__device__ inline unsigned long long block_sum_u64(unsigned long long c) {
  __shared__ unsigned long long red[kThreads];
  red[threadIdx.x] = c;
  __syncthreads();
  for (int o = kThreads / 2; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  return red[0];
}

__global__ __launch_bounds__(kThreads) void k_bbox_partial(const double *__restrict__ xy, int64_t n,
                                                           int has_box, double b0, double b1,
                                                           double b2, double b3,
                                                           double *__restrict__ partial,
                                                           unsigned long long *__restrict__ pcount) {
  double v[4] = {DBL_MAX, DBL_MAX, -DBL_MAX, -DBL_MAX};
  unsigned long long c = 0;
  for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * kThreads) {
    const double a = xy[2 * i], b = xy[2 * i + 1];
    v[0] = fmin(v[0], a);
    v[1] = fmin(v[1], b);
    v[2] = fmax(v[2], a);
    v[3] = fmax(v[3], b);
    c += (a >= b0 && a <= b2 && b >= b1 && b <= b3) ? 1ull : 0ull;
  }
  bbox_block_store(v, partial + 4 * blockIdx.x);
  if (has_box) {
    c = block_sum_u64(c);
    if (threadIdx.x == 0) pcount[blockIdx.x] = c;
  }
}

// out = {x1min, x2min, x1max, x2max} and, with has_box, the count as the
// bits of out[4]; out may be host-mapped memory (the read-back landing).
__global__ __launch_bounds__(kThreads) void k_bbox_final(const double *__restrict__ partial,
                                                         const unsigned long long *__restrict__ pcount,
                                                         int nparts, int has_box,
                                                         double *__restrict__ out) {
  double v[4] = {DBL_MAX, DBL_MAX, -DBL_MAX, -DBL_MAX};
  bbox_merge_parts(partial, nparts, v);
  bbox_block_store(v, out);
  if (has_box) {
    unsigned long long c = 0;
    for (int i = threadIdx.x; i < nparts; i += kThreads) c += pcount[i];
    c = block_sum_u64(c);
    if (threadIdx.x == 0) reinterpret_cast<unsigned long long *>(out)[4] = c;
  }
}

// Bounding boxes of several point sets at once: blockIdx.y = set; partial
// results [set][part][4], then one workgroup per set reduces its parts.
__global__ __launch_bounds__(kThreads) void k_bbox_multi_partial(const BBoxSet *__restrict__ sets,
                                                                 int nparts,
                                                                 double *__restrict__ partial) {
  const BBoxSet S = sets[blockIdx.y];
  double v[4] = {DBL_MAX, DBL_MAX, -DBL_MAX, -DBL_MAX};
  bbox_accumulate(S.xy, S.n, v);
  bbox_block_store(v, partial + ((size_t)blockIdx.y * nparts + blockIdx.x) * 4);
}

__global__ __launch_bounds__(kThreads) void k_bbox_multi_final(const double *__restrict__ partial,
                                                               int nparts, double *__restrict__ out) {
  double v[4] = {DBL_MAX, DBL_MAX, -DBL_MAX, -DBL_MAX};
  bbox_merge_parts(partial + (size_t)blockIdx.x * nparts * 4, nparts, v);
  bbox_block_store(v, out + (size_t)blockIdx.x * 4);
}

// -------------------------------------------------------------------- keys

// Key of point i: its leaf box of the whole level, row-major (stars), or its
// box of the window `win`, clamped to it (explicit rays, adjoint targets).
struct PointKey {
  const double *xy;
  Geometry g;
  Window win;
  int32_t windowed;
  __device__ uint32_t operator()(int64_t i) const {
    const int64_t nb = int64_t(1) << g.L;
    const double s = ldexp(g.side, -g.L);
    int64_t ix = box_coord(xy[2 * i], g.x0, s, nb);
    int64_t iy = box_coord(xy[2 * i + 1], g.y0, s, nb);
    if (!windowed) return (uint32_t)(iy * nb + ix);
    ix -= win.bx0;
    iy -= win.by0;
    ix = ix < 0 ? 0 : (ix >= win.nbx ? win.nbx - 1 : ix);
    iy = iy < 0 ? 0 : (iy >= win.nby ? win.nby - 1 : iy);
    return (uint32_t)(iy * win.nbx + ix);
  }
};

// Keys of every point; also clears the sort's group totals and, with rec,
// packs the point and its charges into a 32-byte record.
__global__ __launch_bounds__(kThreads) void k_keys(PointKey key, int64_t n, uint32_t *__restrict__ keys,
                                                   uint32_t *__restrict__ zero, int64_t nzero,
                                                   const double *__restrict__ q, int qdim,
                                                   double *__restrict__ rec) {
  const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  for (int64_t z = i; z < nzero; z += (int64_t)gridDim.x * kThreads) zero[z] = 0u;
  if (i >= n) return;
  keys[i] = key(i);
  if (rec) {
    double2 *r = reinterpret_cast<double2 *>(rec) + 2 * i;
    r[0] = make_double2(key.xy[2 * i], key.xy[2 * i + 1]);
    r[1] = qdim == 1 ? make_double2(q[i], 0.0) : make_double2(q[2 * i], q[2 * i + 1]);
  }
}

__global__ __launch_bounds__(kThreads) void k_fill_u32(uint32_t *__restrict__ p, int64_t n,
                                                       uint32_t v) {
  for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * kThreads)
    p[i] = v;
}

// ------------------------------------------------------------------ scans

__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t x, int lane) {
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  return x;
}

// Exclusive scan across the first `WAVES` waves of the workgroup of one value
// per thread (called by all of the workgroup); returns the thread's exclusive
// prefix and writes the total to *total.
template <int WAVES>
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t x, uint32_t *sh /*[WAVES]*/,
                                                    uint32_t *total) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const uint32_t incl = wave_incl_scan(x, lane);
  if (lane == 63 && w < WAVES) sh[w] = incl;
  __syncthreads();
  uint32_t woff = 0, tot = 0;
#pragma unroll
  for (int q = 0; q < WAVES; ++q) {
    if (q < w) woff += sh[q];
    tot += sh[q];
  }
  __syncthreads();
  *total = tot;
  return woff + incl - x;
}

// ------------------------------------------------------------- radix sort
// Stable LSD radix sort of (key, index) pairs, 8 bits a pass, two kernels a
// pass: k_radix_count leaves every tile's digit counts and, by atomics, those
// of groups of ~sqrt(tiles) tiles; a workgroup of k_radix_scatter adds up the
// groups before its own and the tiles of its group before it, some tens of
// loads per digit, which replaced two scan kernels a pass (1e6 keys: 8 launches
// of ~5 us less).

// Tiles of kThreads * ITEMS keys: 2048 (twice as many workgroups as 4096-key
// tiles: 1e6 keys 13.4 us a scatter against 14.2) up to kLongSort keys, 4096
// beyond (a digit's run in a tile is then twice as long: 5e6 keys 37 us against
// 42).
constexpr int kSortItems = 8, kLongSortItems = 16;
constexpr int64_t kLongSort = int64_t(1) << 21;
constexpr int kMaxPasses = 4;

template <int ITEMS>
__global__ __launch_bounds__(kThreads) void k_radix_count(const uint32_t *__restrict__ keys,
                                                          int64_t n, int shift,
                                                          uint32_t *__restrict__ counts,
                                                          uint32_t *__restrict__ groups,
                                                          int tiles_per_group) {
  constexpr int TILE = kThreads * ITEMS;
  __shared__ uint32_t h[256];
  h[threadIdx.x] = 0;
  __syncthreads();
  const int64_t base = (int64_t)blockIdx.x * TILE;
#pragma unroll
  for (int it = 0; it < ITEMS; ++it) {
    const int64_t i = base + (int64_t)it * kThreads + threadIdx.x;
    if (i < n) atomicAdd(&h[(keys[i] >> shift) & 255u], 1u);
  }
  __syncthreads();
  const uint32_t c = h[threadIdx.x];
  counts[(size_t)blockIdx.x * 256 + threadIdx.x] = c;
  if (c) atomicAdd(&groups[(size_t)(blockIdx.x / tiles_per_group) * 256 + threadIdx.x], c);
}

// Ranks one key of each lane among the keys with the same digit that its wave
// has taken: `run` counts those of earlier rounds (one entry per digit, this
// wave's), lanes with the same digit are found with ballots on its bits.
template <typename C>
__device__ __forceinline__ uint32_t wave_rank(uint32_t d, bool valid, int lane, C *run) {
  uint64_t peers = __ballot(valid);
#pragma unroll
  for (int b = 0; b < 8; ++b) {
    const bool bit = (d >> b) & 1u;
    const uint64_t bb = __ballot(bit);
    peers &= bit ? bb : ~bb;
  }
  const uint32_t seen = run[d];
  wave_sync();
  // the highest lane of each digit group records the group
  if (valid && (peers >> lane) == 1ull) run[d] = (C)(seen + __popcll(peers));
  wave_sync();
  return seen + (uint32_t)__popcll(peers & ((1ull << lane) - 1ull));
}

// Where the sorted points go: positions [n][2] and, with q, charges
// [n][qdim] (qdim 1: real masses; 2: complex) and the masses rounded to FP32.
struct PointMove {
  const double *xy, *q;
  int32_t qdim;
  double *sxy, *sq;
  float *sq32;
  __device__ void operator()(int64_t i, int64_t j) const {
    const double x = xy[2 * i], y = xy[2 * i + 1];
    sxy[2 * j] = x;
    sxy[2 * j + 1] = y;
    if (!q) return;
    if (qdim == 1) {
      const double m = q[i];
      sq[j] = m;
      if (sq32) sq32[j] = (float)m;
    } else {
      const double a = q[2 * i], b = q[2 * i + 1];
      sq[2 * j] = a;
      sq[2 * j + 1] = b;
    }
  }
};

// Stable scatter of one tile.  A wave takes ITEMS rounds of 64 consecutive
// keys; a key's place in the tile's own sorted order is its digit's first
// place, plus the keys of that digit in earlier waves, in earlier rounds of its
// wave and in lower lanes.  The tile is put in that order in LDS and then
// written out, so that consecutive lanes write a digit's run (1.6e7 pairs 95 us
// a pass; 171 written straight from the lanes that hold them).  first: the
// values are the points' own indices (none are read).
template <int ITEMS>
__global__ __launch_bounds__(kThreads) void k_radix_scatter(
    const uint32_t *__restrict__ kin, const uint32_t *__restrict__ vin, uint32_t *__restrict__ kout,
    uint32_t *__restrict__ vout, int64_t n, int shift, int first, const uint32_t *__restrict__ counts,
    const uint32_t *__restrict__ groups, int ngroups, int tiles_per_group) {
  constexpr int TILE = kThreads * ITEMS;
  __shared__ uint32_t run[kWaves][256];
  __shared__ uint32_t goff[256];  // a digit's place in the output minus that in the tile
  __shared__ uint32_t sh[kWaves];
  __shared__ uint32_t skey[TILE], sval[TILE];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int64_t tile0 = (int64_t)blockIdx.x * TILE, base = tile0 + w * (ITEMS * 64) + lane;
  uint32_t key[ITEMS], val[ITEMS], rank[ITEMS];
#pragma unroll
  for (int it = 0; it < ITEMS; ++it) {
    const int64_t i = base + it * 64;
    key[it] = i < n ? kin[i] : 0u;
    val[it] = first ? (uint32_t)i : (i < n ? vin[i] : 0u);
  }
  // thread t: digit t's keys in earlier groups, earlier tiles of the group,
  // and in all
  const int group = blockIdx.x / tiles_per_group;
  uint32_t before = 0, total = 0;
#pragma unroll 4
  for (int g = 0; g < ngroups; ++g) {
    const uint32_t c = groups[(size_t)g * 256 + t];
    if (g < group) before += c;
    total += c;
  }
#pragma unroll 4
  for (int q = group * tiles_per_group; q < (int)blockIdx.x; ++q) before += counts[(size_t)q * 256 + t];
#pragma unroll
  for (int q = 0; q < kWaves; ++q) run[q][t] = 0u;
  __syncthreads();
#pragma unroll
  for (int it = 0; it < ITEMS; ++it)
    rank[it] = wave_rank((key[it] >> shift) & 255u, base + it * 64 < n, lane, run[w]);
  uint32_t all;
  const uint32_t out0 = block_excl_scan<kWaves>(total, sh, &all) + before;  // (its barriers: ranks are done)
  uint32_t mine = 0;
#pragma unroll
  for (int q = 0; q < kWaves; ++q) mine += run[q][t];
  uint32_t pre = block_excl_scan<kWaves>(mine, sh, &all);
  goff[t] = out0 - pre;
#pragma unroll
  for (int q = 0; q < kWaves; ++q) {
    const uint32_t c = run[q][t];
    run[q][t] = pre;
    pre += c;
  }
  __syncthreads();
#pragma unroll
  for (int it = 0; it < ITEMS; ++it)
    if (base + it * 64 < n) {
      const uint32_t pos = run[w][(key[it] >> shift) & 255u] + rank[it];
      skey[pos] = key[it];
      sval[pos] = val[it];
    }
  __syncthreads();
  const int cnt = (int)(n - tile0 < TILE ? n - tile0 : TILE);
#pragma unroll
  for (int it = 0; it < ITEMS; ++it) {
    const int e = it * kThreads + t;
    if (e < cnt) {
      const uint32_t k = skey[e], pos = goff[(k >> shift) & 255u] + (uint32_t)e;
      kout[pos] = k;
      vout[pos] = sval[e];
    }
  }
}

// The points moved to their sorted places, a thread each (in the last
// scatter's own workgroups the random reads of 5e6 points took twice as long:
// there are more of them in flight here).  It is bound by the cache lines those
// reads touch, one for the position and one for the charge; from packed
// records (rec) it is one (see kPackFrom).
template <bool REC>
__global__ __launch_bounds__(kThreads) void k_move(PointMove move, const double *__restrict__ rec,
                                                   const uint32_t *__restrict__ perm, int64_t n) {
  const int64_t j = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (j >= n) return;
  const int64_t i = perm[j];
  if (!REC) return move(i, j);
  const double2 *r = reinterpret_cast<const double2 *>(rec) + 2 * i;
  const double2 p = r[0], c = r[1];
  reinterpret_cast<double2 *>(move.sxy)[j] = p;
  if (move.qdim == 1) {
    move.sq[j] = c.x;
    if (move.sq32) move.sq32[j] = (float)c.x;
  } else {
    reinterpret_cast<double2 *>(move.sq)[j] = c;
  }
}

// A whole small tree in one workgroup: keys, two radix passes of half the
// key's bits each in LDS, the points moved to their places and the boxes'
// starts.  Up to 8192 points in up to 16384 boxes (a dozen launches of ~4.6 us
// otherwise).
constexpr int kSmallThreads = 1024, kSmallItems = 8;
constexpr int kSmallPoints = kSmallThreads * kSmallItems, kSmallBoxes = 16384;
constexpr size_t kSmallLds = (size_t)kSmallPoints * 6 + (size_t)(kSmallBoxes + kSmallThreads) * 2 + 64;

__global__ __launch_bounds__(kSmallThreads) void k_tree_small(PointKey pkey, int32_t n, int bits,
                                                              int32_t nbox, uint32_t *__restrict__ perm,
                                                              PointMove move,
                                                              int32_t *__restrict__ start) {
  constexpr int W = kSmallThreads / 64;
  extern __shared__ __align__(16) unsigned char small_lds[];
  uint32_t *skey = reinterpret_cast<uint32_t *>(small_lds);
  uint16_t *sval = reinterpret_cast<uint16_t *>(skey + kSmallPoints);
  uint16_t *run = sval + kSmallPoints;  // [W][256] while sorting, then [nbox] counts
  __shared__ uint32_t sh[W];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int db = (bits + 1) / 2;  // digit bits, at most 8 (bits <= 16)
  const uint32_t mask = (1u << db) - 1u;
  // rounds of 64 points per wave, so that every wave has some
  const int rounds = (n + kSmallThreads - 1) / kSmallThreads;
  const int base = w * (rounds * 64) + lane;
  for (int pass = 0; pass < 2; ++pass) {
    uint32_t key[kSmallItems], val[kSmallItems], rank[kSmallItems];
#pragma unroll
    for (int it = 0; it < kSmallItems; ++it) {
      if (it >= rounds) break;
      const int i = base + it * 64;
      key[it] = i < n ? (pass ? skey[i] : pkey(i)) : 0u;
      val[it] = i < n && pass ? sval[i] : (uint32_t)i;
    }
#pragma unroll
    for (int q = 0; q < W * 256 / kSmallThreads; ++q) run[q * kSmallThreads + t] = 0;
    __syncthreads();
#pragma unroll
    for (int it = 0; it < kSmallItems; ++it) {
      if (it >= rounds) break;
      rank[it] = wave_rank((key[it] >> (pass * db)) & mask, base + it * 64 < n, lane, run + w * 256);
    }
    __syncthreads();
    uint32_t total = 0;
    if (t < 256)
#pragma unroll
      for (int q = 0; q < W; ++q) total += run[q * 256 + t];
    uint32_t all;
    uint32_t pre = block_excl_scan<4>(t < 256 ? total : 0u, sh, &all);
    if (t < 256)
#pragma unroll
      for (int q = 0; q < W; ++q) {
        const uint32_t c = run[q * 256 + t];
        run[q * 256 + t] = (uint16_t)pre;
        pre += c;
      }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < kSmallItems; ++it)
      if (it < rounds && base + it * 64 < n) {
        const uint32_t pos = run[w * 256 + ((key[it] >> (pass * db)) & mask)] + rank[it];
        skey[pos] = key[it];
        sval[pos] = (uint16_t)val[it];
      }
    __syncthreads();
  }
  if (!start) {
    for (int j = t; j < n; j += kSmallThreads) {
      perm[j] = sval[j];
      move(sval[j], j);
    }
    return;
  }
  // starts: counts per box (two to a word), then their prefix
  uint32_t *cnt32 = reinterpret_cast<uint32_t *>(run);
  for (int e = t; e < (nbox + 1) / 2; e += kSmallThreads) cnt32[e] = 0u;
  __syncthreads();
  for (int j = t; j < n; j += kSmallThreads) {
    const uint32_t k = skey[j], i = sval[j];
    atomicAdd(&cnt32[k >> 1], k & 1 ? 0x10000u : 1u);
    perm[j] = i;
    move(i, j);
  }
  __syncthreads();
  constexpr int PER = kSmallBoxes / kSmallThreads;
  uint32_t c[PER], sum = 0;
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int b = t * PER + q;
    c[q] = sum;
    sum += b < nbox ? run[b] : 0u;
  }
  uint32_t all;
  const uint32_t ex = block_excl_scan<W>(sum, sh, &all);
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int b = t * PER + q;
    if (b < nbox) start[b] = (int32_t)(ex + c[q]);
  }
  if (t == 0) start[nbox] = n;
}

// ----------------------------------------------------------------- batches

// Several fields' trees in one pass (batched maps): field j's sources are
// elements [off_j, off_j + n_j) of the combined key/value arrays, keyed
// (j << shift) | leaf key, so one stable sort orders every field by leaf box
// (within a field exactly as its own sort would).
__device__ __forceinline__ int tree_job_of(const TreeJob *__restrict__ jobs, int njobs, int64_t g) {
  int lo = 0, hi = njobs - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (jobs[mid].off <= g) lo = mid; else hi = mid - 1;
  }
  return lo;
}

__global__ __launch_bounds__(kThreads) void k_leaf_keys_multi(const TreeJob *__restrict__ jobs,
                                                              int njobs, int64_t total, int shift,
                                                              uint32_t *__restrict__ keys,
                                                              uint32_t *__restrict__ zero, int64_t nzero) {
  const int64_t gi = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  for (int64_t z = gi; z < nzero; z += (int64_t)gridDim.x * kThreads) zero[z] = 0u;
  if (gi >= total) return;
  const int j = tree_job_of(jobs, njobs, gi);
  const TreeJob &t = jobs[j];
  const int64_t i = gi - t.off;
  const int64_t nb = int64_t(1) << t.g.L;
  const double s = ldexp(t.g.side, -t.g.L);
  const int64_t ix = box_coord(t.xy[2 * i], t.g.x0, s, nb);
  const int64_t iy = box_coord(t.xy[2 * i + 1], t.g.y0, s, nb);
  keys[gi] = ((uint32_t)j << shift) | (uint32_t)(iy * nb + ix);
}

// Sorted position gi of the combined arrays: source perm[gi] (an index of the
// combined arrays, in field j) into that field's sorted arrays; the key loses
// its field bits.
__global__ __launch_bounds__(kThreads) void k_gather_multi(const TreeJob *__restrict__ jobs, int njobs,
                                                           int64_t total, uint32_t mask,
                                                           uint32_t *__restrict__ keys,
                                                           const uint32_t *__restrict__ perm) {
  const int64_t gi = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (gi >= total) return;
  const int j = tree_job_of(jobs, njobs, gi);
  const TreeJob &t = jobs[j];
  const int64_t k = gi - t.off;
  const int64_t i = (int64_t)perm[gi] - t.off;
  t.sxy[2 * k] = t.xy[2 * i];
  t.sxy[2 * k + 1] = t.xy[2 * i + 1];
  t.sq[k] = t.q[i];
  if (t.sq32) t.sq32[k] = (float)t.q[i];
  keys[gi] &= mask;
}

// -------------------------------------------------------------- box starts

// start[b] = lower_bound of box b in the sorted keys, b = 0..nbox, in two
// steps: every stride-th box searches the whole array; then a workgroup per
// stride of boxes counts the keys between its two coarse bounds per box
// (LDS histogram) and writes their exclusive prefix, so each key is read once
// and each entry written once, with no per-box search.  The stride is 256
// boxes (one per thread: more workgroups in flight) for trees of up to 2^22
// leaves and 4096 (16 per thread, so the per-workgroup cost stays small
// against its 16 KB of output) beyond; a stride without keys only fills its
// entries (the deep, mostly empty trees of clustered fields: 2.7e8 boxes).
constexpr int64_t kWideStartsFrom = int64_t(1) << 22;

__global__ __launch_bounds__(kThreads) void k_box_starts_coarse(const uint32_t *__restrict__ keys,
                                                                int64_t n, int64_t nbox,
                                                                int64_t stride,
                                                                int32_t *__restrict__ coarse) {
  const int64_t c = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  const int64_t nc = nbox / stride + 1;
  if (c > nc) return;
  const int64_t b = c * stride < nbox ? c * stride : nbox;
  int64_t lo = 0, hi = n;
  while (lo < hi) {
    const int64_t mid = (lo + hi) >> 1;
    if ((int64_t)keys[mid] < b)
      lo = mid + 1;
    else
      hi = mid;
  }
  coarse[c] = (int32_t)lo;
}

template <int ITEMS>
__global__ __launch_bounds__(kThreads) void k_box_starts(const uint32_t *__restrict__ keys,
                                                         int64_t nbox,
                                                         const int32_t *__restrict__ coarse,
                                                         int32_t *__restrict__ start) {
  constexpr int64_t STRIDE = (int64_t)kThreads * ITEMS;
  __shared__ uint32_t cnt[STRIDE];
  __shared__ uint32_t sh[kWaves];
  const int t = threadIdx.x;
  const int64_t c = blockIdx.x, b0 = c * STRIDE;
  // the keys in [lo, hi) are those of boxes [b0, b0 + stride)
  const int32_t lo = coarse[c], hi = coarse[c + 1];
  const int64_t nb = nbox + 1 - b0 < STRIDE ? nbox + 1 - b0 : STRIDE;
  if (lo == hi) {  // no keys: every start is lo (workgroup-uniform)
    for (int64_t j = t; j < nb; j += kThreads) start[b0 + j] = lo;
    return;
  }
  for (int j = t; j < STRIDE; j += kThreads) cnt[j] = 0;
  __syncthreads();
  for (int64_t j = (int64_t)lo + t; j < hi; j += kThreads) atomicAdd(&cnt[keys[j] - b0], 1u);
  __syncthreads();
  // thread t: boxes [t * ITEMS, (t + 1) * ITEMS), prefixed within the
  // thread, then across the workgroup; the prefixes go back to LDS for
  // coalesced stores
  uint32_t v[ITEMS], sum = 0;
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    v[i] = sum;
    sum += cnt[t * ITEMS + i];
  }
  uint32_t tot;
  const uint32_t ex = block_excl_scan<kWaves>(sum, sh, &tot);
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) cnt[t * ITEMS + i] = ex + v[i];
  __syncthreads();
  for (int64_t j = t; j < nb; j += kThreads) start[b0 + j] = lo + (int32_t)cnt[j];
}

inline unsigned blocks_for(int64_t n, int per = kThreads) {
  return (unsigned)((n + per - 1) / per);
}

}  // namespace

// ------------------------------------------------------------- launchers

int bbox_parts(int64_t n) {
  int64_t b = (n + kThreads * 8 - 1) / (kThreads * 8);
  if (b < 1) b = 1;
  if (b > 1024) b = 1024;
  return (int)b;
}

void launch_bbox(const double *xy, int64_t n, double *partial, int nparts, const double *count_box,
                 double *out, hipStream_t stream) {
  const bool has = count_box != nullptr;
  const double b0 = has ? count_box[0] : 0.0, b1 = has ? count_box[1] : 0.0;
  const double b2 = has ? count_box[2] : -1.0, b3 = has ? count_box[3] : -1.0;
  auto *pcount = reinterpret_cast<unsigned long long *>(partial + 4 * (size_t)nparts);
  hipLaunchKernelGGL(k_bbox_partial, dim3(nparts), dim3(kThreads), 0, stream, xy, n, (int)has, b0,
                     b1, b2, b3, partial, pcount);
  hipLaunchKernelGGL(k_bbox_final, dim3(1), dim3(kThreads), 0, stream, partial, pcount, nparts,
                     (int)has, out);
  LENS_HIP(hipGetLastError());
}

void launch_bbox_multi(const BBoxSet *sets_dev, int nsets, int nparts, double *partial,
                       double *out, hipStream_t stream) {
  if (nsets == 0) return;
  hipLaunchKernelGGL(k_bbox_multi_partial, dim3(nparts, nsets), dim3(kThreads), 0, stream, sets_dev,
                     nparts, partial);
  hipLaunchKernelGGL(k_bbox_multi_final, dim3(nsets), dim3(kThreads), 0, stream, partial, nparts,
                     out);
  LENS_HIP(hipGetLastError());
}

void launch_fill_u32(uint32_t *p, int64_t n, uint32_t v, hipStream_t stream) {
  if (n == 0) return;
  int64_t nb = blocks_for(n);
  if (nb > 4096) nb = 4096;
  hipLaunchKernelGGL(k_fill_u32, dim3((unsigned)nb), dim3(kThreads), 0, stream, p, n, v);
  LENS_HIP(hipGetLastError());
}

namespace {

struct SortShape {
  int items, tiles, per_group, groups;
};

SortShape sort_shape(int64_t n) {
  SortShape s;
  s.items = n > kLongSort ? kLongSortItems : kSortItems;
  const int64_t tile = (int64_t)kThreads * s.items;
  s.tiles = (int)((n + tile - 1) / tile);
  s.per_group = 1;
  while ((int64_t)s.per_group * s.per_group < s.tiles) ++s.per_group;
  s.groups = (s.tiles + s.per_group - 1) / s.per_group;
  return s;
}

// Group totals of every pass, behind the tile counts (cleared with the keys).
uint32_t *group_totals(uint32_t *counts, const SortShape &s) { return counts + (size_t)s.tiles * 256; }
int64_t group_totals_len(const SortShape &s) { return (int64_t)kMaxPasses * s.groups * 256; }

// Sorts by the low `bits` bits; keys in k on entry, the values the points'
// own indices.  Returns true if the result is in the tmp buffers.
template <int ITEMS>
bool radix_passes(uint32_t *k, uint32_t *v, uint32_t *k_tmp, uint32_t *v_tmp, int64_t n, int bits,
                  uint32_t *counts, const SortShape &s, hipStream_t stream) {
  bool in_tmp = false;
  uint32_t *groups = group_totals(counts, s);
  for (int shift = 0; shift < bits; shift += 8, groups += (size_t)s.groups * 256) {
    uint32_t *ki = in_tmp ? k_tmp : k, *vi = in_tmp ? v_tmp : v;
    uint32_t *ko = in_tmp ? k : k_tmp, *vo = in_tmp ? v : v_tmp;
    hipLaunchKernelGGL((k_radix_count<ITEMS>), dim3(s.tiles), dim3(kThreads), 0, stream, ki, n, shift,
                       counts, groups, s.per_group);
    hipLaunchKernelGGL((k_radix_scatter<ITEMS>), dim3(s.tiles), dim3(kThreads), 0, stream, ki, vi, ko, vo, n,
                       shift, (int)(shift == 0), counts, groups, s.groups, s.per_group);
    LENS_HIP(hipGetLastError());
    in_tmp = !in_tmp;
  }
  return in_tmp;
}

bool radix_sort(uint32_t *k, uint32_t *v, uint32_t *k_tmp, uint32_t *v_tmp, int64_t n, int bits,
                uint32_t *counts, const SortShape &s, hipStream_t stream) {
  if (s.items == kLongSortItems)
    return radix_passes<kLongSortItems>(k, v, k_tmp, v_tmp, n, bits, counts, s, stream);
  return radix_passes<kSortItems>(k, v, k_tmp, v_tmp, n, bits, counts, s, stream);
}

}  // namespace

// Points from which the records pay for themselves (their 32 bytes are
// written and read once more: keys and move of 1e6 points 41 us against 44, of
// 5e6 166 against 221, of 1.6e7 587 against 738).
constexpr int64_t kPackFrom = int64_t(1) << 19;

size_t tree_rec_len(int64_t n) { return n >= kPackFrom ? (size_t)n * 4 : 0; }

size_t radix_counts_len(int64_t n) {
  const SortShape s = sort_shape(n < 1 ? 1 : n);
  return (size_t)s.tiles * 256 + (size_t)group_totals_len(s);
}

const uint32_t *launch_tree_sort(const TreeSort &a, hipStream_t stream) {
  if (a.n == 0) {
    if (a.start) launch_box_starts(a.k, 0, a.nbox, a.start, a.coarse, stream);  // all zero
    return a.v;
  }
  int bits = 1;
  while ((int64_t(1) << bits) < a.nbox) ++bits;
  const PointKey key{a.xy, a.g, a.win, a.windowed ? 1 : 0};
  const PointMove move{a.xy, a.q, a.qdim, a.sxy, a.sq, a.qdim == 1 ? a.sq32 : nullptr};
  if (a.n <= kSmallPoints && a.nbox <= kSmallBoxes) {
    hipLaunchKernelGGL(k_tree_small, dim3(1), dim3(kSmallThreads), kSmallLds, stream, key, (int32_t)a.n,
                       bits, (int32_t)a.nbox, a.v, move, a.start);
    LENS_HIP(hipGetLastError());
    return a.v;
  }
  const SortShape s = sort_shape(a.n);
  hipLaunchKernelGGL(k_keys, dim3(blocks_for(a.n)), dim3(kThreads), 0, stream, key, a.n, a.k,
                     group_totals(a.cnt, s), group_totals_len(s), a.q, a.qdim, a.q ? a.rec : nullptr);
  const bool in_tmp = radix_sort(a.k, a.v, a.k_tmp, a.v_tmp, a.n, bits, a.cnt, s, stream);
  const uint32_t *perm = in_tmp ? a.v_tmp : a.v;
  if (a.q && a.rec)
    hipLaunchKernelGGL(k_move<true>, dim3(blocks_for(a.n)), dim3(kThreads), 0, stream, move, a.rec, perm, a.n);
  else
    hipLaunchKernelGGL(k_move<false>, dim3(blocks_for(a.n)), dim3(kThreads), 0, stream, move, nullptr, perm,
                       a.n);
  if (a.start) launch_box_starts(in_tmp ? a.k_tmp : a.k, a.n, a.nbox, a.start, a.coarse, stream);
  return perm;
}

bool launch_sort_multi(const TreeJob *jobs, int njobs, int64_t total, int shift, int bits, uint32_t *k,
                       uint32_t *v, uint32_t *k_tmp, uint32_t *v_tmp, uint32_t *counts,
                       hipStream_t stream) {
  if (total == 0) return false;
  const SortShape s = sort_shape(total);
  hipLaunchKernelGGL(k_leaf_keys_multi, dim3(blocks_for(total)), dim3(kThreads), 0, stream, jobs, njobs,
                     total, shift, k, group_totals(counts, s), group_totals_len(s));
  LENS_HIP(hipGetLastError());
  return radix_sort(k, v, k_tmp, v_tmp, total, bits, counts, s, stream);
}

void launch_gather_multi(const TreeJob *jobs, int njobs, int64_t total, uint32_t mask, uint32_t *keys,
                         const uint32_t *perm, hipStream_t stream) {
  if (total == 0) return;
  hipLaunchKernelGGL(k_gather_multi, dim3(blocks_for(total)), dim3(kThreads), 0, stream, jobs, njobs,
                     total, mask, keys, perm);
  LENS_HIP(hipGetLastError());
}

void launch_box_starts(const uint32_t *sorted_keys, int64_t n, int64_t nbox, int32_t *start,
                       int32_t *coarse, hipStream_t stream) {
  const bool wide = nbox >= kWideStartsFrom;
  const int64_t stride = wide ? (int64_t)kThreads * 16 : kThreads;
  const int64_t nc = nbox / stride + 2;
  hipLaunchKernelGGL(k_box_starts_coarse, dim3(blocks_for(nc)), dim3(kThreads), 0, stream,
                     sorted_keys, n, nbox, stride, coarse);
  const dim3 grid((unsigned)(nbox / stride + 1));
  if (wide)
    hipLaunchKernelGGL(k_box_starts<16>, grid, dim3(kThreads), 0, stream, sorted_keys, nbox, coarse, start);
  else
    hipLaunchKernelGGL(k_box_starts<1>, grid, dim3(kThreads), 0, stream, sorted_keys, nbox, coarse, start);
  LENS_HIP(hipGetLastError());
}

int64_t box_starts_coarse_len(int64_t nbox) { return nbox / kThreads + 2; }

}  // namespace lensfmm
