// bh_build.hip -- tree construction on the GPU (gfx950).
//
// The paper builds the oct-tree on the host (Sec. 4.1, and steps 1-3 of the
// flow listed at the end of Sec. 4.4) and suggests parallelising that part
// (Sec. 7).  Here every step runs on the device, as a pipeline of HBM-bound
// passes with no host round trip:
//
//   bbox     root cube: coordinate-wise min, largest extent L       (Sec. 4.1)
//   keys     63-bit Morton key on the 2^21 grid of the cube         (Sec. 5)
//   sort     stable LSD radix sort of (key, index), 8 x 8-bit digits (Sec. 5,
//            localized particle ordering), then gather to Morton order
//   topology compressed oct-tree read off the sorted unique keys; nodes are
//            numbered in depth-first preorder, so more(c) = c+1 and
//            next(c) = c + subtree size (Sec. 4.4, next/more pointers)
//   moments  FP64 mass and centre of mass, children folded left in octant
//            order, one pass per tree level, deepest first (Sec. 4.4), and
//            the distance s of Eq. (2)
//
// Determinism: integer work is exact; the FP64 sums have a fixed order and use
// only correctly rounded +, *, /, sqrt and fma, so the node set and every node
// value are bit-identical from run to run and independent of launch shapes.
#include "bh_internal.h"

namespace bh {

// ---------------------------------------------------------------- helpers
__device__ __forceinline__ int wave_incl_scan(int x, int lane) {
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    int y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  return x;
}

// Exclusive block scan of one value per thread (blockDim.x = nwaves*64).
template <int NT>
__device__ __forceinline__ int block_excl_scan(int v, int* lds, int* total) {
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  int x = wave_incl_scan(v, lane);
  if (lane == 63) lds[w] = x;
  __syncthreads();
  int pre = 0, tot = 0;
#pragma unroll
  for (int k = 0; k < NT / 64; ++k) {
    int s = lds[k];
    pre += (k < w) ? s : 0;
    tot += s;
  }
  __syncthreads();
  *total = tot;
  return pre + x - v;
}

__global__ void k_fill_i32(int32_t* __restrict__ p, int64_t n, int32_t v) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) p[i] = v;
}

// ---------------------------------------------------------------- scan (int32)
// Device-wide exclusive scan: tile sums, scan of tile sums, per-tile apply.
__global__ __launch_bounds__(kScanThreads) void k_scan_reduce(const int32_t* __restrict__ in, int n,
                                                               int32_t* __restrict__ tile_sums) {
  __shared__ int lds[kScanThreads / 64];
  int64_t base = (int64_t)blockIdx.x * kScanTile;
  int s = 0;
#pragma unroll 4
  for (int r = 0; r < kScanItems; ++r) {
    int64_t i = base + r * kScanThreads + threadIdx.x;
    s += (i < n) ? in[i] : 0;
  }
  int tot;
  block_excl_scan<kScanThreads>(s, lds, &tot);
  if (threadIdx.x == 0) tile_sums[blockIdx.x] = tot;
}

// One block: exclusive scan of the tile sums in place; total to *total.
__global__ __launch_bounds__(1024) void k_scan_tiles(int32_t* __restrict__ sums, int ntiles,
                                                     int32_t* __restrict__ total) {
  __shared__ int lds[16];
  const int t = threadIdx.x;
  int per = (ntiles + 1023) / 1024;
  int b = t * per, e = min(ntiles, b + per);
  int s = 0;
  for (int k = b; k < e; ++k) s += sums[k];
  int tot;
  int pre = block_excl_scan<1024>(s, lds, &tot);
  for (int k = b; k < e; ++k) {
    int v = sums[k];
    sums[k] = pre;
    pre += v;
  }
  if (t == 0 && total) *total = tot;
}

__global__ __launch_bounds__(kScanThreads) void k_scan_apply(const int32_t* __restrict__ in, int n,
                                                              const int32_t* __restrict__ tile_offs,
                                                              int32_t* __restrict__ out) {
  __shared__ int tile[kScanTile];
  __shared__ int lds[kScanThreads / 64];
  const int t = threadIdx.x;
  int64_t base = (int64_t)blockIdx.x * kScanTile;
  for (int r = 0; r < kScanItems; ++r) {
    int64_t i = base + r * kScanThreads + t;
    tile[r * kScanThreads + t] = (i < n) ? in[i] : 0;
  }
  __syncthreads();
  int s = 0;
  for (int k = 0; k < kScanItems; ++k) s += tile[t * kScanItems + k];
  int tot;
  int pre = block_excl_scan<kScanThreads>(s, lds, &tot) + tile_offs[blockIdx.x];
  for (int k = 0; k < kScanItems; ++k) {
    int v = tile[t * kScanItems + k];
    tile[t * kScanItems + k] = pre;
    pre += v;
  }
  __syncthreads();
  for (int r = 0; r < kScanItems; ++r) {
    int64_t i = base + r * kScanThreads + t;
    if (i < n) out[i] = tile[r * kScanThreads + t];
  }
}

// k_scan_apply for at most kScanFuseTiles tiles, without the pass over the
// tile sums: each block adds up the sums of the tiles before it itself (at most
// kScanFuseTiles / kScanThreads loads per thread), which saves a launch.
constexpr int kScanFuseTiles = 2048;
__global__ __launch_bounds__(kScanThreads) void k_scan_apply_sum(const int32_t* __restrict__ in, int n,
                                                                  const int32_t* __restrict__ tile_sums,
                                                                  int32_t* __restrict__ out,
                                                                  int32_t* __restrict__ total) {
  __shared__ int tile[kScanTile];
  __shared__ int lds[kScanThreads / 64];
  const int t = threadIdx.x;
  int o = 0;
  for (int k = t; k < (int)blockIdx.x; k += kScanThreads) o += tile_sums[k];
  int off;
  block_excl_scan<kScanThreads>(o, lds, &off);
  int64_t base = (int64_t)blockIdx.x * kScanTile;
  for (int r = 0; r < kScanItems; ++r) {
    int64_t i = base + r * kScanThreads + t;
    tile[r * kScanThreads + t] = (i < n) ? in[i] : 0;
  }
  __syncthreads();
  int s = 0;
  for (int k = 0; k < kScanItems; ++k) s += tile[t * kScanItems + k];
  int tot;
  int pre = block_excl_scan<kScanThreads>(s, lds, &tot) + off;
  for (int k = 0; k < kScanItems; ++k) {
    int v = tile[t * kScanItems + k];
    tile[t * kScanItems + k] = pre;
    pre += v;
  }
  __syncthreads();
  for (int r = 0; r < kScanItems; ++r) {
    int64_t i = base + r * kScanThreads + t;
    if (i < n) out[i] = tile[r * kScanThreads + t];
  }
  if (total && t == 0 && blockIdx.x == gridDim.x - 1) *total = off + tot;
}

hipError_t scan_excl(const int32_t* in, int32_t* out, int n, int32_t* tile_buf, int32_t* total,
                     hipStream_t st) {
  int ntiles = (n + kScanTile - 1) / kScanTile;
  if (ntiles == 0) ntiles = 1;
  k_scan_reduce<<<ntiles, kScanThreads, 0, st>>>(in, n, tile_buf);
  if (ntiles <= kScanFuseTiles) {
    k_scan_apply_sum<<<ntiles, kScanThreads, 0, st>>>(in, n, tile_buf, out, total);
  } else {
    k_scan_tiles<<<1, 1024, 0, st>>>(tile_buf, ntiles, total);
    k_scan_apply<<<ntiles, kScanThreads, 0, st>>>(in, n, tile_buf, out);
  }
  return hipGetLastError();
}

// ---------------------------------------------------------------- start of a build
// What a sort needs beside its keys: the passes' histograms and tickets, and two
// tables of tile words, which the passes use in turn (each clears the other's
// for the next one).
struct SortScratch {
  int32_t* hist;     // [kSortPasses][256]
  int32_t* ticket;   // [kSortPasses]
  uint32_t* tiles[2];
};

__device__ __forceinline__ void clear_sort(int32_t* __restrict__ hist, int32_t* __restrict__ ticket,
                                           uint32_t* __restrict__ tiles, int64_t words) {
  const int64_t i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, step = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = i0; i < kSortPasses * 256; i += step) hist[i] = 0;
  if (i0 <= kSortPasses) ticket[i0] = 0;
  for (int64_t i = i0; i < words; i += step) tiles[i] = 0;
}

__global__ __launch_bounds__(256) void k_clear_sort(int32_t* __restrict__ hist, int32_t* __restrict__ ticket,
                                                    uint32_t* __restrict__ tiles, int64_t words) {
  clear_sort(hist, ticket, tiles, words);
}

// The start of a build: counters, offsets, the sort's words, run ancestors, and
// cluster roots for an empty build (every cluster starts and ends at node 0).
// By every thread of a launch.
__device__ __forceinline__ void init_build(const BuildWs& w, const SortScratch& sc, int64_t n, int64_t words,
                                           int64_t n_anc) {
  const int64_t i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, step = (int64_t)gridDim.x * blockDim.x;
  if (i0 < (int64_t)(sizeof(Counts) / 4)) reinterpret_cast<int32_t*>(w.counts)[i0] = 0;
  if (w.seg_off == w.own_off && i0 < 2) w.own_off[i0] = i0 ? n : 0;
  for (int64_t i = i0; i <= w.n_seg; i += step) w.croot[i] = n > 0 ? -1 : 0;
  for (int64_t i = i0; i < n_anc; i += step) w.anc[i] = -1;
  if (words) clear_sort(sc.hist, sc.ticket, sc.tiles[0], words);
}

__global__ __launch_bounds__(256) void k_init(BuildWs w, SortScratch sc, int64_t n, int64_t words, int64_t n_anc) {
  init_build(w, sc, n, words, n_anc);
}

// ---------------------------------------------------------------- bbox
// Per workgroup the coordinate-wise extremes and whether an input is not finite
// (w.bbox_part [7][gridDim.x]).  The launch also starts the build: nothing else
// reads or counts into what init_build clears before the next launch.  (A launch
// of its own for that took 5 to 6 us of every build.)
template <typename T>
__global__ __launch_bounds__(256) void k_bbox_partial(const T* __restrict__ pos, const T* __restrict__ mass,
                                                      int64_t n, BuildWs ws, SortScratch sc, int64_t words,
                                                      int64_t n_anc) {
  init_build(ws, sc, n, words, n_anc);
  __shared__ double red[6][4];
  double mn[3] = {INFINITY, INFINITY, INFINITY};
  double mx[3] = {-INFINITY, -INFINITY, -INFINITY};
  bool bad = false;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      double v = (double)pos[3 * i + d];
      if (!isfinite(v)) {
        bad = true;
      } else {
        mn[d] = fmin(mn[d], v);
        mx[d] = fmax(mx[d], v);
      }
    }
    if (!isfinite((double)mass[i])) bad = true;
  }
  bad = __syncthreads_or(bad);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    double a = mn[d], b = mx[d];
    for (int o = 32; o > 0; o >>= 1) {
      a = fmin(a, __shfl_xor(a, o, 64));
      b = fmax(b, __shfl_xor(b, o, 64));
    }
    if (lane == 0) {
      red[d][w] = a;
      red[3 + d][w] = b;
    }
  }
  __syncthreads();
  if (threadIdx.x < 6) {
    int k = threadIdx.x;
    double v = red[k][0];
    for (int q = 1; q < 4; ++q) v = (k < 3) ? fmin(v, red[k][q]) : fmax(v, red[k][q]);
    ws.bbox_part[k * gridDim.x + blockIdx.x] = v;
  }
  if (threadIdx.x == 6) ws.bbox_part[6 * gridDim.x + blockIdx.x] = bad ? 1.0 : 0.0;
}

// Root cube from the coordinate-wise extremes: lo = minimum corner, side L =
// largest extent (1 if every particle coincides or there is none).
__device__ void finish_cube(double lo[3], double hi[3], Cube* __restrict__ cube) {
  double L = 0.0;
  for (int d = 0; d < 3; ++d) {
    if (!(lo[d] <= hi[d])) {  // no finite particle at all
      lo[d] = 0.0;
      hi[d] = 0.0;
    }
    double e = hi[d] - lo[d];
    if (e > L) L = e;
  }
  if (L == 0.0) L = 1.0;
  for (int d = 0; d < 3; ++d) cube->lo[d] = lo[d];
  cube->L = L;
  cube->scale = (double)kGrid / L;
}

// One wave per row of the workgroups' extremes (min and max are exact, so the
// order does not matter); the last finds the inputs that are not finite.  (One
// wave for all rows, in turn, took 8.5 us.)
__global__ __launch_bounds__(448) void k_bbox_final(const double* __restrict__ part, int nb, Cube* __restrict__ cube,
                                                    Counts* __restrict__ cnt) {
  __shared__ double ext[6];
  const int lane = threadIdx.x & 63, k = threadIdx.x >> 6;
  double v = k < 3 ? INFINITY : -INFINITY;
#pragma unroll 4
  for (int b = lane; b < nb; b += 64) v = k < 3 ? fmin(v, part[k * nb + b]) : fmax(v, part[k * nb + b]);
  for (int o = 32; o > 0; o >>= 1) {
    const double u = __shfl_xor(v, o, 64);
    v = k < 3 ? fmin(v, u) : fmax(v, u);
  }
  if (lane == 0) {
    if (k < 6)
      ext[k] = v;
    else if (v > 0.0)
      atomicOr(&cnt->bad_input, 1);
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double e[6];
    for (int q = 0; q < 6; ++q) e[q] = ext[q];
    finish_cube(e, e + 3, cube);
  }
}

// Offsets of a forest: off[0] = 0, nondecreasing, off[K] = n.  A violation is
// reported through bad_input; every later pass clamps ranges to [0, n], so a bad
// offset array can give wrong trees but never an access out of bounds.
__global__ __launch_bounds__(256) void k_seg_check(const int64_t* __restrict__ off, int K, int64_t n,
                                                   Counts* __restrict__ cnt) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k > K) return;
  const int64_t v = off[k];
  bool bad = v < 0 || v > n || (k == 0 && v != 0) || (k == K && v != n) || (k < K && off[k + 1] < v);
  if (bad) atomicOr(&cnt->bad_input, 2);
}

__device__ __forceinline__ int64_t clamp_off(int64_t v, int64_t n) { return v < 0 ? 0 : (v > n ? n : v); }

// Cluster of caller index i: the k with off[k] <= i < off[k+1] (off in global
// memory or in an LDS copy).
template <typename P>
__device__ __forceinline__ int seg_of(P off, int K, int64_t i) {
  int lo = 0, hi = K;
  while (hi - lo > 1) {
    int mid = (lo + hi) >> 1;
    if (off[mid] <= i) lo = mid; else hi = mid;
  }
  return lo;
}

// Root cube of every cluster of a forest: one workgroup per cluster.
template <typename T>
__global__ __launch_bounds__(256) void k_bbox_seg(const T* __restrict__ pos, const T* __restrict__ mass,
                                                  const int64_t* __restrict__ off, int64_t n,
                                                  Cube* __restrict__ cube, Counts* __restrict__ cnt) {
  __shared__ double red[6][4];
  const int k = blockIdx.x;
  const int64_t b = clamp_off(off[k], n), e = max(b, clamp_off(off[k + 1], n));
  double v[6] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY};
  bool bad = false;
  for (int64_t i = b + threadIdx.x; i < e; i += blockDim.x) {
    for (int d = 0; d < 3; ++d) {
      double x = (double)pos[3 * i + d];
      if (!isfinite(x)) {
        bad = true;
      } else {
        v[d] = fmin(v[d], x);
        v[3 + d] = fmax(v[3 + d], x);
      }
    }
    if (!isfinite((double)mass[i])) bad = true;
  }
  if (__any(bad) && lane_id() == 0) atomicOr(&cnt->bad_input, 1);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  for (int q = 0; q < 6; ++q) {
    for (int o = 32; o > 0; o >>= 1) {
      double u = __shfl_xor(v[q], o, 64);
      v[q] = q < 3 ? fmin(v[q], u) : fmax(v[q], u);
    }
    if (lane == 0) red[q][w] = v[q];
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int q = 0; q < 6; ++q)
      for (int r = 1; r < 4; ++r) red[q][0] = q < 3 ? fmin(red[q][0], red[q][r]) : fmax(red[q][0], red[q][r]);
    double lo[3] = {red[0][0], red[1][0], red[2][0]}, hi[3] = {red[3][0], red[4][0], red[5][0]};
    finish_cube(lo, hi, cube + k);
  }
}

// ---------------------------------------------------------------- Morton keys
__device__ __forceinline__ uint64_t spread3(uint64_t v) {
  v &= 0x1fffffull;
  v = (v | (v << 32)) & 0x1f00000000ffffull;
  v = (v | (v << 16)) & 0x1f0000ff0000ffull;
  v = (v | (v << 8)) & 0x100f00f00f00f00full;
  v = (v | (v << 4)) & 0x10c30c30c30c30c3ull;
  v = (v | (v << 2)) & 0x1249249249249249ull;
  return v;
}

__device__ __forceinline__ uint32_t compact3(uint64_t v) {
  v &= 0x1249249249249249ull;
  v = (v ^ (v >> 2)) & 0x10c30c30c30c30c3ull;
  v = (v ^ (v >> 4)) & 0x100f00f00f00f00full;
  v = (v ^ (v >> 8)) & 0x1f0000ff0000ffull;
  v = (v ^ (v >> 16)) & 0x1f00000000ffffull;
  v = (v ^ (v >> 32)) & 0x1fffffull;
  return (uint32_t)v;
}

// q_d = clamp(floor((x_d - lo_d) * 2^21/L), 0, 2^21-1); key interleaves the
// bits with x as the most significant bit of each triplet, so the octant of a
// child is 4*bx + 2*by + bz and key order is depth-first (Morton) order.
template <typename T>
__device__ __forceinline__ uint64_t morton_key(const Cube& cube, const T* __restrict__ pos, int i) {
  const double sc = cube.scale;
  uint64_t q[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    double t = floor(((double)pos[3 * (int64_t)i + d] - cube.lo[d]) * sc);
    if (!(t >= 0.0)) t = 0.0;  // also maps a non-finite input to 0 (flagged by bbox)
    if (t > (double)(kGrid - 1)) t = (double)(kGrid - 1);
    q[d] = (uint64_t)t;
  }
  return (spread3(q[0]) << 2) | (spread3(q[1]) << 1) | spread3(q[2]);
}

// ---------------------------------------------------------------- radix sort
// Digit sources of a pass: 8 bits of the key, or 8 bits of the item's cluster.
// The cluster of caller index v is a search over the cluster offsets, staged in
// LDS when they fit (the offsets are sorted and caller order keeps each cluster
// contiguous), else the per-index cluster array, which the key passes leave in
// no useful order, so that lookup is a scattered read.
enum SortDigit { kDigKey = 0, kDigSegLds = 1, kDigSegIdx = 2 };
constexpr int kSegLds = 2048;  // most cluster offsets (K + 1) staged in LDS

template <int kDig>
struct SegTable {
  // off[0..K] when the offsets sit in LDS
  int64_t off[kDig == kDigSegLds ? kSegLds : 1];
  __device__ __forceinline__ void load(const int64_t* __restrict__ g, int K) {
    if constexpr (kDig == kDigSegLds) {
      for (int k = threadIdx.x; k <= K; k += blockDim.x) off[k] = g[k];
    }
  }
  __device__ __forceinline__ uint32_t digit(uint64_t key, int32_t val, const int32_t* __restrict__ seg, int K,
                                            int shift) const {
    if constexpr (kDig == kDigKey) return (uint32_t)(key >> shift) & 255u;
    if constexpr (kDig == kDigSegLds) return ((uint32_t)seg_of(off, K, val) >> shift) & 255u;
    return ((uint32_t)seg[val] >> shift) & 255u;
  }
};

// One launch per pass.  A workgroup takes the next tile (a ticket, so that tiles
// start in order), counts its digits, and learns how many items of each digit
// the tiles before it hold by looking back over what they have published: per
// tile and digit a word with the tile's own count or, once known, the count of
// all tiles up to it ("decoupled look-back", Merrill & Garland 2016).  A word
// carries its own state, so it needs no fence; a tile waits only for tiles that
// started before it.  Where each digit starts comes from the histograms that
// the key kernel has added up for all passes.
//
// The scatter is stable and goes through LDS.  Each wave takes a contiguous
// quarter of the tile and ranks its items in input order (the rank among equal
// digits within 64 items comes from 8 ballots, one per digit bit); the items
// are placed in LDS sorted by digit, and the tile then leaves in that order, so
// that consecutive lanes write consecutive addresses of one digit's run instead
// of 8- and 4-byte pieces all over the output.
//
// A pass moves 24 bytes per particle and, for small sets, is one tile's latency:
// smaller tiles for those, so that more CUs take part (sort_items).  (As a
// histogram, two scan kernels and a scatter a pass took 33 us for 100,000
// particles, 49 for 1M and 64 for 4M; it takes 10, 23 and 54, the digit counts of
// the key kernel 5 more in all, 25 at 4M.)
constexpr uint32_t kTileCount = 1u << 30, kTileTotal = 2u << 30, kTileMask = kTileCount - 1;

template <int kDig, int kItems>
__global__ __launch_bounds__(kSortThreads) void k_rs_pass(const uint64_t* __restrict__ kin,
                                                          const int32_t* __restrict__ vin,
                                                          const int32_t* __restrict__ seg,
                                                          const int64_t* __restrict__ seg_off, int K,
                                                          uint64_t* __restrict__ kout, int32_t* __restrict__ vout, int n,
                                                          int shift, const int32_t* __restrict__ hist,
                                                          uint32_t* tiles, uint32_t* __restrict__ tiles_next,
                                                          int32_t* __restrict__ ticket, int ntiles) {
  constexpr int kWaves = kSortThreads / 64;
  constexpr int kTile = kSortThreads * kItems;
  constexpr int kPerWave = kTile / kWaves;
  __shared__ uint64_t lkey[kTile];
  __shared__ int32_t lval[kTile];
  __shared__ uint8_t ldig[kTile];
  __shared__ uint32_t goff[256];           // output position of the tile's first item of each digit
  __shared__ uint32_t loff[256];           // tile position of the first item of each digit
  __shared__ uint32_t wslot[kWaves][256];  // per wave: its counts, then its first slot per digit
  __shared__ int scan[kWaves];
  __shared__ SegTable<kDig> tab;
  __shared__ int tile_s;
  const int t = threadIdx.x, w = t >> 6, lane = t & 63;
  if (t == 0) tile_s = atomicAdd(ticket, 1);
#pragma unroll
  for (int k = 0; k < kWaves; ++k) wslot[k][t] = 0;
  tab.load(seg_off, K);
  __syncthreads();
  const int tile = tile_s;
  if (tile >= ntiles) return;
  const int64_t tile0 = (int64_t)tile * kTile;
  const int m = (int)min((int64_t)kTile, (int64_t)n - tile0);  // items in this tile
  uint64_t key[kItems];
  int32_t val[kItems];
  uint32_t at[kItems];  // digit << 16 | rank among the wave's items of that digit
#pragma unroll
  for (int r = 0; r < kItems; ++r) {
    const int j = w * kPerWave + r * 64 + lane;
    key[r] = j < m ? kin[tile0 + j] : 0ull;
    val[r] = j < m ? vin[tile0 + j] : 0;
  }
  const uint64_t lt = (1ull << lane) - 1ull;
#pragma unroll
  for (int r = 0; r < kItems; ++r) {
    const bool valid = w * kPerWave + r * 64 + lane < m;
    const uint32_t d = valid ? tab.digit(key[r], val[r], seg, K, shift) : 0u;
    uint64_t peers = ballot(valid);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      const bool bit = (d >> b) & 1u;
      const uint64_t mk = ballot(bit);
      peers &= bit ? mk : ~mk;
    }
    const int leader = valid ? __builtin_ctzll(peers) : lane;
    uint32_t base = 0;
    if (valid && lane == leader) base = atomicAdd(&wslot[w][d], (uint32_t)__popcll(peers));
    at[r] = d << 16 | (__shfl(base, leader, 64) + (uint32_t)__popcll(peers & lt));
  }
  __syncthreads();
  // digit t: the tile's count, published for the tiles after this one
  uint32_t cw[kWaves], c = 0;
#pragma unroll
  for (int k = 0; k < kWaves; ++k) c += cw[k] = wslot[k][t];
  uint32_t* mine = tiles + (int64_t)tile * 256 + t;
  __hip_atomic_store(mine, (tile == 0 ? kTileTotal : kTileCount) | c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  tiles_next[(int64_t)tile * 256 + t] = 0;
  // each digit's first position in the tile and in the output, each wave's first slot
  int tot;
  const uint32_t first = (uint32_t)block_excl_scan<kSortThreads>((int)c, scan, &tot);
  const uint32_t digit0 = (uint32_t)block_excl_scan<kSortThreads>(hist[t], scan, &tot);
  loff[t] = first;
  uint32_t run = first;
#pragma unroll
  for (int k = 0; k < kWaves; ++k) {
    wslot[k][t] = run;
    run += cw[k];
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kItems; ++r) {
    if (w * kPerWave + r * 64 + lane < m) {
      const uint32_t d = at[r] >> 16, q = wslot[w][d] + (at[r] & 0xffffu);
      lkey[q] = key[r];
      lval[q] = val[r];
      ldig[q] = (uint8_t)d;
    }
  }
  // look back, kBack tiles at a time
  constexpr int kBack = 8;
  uint32_t before = 0;
  for (int p = tile - 1; p >= 0;) {
    uint32_t word[kBack];
#pragma unroll
    for (int k = 0; k < kBack; ++k)
      word[k] = p - k >= 0 ? __hip_atomic_load(tiles + (int64_t)(p - k) * 256 + t, __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_AGENT)
                           : 0u;
    bool open = true;  // no tile without a word met yet
#pragma unroll
    for (int k = 0; k < kBack; ++k) {
      if (!open) continue;
      if (word[k] == 0u) {
        open = false;
      } else {
        before += word[k] & kTileMask;
        --p;
        if (word[k] & kTileTotal) {
          p = -1;
          open = false;
        }
      }
    }
    if (p >= 0 && !open) __builtin_amdgcn_s_sleep(1);
  }
  if (tile > 0) __hip_atomic_store(mine, kTileTotal | (before + c), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  goff[t] = digit0 + before;
  __syncthreads();
  // the tile in digit order: position j holds the (j - loff[d])-th item of digit d
#pragma unroll
  for (int r = 0; r < kItems; ++r) {
    const int j = r * kSortThreads + t;
    if (j < m) {
      const uint32_t d = ldig[j];
      const uint32_t q = goff[d] + (uint32_t)j - loff[d];
      kout[q] = lkey[j];
      vout[q] = lval[j];
    }
  }
}

// Adds the digits of one item to the histograms of all passes in LDS
// (h [kSortPasses][256]): key digits, then cluster digits.
__device__ __forceinline__ void count_digits(uint32_t (*h)[256], uint64_t key, int key_passes, uint32_t cluster,
                                             int seg_passes) {
  for (int p = 0; p < key_passes; ++p) atomicAdd(&h[p][(uint32_t)(key >> (8 * p)) & 255u], 1u);
  for (int p = 0; p < seg_passes; ++p) atomicAdd(&h[key_passes + p][(cluster >> (8 * p)) & 255u], 1u);
}
__device__ __forceinline__ void clear_digits(uint32_t (*h)[256], int passes) {
  for (int k = threadIdx.x; k < passes * 256; k += blockDim.x) h[0][k] = 0;
  __syncthreads();
}
__device__ __forceinline__ void store_digits(uint32_t (*h)[256], int passes, int32_t* __restrict__ hist) {
  __syncthreads();
  for (int k = threadIdx.x; k < passes * 256; k += blockDim.x)
    if (h[0][k]) atomicAdd(&hist[k], (int32_t)h[0][k]);
}

// Workgroups of a key kernel: each ends with an atomic per digit and pass, so
// few large ones.
constexpr int kKeyThreads = 512;
static inline int key_blocks(int64_t n) { return (int)min((int64_t)512, max((int64_t)1, (n + 2047) / 2048)); }

template <int kDig>
static void launch_pass(const uint64_t* kin, const int32_t* vin, const BuildWs& w, uint64_t* kout, int32_t* vout, int n,
                        int shift, const SortScratch& sc, int pass, hipStream_t st) {
  const int items = sort_items(n);
  const int ntiles = (int)sort_tiles(n);
  auto go = [&](auto kernel) {
    kernel<<<ntiles, kSortThreads, 0, st>>>(kin, vin, w.seg, w.seg_off, w.n_seg, kout, vout, n, shift,
                                            sc.hist + 256 * pass, sc.tiles[pass & 1], sc.tiles[(pass & 1) ^ 1],
                                            sc.ticket + pass, ntiles);
  };
  if (items == 4)
    go(k_rs_pass<kDig, 4>);
  else if (items == 8)
    go(k_rs_pass<kDig, 8>);
  else
    go(k_rs_pass<kDig, 16>);
}

template <typename T>
__global__ __launch_bounds__(kKeyThreads) void k_keys(const T* __restrict__ pos, int n, const Cube* __restrict__ cubes,
                                                      const int64_t* __restrict__ off, int K, int seg_passes,
                                                      int32_t* __restrict__ seg, uint64_t* __restrict__ keys,
                                                      int32_t* __restrict__ idx, int32_t* __restrict__ hist) {
  __shared__ uint32_t h[kSortPasses][256];
  const int passes = 8 + seg_passes;
  clear_digits(h, passes);
  for (int64_t i = (int64_t)blockIdx.x * kKeyThreads + threadIdx.x; i < n; i += (int64_t)gridDim.x * kKeyThreads) {
    const int k = K > 1 ? seg_of(off, K, i) : 0;
    if (seg) seg[i] = k;
    const uint64_t key = morton_key(cubes[k], pos, (int)i);
    keys[i] = key;
    idx[i] = (int32_t)i;
    count_digits(h, key, 8, (uint32_t)k, seg_passes);
  }
  store_digits(h, passes, hist);
}

__global__ __launch_bounds__(256) void k_copy_kv(const uint64_t* __restrict__ kin, const int32_t* __restrict__ vin,
                                                 uint64_t* __restrict__ kout, int32_t* __restrict__ vout, int n) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  kout[i] = kin[i];
  vout[i] = vin[i];
}

// ---------------------------------------------------------------- gather
template <typename T, typename T4>
__global__ __launch_bounds__(256) void k_gather(const T* __restrict__ pos, const T* __restrict__ mass,
                                                const int32_t* __restrict__ perm, const int32_t* __restrict__ seg,
                                                int n, T4* __restrict__ ps, int32_t* __restrict__ scid) {
  // (Morton neighbours often sit close together in the caller's order, e.g.
  // particles of one cluster: runs of consecutive blocks per XCD keep their
  // source lines in one L2)
  const int k = remap_block(blockIdx.x, gridDim.x, 64) * blockDim.x + threadIdx.x;
  if (k >= n) return;
  int64_t j = perm[k];
  if (scid) scid[k] = seg[j];
  T4 v;
  v.x = pos[3 * j];
  v.y = pos[3 * j + 1];
  v.z = pos[3 * j + 2];
  v.w = mass[j];
  ps[k] = v;
}

// ---------------------------------------------------------------- unique keys
// A leaf per distinct (cluster, key): their keys, first positions and clusters,
// compacted in one pass with the look-back of the sort (one word per tile, 64
// tiles at a time); and the first unique key of every cluster that has particles
// and of the one after it (the sort keeps the clusters one after the other), which
// is what k_pairs reads; k_croot_final finds the other empty clusters'.  (With the
// key's lane writing every empty cluster before it, a build of 2^22 clusters with
// 1000 particles in the last took 141 ms; it takes 13.7.)
// It also clears the counters of k_pairs.  (Flags, two scan kernels and the
// write took 36 us for 1M particles and 80 for 4M; this takes 23 and 52.)
constexpr int kUniqueItems = 8;
constexpr int kUniqueTile = kSortThreads * kUniqueItems;
inline int unique_tiles(int64_t n) { return (int)((n + kUniqueTile - 1) / kUniqueTile); }

__global__ __launch_bounds__(kSortThreads) void k_unique(const uint64_t* __restrict__ keys,
                                                         const int32_t* __restrict__ scid, int n, int K,
                                                         uint64_t* __restrict__ ukey, int32_t* __restrict__ ustart,
                                                         int32_t* __restrict__ ucid, Counts* __restrict__ cnt,
                                                         int32_t* __restrict__ nstart, uint32_t* __restrict__ lmask,
                                                         int32_t* __restrict__ croot, uint32_t* tiles,
                                                         int32_t* __restrict__ ticket, int ntiles) {
  constexpr int kWaves = kSortThreads / 64;
  __shared__ int chunk[kUniqueItems * kWaves];  // unique keys of each 64 items, then those before them in the tile
  __shared__ int tile_s, before_s;
  const int t = threadIdx.x, w = t >> 6, lane = t & 63;
  if (t == 0) tile_s = atomicAdd(ticket, 1);
  __syncthreads();
  const int tile = tile_s;
  if (tile >= ntiles) return;
  const int i0 = tile * kUniqueTile;
  uint64_t key[kUniqueItems], mask[kUniqueItems];
#pragma unroll
  for (int r = 0; r < kUniqueItems; ++r) {
    const int i = i0 + r * kSortThreads + t;
    const bool valid = i < n;
    key[r] = valid ? keys[i] : 0ull;
    const bool fl = valid && (i == 0 || key[r] != keys[i - 1] || (scid && scid[i] != scid[i - 1]));
    mask[r] = ballot(fl);
    if (lane == 0) chunk[r * kWaves + w] = __popcll(mask[r]);
    if (valid) {
      nstart[i] = 0;
      lmask[i] = 0;
    }
  }
  __syncthreads();
  if (w == 0) {
    // the tile's count, the chunks' offsets, and the tiles before this one
    const int c = lane < kUniqueItems * kWaves ? chunk[lane] : 0;
    const int incl = wave_incl_scan(c, lane);
    if (lane < kUniqueItems * kWaves) chunk[lane] = incl - c;
    const uint32_t total = (uint32_t)__shfl(incl, 63, 64);
    if (lane == 0)
      __hip_atomic_store(tiles + tile, (tile == 0 ? kTileTotal : kTileCount) | total, __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
    uint32_t before = 0;
    for (int p = tile - 1; p >= 0;) {
      const uint32_t word = p - lane >= 0 ? __hip_atomic_load(tiles + (p - lane), __ATOMIC_RELAXED,
                                                              __HIP_MEMORY_SCOPE_AGENT)
                                          : kTileTotal;
      // the nearest tiles up to the first that knows its total; all of them must have a word
      const uint64_t totals = ballot((word & kTileTotal) != 0u), empty = ballot(word == 0u);
      const int last = totals ? __builtin_ctzll(totals) : 63;
      const uint64_t need = last == 63 ? ~0ull : (2ull << last) - 1ull;
      if (empty & need) {
        __builtin_amdgcn_s_sleep(1);
        continue;
      }
      uint32_t v = lane <= last ? word & kTileMask : 0u;
      for (int o = 32; o > 0; o >>= 1) v += (uint32_t)__shfl_xor((int)v, o, 64);
      before += v;
      p = totals ? -1 : p - 64;
    }
    if (lane == 0) {
      if (tile > 0)
        __hip_atomic_store(tiles + tile, kTileTotal | (before + total), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      before_s = (int)before;
      if (tile == ntiles - 1) {
        const int U = (int)(before + total);
        cnt->n_unique = U;
        ustart[U] = n;
        nstart[n] = 0;
        lmask[n] = 0;
        croot[scid ? min(max(scid[n - 1], 0), K - 1) + 1 : 1] = U;
      }
    }
  }
  __syncthreads();
  const int before = before_s;
  const uint64_t lt = (1ull << lane) - 1ull;
#pragma unroll
  for (int r = 0; r < kUniqueItems; ++r) {
    if (!((mask[r] >> lane) & 1ull)) continue;
    const int i = i0 + r * kSortThreads + t;
    const int u = before + chunk[r * kWaves + w] + __popcll(mask[r] & lt);
    ukey[u] = key[r];
    ustart[u] = i;
    if (scid) {
      const int c = min(max(scid[i], 0), K - 1), c1 = i > 0 ? min(max(scid[i - 1], 0), K - 1) : -1;
      ucid[u] = c;
      if (c != c1) croot[c1 + 1] = croot[c] = u;
    } else if (i == 0) {
      croot[0] = 0;
    }
  }
}

// Preorder id of the cluster's root: the shallowest node starting at its first
// unique key u, u + #internal nodes starting before u; for k = K the node count.
// And the cluster's first particle; for k = K the particle count.  (An empty
// cluster that k_unique left at -1 takes those of the next one that is not: the
// first key whose cluster is k or more.)
__global__ __launch_bounds__(256) void k_croot_final(int K, const Counts* __restrict__ cnt,
                                                     const int32_t* __restrict__ ucid,
                                                     const int32_t* __restrict__ nexcl,
                                                     const int32_t* __restrict__ ustart, int32_t* __restrict__ croot,
                                                     int32_t* __restrict__ cfirst) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k > K) return;
  int u = croot[k];
  if (u < 0) {
    int hi = cnt->n_unique;
    for (u = 0; u < hi;) {
      const int m = (u + hi) >> 1;
      if (ucid[m] < k) u = m + 1; else hi = m;
    }
  }
  croot[k] = u + nexcl[u];
  cfirst[k] = ustart[u];
}

// ---------------------------------------------------------------- topology
// Level of the deepest cell that holds both keys: 3*level leading bits of the
// 63-bit keys agree.  For distinct keys this is the level of the oct-tree cell
// whose children separate them.
__device__ __forceinline__ int split_level(uint64_t a, uint64_t b) {
  int lcp = __clzll((long long)(a ^ b)) - 1;  // bit 63 is always 0
  return lcp / 3;
}

__device__ __forceinline__ bool same_cell(uint64_t a, uint64_t b, int level) {
  return level == 0 || ((a ^ b) >> (63 - 3 * level)) == 0ull;
}

// Key range [f, l] of the cell of level s that separates the adjacent unique
// keys j (kj) and j + 1 (kj1) of a cluster with unique keys [ulo, uhi), by
// galloping and binary search (keys are sorted, so a range shares a prefix iff
// its ends do); true if j | j + 1 is the cell's first child boundary.  key(m):
// unique key m.
template <typename Key>
__device__ __forceinline__ bool cell_range(int j, int ulo, int uhi, int s, uint64_t kj, uint64_t kj1, Key&& key,
                                           int& f_out, int& l_out) {
  // first key of the cell: smallest f <= j with same_cell(key(f), kj, s)
  int lo = j, step = 1;
  while (true) {
    int cand = j - step;
    if (cand < ulo || !same_cell(key(cand), kj, s)) break;
    lo = cand;
    step <<= 1;
  }
  int a = max(j - step, ulo - 1), b = lo;  // invariant: a outside (or ulo - 1), b inside
  while (b - a > 1) {
    int m = a + (b - a) / 2;
    if (same_cell(key(m), kj, s)) b = m; else a = m;
  }
  const int f = b;
  // last key of the cell: largest l >= j+1 with same_cell(key(l), kj1, s)
  int up = j + 1;
  step = 1;
  while (true) {
    int cand = j + 1 + step;
    if (cand >= uhi || !same_cell(key(cand), kj1, s)) break;
    up = cand;
    step <<= 1;
  }
  int c = up, d = min(j + 1 + step, uhi);  // c inside, d outside (or uhi)
  while (d - c > 1) {
    int m = c + (d - c) / 2;
    if (same_cell(key(m), kj1, s)) c = m; else d = m;
  }
  f_out = f;
  l_out = c;
  return (f == j) || (s < kLevels - 1 && same_cell(key(f), kj, s + 1));
}

// For each pair of adjacent unique keys j, j+1 with split level s, the
// oct-tree cell (s, prefix) exists and has j|j+1 as one of its child
// boundaries.  Its key range [f, l] is found by galloping + binary search
// (keys are sorted, so a range shares a prefix iff its ends do).  The pair is
// the cell's representative iff it is the first child boundary in the range.
//
// Keys of different clusters share no cell: such a pair gets split level -1 and
// bounds every search.
//
// The keys of the block's 256 pairs and of kPairHalo keys on either side are
// staged in LDS first: most cells are small, so most searches stay in the
// tile, and only those that run past it read the key array in memory.
constexpr int kPairHalo = 512;
__global__ __launch_bounds__(256) void k_pairs(const uint64_t* __restrict__ ukey, const int32_t* __restrict__ ucid,
                                               const int32_t* __restrict__ croot,
                                               const Counts* __restrict__ cnt,
                                               int32_t* __restrict__ split, int32_t* __restrict__ rep,
                                               int32_t* __restrict__ pf, int32_t* __restrict__ pl,
                                               int32_t* __restrict__ nstart, uint32_t* __restrict__ lmask, int nmax) {
  __shared__ uint64_t tile[256 + 2 * kPairHalo];
  const int U = cnt->n_unique;
  const int j0 = blockIdx.x * blockDim.x;
  const int tlo = max(j0 - kPairHalo, 0), thi = min(j0 + (int)blockDim.x + kPairHalo, U);  // keys [tlo, thi)
  for (int t = threadIdx.x; t < thi - tlo; t += blockDim.x) tile[t] = ukey[tlo + t];
  __syncthreads();
  auto key = [&](int m) { return (m >= tlo && m < thi) ? tile[m - tlo] : ukey[m]; };
  int j = j0 + threadIdx.x;
  if (j >= nmax) return;
  if (j >= U - 1) {
    rep[j] = 0;
    return;
  }
  // (unique keys [ulo, uhi) are the cluster's: croot holds every cluster's first
  // one at this point; a read of each key's cluster id in the search made the
  // kernel 478 us for a forest of 7.5M particles, it takes 307)
  int ulo = 0, uhi = U;
  if (ucid) {
    const int cj = ucid[j];
    ulo = croot[cj];
    uhi = croot[cj + 1];
  }
  if (j + 1 >= uhi) {
    split[j] = -1;
    rep[j] = 0;
    return;
  }
  const uint64_t kj = key(j), kj1 = key(j + 1);
  const int s = split_level(kj, kj1);
  split[j] = s;
  int f, l;
  const bool is_rep = cell_range(
      j, ulo, uhi, s, kj, kj1, key, f, l);
  rep[j] = is_rep ? 1 : 0;
  if (!is_rep) return;
  pf[j] = f;
  pl[j] = l;
  atomicAdd(&nstart[f], 1);
  atomicOr(&lmask[f], 1u << s);
}

// Preorder: for each unique-key position x, the internal nodes whose first key
// is x (a chain of nested cells, shallowest first) come before leaf x.
//   pre(internal v) = f + #internal nodes starting before f + #shallower nodes starting at f
//   pre(leaf x)     = x + #internal nodes starting at or before x
//   next(v)         = pre(leaf last(v)) + 1
__device__ __forceinline__ Node internal_node(const Cube& cube, uint64_t key, int s, int next, int first, int end) {
  Node nd;
  nd.l = ldexp(cube.L, -s);
  // the cube's centre, in the centre-of-mass fields until the moment passes
  // replace it (they need it for s, and for the centre of a massless cell)
  const uint64_t prefix = (s == 0) ? 0ull : (key >> (63 - 3 * s));
  nd.cx = cube.lo[0] + ((double)compact3(prefix >> 2) + 0.5) * nd.l;
  nd.cy = cube.lo[1] + ((double)compact3(prefix >> 1) + 0.5) * nd.l;
  nd.cz = cube.lo[2] + ((double)compact3(prefix) + 0.5) * nd.l;
  nd.M = 0.0;
  nd.s = 0.0;
  nd.next = next;
  nd.first = first;
  nd.count = end - first;
  nd.meta = s << 8;
  return nd;
}

// Internal node `pre` of level s is an ancestor of the first node of every run
// (walk_segments) that starts inside its subtree.
__device__ __forceinline__ void list_ancestor(int32_t* __restrict__ anc, int r0, int r1, int runs, int pre, int next,
                                              int s) {
  const int len = max(1, (r1 - r0 + runs - 1) / runs);
  const int end = min(next, r1) - r0;
  for (int q = (pre - r0) / len + 1; q < runs && q * len < end; ++q) anc[q * kAncSlots + s] = pre;
}

// The leaf of unique key number x at preorder id `pre`, its particles [first,
// first + count) and its moments.  sl, sr: split levels towards the neighbouring
// keys (-1: none, or another cluster's).
template <typename T4>
__device__ __forceinline__ Node leaf_node(const Cube* __restrict__ cube, int pre, int first, int count, int sl, int sr,
                                          const T4* __restrict__ ps, Mom& mo) {
  // a leaf sits one level below the deeper of its two neighbour splits (split
  // -1 marks a cluster edge, so a cluster's only key is its level-0 root)
  const int level = count > 1 ? kLevels : 1 + max(sl, sr);
  Node nd;
  double M = 0.0, X = 0.0, Y = 0.0, Z = 0.0;
  for (int k = first; k < first + count; ++k) {
    T4 p = ps[k];
    double m = (double)p.w;
    M += m;
    X += m * (double)p.x;
    Y += m * (double)p.y;
    Z += m * (double)p.z;
  }
  if (count == 1) {
    T4 p = ps[first];
    nd.cx = (double)p.x;
    nd.cy = (double)p.y;
    nd.cz = (double)p.z;
  } else if (M != 0.0) {
    nd.cx = X / M;
    nd.cy = Y / M;
    nd.cz = Z / M;
  } else {
    // massless bucket: sit at the cell centre
    const double l = ldexp(cube->L, -level);
    T4 p = ps[first];
    double c[3] = {(double)p.x, (double)p.y, (double)p.z};
    double ctr[3];
    for (int d = 0; d < 3; ++d) {
      double q = floor((c[d] - cube->lo[d]) * cube->scale);
      if (!(q >= 0.0)) q = 0.0;
      if (q > (double)(kGrid - 1)) q = (double)(kGrid - 1);
      ctr[d] = cube->lo[d] + (q + 0.5) * l;
    }
    nd.cx = ctr[0];
    nd.cy = ctr[1];
    nd.cz = ctr[2];
  }
  nd.M = M;
  nd.l = ldexp(cube->L, -level);
  nd.s = 0.0;
  nd.next = pre + 1;
  nd.first = first;
  nd.count = count;
  nd.meta = 1 | (count > 1 ? 2 : 0) | (level << 8);
  mo = Mom{M, X, Y, Z};
  return nd;
}

__global__ __launch_bounds__(256) void k_nodes_internal(const Counts* __restrict__ cnt, const Cube* __restrict__ cubes,
                                                        const int32_t* __restrict__ ucid,
                                                        const int32_t* __restrict__ rep,
                                                        const int32_t* __restrict__ split,
                                                        const int32_t* __restrict__ pf, const int32_t* __restrict__ pl,
                                                        const int32_t* __restrict__ nstart,
                                                        const int32_t* __restrict__ nexcl,
                                                        const uint32_t* __restrict__ lmask,
                                                        const int32_t* __restrict__ ustart,
                                                        const uint64_t* __restrict__ ukey, Node* __restrict__ nodes,
                                                        int32_t* __restrict__ nx, uint8_t* __restrict__ nlev,
                                                        const int32_t* __restrict__ croot,
                                                        const int32_t* __restrict__ cfirst,
                                                        int32_t* __restrict__ anc, int nmax) {
  // (a thread per pair of adjacent unique keys; the pairs that stand for a cell)
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= nmax || j >= cnt->n_unique - 1 || !rep[j]) return;
  const int s = split[j], f = pf[j], l = pl[j];
  const int pre = f + nexcl[f] + __popc(lmask[f] & ((1u << s) - 1u));
  const int cl = ucid ? ucid[f] : 0;
  const Node nd = internal_node(cubes[cl], ukey[f], s, l + nexcl[l] + nstart[l] + 1, ustart[f], ustart[l + 1]);
  nodes[pre] = nd;
  nx[pre] = nd.next;
  nlev[pre] = (uint8_t)s;
  if (anc)
    list_ancestor(anc + (int64_t)cl * kMaxRuns * kAncSlots, croot[cl], croot[cl + 1],
                  walk_segments(cfirst[cl + 1] - cfirst[cl]), pre, nd.next, s);
}

template <typename T4>
__global__ __launch_bounds__(256) void k_nodes_leaf(Counts* __restrict__ cnt, const Cube* __restrict__ cubes,
                                                    const int32_t* __restrict__ ucid,
                                                    const int32_t* __restrict__ split,
                                                    const int32_t* __restrict__ nstart,
                                                    const int32_t* __restrict__ nexcl,
                                                    const int32_t* __restrict__ ustart, const T4* __restrict__ ps,
                                                    Node* __restrict__ nodes, Mom* __restrict__ mom,
                                                    int32_t* __restrict__ nx, uint8_t* __restrict__ nlev, int nmax) {
  int x = blockIdx.x * blockDim.x + threadIdx.x;
  const int U = cnt->n_unique;
  if (x == 0) cnt->n_nodes = U + cnt->n_internal;
  if (x >= nmax || x >= U) return;
  const int pre = x + nexcl[x] + nstart[x];
  Mom mo;
  const Node nd = leaf_node(cubes + (ucid ? ucid[x] : 0), pre, ustart[x], ustart[x + 1] - ustart[x],
                            x > 0 ? split[x - 1] : -1, x < U - 1 ? split[x] : -1, ps, mo);
  nodes[pre] = nd;
  mom[pre] = mo;
  nx[pre] = pre + 1;
  nlev[pre] = (uint8_t)(nd.meta >> 8);
}

// ---------------------------------------------------------------- moments
// The moments of an internal node fold its children's, in octant order (the
// preorder of the children p+1, next(p+1), ... < next(p)).  The fold runs
// bottom-up, with the same arithmetic for every node:
//  * k_moments_chunk: a workgroup loads a chunk of kChunk consecutive preorder
//    nodes (next, level, the leaves' moments) into LDS and folds there, level
//    by level (deepest first), every internal node whose subtree ends inside
//    the chunk.  The others, at most one per level, go to the chunk's slot of
//    their level's list;
//  * k_moments_super and k_moments_final fold the listed nodes.
// A node's children are deeper than it, so each fold reads finished values.

// Per-chunk index in LDS: next of every node, and the internal nodes whose
// subtree ends in the chunk grouped by level.
struct ChunkIndex {
  int32_t nx[kChunk];
  int16_t ord[kChunk];         // chunk offsets of the closed internal nodes, by level
  uint8_t lv[kChunk];
  int32_t start[kLevels + 2];  // ord range of each level
  int32_t fill[kLevels + 1];
  int32_t levels[kLevels + 1]; // the levels that have closed internal nodes, deepest first
  int32_t n_levels;
};

__device__ __forceinline__ bool chunk_leaf(const ChunkIndex& ci, int c0, int i) { return ci.nx[i] == c0 + i + 1; }

// Groups the chunk's closed internal nodes by level (ci.nx and ci.lv loaded,
// then a barrier, by the caller).  Ends with a barrier.
__device__ void chunk_sort(ChunkIndex& ci, int c0, int cn) {
  const int tid = threadIdx.x, c1 = c0 + cn;
  if (tid <= kLevels) ci.fill[tid] = 0;
  __syncthreads();
  for (int i = tid; i < cn; i += blockDim.x)
    if (!chunk_leaf(ci, c0, i) && ci.nx[i] <= c1) atomicAdd(&ci.fill[ci.lv[i]], 1);
  __syncthreads();
  if (tid < kWave) {
    // (one wave: an exclusive scan of the level counts, and the non-empty
    // levels, deepest first)
    const int cntL = tid <= kLevels ? ci.fill[tid] : 0;
    int incl = cntL;
    for (int o = 1; o < kWave; o <<= 1) {
      const int u = __shfl_up(incl, o, kWave);
      if (tid >= o) incl += u;
    }
    if (tid <= kLevels) ci.start[tid] = incl - cntL;
    if (tid == kLevels) ci.start[kLevels + 1] = incl;
    const uint64_t ne = __ballot(tid <= kLevels && cntL > 0);
    if (tid <= kLevels && cntL > 0) ci.levels[__popcll(ne >> (tid + 1))] = tid;
    if (tid == 0) ci.n_levels = __popcll(ne);
  }
  __syncthreads();
  if (tid <= kLevels) ci.fill[tid] = 0;
  __syncthreads();
  for (int i = tid; i < cn; i += blockDim.x) {
    if (chunk_leaf(ci, c0, i) || ci.nx[i] > c1) continue;
    const int L = ci.lv[i];
    ci.ord[ci.start[L] + atomicAdd(&ci.fill[L], 1)] = (int16_t)i;
  }
  __syncthreads();
}

__device__ __forceinline__ void add_mom(Mom& s, const Mom& q) {
  s.M += q.M;
  s.X += q.X;
  s.Y += q.Y;
  s.Z += q.Z;
}

// Centre of mass and s of node p from its folded moments q and its cube's
// centre ctr (which the node record holds until here).
__device__ __forceinline__ void finish_node(int p, const Mom& q, const double ctr[3], Node* __restrict__ nodes,
                                            Mom* __restrict__ mom) {
  double com[3];
  if (q.M != 0.0) {
    com[0] = q.X / q.M;
    com[1] = q.Y / q.M;
    com[2] = q.Z / q.M;
  } else {
    com[0] = ctr[0];
    com[1] = ctr[1];
    com[2] = ctr[2];
  }
  const double dx = ctr[0] - com[0], dy = ctr[1] - com[1], dz = ctr[2] - com[2];
  nodes[p].cx = com[0];
  nodes[p].cy = com[1];
  nodes[p].cz = com[2];
  nodes[p].M = q.M;
  nodes[p].s = sqrt(fma(dz, dz, fma(dy, dy, dx * dx)));
  mom[p] = q;
}

__global__ __launch_bounds__(kChunkThreads) void k_moments_chunk(const Counts* __restrict__ cnt,
                                                                 const int32_t* __restrict__ nx,
                                                                 const uint8_t* __restrict__ nlev,
                                                                 Node* __restrict__ nodes, Mom* __restrict__ mom,
                                                                 int32_t* __restrict__ obkt, int nchunks) {
  constexpr int kItems = kChunk / kChunkThreads;
  __shared__ ChunkIndex ci;
  __shared__ Mom sm[kChunk];
  const int n_nodes = cnt->n_nodes;
  const int c0 = blockIdx.x * kChunk;
  if (c0 >= n_nodes) return;
  const int cn = min(kChunk, n_nodes - c0), c1 = c0 + cn;
  const int tid = threadIdx.x;
  int nxt[kItems];
#pragma unroll
  for (int t = 0; t < kItems; ++t) {
    const int i = tid + t * kChunkThreads;
    nxt[t] = i < cn ? nx[c0 + i] : 0;
  }
#pragma unroll
  for (int t = 0; t < kItems; ++t) {
    const int i = tid + t * kChunkThreads;
    if (i >= cn) continue;
    ci.nx[i] = nxt[t];
    ci.lv[i] = (uint8_t)min((int)nlev[c0 + i], kLevels);
    if (nxt[t] == c0 + i + 1) sm[i] = mom[c0 + i];  // a leaf
  }
  // the cube centres of this thread's closed internal nodes, for the end
  double ctr[kItems][3];
#pragma unroll
  for (int t = 0; t < kItems; ++t) {
    const int i = tid + t * kChunkThreads;
    const bool closed = i < cn && nxt[t] != c0 + i + 1 && nxt[t] <= c1;
    ctr[t][0] = closed ? nodes[c0 + i].cx : 0.0;
    ctr[t][1] = closed ? nodes[c0 + i].cy : 0.0;
    ctr[t][2] = closed ? nodes[c0 + i].cz : 0.0;
  }
  // this chunk's slot of each level's list of straddling nodes: none yet
  if (tid < kLevels) obkt[tid * nchunks + blockIdx.x] = -1;
  __syncthreads();
  chunk_sort(ci, c0, cn);
  for (int t = 0; t < ci.n_levels; ++t) {
    const int L = ci.levels[t];
    for (int j = ci.start[L] + tid; j < ci.start[L + 1]; j += kChunkThreads) {
      const int i = ci.ord[j];
      const int end = ci.nx[i] - c0;
      Mom q{0.0, 0.0, 0.0, 0.0};
      int c = i + 1;
      for (int k = 0; k < 8 && c < end; ++k, c = max(ci.nx[c] - c0, c + 1)) add_mom(q, sm[c]);
      sm[i] = q;
    }
    __syncthreads();
  }
#pragma unroll
  for (int t = 0; t < kItems; ++t) {
    const int i = tid + t * kChunkThreads;
    if (i >= cn || nxt[t] == c0 + i + 1) continue;
    if (nxt[t] <= c1) {
      finish_node(c0 + i, sm[i], ctr[t], nodes, mom);
    } else {
      // crosses the chunk's end (an ancestor of the next chunk's first node,
      // the only one of its level here): list it for its level's pass
      obkt[min((int)ci.lv[i], kLevels - 1) * nchunks + blockIdx.x] = c0 + i;
    }
  }
}

// The straddling nodes, in two launches.  k_moments_super: a workgroup takes
// kSuper consecutive chunks, one thread per (level, chunk) slot; it lists its
// node's children (along next, which past the chunk's end continues in memory;
// the second moments read the list too), and the nodes whose subtree ends
// inside the workgroup's chunks are folded level by level, deepest first, a
// barrier apart.  What still straddles, at most one node per level and
// workgroup, is listed for k_moments_final, one workgroup that does the same
// over all of them.  (One launch per level, 21 of some 5 us, and one for the
// lists took 79 us for 100,000 particles, 122 for 1M and 157 for 4M; the two take
// 39, 50 and 159.)
constexpr int kSuper = kSuperChunks;
constexpr int kSuperSlots = kSuper * kLevels;
constexpr int kSuperThreads = (kSuperSlots + kWave - 1) / kWave * kWave;
constexpr int kFinalThreads = 1024;

// Levels that some thread asks for (level < 0: none), as a mask (LDS word `m`).
__device__ __forceinline__ uint32_t level_mask(uint32_t* m, int level) {
  if (threadIdx.x == 0) *m = 0;
  __syncthreads();
  if (level >= 0) atomicOr(m, 1u << level);
  __syncthreads();
  return *m;
}

// The slots of one workgroup of the super launches: calls fold(p, kids) for
// every node that ends inside the workgroup's chunks, deepest level first.
// load(slot, p, kids): the children of the slot's node; open(L, slot): a node
// that is left over.
template <typename Load, typename Open, typename Fold>
__device__ __forceinline__ void fold_super(const Counts* __restrict__ cnt, const int32_t* __restrict__ obkt,
                                           const int32_t* __restrict__ nx, int nchunks, Load&& load, Open&& open,
                                           Fold&& fold) {
  __shared__ uint32_t mask;
  const int n_nodes = cnt->n_nodes;
  const int L = threadIdx.x / kSuper, j = blockIdx.x * kSuper + threadIdx.x % kSuper;
  if ((int64_t)blockIdx.x * kSuper * kChunk >= n_nodes) return;  // (the whole workgroup)
  const int64_t end = min((int64_t)(blockIdx.x + 1) * kSuper * kChunk, (int64_t)n_nodes);
  int p = -1, kids[8];
  if (L < kLevels && j < nchunks && (int64_t)j * kChunk < n_nodes) {
    const int slot = L * nchunks + j;
    p = obkt[slot];
    if (p >= n_nodes) p = -1;
    if (p >= 0) {
      load(slot, p, kids);
      if (nx[p] > end) {
        open(L, slot);
        p = -1;
      }
    }
  }
  for (uint32_t left = level_mask(&mask, p >= 0 ? L : -1); left;) {
    const int lv = 31 - __clz((int)left);
    left &= ~(1u << lv);
    if (p >= 0 && L == lv) fold(p, kids);
    __syncthreads();
  }
}

// The slots left over (sbkt [kLevels][nsuper]; -1: none), by one workgroup; the
// lists of the next level's nodes are read before the barrier of the current
// one.
template <typename Fold>
__device__ __forceinline__ void fold_final(const Counts* __restrict__ cnt, const int32_t* __restrict__ obkt,
                                           const int32_t* __restrict__ okids, const int32_t* __restrict__ sbkt,
                                           int nsuper, Fold&& fold) {
  const int n_nodes = cnt->n_nodes;
  const int m = (int)min((int64_t)nsuper, ((int64_t)n_nodes + kSuper * kChunk - 1) / (kSuper * kChunk));
  int p = -1, kids[8];
  auto read = [&](int L, int j) {
    p = -1;
    const int slot = L >= 0 && j < m ? sbkt[L * nsuper + j] : -1;
    if (slot < 0) return;
    p = obkt[slot];
    for (int k = 0; k < 8; ++k) kids[k] = okids[8 * (int64_t)slot + k];
  };
  read(kLevels - 1, threadIdx.x);
  for (int L = kLevels - 1; L >= 0; --L) {
    if (p >= 0) fold(p, kids);
    for (int j = threadIdx.x + kFinalThreads; j < m; j += kFinalThreads) {
      read(L, j);
      if (p >= 0) fold(p, kids);
    }
    read(L - 1, threadIdx.x);
    __syncthreads();
  }
}

__device__ __forceinline__ void fold_moments(int p, const int (&kids)[8], int n_nodes, Node* __restrict__ nodes,
                                             Mom* __restrict__ mom) {
  Mom c[8];
  const double ctr[3] = {nodes[p].cx, nodes[p].cy, nodes[p].cz};
  int n = 0;
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const bool ok = n == k && kids[k] > p && kids[k] < n_nodes;
    if (ok) c[k] = mom[kids[k]];
    n += ok ? 1 : 0;
  }
  Mom q{0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int k = 0; k < 8; ++k)
    if (k < n) add_mom(q, c[k]);
  finish_node(p, q, ctr, nodes, mom);
}

__global__ __launch_bounds__(kSuperThreads) void k_moments_super(const Counts* __restrict__ cnt,
                                                                 const int32_t* __restrict__ obkt,
                                                                 const int32_t* __restrict__ nx, int nchunks,
                                                                 Node* nodes, Mom* mom, int32_t* __restrict__ okids,
                                                                 int32_t* __restrict__ sbkt, int nsuper) {
  const int n_nodes = cnt->n_nodes;
  if (threadIdx.x < kLevels) sbkt[threadIdx.x * nsuper + blockIdx.x] = -1;
  __syncthreads();
  fold_super(
      cnt, obkt, nx, nchunks,
      [&](int slot, int p, int (&kids)[8]) {
        const int end = min(nx[p], n_nodes);
        int c = p + 1;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          kids[k] = c < end ? c : -1;
          if (c < end) c = max(nx[c], c + 1);
          okids[8 * (int64_t)slot + k] = kids[k];
        }
      },
      [&](int L, int slot) { sbkt[L * nsuper + blockIdx.x] = slot; },
      [&](int p, const int (&kids)[8]) { fold_moments(p, kids, n_nodes, nodes, mom); });
}

__global__ __launch_bounds__(kFinalThreads) void k_moments_final(const Counts* __restrict__ cnt,
                                                                 const int32_t* __restrict__ obkt,
                                                                 const int32_t* __restrict__ okids,
                                                                 const int32_t* __restrict__ sbkt, int nsuper,
                                                                 Node* nodes, Mom* mom) {
  const int n_nodes = cnt->n_nodes;
  fold_final(cnt, obkt, okids, sbkt, nsuper,
             [&](int p, const int (&kids)[8]) { fold_moments(p, kids, n_nodes, nodes, mom); });
}

// ---------------------------------------------------------------- driver
static inline int nblk(int64_t n, int t) { return (int)((n + t - 1) / t) > 0 ? (int)((n + t - 1) / t) : 1; }

template <typename T4>
static hipError_t hilbert_impl(int n, const BuildWs& w, hipStream_t st);

static inline int clear_blocks(int64_t n) { return (int)min((int64_t)1024, max((int64_t)8, n / 4096)); }

template <typename T, typename T4>
static hipError_t build_impl(const T* pos, const T* mass, int n, const BuildWs& w, const BuildFork* fork,
                             hipStream_t st) {
  hipError_t e;
  const int K = w.n_seg;
  // the start, and the root cubes (of one cluster: in the launch of the start)
  {
    const SortScratch sc{w.hist, w.ticket, {w.tiles, nullptr}};
    const int64_t words = n > 0 ? 256 * sort_tiles(n) : 0, n_anc = w.anc ? (int64_t)K * kMaxRuns * kAncSlots : 0;
    const int nbb = min(kBboxBlocks, nblk(n, 256));
    if (K == 1 && n > 0)
      k_bbox_partial<T><<<nbb, 256, 0, st>>>(pos, mass, n, w, sc, words, n_anc);
    else
      k_init<<<clear_blocks(n), 256, 0, st>>>(w, sc, n, words, n_anc);
    if (w.seg_off != w.own_off) k_seg_check<<<nblk(K + 1, 256), 256, 0, st>>>(w.seg_off, K, n, w.counts);
    if (n == 0) return hipGetLastError();
    if (K == 1)
      k_bbox_final<<<1, 448, 0, st>>>(w.bbox_part, nbb, w.cube, w.counts);
    else
      k_bbox_seg<T><<<K, 256, 0, st>>>(pos, mass, w.seg_off, n, w.cube, w.counts);
  }
  // keys and stable sort by (cluster, key): 8 key passes, then the cluster digits
  // cluster ids are kept only for a forest (a single tree's are all 0)
  int32_t* seg = K > 1 ? w.seg : nullptr;
  int32_t* scid = K > 1 ? w.scid : nullptr;
  int32_t* ucid = K > 1 ? w.ucid : nullptr;
  int seg_passes = 0;
  for (unsigned r = (unsigned)(K - 1); r; r >>= 8) ++seg_passes;
  const SortScratch sc{w.hist, w.ticket, {w.tiles, w.tiles + 256 * sort_tiles(n)}};
  k_keys<T><<<key_blocks(n), kKeyThreads, 0, st>>>(pos, n, w.cube, w.seg_off, K, seg_passes, seg, w.key_a, w.idx_a,
                                                   w.hist);
  uint64_t *kin = w.key_a, *kout = w.key_b;
  int32_t *vin = w.idx_a, *vout = w.idx_b;
  for (int pass = 0; pass < 8 + seg_passes; ++pass) {
    if (pass < 8)
      launch_pass<kDigKey>(kin, vin, w, kout, vout, n, 8 * pass, sc, pass, st);
    else if (K + 1 <= kSegLds)
      launch_pass<kDigSegLds>(kin, vin, w, kout, vout, n, 8 * (pass - 8), sc, pass, st);
    else
      launch_pass<kDigSegIdx>(kin, vin, w, kout, vout, n, 8 * (pass - 8), sc, pass, st);
    uint64_t* tk = kin; kin = kout; kout = tk;
    int32_t* tv = vin; vin = vout; vout = tv;
  }
  // the sorted data must end in key_a / idx_a
  if (kin != w.key_a) k_copy_kv<<<nblk(n, 256), 256, 0, st>>>(kin, vin, w.key_a, w.idx_a, n);
  k_gather<T, T4><<<nblk(n, 256), 256, 0, st>>>(pos, mass, w.idx_a, seg, n, reinterpret_cast<T4*>(w.ps), scid);
  if (fork) {
    if ((e = hipEventRecord(fork->fork, st)) != hipSuccess) return e;
    if ((e = hipStreamWaitEvent(fork->side, fork->fork, 0)) != hipSuccess) return e;
    if ((e = hilbert_impl<T4>(n, w, fork->side)) != hipSuccess) return e;
    if ((e = hipEventRecord(fork->join, fork->side)) != hipSuccess) return e;
  }
  // unique (cluster, key) pairs (the sort's last pass left the words of its next one cleared)
  const int ut = unique_tiles(n);
  k_unique<<<ut, kSortThreads, 0, st>>>(w.key_a, scid, n, K, w.ukey, w.ustart, ucid, w.counts, w.nstart, w.lmask,
                                        w.croot, sc.tiles[(8 + seg_passes) & 1], w.ticket + kSortPasses, ut);
  // internal nodes
  k_pairs<<<nblk(n, 256), 256, 0, st>>>(w.ukey, ucid, w.croot, w.counts, w.split, w.flag, w.pf, w.pl, w.nstart, w.lmask,
                                        n);
  if ((e = scan_excl(w.nstart, w.nexcl, n + 1, w.scan_tiles, &w.counts->n_internal, st)) != hipSuccess) return e;
  k_croot_final<<<nblk(K + 1, 256), 256, 0, st>>>(K, w.counts, ucid, w.nexcl, w.ustart, w.croot, w.cfirst);
  k_nodes_internal<<<nblk(n, 256), 256, 0, st>>>(w.counts, w.cube, ucid, w.flag, w.split, w.pf, w.pl, w.nstart, w.nexcl,
                                                 w.lmask, w.ustart, w.ukey, w.nodes, w.nx, w.nlev, w.croot, w.cfirst,
                                                 w.anc, n);
  k_nodes_leaf<T4><<<nblk(n, 256), 256, 0, st>>>(w.counts, w.cube, ucid, w.split, w.nstart, w.nexcl, w.ustart,
                                                 reinterpret_cast<const T4*>(w.ps), w.nodes, w.mom, w.nx, w.nlev, n);
  // moments: chunks of the preorder (2n nodes at most), then the straddling
  // internal nodes
  const int nch = (int)n_chunks(n);
  k_moments_chunk<<<nch, kChunkThreads, 0, st>>>(w.counts, w.nx, w.nlev, w.nodes, w.mom, w.obkt, nch);
  const int nsup = n_super(n);
  k_moments_super<<<nsup, kSuperThreads, 0, st>>>(w.counts, w.obkt, w.nx, nch, w.nodes, w.mom, w.okids, w.sbkt, nsup);
  // (a node that straddles no workgroup's chunks is done)
  if (nsup > 1)
    k_moments_final<<<1, kFinalThreads, 0, st>>>(w.counts, w.obkt, w.okids, w.sbkt, nsup, w.nodes, w.mom);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if (fork) return hipStreamWaitEvent(st, fork->join, 0);
  return hipSuccess;
}

hipError_t fill_i32(int32_t* p, int64_t n, int32_t v, hipStream_t st) {
  k_fill_i32<<<nblk(n, 256), 256, 0, st>>>(p, n, v);
  return hipGetLastError();
}

__global__ __launch_bounds__(256) void k_rank(const int32_t* __restrict__ perm, int n, int32_t* __restrict__ rank) {
  int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k < n) rank[perm[k]] = k;
}

hipError_t make_rank(const int32_t* perm, int n, int32_t* rank, hipStream_t st) {
  k_rank<<<nblk(n, 256), 256, 0, st>>>(perm, n, rank);
  return hipGetLastError();
}

// ---------------------------------------------------------------- Hilbert walk order
// The walk's targets go in groups of 64 consecutive positions of an order.  In
// Morton order a group that straddles the edge of a large cell is split between
// distant cells, which widens the group's union walk; in Hilbert order a group
// is a face-connected run of cells.  Only the coarse levels matter (measured:
// 10 levels give the full-depth order's walk on a clumpy 4M field), so the
// order sorts Morton positions by (cluster, Hilbert index of the cell
// hilbert_levels(K) below the cluster's root cube), ties in Morton order, in as
// few 8-bit passes as the key needs.

// Hilbert index of the cell (x, y, z) of a 2^b grid, by Skilling's transform
// ("Programming the Hilbert curve", AIP Conf. Proc. 707, 2004): undo the
// excess work of the Gray-code walk level by level, Gray-encode, then
// interleave with x as the most significant bit of each triplet.
__device__ __forceinline__ uint32_t hilbert3(uint32_t x, uint32_t y, uint32_t z, int b) {
  uint32_t X[3] = {x, y, z};
  const uint32_t top = 1u << (b - 1);
  for (uint32_t q = top; q > 1; q >>= 1) {
    const uint32_t low = q - 1;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      if (X[i] & q) {
        X[0] ^= low;
      } else {
        const uint32_t t = (X[0] ^ X[i]) & low;
        X[0] ^= t;
        X[i] ^= t;
      }
    }
  }
  X[1] ^= X[0];
  X[2] ^= X[1];
  uint32_t t = 0;
  for (uint32_t q = top; q > 1; q >>= 1)
    if (X[2] & q) t ^= q - 1;
  uint32_t h = 0;
  for (int j = b - 1; j >= 0; --j)
    h = (h << 3) | ((((X[0] ^ t) >> j) & 1u) << 2) | ((((X[1] ^ t) >> j) & 1u) << 1) | (((X[2] ^ t) >> j) & 1u);
  return h;
}

static int bits_of(unsigned v) {
  int b = 0;
  for (; v; v >>= 1) ++b;
  return b;
}

// Levels of the Hilbert cells: 10 for a single tree (four passes; 8 levels in
// three passes walked 2 % slower), fewer in a forest so that the cluster id and
// the index share 32 bits where they can.
static int hilbert_levels(int K) {
  const int cbits = bits_of((unsigned)(K - 1));
  return max(5, min(10, (32 - cbits) / 3));
}

// Sort key of Morton position k: its cluster above the Hilbert index of its
// particle's cell `levels` below the cluster's root cube (the grid coordinates
// are those of the Morton keys).
template <typename T4>
__device__ __forceinline__ uint32_t hilbert_key(const Cube& cube, const T4& p, int levels) {
  const double c[3] = {(double)p.x, (double)p.y, (double)p.z};
  uint32_t q[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    double t = floor((c[d] - cube.lo[d]) * cube.scale);
    if (!(t >= 0.0)) t = 0.0;
    if (t > (double)(kGrid - 1)) t = (double)(kGrid - 1);
    q[d] = (uint32_t)t >> (kLevels - levels);
  }
  return hilbert3(q[0], q[1], q[2], levels);
}

template <typename T4>
__global__ __launch_bounds__(kKeyThreads) void k_hkeys(const T4* __restrict__ ps, int n, const Cube* __restrict__ cubes,
                                                       const int32_t* __restrict__ scid, int levels, int passes,
                                                       uint64_t* __restrict__ keys, int32_t* __restrict__ idx,
                                                       int32_t* __restrict__ hist) {
  __shared__ uint32_t h[kSortPasses][256];
  clear_digits(h, passes);
  for (int64_t k = (int64_t)blockIdx.x * kKeyThreads + threadIdx.x; k < n; k += (int64_t)gridDim.x * kKeyThreads) {
    const int cl = scid ? scid[k] : 0;
    const uint64_t key = ((uint64_t)(uint32_t)cl << (3 * levels)) | hilbert_key(cubes[cl], ps[k], levels);
    keys[k] = key;
    idx[k] = (int32_t)k;
    count_digits(h, key, passes, 0u, 0);
  }
  store_digits(h, passes, hist);
}

template <typename T4>
static hipError_t hilbert_impl(int n, const BuildWs& w, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  const int K = w.n_seg;
  const int levels = hilbert_levels(K);
  const int passes = (3 * levels + bits_of((unsigned)(K - 1)) + 7) / 8;
  const SortScratch sc{w.hhist, w.hticket, {w.htiles, w.htiles + 256 * sort_tiles(n)}};
  // (formed once per build, beside it or later: its words are cleared here)
  k_clear_sort<<<clear_blocks(n), 256, 0, st>>>(sc.hist, sc.ticket, sc.tiles[0], 256 * sort_tiles(n));
  k_hkeys<T4><<<key_blocks(n), kKeyThreads, 0, st>>>(reinterpret_cast<const T4*>(w.ps), n, w.cube,
                                                     K > 1 ? w.scid : nullptr, levels, passes, w.hkey_a, w.horder,
                                                     w.hhist);
  uint64_t *kin = w.hkey_a, *kout = w.hkey_b;
  int32_t *vin = w.horder, *vout = w.hidx;
  for (int pass = 0; pass < passes; ++pass) {
    launch_pass<kDigKey>(kin, vin, w, kout, vout, n, 8 * pass, sc, pass, st);
    uint64_t* tk = kin; kin = kout; kout = tk;
    int32_t* tv = vin; vin = vout; vout = tv;
  }
  if (vin != w.horder) k_copy_kv<<<nblk(n, 256), 256, 0, st>>>(kin, vin, kout, w.horder, n);
  return hipGetLastError();
}

// ---------------------------------------------------------------- small trees
// The whole build of a single tree of at most kSmallBuild particles by one
// workgroup: the same steps as the kernels above with the keys, the topology
// and the level lists in LDS (keys, indices, node links and lists fill 152 KB
// of it), a barrier where they have a launch.  It ends with the Hilbert walk
// order.  As a sequence of kernels a small build is bound by its launches, some
// 95 of about 4 us (340 us for 1000 particles, 390 us for 4096 in FP64); here it
// is bound by the latency of one workgroup's steps: 54 and 131 us.  More
// particles do not fit the LDS.
constexpr int kSmallThreads = 1024;
constexpr int kSmallWaves = kSmallThreads / kWave;
constexpr int kSmallItems = kSmallBuild / kSmallThreads;
constexpr int kSmallRun = 16;

struct SmallLds {
  union {
    struct {
      uint64_t key[2][kSmallBuild];
      int32_t idx[2][kSmallBuild];
      uint32_t hist[kSmallWaves][256];
    } sort;
    struct {
      int32_t nx[2 * kSmallBuild];     // (over key[0], which holds the sorted keys until ukey is written)
      uint64_t ukey[kSmallBuild];      // (over key[1])
      int32_t nstart[kSmallBuild + 4]; // (from here over idx and hist, free once the particles are gathered)
      int32_t nexcl[kSmallBuild + 4];
      uint32_t lmask[kSmallBuild];
    } topo;
  };
  int32_t ustart[kSmallBuild + 4];
  uint16_t ord[kSmallBuild];           // internal nodes by level
  int8_t split[kSmallBuild];
  uint8_t lv[2 * kSmallBuild];
  int32_t start[kLevels + 2], fill[kLevels + 1];
  int32_t scan[kSmallWaves];
  double red[6][kSmallWaves];
  Cube cube;
  int32_t bad, long_run;
};
static_assert(sizeof(SmallLds) <= 160 * 1024, "the small build's arrays must fit the LDS");

// One stable pass by the 8-bit digit at `shift`, buffer b to buffer b ^ 1: each
// wave ranks its contiguous share in input order (as k_rs_pass does), then
// the counts are scanned digit by digit, wave by wave.
__device__ __forceinline__ void small_sort_pass(SmallLds& s, int n, int shift, int b) {
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  for (int k = t; k < kSmallWaves * 256; k += kSmallThreads) s.sort.hist[0][k] = 0;
  __syncthreads();
  constexpr int kRounds = kSmallBuild / kSmallThreads;
  const int rounds = (n + kSmallThreads - 1) / kSmallThreads;  // 64 items of each wave
  uint64_t key[kRounds];
  int32_t val[kRounds];
  uint32_t rank[kRounds];
  const uint64_t lt = (1ull << lane) - 1ull;
#pragma unroll
  for (int r = 0; r < kRounds; ++r) {
    if (r >= rounds) break;
    const int j = (w * rounds + r) * kWave + lane;
    const bool valid = j < n;
    key[r] = valid ? s.sort.key[b][j] : 0ull;
    val[r] = valid ? s.sort.idx[b][j] : 0;
    const uint32_t d = (uint32_t)(key[r] >> shift) & 255u;
    uint64_t peers = ballot(valid);
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const bool bit = (d >> q) & 1u;
      const uint64_t mk = ballot(bit);
      peers &= bit ? mk : ~mk;
    }
    const int leader = valid ? __builtin_ctzll(peers) : lane;
    uint32_t base = 0;
    if (valid && lane == leader) base = atomicAdd(&s.sort.hist[w][d], (uint32_t)__popcll(peers));
    rank[r] = __shfl(base, leader, 64) + (uint32_t)__popcll(peers & lt);
  }
  __syncthreads();
  uint32_t h[kSmallWaves], c = 0;
  if (t < 256)
#pragma unroll
    for (int k = 0; k < kSmallWaves; ++k) c += h[k] = s.sort.hist[k][t];
  int tot;
  uint32_t run = (uint32_t)block_excl_scan<kSmallThreads>((int)c, s.scan, &tot);
  if (t < 256)
#pragma unroll
    for (int k = 0; k < kSmallWaves; ++k) {
      s.sort.hist[k][t] = run;
      run += h[k];
    }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kRounds; ++r) {
    const int j = (w * rounds + r) * kWave + lane;
    if (r < rounds && j < n) {
      const uint32_t q = s.sort.hist[w][(uint32_t)(key[r] >> shift) & 255u] + rank[r];
      s.sort.key[b ^ 1][q] = key[r];
      s.sort.idx[b ^ 1][q] = val[r];
    }
  }
  __syncthreads();
}

struct SmallArgs {
  int n;
  Cube* cube;
  Counts* counts;
  const int64_t* seg_off;  // the caller's offsets {0, n}, to be checked (null: none)
  int64_t* own_off;        // the tree's own, to be written
  int32_t *croot, *cfirst;
  int32_t* perm;
  void* ps;
  Node* nodes;
  Mom* mom;
  int32_t* nx;
  uint8_t* nlev;
  int32_t *obkt, *okids;
  int32_t* anc;
  int32_t* horder;
  int nchunks, hlevels;
};

template <typename T, typename T4>
__global__ __launch_bounds__(kSmallThreads) void k_build_small(const T* __restrict__ pos, const T* __restrict__ mass,
                                                               SmallArgs a) {
  __shared__ SmallLds s;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6, n = a.n;
  T4* ps = reinterpret_cast<T4*>(a.ps);

  // root cube
  {
    double v[6] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY};
    bool bad = false;
    for (int i = t; i < n; i += kSmallThreads) {
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        const double x = (double)pos[3 * i + d];
        if (!isfinite(x)) {
          bad = true;
        } else {
          v[d] = fmin(v[d], x);
          v[3 + d] = fmax(v[3 + d], x);
        }
      }
      if (!isfinite((double)mass[i])) bad = true;
    }
    if (t == 0) s.bad = s.long_run = 0;
#pragma unroll
    for (int q = 0; q < 6; ++q) {
      for (int o = 32; o > 0; o >>= 1) {
        const double u = __shfl_xor(v[q], o, 64);
        v[q] = q < 3 ? fmin(v[q], u) : fmax(v[q], u);
      }
      if (lane == 0) s.red[q][w] = v[q];
    }
    for (int k = t; k < kMaxRuns * kAncSlots; k += kSmallThreads) a.anc[k] = -1;
    for (int k = t; k < kLevels * a.nchunks; k += kSmallThreads) a.obkt[k] = -1;
    __syncthreads();
    if (bad) atomicOr(&s.bad, 1);
    if (t == 0) {
      double lo[3], hi[3];
      for (int d = 0; d < 3; ++d) {
        lo[d] = s.red[d][0];
        hi[d] = s.red[3 + d][0];
        for (int k = 1; k < kSmallWaves; ++k) {
          lo[d] = fmin(lo[d], s.red[d][k]);
          hi[d] = fmax(hi[d], s.red[3 + d][k]);
        }
      }
      finish_cube(lo, hi, &s.cube);
      if (a.seg_off) {
        if (a.seg_off[0] != 0 || a.seg_off[1] != n) atomicOr(&s.bad, 2);
      } else {
        a.own_off[0] = 0;
        a.own_off[1] = n;
      }
    }
    __syncthreads();
  }
  const Cube cube = s.cube;

  // keys, stable sort, gather
  for (int i = t; i < n; i += kSmallThreads) {
    s.sort.key[0][i] = morton_key(cube, pos, i);
    s.sort.idx[0][i] = i;
  }
  __syncthreads();
  // By the upper 32 key bits first, four passes instead of eight: few particles
  // of a small set share them (a cell ten levels down), and where they do, the
  // first of them puts them into order by the whole key.  Longer runs of one cell
  // take the other digits as well; a stable sort from the lowest digit up may
  // start from any order that keeps equal keys by index.
  for (int pass = 0; pass < 4; ++pass) small_sort_pass(s, n, 31 + 8 * pass, pass & 1);
  for (int j = t; j < n; j += kSmallThreads) {
    const uint64_t hi = s.sort.key[0][j] >> 31;
    if (j > 0 && s.sort.key[0][j - 1] >> 31 == hi) continue;
    int e = j + 1;
    while (e < n && e - j <= kSmallRun && s.sort.key[0][e] >> 31 == hi) ++e;
    if (e - j > kSmallRun) {
      s.long_run = 1;
      continue;
    }
    for (int i = j + 1; i < e; ++i) {
      const uint64_t key = s.sort.key[0][i];
      const int32_t id = s.sort.idx[0][i];
      int q = i;
      for (; q > j && s.sort.key[0][q - 1] > key; --q) {
        s.sort.key[0][q] = s.sort.key[0][q - 1];
        s.sort.idx[0][q] = s.sort.idx[0][q - 1];
      }
      s.sort.key[0][q] = key;
      s.sort.idx[0][q] = id;
    }
  }
  __syncthreads();
  if (s.long_run) {
    for (int pass = 0; pass < 4; ++pass) small_sort_pass(s, n, 8 * pass, pass & 1);
    for (int pass = 0; pass < 4; ++pass) small_sort_pass(s, n, 31 + 8 * pass, pass & 1);
  }
  for (int k = t; k < n; k += kSmallThreads) {
    const int j = s.sort.idx[0][k];
    a.perm[k] = j;
    T4 v;
    v.x = pos[3 * j];
    v.y = pos[3 * j + 1];
    v.z = pos[3 * j + 2];
    v.w = mass[j];
    ps[k] = v;
  }

  // unique keys, kSmallItems consecutive positions per thread
  int U;
  {
    uint64_t key[kSmallItems];
    bool fl[kSmallItems];
    int c = 0;
#pragma unroll
    for (int k = 0; k < kSmallItems; ++k) {
      const int j = t * kSmallItems + k;
      key[k] = j < n ? s.sort.key[0][j] : 0ull;
      fl[k] = j < n && (j == 0 || key[k] != s.sort.key[0][j - 1]);
      c += fl[k] ? 1 : 0;
    }
    int u = block_excl_scan<kSmallThreads>(c, s.scan, &U);  // (its barriers end the reads of idx and hist)
#pragma unroll
    for (int k = 0; k < kSmallItems; ++k)
      if (fl[k]) {
        s.topo.ukey[u] = key[k];
        s.ustart[u] = t * kSmallItems + k;
        ++u;
      }
    if (t == 0) s.ustart[U] = n;
    for (int k = t; k <= U; k += kSmallThreads) s.topo.nstart[k] = 0;
    for (int k = t; k < U; k += kSmallThreads) s.topo.lmask[k] = 0;
    if (t <= kLevels) s.fill[t] = 0;
  }
  __syncthreads();

  // internal nodes: the pairs that are their cell's first child boundary
  int nf[kSmallItems], nl[kSmallItems], ns[kSmallItems];  // first and last key, level (-1: none)
#pragma unroll
  for (int k = 0; k < kSmallItems; ++k) {
    const int j = t + k * kSmallThreads;
    ns[k] = -1;
    nf[k] = nl[k] = 0;
    if (j >= U - 1) continue;
    const uint64_t kj = s.topo.ukey[j], kj1 = s.topo.ukey[j + 1];
    const int lev = split_level(kj, kj1);
    s.split[j] = (int8_t)lev;
    if (cell_range(
            j, 0, U, lev, kj, kj1, [&](int m) { return s.topo.ukey[m]; }, nf[k], nl[k])) {
      ns[k] = lev;
      atomicAdd(&s.topo.nstart[nf[k]], 1);
      atomicOr(&s.topo.lmask[nf[k]], 1u << lev);
      atomicAdd(&s.fill[lev], 1);
    }
  }
  __syncthreads();
  int I;
  {
    int v[kSmallItems], c = 0;
#pragma unroll
    for (int k = 0; k < kSmallItems; ++k) {
      const int x = t * kSmallItems + k;
      v[k] = x < U ? s.topo.nstart[x] : 0;
      c += v[k];
    }
    int e = block_excl_scan<kSmallThreads>(c, s.scan, &I);
#pragma unroll
    for (int k = 0; k < kSmallItems; ++k) {
      const int x = t * kSmallItems + k;
      if (x < U) s.topo.nexcl[x] = e;
      e += v[k];
    }
    if (t == 0) {
      int run = 0;
      for (int L = 0; L <= kLevels; ++L) {
        s.start[L] = run;
        run += s.fill[L];
        s.fill[L] = 0;
      }
      s.start[kLevels + 1] = run;
      a.croot[0] = 0;
      a.croot[1] = U + I;
      a.cfirst[0] = 0;
      a.cfirst[1] = n;
      *a.cube = cube;
      Counts cn{};
      cn.n_unique = U;
      cn.n_internal = I;
      cn.n_nodes = U + I;
      cn.bad_input = s.bad;
      *a.counts = cn;
    }
  }
  __syncthreads();

  // node records (the sorted keys in key[0] are no longer needed: nx takes their place)
  const int m = U + I;
#pragma unroll
  for (int k = 0; k < kSmallItems; ++k) {
    if (ns[k] < 0) continue;
    const int f = nf[k], l = nl[k], lev = ns[k];
    const int pre = f + s.topo.nexcl[f] + __popc(s.topo.lmask[f] & ((1u << lev) - 1u));
    const Node nd = internal_node(cube, s.topo.ukey[f], lev, l + s.topo.nexcl[l] + s.topo.nstart[l] + 1, s.ustart[f],
                                  s.ustart[l + 1]);
    a.nodes[pre] = nd;
    a.nx[pre] = s.topo.nx[pre] = nd.next;
    a.nlev[pre] = s.lv[pre] = (uint8_t)lev;
    s.ord[s.start[lev] + atomicAdd(&s.fill[lev], 1)] = (uint16_t)pre;
    list_ancestor(a.anc, 0, m, walk_segments(n), pre, nd.next, lev);
    // (one node of a level straddles a chunk's end at most: the second moments' lists)
    const int ch = pre / kChunk;
    if (nd.next > (ch + 1) * kChunk) a.obkt[min(lev, kLevels - 1) * a.nchunks + ch] = pre;
  }
  for (int x = t; x < U; x += kSmallThreads) {
    const int pre = x + s.topo.nexcl[x] + s.topo.nstart[x];
    Mom mo;
    const Node nd = leaf_node(&s.cube, pre, s.ustart[x], s.ustart[x + 1] - s.ustart[x], x > 0 ? s.split[x - 1] : -1,
                              x < U - 1 ? s.split[x] : -1, ps, mo);
    a.nodes[pre] = nd;
    a.mom[pre] = mo;
    a.nx[pre] = s.topo.nx[pre] = pre + 1;
    a.nlev[pre] = s.lv[pre] = (uint8_t)(nd.meta >> 8);
  }
  __syncthreads();

  // moments, deepest level first, and the straddling nodes' children
  for (int L = kLevels; L >= 0; --L) {
    const int b = s.start[L], e = s.start[L + 1];
    if (b == e) continue;
    for (int j = b + t; j < e; j += kSmallThreads) {
      const int p = s.ord[j], end = s.topo.nx[p];
      Mom q{0.0, 0.0, 0.0, 0.0};
      int c = p + 1;
      for (int k = 0; k < 8 && c < end; ++k, c = max(s.topo.nx[c], c + 1)) add_mom(q, a.mom[c]);
      const double ctr[3] = {a.nodes[p].cx, a.nodes[p].cy, a.nodes[p].cz};
      finish_node(p, q, ctr, a.nodes, a.mom);
    }
    __syncthreads();
  }
  for (int slot = t; slot < kLevels * a.nchunks; slot += kSmallThreads) {
    const int p = a.obkt[slot];
    if (p < 0) continue;
    const int end = s.topo.nx[p];
    int k = 0;
    for (int c = p + 1; k < 8 && c < end; ++k, c = max(s.topo.nx[c], c + 1)) a.okids[8 * slot + k] = c;
    for (; k < 8; ++k) a.okids[8 * slot + k] = -1;
  }
  __syncthreads();

  // Hilbert walk order
  for (int k = t; k < n; k += kSmallThreads) {
    s.sort.key[0][k] = hilbert_key(cube, ps[k], a.hlevels);
    s.sort.idx[0][k] = k;
  }
  __syncthreads();
  int b = 0;
  for (int shift = 0; shift < 3 * a.hlevels; shift += 8, b ^= 1) small_sort_pass(s, n, shift, b);
  for (int k = t; k < n; k += kSmallThreads) a.horder[k] = s.sort.idx[b][k];
}

template <typename T, typename T4>
static hipError_t build_small_impl(const T* pos, const T* mass, int n, const BuildWs& w, hipStream_t st) {
  if (n < 1 || n > kSmallBuild || w.n_seg != 1 || !w.anc) return hipErrorInvalidValue;
  SmallArgs a{n,       w.cube, w.counts, w.seg_off == w.own_off ? nullptr : w.seg_off, w.own_off, w.croot, w.cfirst,
              w.idx_a, w.ps,   w.nodes,  w.mom, w.nx, w.nlev, w.obkt, w.okids, w.anc, w.horder, (int)n_chunks(n),
              hilbert_levels(1)};
  k_build_small<T, T4><<<1, kSmallThreads, 0, st>>>(pos, mass, a);
  return hipGetLastError();
}

hipError_t build_small_f32(const float* pos, const float* mass, int n, const BuildWs& w, hipStream_t st) {
  return build_small_impl<float, float4>(pos, mass, n, w, st);
}

hipError_t build_small_f64(const double* pos, const double* mass, int n, const BuildWs& w, hipStream_t st) {
  return build_small_impl<double, double4>(pos, mass, n, w, st);
}

// The walk order of the targets as caller indices: out[k] = perm[order[k]]
// (order: Morton positions in walk order; null = Morton order itself).
__global__ __launch_bounds__(256) void k_walk_order(const int32_t* __restrict__ order, const int32_t* __restrict__ perm,
                                                    int n, int32_t* __restrict__ out) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k < n) out[k] = perm[order ? order[k] : k];
}

hipError_t launch_walk_order(const int32_t* order, const int32_t* perm, int n, int32_t* out, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  k_walk_order<<<nblk(n, 256), 256, 0, st>>>(order, perm, n, out);
  return hipGetLastError();
}

hipError_t hilbert_order(bool f64, int n, const BuildWs& w, hipStream_t st) {
  return f64 ? hilbert_impl<double4>(n, w, st) : hilbert_impl<float4>(n, w, st);
}

// ---------------------------------------------------------------- second moments
// Quadrupole cell terms (walks of order 2) need each node's second moments
// about its centre of mass.  A leaf sums over its particles (one particle: 0);
// a cell takes its children's moments shifted to its own centre of mass by the
// parallel-axis theorem, B = sum_c (B_c + M_c d_c d_c^T) with d_c = com_c -
// com, children in octant order, one pass per level, deepest first.
__device__ __forceinline__ void put_quad(QuadRec* __restrict__ qr, int p, const double b[6]) {
  QuadRec q;
  q.bxx = b[0];
  q.bxy = b[1];
  q.bxz = b[2];
  q.byy = b[3];
  q.byz = b[4];
  q.bzz = b[5];
  const double T = b[0] + b[3] + b[5];
  q.t05 = 0.5 * T;
  q.nt15 = -1.5 * T;
  qr[p] = q;
}

// Second moments of leaf c (over its particles; one particle: zero).
template <typename T4>
__device__ __forceinline__ void leaf_quad(const Node& nd, const T4* __restrict__ ps, double b[6]) {
  for (int t = 0; t < 6; ++t) b[t] = 0.0;
  if (nd.count <= 1) return;
  for (int k = nd.first; k < nd.first + nd.count; ++k) {
    const T4 q = ps[k];
    const double m = (double)q.w;
    const double y0 = (double)q.x - nd.cx, y1 = (double)q.y - nd.cy, y2 = (double)q.z - nd.cz;
    b[0] += m * y0 * y0;
    b[1] += m * y0 * y1;
    b[2] += m * y0 * y2;
    b[3] += m * y1 * y1;
    b[4] += m * y1 * y2;
    b[5] += m * y2 * y2;
  }
}

// Child c's term of the parallel-axis fold into a parent with centre of mass
// (px, py, pz).
__device__ __forceinline__ void quad_fold(double b[6], const double cb[6], double cx, double cy, double cz, double cM,
                                          double px, double py, double pz) {
  const double d0 = cx - px, d1 = cy - py, d2 = cz - pz;
  const double m0 = cM * d0, m1 = cM * d1, m2 = cM * d2;
  b[0] += cb[0] + m0 * d0;
  b[1] += cb[1] + m0 * d1;
  b[2] += cb[2] + m0 * d2;
  b[3] += cb[3] + m1 * d1;
  b[4] += cb[4] + m1 * d2;
  b[5] += cb[5] + m2 * d2;
}

// The launches of the first moments (k_moments_chunk, k_moments_super,
// k_moments_final), for the second, over the same chunks: the chunk launch forms the leaves' moments
// from their particles and folds the chunk's closed nodes in LDS; the
// straddling nodes and their children are the lists the build made.
template <typename T4>
__global__ __launch_bounds__(kChunkThreads) void k_quad_chunk(const Counts* __restrict__ cnt, const int32_t* __restrict__ nx,
                                                    const uint8_t* __restrict__ nlev, const Node* __restrict__ nodes,
                                                    const T4* __restrict__ ps, QuadRec* __restrict__ qr) {
  __shared__ ChunkIndex ci;
  __shared__ double sb[kChunk][6];
  __shared__ double sc[kChunk][4];
  const int n_nodes = cnt->n_nodes;
  const int c0 = blockIdx.x * kChunk;
  if (c0 >= n_nodes) return;
  const int cn = min(kChunk, n_nodes - c0), c1 = c0 + cn;
  const int tid = threadIdx.x;
  for (int i = tid; i < cn; i += blockDim.x) {
    const int nxt = nx[c0 + i];
    const Node nd = nodes[c0 + i];
    ci.nx[i] = nxt;
    ci.lv[i] = (uint8_t)min((int)nlev[c0 + i], kLevels);
    sc[i][0] = nd.cx;
    sc[i][1] = nd.cy;
    sc[i][2] = nd.cz;
    sc[i][3] = nd.M;
    if (nxt == c0 + i + 1) {
      double b[6];
      leaf_quad(nd, ps, b);
      for (int t = 0; t < 6; ++t) sb[i][t] = b[t];
      put_quad(qr, c0 + i, b);
    }
  }
  __syncthreads();
  chunk_sort(ci, c0, cn);
  for (int t = 0; t < ci.n_levels; ++t) {
    const int L = ci.levels[t];
    for (int j = ci.start[L] + tid; j < ci.start[L + 1]; j += kChunkThreads) {
      const int i = ci.ord[j];
      const int end = ci.nx[i] - c0;
      double b[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
      int c = i + 1;
      for (int k = 0; k < 8 && c < end; ++k, c = max(ci.nx[c] - c0, c + 1))
        quad_fold(b, sb[c], sc[c][0], sc[c][1], sc[c][2], sc[c][3], sc[i][0], sc[i][1], sc[i][2]);
      for (int q = 0; q < 6; ++q) sb[i][q] = b[q];
    }
    __syncthreads();
  }
  for (int i = tid; i < cn; i += blockDim.x)
    if (!chunk_leaf(ci, c0, i) && ci.nx[i] <= c1) put_quad(qr, c0 + i, sb[i]);
}

__device__ __forceinline__ void fold_quad(int p, const int (&kids)[8], int n_nodes, const Node* __restrict__ nodes,
                                          QuadRec* qr) {
  const double px = nodes[p].cx, py = nodes[p].cy, pz = nodes[p].cz;
  double b[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const int c = kids[k];
    if (c <= p || c >= n_nodes) break;
    const QuadRec q = qr[c];
    const double cb[6] = {q.bxx, q.bxy, q.bxz, q.byy, q.byz, q.bzz};
    quad_fold(b, cb, nodes[c].cx, nodes[c].cy, nodes[c].cz, nodes[c].M, px, py, pz);
  }
  put_quad(qr, p, b);
}

__global__ __launch_bounds__(kSuperThreads) void k_quad_super(const Counts* __restrict__ cnt,
                                                              const int32_t* __restrict__ obkt,
                                                              const int32_t* __restrict__ nx, int nchunks,
                                                              const Node* __restrict__ nodes,
                                                              const int32_t* __restrict__ okids, QuadRec* qr) {
  const int n_nodes = cnt->n_nodes;
  fold_super(
      cnt, obkt, nx, nchunks,
      [&](int slot, int, int (&kids)[8]) {
#pragma unroll
        for (int k = 0; k < 8; ++k) kids[k] = okids[8 * (int64_t)slot + k];
      },
      [](int, int) {}, [&](int p, const int (&kids)[8]) { fold_quad(p, kids, n_nodes, nodes, qr); });
}

__global__ __launch_bounds__(kFinalThreads) void k_quad_final(const Counts* __restrict__ cnt,
                                                              const int32_t* __restrict__ obkt,
                                                              const int32_t* __restrict__ okids,
                                                              const int32_t* __restrict__ sbkt, int nsuper,
                                                              const Node* __restrict__ nodes, QuadRec* qr) {
  const int n_nodes = cnt->n_nodes;
  fold_final(cnt, obkt, okids, sbkt, nsuper,
             [&](int p, const int (&kids)[8]) { fold_quad(p, kids, n_nodes, nodes, qr); });
}

template <typename T4>
static hipError_t quad_impl(int n, const BuildWs& w, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  const int nch = (int)n_chunks(n);
  k_quad_chunk<T4><<<nch, kChunkThreads, 0, st>>>(w.counts, w.nx, w.nlev, w.nodes, reinterpret_cast<const T4*>(w.ps),
                                                  w.qrec);
  const int nsup = n_super(n);
  k_quad_super<<<nsup, kSuperThreads, 0, st>>>(w.counts, w.obkt, w.nx, nch, w.nodes, w.okids, w.qrec);
  if (nsup > 1)
    k_quad_final<<<1, kFinalThreads, 0, st>>>(w.counts, w.obkt, w.okids, w.sbkt, nsup, w.nodes, w.qrec);
  return hipGetLastError();
}

hipError_t quad_moments(bool f64, int n, const BuildWs& w, hipStream_t st) {
  return f64 ? quad_impl<double4>(n, w, st) : quad_impl<float4>(n, w, st);
}

hipError_t build_tree_f32(const float* pos, const float* mass, int n, const BuildWs& w, const BuildFork* fork,
                          hipStream_t st) {
  return build_impl<float, float4>(pos, mass, n, w, fork, st);
}

hipError_t build_tree_f64(const double* pos, const double* mass, int n, const BuildWs& w, const BuildFork* fork,
                          hipStream_t st) {
  return build_impl<double, double4>(pos, mass, n, w, fork, st);
}

}  // namespace bh
