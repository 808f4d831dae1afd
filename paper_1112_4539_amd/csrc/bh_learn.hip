// bh_learn.hip -- the learned opening parameter (gfx950): group features, the
// per-group force error that labels them, and the small MLP that maps features
// to theta, with its training step.  None of this is in the paper: the paper
// uses one fixed theta (Eq. (2)); here each walk group of 64 targets may get
// its own, predicted from the group's geometry and the tree around it.
//
// MLP: 8 -> 64 -> 64 -> 1, tanh-form GELU, theta = 0.2 + 0.8 sigmoid(z).
// Matrix products run on the matrix cores (v_mfma_f32_16x16x32_bf16): bf16
// operands, FP32 accumulation.  Weights are kept in FP32 (Adam state) and
// rounded to bf16 copies after every step; biases stay FP32.  A workgroup
// handles a tile of 32 rows (two 16-row MFMA blocks), staging activations and
// their transposes in LDS so that every operand fragment is one 16-byte read.
#include "bh_internal.h"

namespace bh {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------- bf16
// Round to nearest bfloat16, ties to even (NaN stays NaN).
__device__ __forceinline__ uint16_t to_bf16(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return 0x7fc0;
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float from_bf16(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

__device__ __forceinline__ bf16x8 frag(const uint16_t* p) {  // 8 consecutive bf16, 16-byte aligned
  const uint4 u = *reinterpret_cast<const uint4*>(p);
  return __builtin_bit_cast(bf16x8, u);
}
__device__ __forceinline__ bf16x8 zero8() { return __builtin_bit_cast(bf16x8, make_uint4(0, 0, 0, 0)); }

// D += A B for 16x16 tiles with K = 32.  Lane l supplies A[l%16][k], B[k][l%16]
// for its eight k of the lane group l/16 (the same k for A and B), and holds
// D[4 (l/16) + i][l%16], i = 0..3.
__device__ __forceinline__ f32x4 mma(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

constexpr float kGeluC = 0.7978845608028654f;  // sqrt(2/pi)
constexpr float kGeluA = 0.044715f;
__device__ __forceinline__ float gelu(float x) {
  return 0.5f * x * (1.0f + tanhf(kGeluC * (x + kGeluA * x * x * x)));
}
__device__ __forceinline__ float gelu_grad(float x) {
  const float t = tanhf(kGeluC * (x + kGeluA * x * x * x));
  return 0.5f * (1.0f + t) + 0.5f * x * (1.0f - t * t) * kGeluC * (1.0f + 3.0f * kGeluA * x * x);
}

// ---------------------------------------------------------------- features
// Eight scale-free descriptors of walk group g (the Morton positions at
// [64g, 64g+64) of the walk order `order`; null: the positions themselves):
//   0 log2(h / h_typ), h the AABB half-width, h_typ = L (64/N)^(1/3) / 2
//   1 |centre of mass - centre of mass of c| / l_c, c the smallest cell
//     holding the group, l_c its side
//   2 the same against the ancestor of c three levels up (or the root)
//   3 mass-weighted RMS radius about the centre of mass, / h
//   4 |centre of mass - AABB centre| / h
//   5 log10(density of the smallest cell holding the group / M_tot L^-3)
//   6 the same for that cell's parent
//   7 log2(side of that cell / h)
// N, L, M_tot are those of the cluster of the group's first Morton position
// (the whole set for one tree).
//
// A workgroup takes kFeatGroups groups.  A wave reads a group's particles, one
// per lane, into LDS, and one lane per group then forms the sums over them in
// order and descends the tree.  (With one thread per group reading its particles
// itself, 64 scattered loads three times over on a quarter of the CUs, the
// kernel took 117 us for 1M particles; it takes 60, most of it the descent.)
constexpr int kFeatGroups = 32, kFeatWaves = 4, kFeatPerWave = kFeatGroups / kFeatWaves;

template <typename T4>
__global__ __launch_bounds__(64 * kFeatWaves) void k_features(
    const Node* __restrict__ nodes, const T4* __restrict__ ps, const Cube* __restrict__ cubes,
    const int32_t* __restrict__ scid, const int32_t* __restrict__ croot, const int64_t* __restrict__ seg_off, int n_seg,
    int n, const int32_t* __restrict__ order, float* __restrict__ X) {
  __shared__ T4 part[kFeatGroups][64 + 1];
  __shared__ int2 range[kFeatGroups];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  for (int r = 0; r < kFeatPerWave; ++r) {
    const int q = w * kFeatPerWave + r;
    const int s = 64 * (blockIdx.x * kFeatGroups + q) + lane;
    int lo = n, hi = 0;
    if (s < n) {
      const int m = order ? min(max(order[s], 0), n - 1) : s;
      part[q][lane] = ps[m];
      lo = m;
      hi = m + 1;
    }
    for (int o = 32; o > 0; o >>= 1) {
      lo = min(lo, __shfl_xor(lo, o, 64));
      hi = max(hi, __shfl_xor(hi, o, 64));
    }
    if (lane == 0) range[q] = make_int2(lo, hi);
  }
  __syncthreads();
  if (lane >= kFeatPerWave) return;
  const int slot = w * kFeatPerWave + lane;
  const int g = blockIdx.x * kFeatGroups + slot;
  const int s0 = 64 * g;
  if (s0 >= n) return;
  const int cnt = min(n - s0, 64);
  const T4* mem = part[slot];
  // the group's Morton range [a, b)
  const int a = range[slot].x, b = range[slot].y;
  const int k = scid ? min(max(scid[a], 0), n_seg - 1) : 0;
  const double L = cubes[k].L;
  const int64_t nk64 = seg_off[k + 1] - seg_off[k];
  const double Nk = (double)(nk64 > 0 ? nk64 : 1);
  const int cap = 2 * n;
  const int root = min(max(croot[k], 0), cap - 1);
  const double Mtot = nodes[root].M;
  double lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
  double M = 0.0, Sx = 0.0, Sy = 0.0, Sz = 0.0;
  for (int s = 0; s < cnt; ++s) {
    const T4 p = mem[s];
    const double x = (double)p.x, y = (double)p.y, z = (double)p.z, m = (double)p.w;
    lo[0] = fmin(lo[0], x); hi[0] = fmax(hi[0], x);
    lo[1] = fmin(lo[1], y); hi[1] = fmax(hi[1], y);
    lo[2] = fmin(lo[2], z); hi[2] = fmax(hi[2], z);
    M += m;
    Sx += m * x; Sy += m * y; Sz += m * z;
  }
  double h = fmax(fmax(hi[0] - lo[0], hi[1] - lo[1]), hi[2] - lo[2]) * 0.5;
  h = fmax(h, ldexp(L, -22));
  const double gc[3] = {0.5 * (lo[0] + hi[0]), 0.5 * (lo[1] + hi[1]), 0.5 * (lo[2] + hi[2])};
  double com[3] = {gc[0], gc[1], gc[2]};
  if (M > 0.0) {
    com[0] = Sx / M; com[1] = Sy / M; com[2] = Sz / M;
  }
  double R2 = 0.0;
  for (int s = 0; s < cnt; ++s) {
    const T4 p = mem[s];
    const double dx = (double)p.x - com[0], dy = (double)p.y - com[1], dz = (double)p.z - com[2];
    R2 += (double)p.w * (dx * dx + dy * dy + dz * dz);
  }
  const double rms = M > 0.0 ? sqrt(R2 / M) : 0.0;
  // smallest cell holding the group's Morton range [a, b): descend from the cluster's root while a
  // child holds the whole range (at most 21 levels of at most 8 children)
  // (path[0] = c, path[1] = its parent, ... path[3] = three levels up)
  int path[4] = {root, root, root, root};
  int c = root;
  const Node& r0 = nodes[root];
  if (r0.first <= a && r0.first + r0.count >= b) {
    for (int depth = 0; depth < 2 * kLevels && !(nodes[c].meta & 1); ++depth) {
      const int end = min(nodes[c].next, cap);
      int ch = c + 1, found = -1;
      for (int s = 0; s < 8 && ch < end; ++s) {
        const Node& nd = nodes[ch];
        if (nd.first <= a && nd.first + nd.count >= b) {
          found = ch;
          break;
        }
        ch = max(nd.next, ch + 1);
      }
      if (found < 0) break;
      path[3] = path[2];
      path[2] = path[1];
      path[1] = c;
      c = found;
      path[0] = c;
    }
  }
  const int par = path[1], anc = path[3];
  const double rho_mean = fmax(Mtot, 1e-300) / (L * L * L);
  const double lc = nodes[c].l, lp = nodes[par].l;
  float* o = X + 8 * (int64_t)g;
  o[0] = (float)log2(h / (0.5 * L * cbrt(64.0 / Nk)));
  {
    const Node& nc = nodes[c];
    const Node& na = nodes[anc];
    const double cx = com[0] - nc.cx, cy = com[1] - nc.cy, cz = com[2] - nc.cz;
    const double ax = com[0] - na.cx, ay = com[1] - na.cy, az = com[2] - na.cz;
    o[1] = (float)(sqrt(cx * cx + cy * cy + cz * cz) / nc.l);
    o[2] = (float)(sqrt(ax * ax + ay * ay + az * az) / na.l);
  }
  o[3] = (float)(rms / h);
  const double ex = com[0] - gc[0], ey = com[1] - gc[1], ez = com[2] - gc[2];
  o[4] = (float)(sqrt(ex * ex + ey * ey + ez * ez) / h);
  o[5] = (float)log10(fmax(nodes[c].M, 1e-300) / (lc * lc * lc) / rho_mean);
  o[6] = (float)log10(fmax(nodes[par].M, 1e-300) / (lp * lp * lp) / rho_mean);
  o[7] = (float)log2(lc / h);
}

hipError_t launch_features(bool f64, const Node* nodes, const void* ps, const Cube* cubes, const int32_t* scid,
                           const int32_t* croot, const int64_t* seg_off, int n_seg, int n, const int32_t* order,
                           float* X, hipStream_t st) {
  const int G = (n + 63) / 64;
  if (G == 0) return hipSuccess;
  const int blocks = (G + kFeatGroups - 1) / kFeatGroups;
  if (f64)
    k_features<double4><<<blocks, 64 * kFeatWaves, 0, st>>>(nodes, static_cast<const double4*>(ps), cubes, scid, croot,
                                                            seg_off, n_seg, n, order, X);
  else
    k_features<float4><<<blocks, 64 * kFeatWaves, 0, st>>>(nodes, static_cast<const float4*>(ps), cubes, scid, croot,
                                                           seg_off, n_seg, n, order, X);
  return hipGetLastError();
}

// ---------------------------------------------------------------- group error
// RMS over walk group g's particles (as in k_features) of |a - a_ref| / |a_ref|;
// where it is within `target`, label[g] = max(label[g], theta) (labels start
// at the grid minimum).
template <typename R>
__global__ __launch_bounds__(256) void k_group_error(const R* __restrict__ acc, const double* __restrict__ ref,
                                                     const int32_t* __restrict__ perm,
                                                     const int32_t* __restrict__ order, int n, double theta,
                                                     double target, double* __restrict__ rms,
                                                     float* __restrict__ label) {
  const int g = blockIdx.x * blockDim.x + threadIdx.x;
  const int s0 = 64 * g;
  if (s0 >= n) return;
  const int s1 = min(n, s0 + 64);
  // (a particle whose reference force is exactly zero has no relative error:
  // it is left out, and a group of only such particles has RMS 0)
  double s = 0.0;
  int m = 0;
  for (int j = s0; j < s1; ++j) {
    const int64_t o = perm[order ? min(max(order[j], 0), n - 1) : j];
    const double rx = ref[3 * o], ry = ref[3 * o + 1], rz = ref[3 * o + 2];
    const double dx = (double)acc[3 * o] - rx, dy = (double)acc[3 * o + 1] - ry, dz = (double)acc[3 * o + 2] - rz;
    const double r2 = rx * rx + ry * ry + rz * rz;
    if (r2 > 0.0) {
      s += (dx * dx + dy * dy + dz * dz) / r2;
      ++m;
    }
  }
  const double r = m > 0 ? sqrt(s / (double)m) : 0.0;
  if (rms) rms[g] = r;
  if (label && r <= target) label[g] = fmaxf(label[g], (float)theta);
}

hipError_t launch_group_error(bool f64, const void* acc, const double* ref, const int32_t* perm,
                              const int32_t* order, int n, double theta, double target, double* rms, float* label,
                              hipStream_t st) {
  const int G = (n + 63) / 64;
  if (G == 0) return hipSuccess;
  if (f64)
    k_group_error<double><<<(G + 255) / 256, 256, 0, st>>>(static_cast<const double*>(acc), ref, perm, order, n,
                                                           theta, target, rms, label);
  else
    k_group_error<float><<<(G + 255) / 256, 256, 0, st>>>(static_cast<const float*>(acc), ref, perm, order, n,
                                                          theta, target, rms, label);
  return hipGetLastError();
}

// ---------------------------------------------------------------- MLP
struct MlpArgs {
  const float* P;        // [kMlpParams] FP32 master parameters
  const uint16_t* wb;    // [kMlpWb] bf16 copies: W1, W2, W2^T, w3
  const float* norm;     // [16]: mu[8], 1/sd[8]
};

// A workgroup of four waves takes a tile of 32 rows, each wave 16 of the 64
// hidden columns: a tile is a serial chain of small matrix products and about
// 4000 tanh, and a batch has few tiles (128 at 4096 rows), so what it costs is
// the length of that chain.  (With one wave per tile the gradient of 4096 rows
// took 25 us and inference of 16,384 rows 16 us.)
constexpr int kMlpWaves = 4;

// LDS of one workgroup: a 32-row tile, row-major and transposed copies.
struct alignas(16) TileLds {
  uint16_t xb[32][8];
  uint16_t xT[8][32];
  uint16_t h1[32][64];
  uint16_t h1T[64][32];
  uint16_t h2[32][64];
  uint16_t dp2[32][64];
  uint16_t dp2T[64][32];
  uint16_t dp1T[64][32];
  float gd1[32][64];   // gelu'(pre-activation) of the two hidden layers (gradient pass)
  float gd2[32][64];
  float dz[32];
  float tgt[32];
};

// Normalised bf16 inputs of the tile's rows, one feature per thread (rows past
// `rows` are zero).
template <bool kT>
__device__ __forceinline__ void load_rows(const MlpArgs& w, const float* __restrict__ X, int64_t rows, int64_t row0,
                                          const int32_t* __restrict__ idx, TileLds& s, const float* __restrict__ T) {
  const int j = threadIdx.x >> 3, k = threadIdx.x & 7;
  const int64_t row = row0 + j;
  const bool valid = row < rows;
  const int64_t src = valid ? (idx ? (int64_t)idx[row] : row) : 0;
  const float v = valid ? (X[8 * src + k] - w.norm[k]) * w.norm[8 + k] : 0.0f;
  const uint16_t hb = valid ? to_bf16(v) : (uint16_t)0;
  s.xb[j][k] = hb;
  if constexpr (kT) {
    s.xT[k][j] = hb;
    if (k == 0) s.tgt[j] = valid ? T[src] : 0.0f;
  }
}

// The hidden layers of the tile's columns 16q..16q+15: states (and, for the
// gradient pass, their transposes and the GELU slopes) to LDS.  Ends with a
// barrier.
template <bool kT>
__device__ __forceinline__ void fwd_hidden(const MlpArgs& w, TileLds& s, int q, int lane) {
  const int r = lane & 15, g = lane >> 4;
  const int col = 16 * q + r;
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  // layer 1: K = 8 features, padded to 32 with zeros
  const bf16x8 bw1 = g == 0 ? frag(w.wb + kMlpW1b + col * 8) : zero8();
  const float bias1 = w.P[kMlpB1 + col];
  const bf16x8 bw2a = frag(w.wb + kMlpW2b + col * 64 + 8 * g);
  const bf16x8 bw2b = frag(w.wb + kMlpW2b + col * 64 + 32 + 8 * g);
  const float bias2 = w.P[kMlpB2 + col];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const bf16x8 ax = g == 0 ? frag(&s.xb[16 * h + r][0]) : zero8();
    const f32x4 d = mma(ax, bw1, zero);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = 16 * h + 4 * g + i;
      const float v = d[i] + bias1;
      const uint16_t hb = to_bf16(gelu(v));
      s.h1[row][col] = hb;
      if constexpr (kT) {
        s.h1T[col][row] = hb;
        s.gd1[row][col] = gelu_grad(v);
      }
    }
  }
  __syncthreads();
  // layer 2: K = 64
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    f32x4 d = mma(frag(&s.h1[16 * h + r][8 * g]), bw2a, zero);
    d = mma(frag(&s.h1[16 * h + r][32 + 8 * g]), bw2b, d);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float v = d[i] + bias2;
      s.h2[16 * h + 4 * g + i][col] = to_bf16(gelu(v));
      if constexpr (kT) s.gd2[16 * h + 4 * g + i][col] = gelu_grad(v);
    }
  }
  __syncthreads();
}

// The output layer of rows 16h..16h+15: z in the lanes with l%16 == 0 (rows
// 16h + 4(l/16) + i).
__device__ __forceinline__ f32x4 fwd_out(const MlpArgs& w, const TileLds& s, int h, int lane) {
  const int r = lane & 15, g = lane >> 4;
  // one output column (B is zero outside column 0)
  f32x4 d = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int ks = 0; ks < 2; ++ks)
    d = mma(frag(&s.h2[16 * h + r][32 * ks + 8 * g]), r == 0 ? frag(w.wb + kMlpw3b + 32 * ks + 8 * g) : zero8(), d);
  const float b3 = w.P[kMlpB3];
#pragma unroll
  for (int i = 0; i < 4; ++i) d[i] += b3;
  return d;
}

// theta for every row of X: 0.2 + 0.8 sigmoid(z), times alpha, at most `cap`;
// a non-finite result is replaced by `fallback`.
__global__ __launch_bounds__(64 * kMlpWaves) void k_mlp_infer(MlpArgs w, const float* __restrict__ X, int64_t rows,
                                                              float alpha, float fallback, float cap,
                                                              float* __restrict__ theta) {
  __shared__ TileLds s;
  const int lane = threadIdx.x & 63, q = uniform(threadIdx.x >> 6);
  const int r = lane & 15, g = lane >> 4;
  for (int64_t tile = blockIdx.x; tile * 32 < rows; tile += gridDim.x) {
    load_rows<false>(w, X, rows, tile * 32, nullptr, s, nullptr);
    __syncthreads();
    fwd_hidden<false>(w, s, q, lane);
    if (q < 2) {
      const f32x4 z = fwd_out(w, s, q, lane);
      if (r == 0) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int64_t row = tile * 32 + 16 * q + 4 * g + i;
          if (row < rows) {
            float th = (0.2f + 0.8f / (1.0f + expf(-z[i]))) * alpha;
            if (!isfinite(th)) th = fallback;
            theta[row] = fminf(th, cap);
          }
        }
      }
    }
    __syncthreads();
  }
}

// Gradient of the batch loss mean((sigmoid(z) - t)^2) over the rows idx[0..B):
// every workgroup accumulates its tiles' contributions (weight gradients in
// MFMA accumulators, wave q those of rows 16q..16q+15 of W1 and W2) and writes
// one partial vector; k_mlp_reduce sums them in a fixed order.
__global__ __launch_bounds__(64 * kMlpWaves) void k_mlp_grad(MlpArgs w, const float* __restrict__ X,
                                                             const float* __restrict__ T,
                                                             const int32_t* __restrict__ idx, int batch,
                                                             float* __restrict__ partial) {
  __shared__ TileLds s;
  __shared__ float loss2[2];
  const int lane = threadIdx.x & 63, q = uniform(threadIdx.x >> 6);
  const int r = lane & 15, g = lane >> 4;
  const int col = 16 * q + r;
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  f32x4 gW2[4], gW1 = zero;
#pragma unroll
  for (int b = 0; b < 4; ++b) gW2[b] = zero;
  float gb1 = 0.f, gb2 = 0.f, gw3 = 0.f, gb3 = 0.f, loss = 0.f;
  const float scale = 2.0f / (float)batch;
  const float w3c = from_bf16(w.wb[kMlpw3b + col]);
  for (int64_t tile = blockIdx.x; tile * 32 < batch; tile += gridDim.x) {
    load_rows<true>(w, X, batch, tile * 32, idx, s, T);
    __syncthreads();
    fwd_hidden<true>(w, s, q, lane);
    // output error, half a tile per wave
    if (q < 2) {
      const f32x4 z = fwd_out(w, s, q, lane);
      if (r == 0) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int row = 16 * q + 4 * g + i;
          const bool valid = tile * 32 + row < batch;
          const float y = 1.0f / (1.0f + expf(-z[i]));
          const float e = y - s.tgt[row];
          s.dz[row] = valid ? scale * e * y * (1.0f - y) : 0.0f;
          loss += valid ? e * e : 0.0f;
        }
      }
    }
    __syncthreads();
    // last layer: lane l of wave 2 owns w3[l], wave 3 the bias
    if (q == 2) {
      for (int row = 0; row < 32; ++row) gw3 += s.dz[row] * from_bf16(s.h2[row][lane]);
    } else if (q == 3) {
      gb3 += lane < 32 ? s.dz[lane] : 0.0f;
    }
    // error of the second hidden layer
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int row = 16 * h + 4 * g + i;
        const float dp = s.dz[row] * w3c * s.gd2[row][col];
        gb2 += dp;
        const uint16_t hb = to_bf16(dp);
        s.dp2[row][col] = hb;
        s.dp2T[col][row] = hb;
      }
    __syncthreads();
    // error of the first hidden layer: dh1 = bf16(dpre2) W2
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      f32x4 d = zero;
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
        d = mma(frag(&s.dp2[16 * h + r][32 * ks + 8 * g]), frag(w.wb + kMlpW2Tb + col * 64 + 32 * ks + 8 * g), d);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int row = 16 * h + 4 * g + i;
        const float dp = d[i] * s.gd1[row][col];
        gb1 += dp;
        s.dp1T[col][row] = to_bf16(dp);
      }
    }
    // dW2 += bf16(dpre2)^T h1 (contraction over the tile's 32 rows)
#pragma unroll
    for (int nt = 0; nt < 4; ++nt)
      gW2[nt] = mma(frag(&s.dp2T[col][8 * g]), frag(&s.h1T[16 * nt + r][8 * g]), gW2[nt]);
    __syncthreads();
    // dW1 += bf16(dpre1)^T x'
    gW1 = mma(frag(&s.dp1T[col][8 * g]), r < 8 ? frag(&s.xT[r][8 * g]) : zero8(), gW1);
    __syncthreads();
  }
  // this workgroup's partial gradient
  float* out = partial + (int64_t)blockIdx.x * kMlpGradLen;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int o = 16 * q + 4 * g + i;
    if (r < 8) out[kMlpW1 + o * 8 + r] = gW1[i];
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) out[kMlpW2 + o * 64 + 16 * nt + r] = gW2[nt][i];
  }
  gb1 += __shfl_xor(gb1, 16, 64);
  gb1 += __shfl_xor(gb1, 32, 64);
  gb2 += __shfl_xor(gb2, 16, 64);
  gb2 += __shfl_xor(gb2, 32, 64);
  if (g == 0) {
    out[kMlpB1 + col] = gb1;
    out[kMlpB2 + col] = gb2;
  }
  if (q == 2) out[kMlpw3 + lane] = gw3;
  if (q == 3) {
    for (int o = 1; o < 32; o <<= 1) gb3 += __shfl_xor(gb3, o, 64);
    if (lane == 0) out[kMlpB3] = gb3;
  }
  loss += __shfl_xor(loss, 16, 64);
  loss += __shfl_xor(loss, 32, 64);
  if (q < 2 && lane == 0) loss2[q] = loss;
  __syncthreads();
  if (threadIdx.x == 0) out[kMlpParams] = loss2[0] + loss2[1];
}

// The partial vectors' sum, FP64, in a fixed order: a workgroup takes 32
// parameters, eight threads each an eighth of the vectors.  (One thread per
// parameter read 128 vectors one after the other on 19 workgroups: 32 us.)
constexpr int kReduceParams = 32, kReduceSlices = 8;
__global__ __launch_bounds__(kReduceParams * kReduceSlices) void k_mlp_reduce(const float* __restrict__ partial,
                                                                              int nparts, int batch,
                                                                              float* __restrict__ grad) {
  __shared__ double red[kReduceSlices][kReduceParams];
  const int c = threadIdx.x % kReduceParams, sl = threadIdx.x / kReduceParams;
  const int p = blockIdx.x * kReduceParams + c;
  double s = 0.0;
  if (p < kMlpGradLen) {
    const int per = (nparts + kReduceSlices - 1) / kReduceSlices;
    const int b1 = min((sl + 1) * per, nparts);
#pragma unroll 8
    for (int b = sl * per; b < b1; ++b) s += (double)partial[(int64_t)b * kMlpGradLen + p];
  }
  red[sl][c] = s;
  __syncthreads();
  if (sl != 0 || p >= kMlpGradLen) return;
  for (int k = 1; k < kReduceSlices; ++k) s += red[k][c];
  grad[p] = (float)(p == kMlpParams ? s / (double)batch : s);
}

// bf16 copies of the weights (W1, W2, W2 transposed, w3) from the FP32 masters.
__device__ __forceinline__ void write_bf16_copy(const float* __restrict__ P, uint16_t* __restrict__ wb, int p) {
  if (p < kMlpB1) {
    wb[kMlpW1b + p] = to_bf16(P[p]);
  } else if (p >= kMlpW2 && p < kMlpB2) {
    const int q = p - kMlpW2, o = q / 64, i = q % 64;
    const uint16_t v = to_bf16(P[p]);
    wb[kMlpW2b + q] = v;
    wb[kMlpW2Tb + i * 64 + o] = v;
  } else if (p >= kMlpw3 && p < kMlpB3) {
    wb[kMlpw3b + (p - kMlpw3)] = to_bf16(P[p]);
  }
}

__global__ __launch_bounds__(256) void k_mlp_prepare(const float* __restrict__ P, uint16_t* __restrict__ wb) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p < kMlpParams) write_bf16_copy(P, wb, p);
}

// One Adam step (Kingma & Ba): c1 = 1 - beta1^t, c2 = 1 - beta2^t.
__global__ __launch_bounds__(256) void k_mlp_adam(float* __restrict__ P, const float* __restrict__ grad,
                                                  float* __restrict__ m, float* __restrict__ v, float lr, float beta1,
                                                  float beta2, float eps, float c1, float c2,
                                                  uint16_t* __restrict__ wb) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= kMlpParams) return;
  const float gr = grad[p];
  const float mm = beta1 * m[p] + (1.0f - beta1) * gr;
  const float vv = beta2 * v[p] + (1.0f - beta2) * gr * gr;
  m[p] = mm;
  v[p] = vv;
  P[p] = P[p] - lr * (mm / c1) / (sqrtf(vv / c2) + eps);
  write_bf16_copy(P, wb, p);
}

static inline int blocks(int64_t n, int t) { return (int)((n + t - 1) / t); }

hipError_t launch_mlp_prepare(const float* P, uint16_t* wb, hipStream_t st) {
  k_mlp_prepare<<<blocks(kMlpParams, 256), 256, 0, st>>>(P, wb);
  return hipGetLastError();
}

hipError_t launch_mlp_infer(const float* P, const uint16_t* wb, const float* norm, const float* X, int64_t rows,
                            float alpha, float fallback, float cap, float* theta, hipStream_t st) {
  if (rows <= 0) return hipSuccess;
  MlpArgs w{P, wb, norm};
  const int64_t tiles = (rows + 31) / 32;
  const int grid = (int)(tiles < 4096 ? tiles : 4096);
  k_mlp_infer<<<grid, 64 * kMlpWaves, 0, st>>>(w, X, rows, alpha, fallback, cap, theta);
  return hipGetLastError();
}

int mlp_grad_parts(int batch) {
  const int tiles = (batch + 31) / 32;
  return tiles < kMlpMaxParts ? tiles : kMlpMaxParts;
}

hipError_t launch_mlp_grad(const float* P, const uint16_t* wb, const float* norm, const float* X, const float* T,
                           const int32_t* idx, int batch, float* partial, float* grad, hipStream_t st) {
  MlpArgs w{P, wb, norm};
  const int parts = mlp_grad_parts(batch);
  k_mlp_grad<<<parts, 64 * kMlpWaves, 0, st>>>(w, X, T, idx, batch, partial);
  k_mlp_reduce<<<blocks(kMlpGradLen, kReduceParams), kReduceParams * kReduceSlices, 0, st>>>(partial, parts, batch, grad);
  return hipGetLastError();
}

hipError_t launch_mlp_adam(float* P, const float* grad, float* m, float* v, float lr, float beta1, float beta2,
                           float eps, float c1, float c2, uint16_t* wb, hipStream_t st) {
  k_mlp_adam<<<blocks(kMlpParams, 256), 256, 0, st>>>(P, grad, m, v, lr, beta1, beta2, eps, c1, c2, wb);
  return hipGetLastError();
}

}  // namespace bh
