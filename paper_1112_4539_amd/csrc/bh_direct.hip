// bh_direct.hip -- brute-force O(N^2) sum of Eq. (1) for a list of targets (gfx950).
//
// Used as the accuracy judge of the tree walk (the paper compares its tree
// forces with a brute-force sum, Sec. 5, Eq. (4)), for the labels of the
// learned opening parameter, and for the tree versus brute-force crossover.
//
// Bound: VALU issue, about 20 FP64 (14 FP32) instructions and one hardware
// root per pair.  A workgroup takes 64 / kSub targets; its waves cut the
// sources into contiguous ranges, and kSub lanes share a target, taking the
// wave's range in turn.  The partial sums meet in LDS, lanes first, then the
// waves in order, so that results are the same from run to run.
//   kSub = 1   many targets: a source is the same for the whole wave, read
//              four at a time with scalar loads straight into the
//              instructions' scalar operands (no LDS, no barrier);
//   kSub > 1   few targets: 64 / kSub of them are enough for a workgroup of up
//              to 16 waves, so that some hundred targets fill the chip.
// Four (two) sources are in flight per lane, which hides the chain from r^2
// through the root to the sums: 13.4 ms for 65,536 targets of 262,147 particles
// in FP64, 123 cycles per wave and source (7.1 ms, 65 cycles, in FP32).  (One thread per target over LDS tiles of 256
// sources, with an IEEE root and division per pair in FP64, took 54.1 ms, 494 cycles.)
#include "bh_internal.h"

namespace bh {

namespace {

constexpr int kDirectMaxWaves = 16;

struct DirectArgs {
  const void* pos;         // [n][3]
  const void* mass;        // [n]
  const int64_t* targets;  // [nt]
  int n, nt;
  double eps2;
  void* acc;               // [nt][3]
  void* pot;               // [nt]
};

template <typename R>
struct DirectSum {
  R ax, ay, az, p;
  // r^2 + eps^2 of a source at offset d.
  static __device__ __forceinline__ R dist2(R dx, R dy, R dz, R e2) {
    if constexpr (std::is_same<R, double>::value)
      return fma(dz, dz, fma(dy, dy, dx * dx)) + e2;
    else
      return fmaf(dz, dz, fmaf(dy, dy, fmaf(dx, dx, e2)));
  }
  // One source: offset d, mass m.  kSoft: eps > 0, so r^2 > 0.  Without softening a
  // pair at r = 0 adds nothing: in FP32 the root's place is taken by 0, in FP64
  // the caller leaves the pair out, whatever its mass.
  template <bool kSoft>
  __device__ __forceinline__ void add(R dx, R dy, R dz, R m, R e2) {
    const R r2 = dist2(dx, dy, dz, e2);
    R ri;
    if constexpr (std::is_same<R, double>::value) {
      ri = inv_sqrt_f64(r2);
    } else {
      ri = __builtin_amdgcn_rsqf(r2);
      if (!kSoft) ri = r2 > 0.f ? ri : 0.f;
    }
    const R mr = m * ri;
    const R mr3 = (mr * ri) * ri;
    ax = fma_(mr3, dx, ax);
    ay = fma_(mr3, dy, ay);
    az = fma_(mr3, dz, az);
    p -= mr;
  }
  static __device__ __forceinline__ float fma_(float a, float b, float c) { return fmaf(a, b, c); }
  static __device__ __forceinline__ double fma_(double a, double b, double c) { return fma(a, b, c); }
};

#define BH_CONST __attribute__((address_space(4)))

// A batch of kBatch sources whose pairs at r = 0 are to be left out (FP64 without
// softening): source k at q[3k..3k+2], not to be taken where own(k).  Such pairs
// are rare, so that one branch for the wave tells batches without any; the test is
// one for zero, since a position that is not a number has to reach the sums.
template <int kBatch, typename Own>
__device__ __forceinline__ void add_unequal(DirectSum<double>& s, const double* q, const double* m, double xi,
                                            double yi, double zi, Own&& own) {
  double dx[kBatch], dy[kBatch], dz[kBatch], r2[kBatch];
  uint64_t out = 0;
#pragma unroll
  for (int k = 0; k < kBatch; ++k) {
    dx[k] = q[3 * k] - xi;
    dy[k] = q[3 * k + 1] - yi;
    dz[k] = q[3 * k + 2] - zi;
    r2[k] = DirectSum<double>::dist2(dx[k], dy[k], dz[k], 0.0);
    out |= ballot(own(k)) | __builtin_amdgcn_fcmp(r2[k], 0.0, 1);  // ordered ==
  }
  if (out == 0ull) {
#pragma unroll
    for (int k = 0; k < kBatch; ++k) s.add<false>(dx[k], dy[k], dz[k], m[k], 0.0);
  } else {
#pragma unroll
    for (int k = 0; k < kBatch; ++k)
      if (!own(k) && r2[k] != 0.0) s.add<false>(dx[k], dy[k], dz[k], m[k], 0.0);
  }
}

template <bool kF64, bool kSoft, int kSub>
__global__ __launch_bounds__(64 * kDirectMaxWaves) void k_direct(DirectArgs a) {
  using R = typename std::conditional<kF64, double, float>::type;
  constexpr int kTargets = 64 / kSub;
  __shared__ double part[kDirectMaxWaves][kTargets][4];
  const R* pos = reinterpret_cast<const R*>(a.pos);
  const R* mass = reinterpret_cast<const R*>(a.mass);
  const int lane = threadIdx.x & 63, w = uniform(threadIdx.x >> 6), nw = blockDim.x >> 6;
  const int slot = lane / kSub, sub = lane % kSub;
  const int t = blockIdx.x * kTargets + slot;
  const int64_t ti = t < a.nt ? a.targets[t] : -1;
  const bool valid = ti >= 0 && ti < a.n;  // an index outside [0, n) yields NaN outputs
  const int i = valid ? (int)ti : -1;
  R xi = 0, yi = 0, zi = 0;
  if (valid) {
    xi = pos[3 * (int64_t)i];
    yi = pos[3 * (int64_t)i + 1];
    zi = pos[3 * (int64_t)i + 2];
  }
  const R e2 = (R)a.eps2;
  DirectSum<R> s{0, 0, 0, 0};
  constexpr bool kUnequal = kF64 && !kSoft;
  const int len = (a.n + nw - 1) / nw;
  const int j0 = min(w * len, a.n), j1 = min(j0 + len, a.n);
  if constexpr (kSub == 1) {
    constexpr int kBatch = 4;
    const BH_CONST R* ps = (const BH_CONST R*)(uintptr_t)pos;
    const BH_CONST R* pm = (const BH_CONST R*)(uintptr_t)mass;
    int j = j0;
    for (; j + kBatch <= j1; j += kBatch) {
      R q[3 * kBatch], m[kBatch];
#pragma unroll
      for (int k = 0; k < 3 * kBatch; ++k) q[k] = ps[3 * (int64_t)j + k];
#pragma unroll
      for (int k = 0; k < kBatch; ++k) m[k] = pm[(int64_t)j + k];
      // (a batch that holds a lane's own particle is rare: one test per batch)
      if constexpr (kUnequal) {
        add_unequal<kBatch>(s, q, m, xi, yi, zi, [&](int k) { return j + k == i; });
      } else if (ballot((unsigned)(i - j) < (unsigned)kBatch) == 0ull) {
#pragma unroll
        for (int k = 0; k < kBatch; ++k)
          s.template add<kSoft>(q[3 * k] - xi, q[3 * k + 1] - yi, q[3 * k + 2] - zi, m[k], e2);
      } else {
#pragma unroll
        for (int k = 0; k < kBatch; ++k)
          if (j + k != i) s.template add<kSoft>(q[3 * k] - xi, q[3 * k + 1] - yi, q[3 * k + 2] - zi, m[k], e2);
      }
    }
    for (; j < j1; ++j) {
      const int64_t b = 3 * (int64_t)j;
      if constexpr (kUnequal) {
        const R q[3] = {ps[b], ps[b + 1], ps[b + 2]}, m = pm[j];
        add_unequal<1>(s, q, &m, xi, yi, zi, [&](int) { return j == i; });
      } else {
        if (j != i) s.template add<kSoft>(ps[b] - xi, ps[b + 1] - yi, ps[b + 2] - zi, pm[j], e2);
      }
    }
  } else {
    constexpr int kBatch = 2;
    int j = j0 + sub;
    for (; j + (kBatch - 1) * kSub < j1; j += kBatch * kSub) {
      R q[3 * kBatch], m[kBatch];
#pragma unroll
      for (int k = 0; k < kBatch; ++k) {
        const int64_t b = (int64_t)j + k * kSub;
        q[3 * k] = pos[3 * b];
        q[3 * k + 1] = pos[3 * b + 1];
        q[3 * k + 2] = pos[3 * b + 2];
        m[k] = mass[b];
      }
      if constexpr (kUnequal) {
        add_unequal<kBatch>(s, q, m, xi, yi, zi, [&](int k) { return j + k * kSub == i; });
      } else {
#pragma unroll
        for (int k = 0; k < kBatch; ++k)
          if (j + k * kSub != i) s.template add<kSoft>(q[3 * k] - xi, q[3 * k + 1] - yi, q[3 * k + 2] - zi, m[k], e2);
      }
    }
    for (; j < j1; j += kSub) {
      const int64_t b = 3 * (int64_t)j;
      if constexpr (kUnequal) {
        const R q[3] = {pos[b], pos[b + 1], pos[b + 2]}, m = mass[j];
        add_unequal<1>(s, q, &m, xi, yi, zi, [&](int) { return j == i; });
      } else {
        if (j != i) s.template add<kSoft>(pos[b] - xi, pos[b + 1] - yi, pos[b + 2] - zi, mass[j], e2);
      }
    }
  }
  double v[4] = {(double)s.ax, (double)s.ay, (double)s.az, (double)s.p};
#pragma unroll
  for (int o = 1; o < kSub; o <<= 1)
#pragma unroll
    for (int c = 0; c < 4; ++c) v[c] += __shfl_xor(v[c], o, 64);
  if (sub == 0)
#pragma unroll
    for (int c = 0; c < 4; ++c) part[w][slot][c] = v[c];
  __syncthreads();
  const int u = threadIdx.x;  // output u / 4 of the workgroup, component u % 4
  if (u >= 4 * kTargets) return;
  const int k = u >> 2, c = u & 3, out = blockIdx.x * kTargets + k;
  if (out >= a.nt) return;
  double sum = part[0][k][c];
  for (int q = 1; q < nw; ++q) sum += part[q][k][c];
  const int64_t to = a.targets[out];
  if (!(to >= 0 && to < a.n)) sum = NAN;
  if (c < 3)
    reinterpret_cast<R*>(a.acc)[3 * (int64_t)out + c] = (R)sum;
  else
    reinterpret_cast<R*>(a.pot)[out] = (R)sum;
}

template <bool kF64, bool kSoft>
void launch_sub(const DirectArgs& a, int sub, int blocks, int threads, hipStream_t st) {
  if (sub == 1)
    k_direct<kF64, kSoft, 1><<<blocks, threads, 0, st>>>(a);
  else if (sub == 8)
    k_direct<kF64, kSoft, 8><<<blocks, threads, 0, st>>>(a);
  else
    k_direct<kF64, kSoft, 32><<<blocks, threads, 0, st>>>(a);
}

}  // namespace

hipError_t launch_direct(bool f64, const void* pos, const void* mass, int n, const int64_t* targets, int nt,
                         double eps, void* acc, void* pot, hipStream_t st) {
  if (nt <= 0) return hipSuccess;
  const DirectArgs a{pos, mass, targets, n, nt, eps * eps, acc, pot};
  // (FP64, 100,000 sources: one lane per target takes 1.37 ms for up to 16,384
  // targets, a workgroup on every CU; eight lanes, whose vector loads make a
  // pair 1.7 times as dear, 0.14 us per target: equal at 9,900.  Below 2048
  // targets eight lanes no longer fill the chip.)
  const int sub = nt >= 10240 ? 1 : nt >= 2048 ? 8 : 32;
  const int blocks = (int)(((int64_t)nt * sub + 63) / 64);
  // waves: about eight per SIMD on the whole chip (the sum of the targets of a
  // workgroup uses 4 * 64 / kSub threads), each with 64 sources or more
  int waves = 4;
  while (waves < kDirectMaxWaves && (int64_t)blocks * waves < 8192 && (int64_t)waves * 128 <= n) waves *= 2;
  const bool soft = f64 ? a.eps2 > 0.0 : (float)a.eps2 > 0.f;
  if (f64)
    soft ? launch_sub<true, true>(a, sub, blocks, 64 * waves, st) : launch_sub<true, false>(a, sub, blocks, 64 * waves, st);
  else
    soft ? launch_sub<false, true>(a, sub, blocks, 64 * waves, st)
         : launch_sub<false, false>(a, sub, blocks, 64 * waves, st);
  return hipGetLastError();
}

}  // namespace bh
