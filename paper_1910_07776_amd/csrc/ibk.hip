// Instance-based Tier 2 model (IBK, Section 3.4): k nearest neighbours of a
// standardised feature vector among the stored before/after samples of one
// optimisation, by Euclidean distance; the prediction is the mean of their
// labels.  Candidates come from |q - t|^2 = |q|^2 + |t|^2 - 2 q.t with the
// products on the matrix cores, each vector split into two FP16 halves
// (hi + lo carries 23 bits; hi.hi + hi.lo + lo.hi, accumulated in FP32), one
// 32 x 32 block of (sample, query) pairs per v_mfma_f32_32x32x16_f16 sweep
// over the features; the final distances are FP64.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <type_traits>
#include <cmath>

#include "common.hpp"
#include "ibk.hpp"
#include "path_impl.hpp"

namespace sugg {

typedef float floatx16 __attribute__((ext_vector_type(16)));

// ---- standardised rows, zero-padded to Epad columns -------------------------
// 16 lanes a row, VW columns at a time (16 bytes where the rows are aligned).
// zero (nullable) is cleared: the count of uncertified queries of the search
// that follows.
template <typename T, int VW>
__global__ void __launch_bounds__(256) ibk_z_kernel(const T* __restrict__ c, const T* __restrict__ cyc, int64_t N,
                                                    int E, int Epad, const double* __restrict__ mu,
                                                    const double* __restrict__ sig, float* __restrict__ z,
                                                    int32_t* status, int32_t* zero) {
  const int l16 = threadIdx.x & 15;
  const int64_t g0 = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 4;
  const int64_t ng = ((int64_t)gridDim.x * blockDim.x) >> 4;
  if (zero && blockIdx.x == 0 && threadIdx.x == 0) *zero = 0;
  bool bad = false;
  for (int64_t r = g0; r < N; r += ng) {
    const T lc = dlog<T>(cyc[r]);
    for (int j = l16 * VW; j < Epad; j += 16 * VW) {
      VecN<T, VW> q;
      if (j < E) q = *reinterpret_cast<const VecN<T, VW>*>(c + r * E + j);
      VecN<float, VW> o;
#pragma unroll
      for (int u = 0; u < VW; ++u) {
        o.v[u] = 0.0f;
        if (j < E) {
          const T x = dlog<T>(q.v[u]) - lc;
          bad |= !__builtin_isfinite(x);
          o.v[u] = (float)(((double)x - mu[j + u]) / sig[j + u]);
        }
      }
      *reinterpret_cast<VecN<float, VW>*>(z + r * Epad + j) = o;
    }
  }
  if (__ballot(bad) != 0 && (threadIdx.x & 63) == 0) atomicOr(status, (int)kStatusBadCounter);
}

template <typename T>
hipError_t launch_ibk_z(const T* counters, const T* cycles, int64_t N, int32_t E, int32_t Epad,
                        const double* mu, const double* sig, float* z, int32_t* status, int32_t* zero,
                        hipStream_t s) {
  if (N <= 0) return hipSuccess;
  int64_t blocks = (N + 15) / 16;
  if (blocks > 16384) blocks = 16384;
  constexpr int VEC = 16 / sizeof(T);
  (void)hipGetLastError();
  if (E % VEC == 0 && reinterpret_cast<uintptr_t>(counters) % 16 == 0)
    hipLaunchKernelGGL((ibk_z_kernel<T, VEC>), dim3((unsigned)blocks), dim3(256), 0, s, counters, cycles, N, (int)E,
                       (int)Epad, mu, sig, z, status, zero);
  else
    hipLaunchKernelGGL((ibk_z_kernel<T, 1>), dim3((unsigned)blocks), dim3(256), 0, s, counters, cycles, N, (int)E,
                       (int)Epad, mu, sig, z, status, zero);
  return hipGetLastError();
}

// ---- labels: measured log-speedup of every stored pair, in FP64 -------------
template <typename T>
__global__ void __launch_bounds__(256) ibk_label_kernel(const T* __restrict__ cyc, const int32_t* __restrict__ before,
                                                        const int32_t* __restrict__ after, int64_t Ns,
                                                        double* __restrict__ y) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < Ns; i += (int64_t)gridDim.x * blockDim.x)
    y[i] = log((double)cyc[before[i]]) - log((double)cyc[after[i]]);
}

template <typename T>
hipError_t launch_ibk_labels(const T* cycles, const int32_t* before, const int32_t* after, int64_t Ns, double* y,
                             hipStream_t s) {
  if (Ns <= 0) return hipSuccess;
  int64_t blocks = (Ns + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  (void)hipGetLastError();
  hipLaunchKernelGGL(ibk_label_kernel<T>, dim3((unsigned)blocks), dim3(256), 0, s, cycles, before, after, Ns, y);
  return hipGetLastError();
}

// ---- samples in matrix-core order ------------------------------------------------
// hi + lo of x (already scaled): the nearest FP16 and the nearest FP16 of the
// rest; |x - hi - lo| <= 2^-23 |x| + 2^-25 (the second part where lo is below
// FP16's normal range).
__device__ __forceinline__ void split_f16(float x, _Float16& hi, _Float16& lo) {
  hi = (_Float16)x;
  lo = (_Float16)(x - (float)hi);
}

// The samples of an optimisation in tiles of 32 (the last one filled with
// zero vectors of infinite norm), spread: slot i holds sample i * step mod n,
// step coprime to n and near 0.618 n, so that any run of slots is an even
// subsample.  In stored order a training kernel's versions are neighbours, and
// a kernel nearer than those before it brings a burst of candidates (the
// search took 604 us in that order, 485 us in this).  A tile is Epad / 16 feature steps of two
// operands, hi then lo, each in the lane order of v_mfma_f32_32x32x16_f16:
// lane l holds features (l / 32) * 8 + 0..7 of the step of sample l % 32, 16
// bytes.  One 16-lane group per sample row; the scale is a power of two that
// takes the largest stored value to at most 2^15.
__global__ void __launch_bounds__(256) ibk_pack_kernel(const float* __restrict__ Z, const int32_t* __restrict__ srow,
                                                       const int64_t* __restrict__ off,
                                                       const int32_t* __restrict__ toff,
                                                       const int32_t* __restrict__ step, int D, int64_t n_tiles,
                                                       int Epad, float scale, halfx8* __restrict__ Zt,
                                                       float* __restrict__ norm, int32_t* __restrict__ sidx) {
  const int l16 = threadIdx.x & 15;
  const int64_t i = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 4;   // padded sample slot
  if (i >= n_tiles * kIbkTile) return;
  const int64_t t = i / kIbkTile;
  const int row = (int)(i % kIbkTile);
  int o = 0;
  while (o + 1 < D && toff[o + 1] <= t) ++o;   // (an id without samples has no tiles)
  const uint64_t n = (uint64_t)(off[o + 1] - off[o]);
  const uint64_t slot = (uint64_t)(t - toff[o]) * kIbkTile + row;
  const bool live = slot < n;
  const int64_t s = live ? off[o] + (int64_t)(slot * (uint64_t)step[o] % n) : 0;
  const float* z = Z + (live ? (int64_t)srow[s] : 0) * Epad;
  double acc = 0.0;
  for (int k = l16; k < Epad / 8; k += 16) {   // eight features per lane
    halfx8 h, l;
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const float v = live ? z[8 * k + u] : 0.0f;
      _Float16 a, b;
      split_f16(v * scale, a, b);
      h[u] = a;
      l[u] = b;
      acc = fma((double)v, (double)v, acc);
    }
    halfx8* p = Zt + ((t * (Epad / 16) + k / 2) * 2) * 64 + (k & 1) * 32 + row;
    p[0] = h;
    p[64] = l;
  }
  acc = row_sum16(acc);
  if (l16 == 0) {
    norm[i] = live ? (float)acc : INFINITY;
    sidx[i] = live ? (int32_t)(s - off[o]) : -1;
  }
}

hipError_t launch_ibk_pack(const float* Z, const int32_t* srow, const int64_t* off, const int32_t* toff,
                           const int32_t* step, int32_t D, int64_t n_tiles, int32_t Epad, float scale, halfx8* Zt,
                           float* norm, int32_t* sidx, hipStream_t s) {
  if (n_tiles <= 0) return hipSuccess;
  const int64_t blocks = (n_tiles * kIbkTile * 16 + 255) / 256;
  (void)hipGetLastError();
  hipLaunchKernelGGL(ibk_pack_kernel, dim3((unsigned)blocks), dim3(256), 0, s, Z, srow, off, toff, step, (int)D,
                     n_tiles, (int)Epad, scale, Zt, norm, sidx);
  return hipGetLastError();
}

// ---- the FP32 rounding of the stored vectors, per column, and their largest value
// Non-negative floats order as their bit patterns, so a column maximum is an
// unsigned maximum; each workgroup reduces its rows in LDS first.
__global__ void __launch_bounds__(256) ibk_dz_kernel(const float* __restrict__ z32, int Epad,
                                                     const double* __restrict__ z64, int64_t N, int E,
                                                     uint32_t* __restrict__ out) {
  __shared__ uint32_t m[257];
  for (int j = threadIdx.x; j <= E; j += blockDim.x) m[j] = 0u;
  __syncthreads();
  const int64_t total = N * E;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t r = i / E;
    const int j = (int)(i - r * E);
    const float zv = z32[r * Epad + j];
    if (__builtin_isfinite(zv)) atomicMax(&m[E], __float_as_uint(fabsf(zv)));
    const double d = fabs((double)zv - z64[i]);
    const float f = __builtin_isfinite(d) ? (float)d : INFINITY;
    // round up so the float never understates the double
    const float fu = (double)f < d ? __uint_as_float(__float_as_uint(f) + 1u) : f;   // next float up
    atomicMax(&m[j], __float_as_uint(fu));
  }
  __syncthreads();
  for (int j = threadIdx.x; j <= E; j += blockDim.x)
    if (m[j]) atomicMax(&out[j], m[j]);
}

hipError_t launch_ibk_dz(const float* z32, int32_t Epad, const double* z64, int64_t N, int32_t E, uint32_t* out,
                         hipStream_t s) {
  if (N <= 0) return hipSuccess;
  int64_t blocks = (N * E + 255) / 256;
  if (blocks > 2048) blocks = 2048;
  (void)hipGetLastError();
  hipLaunchKernelGGL(ibk_dz_kernel, dim3((unsigned)blocks), dim3(256), 0, s, z32, (int)Epad, z64, N, (int)E, out);
  return hipGetLastError();
}

// ---- the k-nearest-neighbour search ------------------------------------------
// A candidate is a 64-bit key read as a double: the (non-negative) distance's
// bits, shifted into the normal range, in the high word, the sample's slot in
// the low word.  Such doubles order as (distance, slot), so one v_min_f64 or
// v_max_f64 compares and selects a candidate.  A distance below zero (rounding
// of a distance near zero) is taken as zero.
constexpr uint32_t kKeyBias = 0x00100000u;
__device__ __forceinline__ double knn_key(float d, int s) {
  return __hiloint2double((int)(__float_as_uint(fmaxf(d, 0.0f)) + kKeyBias), s);
}
__device__ __forceinline__ float knn_key_d(double k) { return __uint_as_float((uint32_t)__double2hiint(k) - kKeyBias); }
__device__ __forceinline__ int knn_key_s(double k) { return __double2loint(k); }
__device__ __forceinline__ double knn_empty() { return knn_key(INFINITY, INT_MAX); }

// Insertion into an ascending list of KT keys (the last one drops out): entry
// j becomes min(l[j], max(l[j-1], key)).
template <int KT>
__device__ __forceinline__ void knn_insert(double (&l)[KT], double key) {
#pragma unroll
  for (int j = KT - 1; j > 0; --j) l[j] = fmin(l[j], fmax(l[j - 1], key));
  l[0] = fmin(l[0], key);
}

// One workgroup: up to 256 queries of one optimisation (wave w owns queries
// 64 w .. 64 w + 63, two matrix-core columns of 32), sweeping one of `split`
// shares of its samples in tiles of 32, copied straight into LDS (already in
// operand order) while the tile before is multiplied.  v_permlane32_swap then
// gives every lane all 32 products of its own query: entry r of the first
// (second) half is sample (r / 4) * 8 (+ 4) + r % 4.  A candidate below the
// lane's worst kept one goes to a queue in LDS; a wave merges its queues into
// its lists when one of them could overflow.
//
// Per 64 queries x 32 samples x 128 features: 48 matrix operations of 32
// cycles, and about as many vector cycles for distances and comparisons of
// the wave that shares the SIMD: with FP32 operations (64 of 64 cycles per 32
// queries) and a 64-bit integer insertion (123 instructions; this one has 31)
// the search of 32,256 queries over 16,384 samples each took 1.72 ms; now
// 0.49 ms, of which 0.33 ms remain without any insertion (1.2 PFLOP/s of FP16
// products; a large bf16 library product reaches 1.36 here).  Against FP64
// the split's distances are closer than the FP32 products' were: on normal
// vectors, rms error 1.2e-5 against 1.7e-5 at 128 features, 2.4e-5 against
// 4.0e-5 at 256, 3.2e-6 against 3.7e-6 at 32 (the norms are summed in FP64); on
// the features of twelve batches of perf/cases.py's ranges (40 to 128 events, a
// query's nearest samples and random ones) its rms error is 0.61 to 0.86 of theirs.
// Two workgroups per compute unit where the registers allow it without
// spilling (up to 128 events with lists of at most 16), else one.
template <int ES, int KT>
constexpr int ibk_knn_waves() { return ES <= 4 || (ES <= 8 && KT <= 16) ? 2 : 1; }

template <int ES, int KT>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(ibk_knn_waves<ES, KT>())))
ibk_knn_kernel(const IbkKnnArgs a) {
  constexpr int EP = 16 * ES;                  // features; ES steps of 16
  constexpr int TB = ES * 2 * 64;              // halfx8 per tile
  __shared__ __align__(16) halfx8 ta[TB];
  __shared__ __align__(16) halfx8 tb_[TB];
  // per-lane queue of candidates that beat the list's last entry as of the
  // latest merge (entry j of thread t at [j * 256 + t])
  __shared__ double qk[kIbkQueue * 256];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int col = lane & 31, h = lane >> 5;
  const int tile = blockIdx.x / a.split, part = blockIdx.x - tile * a.split;
  const int o = a.tiles[tile * 4 + 0];
  const int q0 = a.tiles[tile * 4 + 1];
  const int nq = a.tiles[tile * 4 + 2];
  // this workgroup's share of the samples: whole tiles
  const int ntl = a.toff[o + 1] - a.toff[o], per = (ntl + a.split - 1) / a.split;
  const int tb = min(ntl, part * per), te = min(ntl, (part + 1) * per);
  const halfx8* Zo = a.Zt + (int64_t)a.toff[o] * TB;
  // constant address space: the norms are read through the scalar cache (as
  // vector loads they would wait for the tile copies issued before them)
  const auto* No = (const __attribute__((address_space(4))) float*)(uintptr_t)(a.norm + (int64_t)a.toff[o] * kIbkTile);
  const int qloc = wave * 64 + lane;
  const bool wave_live = wave * 64 < nq;

  // tile t into a buffer: wave w copies its quarter, 1 KB per operation
  auto copy = [&](halfx8* dst, int t) {
    const halfx8* src = Zo + (int64_t)t * TB;
#pragma unroll
    for (int i = 0; i < TB / 256; ++i) {
      const int at = (i * 4 + wave) * 64;
      __builtin_amdgcn_global_load_lds(
          (const __attribute__((address_space(1))) uint32_t*)(const void*)(src + at + lane),
          (__attribute__((address_space(3))) uint32_t*)(void*)(dst + at), 16, 0, 0);
    }
  };
  if (tb < te) copy(ta, tb);

  // query operands: lane l holds features (l / 32) * 8 + 0..7 of every step of
  // query l % 32 of either column, scaled by a power of two that takes the
  // query's largest value to [2^14, 2^15)
  halfx8 qh[2][ES], ql[2][ES];
  float qn = 0.0f, cq = 0.0f;   // of this lane's own query: |q|^2 and -2 / (both scales)
#pragma unroll
  for (int g = 0; g < 2; ++g) {
    const int qi = wave * 64 + g * 32 + col;
    const int32_t qrow = a.q_src[q0 + (qi < nq ? qi : 0)];
    const float* qp = a.zq + (int64_t)qrow * EP + h * 8;
    float v[ES][8], mx = 0.0f;
    double nn = 0.0;   // (the norms' rounding would outweigh the split's)
#pragma unroll
    for (int k = 0; k < ES; ++k) {
      const float4 x = *reinterpret_cast<const float4*>(qp + 16 * k);
      const float4 y = *reinterpret_cast<const float4*>(qp + 16 * k + 4);
      v[k][0] = x.x; v[k][1] = x.y; v[k][2] = x.z; v[k][3] = x.w;
      v[k][4] = y.x; v[k][5] = y.y; v[k][6] = y.z; v[k][7] = y.w;
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        mx = fmaxf(mx, fabsf(v[k][u]));
        nn = fma((double)v[k][u], (double)v[k][u], nn);
      }
    }
    mx = fmaxf(mx, __shfl_xor(mx, 32, kWave));
    nn += __shfl_xor(nn, 32, kWave);
    // 2^(14 - exponent), the exponent held within 100 of 14 (a zero or a huge
    // vector keeps a finite scale)
    int e = (int)((__float_as_uint(mx) >> 23) & 255u) - 127;
    e = e < -86 ? -86 : e > 114 ? 114 : e;
    const float sc = __uint_as_float((uint32_t)(14 - e + 127) << 23);
    if (h == g) {
      qn = (float)nn;
      cq = -2.0f * __uint_as_float((uint32_t)(e - 14 + 127) << 23) * a.inv_scale;
    }
#pragma unroll
    for (int k = 0; k < ES; ++k)
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        _Float16 x, y;
        split_f16(v[k][u] * sc, x, y);
        qh[g][k][u] = x;
        ql[g][k][u] = y;
      }
  }
  double lk[KT];
#pragma unroll
  for (int j = 0; j < KT; ++j) lk[j] = knn_empty();
  // lanes without a query take nothing
  float worst = qloc < nq ? INFINITY : -INFINITY;
  int qc = 0;
  auto flush = [&]() {
    // four entries read at a time (slots past qc read as the empty key, which
    // changes nothing): one LDS wait per four insertions
#pragma unroll 1
    for (int j = 0; __any(j < qc); j += 4) {
      double key[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int q = j + u < kIbkQueue ? j + u : kIbkQueue - 1;   // in bounds even if read unconditionally
        const double k = qk[q * 256 + tid];
        key[u] = j + u < qc ? k : knn_empty();
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) knn_insert<KT>(lk, key[u]);
    }
    qc = 0;
    if (qloc < nq) worst = knn_key_d(lk[KT - 1]);
  };
  auto sweep = [&](const halfx8* buf, int t) {
    // the tile's norms, uniform over the wave (scalar loads)
    float tn[kIbkTile];
#pragma unroll
    for (int i = 0; i < kIbkTile; ++i) tn[i] = No[t * kIbkTile + i];
    floatx16 acc0, acc1;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      acc0[r] = 0.0f;
      acc1[r] = 0.0f;
    }
    halfx8 th = buf[lane], tl = buf[64 + lane];
#pragma unroll
    for (int k = 0; k < ES; ++k) {
      // the next step's operands are read while this one's are multiplied
      const halfx8 h0 = th, l0 = tl;
      if (k + 1 < ES) {
        th = buf[(2 * k + 2) * 64 + lane];
        tl = buf[(2 * k + 3) * 64 + lane];
      }
      acc0 = __builtin_amdgcn_mfma_f32_32x32x16_f16(l0, qh[0][k], acc0, 0, 0, 0);
      acc1 = __builtin_amdgcn_mfma_f32_32x32x16_f16(l0, qh[1][k], acc1, 0, 0, 0);
      acc0 = __builtin_amdgcn_mfma_f32_32x32x16_f16(h0, ql[0][k], acc0, 0, 0, 0);
      acc1 = __builtin_amdgcn_mfma_f32_32x32x16_f16(h0, ql[1][k], acc1, 0, 0, 0);
      acc0 = __builtin_amdgcn_mfma_f32_32x32x16_f16(h0, qh[0][k], acc0, 0, 0, 0);
      acc1 = __builtin_amdgcn_mfma_f32_32x32x16_f16(h0, qh[1][k], acc1, 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
    // padded samples have an infinite norm and never enter a list
#pragma unroll
    for (int half = 0; half < 2; ++half) {
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        float d[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int r = 4 * g + u;
          if (half == 0) {
            const auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(acc0[r]), __float_as_uint(acc1[r]), false,
                                                            false);
            acc0[r] = __uint_as_float(p[0]);
            acc1[r] = __uint_as_float(p[1]);
          }
          d[u] = fmaf(cq, half == 0 ? acc0[r] : acc1[r], qn + tn[g * 8 + half * 4 + u]);
        }
        // four at a time: usually no lane of the wave takes any
        if (__any(fminf(fminf(d[0], d[1]), fminf(d[2], d[3])) < worst)) {
#pragma unroll
          for (int u = 0; u < 4; ++u)
            if (d[u] < worst) {
              qk[qc * 256 + tid] = knn_key(d[u], t * kIbkTile + g * 8 + half * 4 + u);
              ++qc;
            }
        }
      }
      // merge before a queue could overflow on the next 16 (a wave pays for
      // its fullest lane, once for all of them)
      if (__any(qc > kIbkQueue - 16)) flush();
    }
  };
  __syncthreads();
  for (int t = tb; t < te; t += 2) {   // uniform over the workgroup
    if (t + 1 < te) copy(tb_, t + 1);
    if (wave_live) sweep(ta, t);
    __syncthreads();   // the next tile has arrived, this one is consumed
    if (t + 1 >= te) break;
    if (t + 2 < te) copy(ta, t + 2);
    if (wave_live) sweep(tb_, t + 1);
    __syncthreads();
  }
  // the candidate list of this share, entry by entry over the queries
  // (re-ranked in FP64 by ibk_refine_kernel after the shares are merged)
  if (!wave_live) return;
  flush();
  if (qloc < nq) {
    double* out = a.part + (int64_t)part * KT * a.n_queries + q0 + qloc;
#pragma unroll
    for (int j = 0; j < KT; ++j) out[j * a.n_queries] = lk[j];
  }
}

// Merge of the shares' candidate lists of one query (one thread per query):
// the KT best over all shares, written over share 0's list.
template <int KT>
__global__ void __launch_bounds__(64) ibk_merge_kernel(const IbkKnnArgs a) {
  const int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (q >= a.n_queries) return;
  double* p0 = a.part + q;
  double lk[KT];
#pragma unroll
  for (int j = 0; j < KT; ++j) lk[j] = p0[j * a.n_queries];
  for (int p = 1; p < a.split; ++p) {
    const double* src = a.part + (int64_t)p * KT * a.n_queries + q;
    double key[KT];
#pragma unroll
    for (int j = 0; j < KT; ++j) key[j] = src[j * a.n_queries];
    // the KT best of two ascending lists are min(l[i], key[KT-1-i]); sorting
    // them is left to the insertions, which stop where nothing enters
#pragma unroll
    for (int j = 0; j < KT; ++j)
      if (__any(key[j] < lk[KT - 1])) knn_insert<KT>(lk, key[j]);
  }
#pragma unroll
  for (int j = 0; j < KT; ++j) p0[j * a.n_queries] = lk[j];
}

// The global optimisation of query q: the tile that holds it (tiles ascend in q).
__device__ __forceinline__ int ibk_query_opt(const IbkKnnArgs& a, int64_t q) {
  int lo = 0, hi = a.n_tiles - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (a.tiles[mid * 4 + 1] <= q) lo = mid;
    else hi = mid - 1;
  }
  return a.tiles[lo * 4 + 0];
}

constexpr int kIbkMaxCols = 16;   // FP64 feature columns per lane (16 lanes x 16 = 256 events); NC of them in use

// A lane's columns of a row: (l16 + 16 i) VW + u, i < NC / VW, u < VW.  VW 2
// (16-byte loads) where rows of E doubles stay aligned, else 1.

// This lane's FP64 standardised features of plan row r (zero past E):
// z = (ln c - ln cyc - mu) / sigma, as the training rows.
template <typename T, int NC, int VW>
__device__ __forceinline__ void ibk_query64(const IbkKnnArgs& a, int64_t r, int l16, double (&q)[NC]) {
  const T* c = reinterpret_cast<const T*>(a.counters) + r * a.E;
  const double lc = flog64((double)reinterpret_cast<const T*>(a.cycles)[r]);
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    const int j = (l16 + 16 * (i / VW)) * VW + i % VW;
    q[i] = j < a.E ? (flog64((double)c[j]) - lc - a.mu64[j]) / a.sig64[j] : 0.0;
  }
}

// A training row's columns, and their squared FP64 distance from the query's,
// summed over the 16 lanes of the group (every lane receives it).
template <int NC, int VW>
__device__ __forceinline__ void ibk_row64(const IbkKnnArgs& a, int32_t row, int l16, double (&t)[NC]) {
  const double* p = a.Z64 + (int64_t)row * a.E;
#pragma unroll
  for (int i = 0; i < NC; i += VW) {
    const int j = (l16 + 16 * (i / VW)) * VW;
    VecN<double, VW> v;
#pragma unroll
    for (int u = 0; u < VW; ++u) v.v[u] = 0.0;
    if (j < a.E) v = *reinterpret_cast<const VecN<double, VW>*>(p + j);
#pragma unroll
    for (int u = 0; u < VW; ++u) t[i + u] = v.v[u];
  }
}
template <int NC>
__device__ __forceinline__ double ibk_dist64(const double (&q)[NC], const double (&t)[NC]) {
  double acc = 0.0;
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    const double d = q[i] - t[i];
    acc = fma(d, d, acc);
  }
  return row_sum16(acc);
}

// Re-ranking (16 lanes per query): the candidates' exact FP64 distances, the
// k nearest of them by (distance, sample index), and the mean of their
// labels.  Every sample outside the candidates has a search distance of at
// least the list's last, dlast; its FP64 distance then exceeds dlast -
// err(dlast), err bounding the search's error (the features' FP32 rounding,
// the FP16 split, and the accumulation in |q|^2 + |t|^2 - 2 q.t), so when the
// k-th FP64 distance lies below that the k nearest are certain.  Otherwise
// the query goes to the queue of ibk_exact_kernel.  By the same bound a
// candidate whose search distance lies past the k-th FP64 distance so far
// plus err, and all after it, need not be read.
//
// Bound by the candidates' rows (1 KB each at 128 events, spread over the
// 34 MB of a 512-kernel training set): all 16 read one after another, and
// sorted in every lane, took 166 us for 32,256 queries; the first k in groups
// of four and the rest as needed, ranked one candidate per lane, 51 us.
template <typename T, int KT, int NC, int VW>
__global__ void __launch_bounds__(256) ibk_refine_kernel(const IbkKnnArgs a) {
  constexpr int SL = (KT + 15) / 16;   // candidates per lane: l16 + 16 i
  constexpr int G = 4;                 // rows in flight
  const int lane = threadIdx.x & 63, l16 = lane & 15, g0 = lane & 48;
  const int64_t q = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 4;
  if (q >= a.n_queries) return;   // whole 16-lane groups leave together
  const int o = ibk_query_opt(a, q);
  const int64_t s0 = a.off[o];
  const int ns = (int)(a.off[o + 1] - s0);
  const int kk = a.k < ns ? a.k : ns;
  const int64_t qr = a.q_src[q];
  // this lane's candidates
  float d32[SL];
  int samp[SL], row[SL];
  double d64[SL];
  bool full = true;
#pragma unroll
  for (int i = 0; i < SL; ++i) {
    const int j = l16 + 16 * i;
    const double key = j < KT ? a.part[j * a.n_queries + q] : knn_empty();
    d32[i] = knn_key_d(key);
    const int slot = knn_key_s(key);
    const bool ok = slot != INT_MAX;
    samp[i] = ok ? a.sidx[(int64_t)a.toff[o] * kIbkTile + slot] : INT_MAX;
    row[i] = ok ? a.srow[s0 + samp[i]] : -1;
    d64[i] = INFINITY;
    full = full && (ok || j >= KT);
  }
  full = ((__ballot(full) >> g0) & 0xffffull) == 0xffffull;
  double qv[NC];
  ibk_query64<T, NC, VW>(a, qr, l16, qv);
  // err(u) = 2 sqrt(u) Dz + Dz^2 + eps span(u)^2 + 1e-12 (1 + u): Dz bounds
  // the rounding of query minus sample vectors (the query's FP32 rounding,
  // measured here, plus the stored vectors' worst, with their halves' loss
  // below FP16's normal range, plus 2^-22.4 of both for the split; a query has
  // a scale of its own, so its loss there is below 2^-34 of it), span the sum
  // of the two vectors' norms.  eps: 2^-24 per FP32
  // addition, three products per feature (2 q.t <= span^2 / 2, every addition
  // allowed twice the rounding), the two norms' sums and two more; lo.lo,
  // left out, is at most 2^-22 span^2 / 2.
  double qn = 0.0, dq = 0.0;
  {
    const float* zr = a.zq + qr * a.Epad;
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      const int j = (l16 + 16 * (i / VW)) * VW + i % VW;
      qn = fma(qv[i], qv[i], qn);
      if (j < a.E) {
        const double e = (double)zr[j] - qv[i];
        dq = fma(e, e, dq);
      }
    }
    qn = row_sum16(qn);
    dq = row_sum16(dq);
  }
  const double rq = sqrt(qn), D0 = sqrt(dq) * (1.0 + 1e-12) + a.dt_norm;
  const double eps = 1.01 * ((double)(4 * a.Epad + 32) * 5.9604644775390625e-8 + 1.2e-7);
  const auto err = [&](double u) -> double {
    const double ru = sqrt(u), span = (2.0 * rq + ru + D0) * (1.0 + 1e-6), Dz = D0 + 1.8e-7 * span;
    return 2.0 * ru * Dz + Dz * Dz + eps * span * span + 1e-12 * (1.0 + u);
  };
  // candidates in search order, G at a time; the largest of the first kk
  // distances bounds the k-th from above, and past kk candidates the groups
  // that need no more of theirs drop out
  double top = 0.0, limit = INFINITY;
#pragma unroll
  for (int j0 = 0; j0 < KT; j0 += G) {
    int rj[G];
    bool any = false;
#pragma unroll
    for (int u = 0; u < G; ++u) {
      const int j = j0 + u, i = j / 16;
      rj[u] = __shfl(row[i], g0 + (j & 15), kWave);
      const float dj = __shfl(d32[i], g0 + (j & 15), kWave);
      if (j >= kk && !((double)dj <= limit)) rj[u] = -1;
      any = any || rj[u] >= 0;
    }
    if (!any) continue;   // uniform per group
    double t[G][NC];
#pragma unroll
    for (int u = 0; u < G; ++u) ibk_row64<NC, VW>(a, rj[u] >= 0 ? rj[u] : 0, l16, t[u]);
#pragma unroll
    for (int u = 0; u < G; ++u) {
      const int j = j0 + u, i = j / 16;
      const double d = ibk_dist64<NC>(qv, t[u]);
      if (rj[u] >= 0) {
        if (l16 == (j & 15)) d64[i] = d;
        if (j < kk) top = d > top ? d : top;
      }
      if (j == kk - 1 && __builtin_isfinite(top)) limit = top + err(top);
    }
  }
  // ranks by (distance, sample): candidates not read are past the k nearest
  int rank[SL];
#pragma unroll
  for (int i = 0; i < SL; ++i) rank[i] = 0;
#pragma unroll
  for (int j = 0; j < KT; ++j) {
    const double dj = __shfl(d64[j / 16], g0 + (j & 15), kWave);
    const int sj = __shfl(samp[j / 16], g0 + (j & 15), kWave);
#pragma unroll
    for (int i = 0; i < SL; ++i) rank[i] += (dj < d64[i]) | ((dj == d64[i]) & (sj < samp[i])) ? 1 : 0;
  }
  double dk = 0.0, sum = 0.0;
  int got = 0;
#pragma unroll
  for (int i = 0; i < SL; ++i)
    if (l16 + 16 * i < KT && rank[i] < kk && samp[i] != INT_MAX && d64[i] < INFINITY) {
      ++got;
      dk = d64[i] > dk ? d64[i] : dk;
      sum += a.y[s0 + samp[i]];
    }
  sum = row_sum16(sum);
#pragma unroll
  for (int m = 1; m < 16; m <<= 1) {
    got += __shfl_xor(got, m, kWave);
    dk = fmax(dk, __shfl_xor(dk, m, kWave));
  }
  const bool have = got == kk;
  // every sample is a candidate where there are no more than the list holds
  bool certain = ns <= KT;
  if (!certain && full && have) {
    const double dlast = (double)__shfl(d32[(KT - 1) / 16], g0 + ((KT - 1) & 15), kWave);
    const double e = err(dk);
    certain = __builtin_isfinite(dlast) && __builtin_isfinite(e) && dk + e < dlast;
  }
  if (l16 == 0) {
    if (certain) {
      reinterpret_cast<T*>(a.out)[a.q_dst[q]] = have ? (T)(sum / (double)kk) : qnan<T>();
    } else {
      const int slot = atomicAdd(a.exact_n, 1);
      a.exact_q[slot] = (int32_t)q;
    }
  }
}

// FP64 search over every sample of the query's optimisation for the queries
// whose candidates were not certain (queue from ibk_refine_kernel); one
// workgroup per query, taken in turn; 16 groups of 16 lanes each keep the
// k nearest of every 16th sample, merged by one thread at the end.
template <typename T>
__global__ void __launch_bounds__(256) ibk_exact_kernel(const IbkKnnArgs a) {
  __shared__ double sd[16 * kIbkMaxK];
  __shared__ int si[16 * kIbkMaxK];
  const int tid = threadIdx.x, l16 = tid & 15, g = tid >> 4;
  const int n = *a.exact_n;
  for (int w = blockIdx.x; w < n; w += gridDim.x) {
    const int64_t q = a.exact_q[w];
    const int o = ibk_query_opt(a, q);
    const int64_t s0 = a.off[o];
    const int ns = (int)(a.off[o + 1] - s0);
    const int kk = a.k < ns ? a.k : ns;
    double qv[kIbkMaxCols], t[kIbkMaxCols];
    ibk_query64<T, kIbkMaxCols, 1>(a, a.q_src[q], l16, qv);
    double ld[kIbkMaxK];
    int li[kIbkMaxK];
#pragma unroll
    for (int j = 0; j < kIbkMaxK; ++j) {
      ld[j] = INFINITY;
      li[j] = INT_MAX;
    }
    for (int s = g; s < ns; s += 16) {   // uniform within the 16-lane group
      ibk_row64<kIbkMaxCols, 1>(a, a.srow[s0 + s], l16, t);
      const double d = ibk_dist64<kIbkMaxCols>(qv, t);
      if (d < ld[kIbkMaxK - 1] || (d == ld[kIbkMaxK - 1] && s < li[kIbkMaxK - 1])) {
        ld[kIbkMaxK - 1] = d;
        li[kIbkMaxK - 1] = s;
#pragma unroll
        for (int j = kIbkMaxK - 1; j > 0; --j) {
          const bool sw = ld[j] < ld[j - 1] || (ld[j] == ld[j - 1] && li[j] < li[j - 1]);
          const double td = ld[j - 1];
          const int ti = li[j - 1];
          ld[j - 1] = sw ? ld[j] : td;
          li[j - 1] = sw ? li[j] : ti;
          ld[j] = sw ? td : ld[j];
          li[j] = sw ? ti : li[j];
        }
      }
    }
    if (l16 == 0)
#pragma unroll
      for (int j = 0; j < kIbkMaxK; ++j) {
        sd[g * kIbkMaxK + j] = ld[j];
        si[g * kIbkMaxK + j] = li[j];
      }
    __syncthreads();
    if (tid == 0) {
      // the k nearest of the 16 group lists: repeated minimum over the heads
      int head[16];
      for (int h = 0; h < 16; ++h) head[h] = 0;
      double sum = 0.0;
      bool ok = true;
      for (int j = 0; j < kk; ++j) {
        int best = -1;
        for (int h = 0; h < 16; ++h) {
          if (head[h] >= kIbkMaxK) continue;
          const double d = sd[h * kIbkMaxK + head[h]];
          const int i = si[h * kIbkMaxK + head[h]];
          if (best < 0) {
            best = h;
            continue;
          }
          const double bd = sd[best * kIbkMaxK + head[best]];
          const int bi = si[best * kIbkMaxK + head[best]];
          if (d < bd || (d == bd && i < bi)) best = h;
        }
        const int i = si[best * kIbkMaxK + head[best]];
        ok = ok && i != INT_MAX;
        sum += i != INT_MAX ? a.y[s0 + i] : 0.0;
        ++head[best];
      }
      reinterpret_cast<T*>(a.out)[a.q_dst[q]] = ok ? (T)(sum / (double)kk) : qnan<T>();
    }
    __syncthreads();   // the lists are read before the next query writes them
  }
}

template <int ES, int KT, typename T>
hipError_t launch_knn_kt(const IbkKnnArgs& a, int n_tiles, hipStream_t s) {
  hipLaunchKernelGGL((ibk_knn_kernel<ES, KT>), dim3(n_tiles * a.split), dim3(256), 0, s, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (a.split > 1) {
    hipLaunchKernelGGL((ibk_merge_kernel<KT>), dim3((unsigned)((a.n_queries + 63) / 64)), dim3(64), 0, s, a);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  const dim3 grid((unsigned)((a.n_queries * 16 + 255) / 256));
  if (a.E % 2 == 0) hipLaunchKernelGGL((ibk_refine_kernel<T, KT, ES, 2>), grid, dim3(256), 0, s, a);
  else hipLaunchKernelGGL((ibk_refine_kernel<T, KT, ES, 1>), grid, dim3(256), 0, s, a);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((ibk_exact_kernel<T>), dim3(256), dim3(256), 0, s, a);
  return hipGetLastError();
}

// Sample shares per query tile: enough workgroups for one round of two per
// compute unit (the search's occupancy), a power of two, at most one share
// per 128 samples of the largest optimisation.  Workgroups go to the eight
// XCDs in turn (workgroup w to XCD w mod 8) and workgroup w takes share w mod
// split of its tile, so with up to eight shares the L2s of the XCDs s, s +
// split, ... serve share s to all of the optimisation's tiles.
int ibk_split(int64_t max_samples, int n_tiles, int cus) {
  const double want = 2.0 * cus / std::max(1, n_tiles);
  int split = 1;
  while (2 * split <= want * 1.5 && 2 * split * 128 <= max_samples && split < 64) split *= 2;
  return split;
}

template <int ES, typename T>
hipError_t launch_knn_es(const IbkKnnArgs& a, int n_tiles, hipStream_t s) {
  if (a.kt == 8) return launch_knn_kt<ES, 8, T>(a, n_tiles, s);
  if (a.kt == 16) return launch_knn_kt<ES, 16, T>(a, n_tiles, s);
  return launch_knn_kt<ES, 24, T>(a, n_tiles, s);
}

template <typename T>
hipError_t launch_ibk_knn(const IbkKnnArgs& a, int n_tiles, hipStream_t s) {
  if (n_tiles <= 0) return hipSuccess;
  if (a.kt != ibk_kt(a.k) || a.E > 16 * kIbkMaxCols || a.k > kIbkMaxK) return hipErrorInvalidValue;
  (void)hipGetLastError();
  switch (a.Epad) {
    case 32: return launch_knn_es<2, T>(a, n_tiles, s);
    case 64: return launch_knn_es<4, T>(a, n_tiles, s);
    case 128: return launch_knn_es<8, T>(a, n_tiles, s);
    case 256: return launch_knn_es<16, T>(a, n_tiles, s);
    default: return hipErrorInvalidValue;
  }
}

// ---- composition along the ascending chain, then the top-n ------------------
// L(S) = L(S without its highest bit b) + step(S), step(S) = the prediction of
// adding b to S without it (the same sum, in the same order, as adding the
// steps of the chain from the baseline one by one), in TE; outputs in TO.
// One wave per kernel.
template <typename TE, typename TO, int KT>
__global__ void __launch_bounds__(64) ibk_compose_kernel(const TE* __restrict__ edges, const TO* __restrict__ grid,
                                                         int grid_ld, const int64_t* __restrict__ row_off,
                                                         const int32_t* __restrict__ nopts, int K, TO* table,
                                                         int32_t* idx_out, TO* score_out, int32_t* count_out, int n,
                                                         TE tau) {
  extern __shared__ __align__(16) unsigned char smem[];
  TE* L = reinterpret_cast<TE*>(smem);
  const int k = blockIdx.x, lane = threadIdx.x;
  if (k >= K) return;
  const int B = nopts[k];
  const int64_t r0 = row_off[k];
  if (lane == 0) L[0] = TE(0);
  __syncthreads();
  for (int b = 0; b < B; ++b) {
    const int lo = 1 << b;
    for (int S = lo + lane; S < 2 * lo; S += kWave) {
      const TE e = edges ? edges[r0 + S] : (TE)grid[(r0 + S - lo) * grid_ld + b];
      L[S] = L[S - lo] + e;
    }
    __syncthreads();
  }
  Entry<TE> lst[KT];
#pragma unroll
  for (int i = 0; i < KT; ++i) lst[i] = empty_entry<TE>();
  for (int S = lane; S < (1 << B); S += kWave) {
    const TE v = L[S];
    if (table) table[r0 + S] = (TO)v;
    if (S != 0 && v > tau) {
      Entry<TE> e;
      e.v = v;
      e.s = S;
      list_insert<TE, KT>(lst, e);
    }
  }
  if (idx_out) {
    group_merge<TE, KT>(lst, kWave);
    if (lane == 0) {
      int cnt = 0;
#pragma unroll
      for (int i = 0; i < KT; ++i)
        if (i < n) {
          const bool ok = lst[i].s >= 0;
          idx_out[(int64_t)k * n + i] = ok ? lst[i].s : -1;
          score_out[(int64_t)k * n + i] = ok ? (TO)lst[i].v : qnan<TO>();
          cnt += ok ? 1 : 0;
        }
      count_out[k] = cnt;
    }
  }
}

template <typename TE, typename TO>
hipError_t launch_ibk_compose(const TE* edges, const TO* grid, int32_t grid_ld, const int64_t* row_off,
                              const int32_t* nopts, int32_t K, int32_t Bmax, TO* table, int32_t* idx_out,
                              TO* score_out, int32_t* count_out, int32_t n, TE tau, hipStream_t s) {
  if (K <= 0) return hipSuccess;
  const size_t smem = sizeof(TE) * ((size_t)1 << Bmax);
  (void)hipGetLastError();
  if (n <= 4)
    hipLaunchKernelGGL((ibk_compose_kernel<TE, TO, 4>), dim3(K), dim3(64), smem, s, edges, grid, grid_ld, row_off,
                       nopts, K, table, idx_out, score_out, count_out, n, tau);
  else
    hipLaunchKernelGGL((ibk_compose_kernel<TE, TO, 8>), dim3(K), dim3(64), smem, s, edges, grid, grid_ld, row_off,
                       nopts, K, table, idx_out, score_out, count_out, n, tau);
  return hipGetLastError();
}

// ---- NaN fill (grid entries that are not predictions) ----------------------
template <typename T>
__global__ void __launch_bounds__(256) ibk_nan_kernel(T* p, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    p[i] = qnan<T>();
}

template <typename T>
hipError_t launch_ibk_nan(T* p, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  int64_t blocks = (n + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  (void)hipGetLastError();
  hipLaunchKernelGGL(ibk_nan_kernel<T>, dim3((unsigned)blocks), dim3(256), 0, s, p, n);
  return hipGetLastError();
}

#define SUGG_INST(T)                                                                                        \
  template hipError_t launch_ibk_z<T>(const T*, const T*, int64_t, int32_t, int32_t, const double*,          \
                                      const double*, float*, int32_t*, int32_t*, hipStream_t);               \
  template hipError_t launch_ibk_labels<T>(const T*, const int32_t*, const int32_t*, int64_t, double*,       \
                                           hipStream_t);                                                     \
  template hipError_t launch_ibk_knn<T>(const IbkKnnArgs&, int, hipStream_t);                                \
  template hipError_t launch_ibk_compose<T, T>(const T*, const T*, int32_t, const int64_t*, const int32_t*,  \
                                               int32_t, int32_t, T*, int32_t*, T*, int32_t*, int32_t, T,     \
                                               hipStream_t);                                                 \
  template hipError_t launch_ibk_nan<T>(T*, int64_t, hipStream_t);
SUGG_INST(float)
SUGG_INST(double)
#undef SUGG_INST
template hipError_t launch_ibk_compose<double, float>(const double*, const float*, int32_t, const int64_t*,
                                                      const int32_t*, int32_t, int32_t, float*, int32_t*, float*,
                                                      int32_t*, int32_t, double, hipStream_t);

}  // namespace sugg
