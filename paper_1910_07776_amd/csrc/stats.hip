// Tier 1 statistics and feature kernels (Section 2: counters divided by the
// cycle count, then standardised per column), the generic Tier 3 ranking
// kernel, and small utilities.
#include "kernels.hpp"
#include "path_impl.hpp"

namespace sugg {

__global__ void fill_i32_kernel(int32_t* p, int32_t v, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    p[i] = v;
}

hipError_t launch_fill_i32(int32_t* p, int32_t v, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  int blocks = (int)((n + 255) / 256);
  if (blocks > 1024) blocks = 1024;
  (void)hipGetLastError();  // report only this launch's status
  hipLaunchKernelGGL(fill_i32_kernel, dim3(blocks), dim3(256), 0, s, p, v, n);
  return hipGetLastError();
}

// ---- column statistics in FP64 -------------------------------------------
// Each workgroup owns a contiguous chunk of rows; 16 lanes share a row and
// each lane owns VPL columns, read VW at a time (16 bytes where the rows are
// aligned).  Sums of d = x - x(row 0) and d^2 are accumulated per lane,
// combined across the 16 row groups in a fixed order, and the chunks are
// combined in a fixed order by the final kernel, so the result is
// bit-reproducible.  With lcyc, ln(cycles) of every row is written too.
//
// Bound by the FP64 logarithms (one per counter): with the library's log,
// 16 columns a lane whatever E is and scalar loads, 4.8 M rows x 128 took
// 3.06 ms and 32,768 rows 62 us; with flog64, VPL columns and vector loads
// 1.11 ms and 15.9 us.
constexpr int kStatThreads = 256;

// Chunks of at least 64 rows (four per row group): 32,768 rows then give two
// workgroups per compute unit; at most 1024, which bounds the partials.
int colstats_chunks(int64_t N) {
  int64_t c = (N + 63) / 64;
  if (c > 1024) c = 1024;
  if (c < 1) c = 1;
  return (int)c;
}

template <typename T, int VPL, int VW>
__global__ void __launch_bounds__(kStatThreads) colstats_partial_kernel(
    const T* __restrict__ c, const T* __restrict__ cyc, int64_t N, int E, int64_t rows_per_chunk,
    double* __restrict__ partial, double* __restrict__ lcyc, int32_t* status) {
  constexpr int NCH = VPL / VW;
  const int tid = threadIdx.x, l16 = tid & 15, grp = tid >> 4;
  const int64_t r0 = blockIdx.x * rows_per_chunk;
  const int64_t r1 = r0 + rows_per_chunk < N ? r0 + rows_per_chunk : N;
  __shared__ double red[16][16 * VW][2];
  auto load = [&](int64_t r, T (&v)[NCH][VW]) {
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch) {
      const int c0 = (l16 + 16 * ch) * VW;
      if (c0 < E) {
        const VecN<T, VW> q = *reinterpret_cast<const VecN<T, VW>*>(c + r * E + c0);
#pragma unroll
        for (int v2 = 0; v2 < VW; ++v2) v[ch][v2] = q.v[v2];
      } else {
#pragma unroll
        for (int v2 = 0; v2 < VW; ++v2) v[ch][v2] = T(1);
      }
    }
  };
  double sh[NCH][VW], s1[NCH][VW], s2[NCH][VW];
  T cur[NCH][VW], nxt[NCH][VW];
  load(0, cur);
  const double lc0 = flog64((double)cyc[0]);
#pragma unroll
  for (int ch = 0; ch < NCH; ++ch)
#pragma unroll
    for (int v = 0; v < VW; ++v) {
      sh[ch][v] = flog64((double)cur[ch][v]) - lc0;
      s1[ch][v] = 0.0;
      s2[ch][v] = 0.0;
    }
  bool bad = false;
  int64_t r = r0 + grp;
  T cy = cyc[r < r1 ? r : r0], cyn = cy;
  load(r < r1 ? r : r0, cur);
  for (; r < r1; r += 16) {
    const int64_t rn = r + 16 < r1 ? r + 16 : r;   // the next row's loads overlap this row's logarithms
    load(rn, nxt);
    cyn = cyc[rn];
    const double lc = flog64((double)cy);
    if (lcyc && l16 == 0) lcyc[r] = lc;
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch) {
      const bool live = (l16 + 16 * ch) * VW < E;
#pragma unroll
      for (int v = 0; v < VW; ++v) {
        const double x = flog64((double)cur[ch][v]) - lc;
        bad |= live & !__builtin_isfinite(x);
        const double d = x - sh[ch][v];
        s1[ch][v] += d;
        s2[ch][v] = fma(d, d, s2[ch][v]);
        cur[ch][v] = nxt[ch][v];
      }
    }
    cy = cyn;
  }
  if (__ballot(bad) != 0 && (tid & 63) == 0) atomicOr(status, (int)kStatusBadCounter);
  double* out = partial + (int64_t)blockIdx.x * 2 * E;
#pragma unroll
  for (int ch = 0; ch < NCH; ++ch) {
    if (16 * ch * VW >= E) break;
#pragma unroll
    for (int v = 0; v < VW; ++v) {
      red[grp][l16 * VW + v][0] = s1[ch][v];
      red[grp][l16 * VW + v][1] = s2[ch][v];
    }
    __syncthreads();
    if (tid < 16 * VW) {
      double a = 0.0, b = 0.0;
      for (int g = 0; g < 16; ++g) {
        a += red[g][tid][0];
        b += red[g][tid][1];
      }
      const int col = 16 * ch * VW + tid;
      if (col < E) {
        out[col] = a;
        out[E + col] = b;
      }
    }
    __syncthreads();
  }
}

// One workgroup per 8 columns: 32 threads a column sum every 32nd chunk each
// (four loads in flight), then their sums are added in order.
template <typename T>
__global__ void __launch_bounds__(256) colstats_final_kernel(const T* __restrict__ c, const T* __restrict__ cyc, int64_t N,
                                      int E, const double* __restrict__ partial, int nchunks,
                                      double* mu64, double* sig64, T* mu_t, T* isg_t, double* isg64, float* mu32,
                                      float* isg32) {
  __shared__ double red[32][8][2];
  const int jl = threadIdx.x & 7, sl = threadIdx.x >> 3;
  const int j = blockIdx.x * 8 + jl;
  double a = 0.0, b = 0.0;
  if (j < E) {
#pragma unroll 4
    for (int q = sl; q < nchunks; q += 32) {
      a += partial[(int64_t)q * 2 * E + j];
      b += partial[(int64_t)q * 2 * E + E + j];
    }
  }
  red[sl][jl][0] = a;
  red[sl][jl][1] = b;
  __syncthreads();
  if (sl != 0 || j >= E) return;
  a = b = 0.0;
  for (int q = 0; q < 32; ++q) {
    a += red[q][jl][0];
    b += red[q][jl][1];
  }
  const double sh = flog64((double)c[j]) - flog64((double)cyc[0]);
  const double m = a / (double)N;
  double var = b / (double)N - m * m;
  if (var < 0.0) var = 0.0;
  double sg = sqrt(var);
  if (sg < 1e-12) sg = 1.0;
  const double mu = sh + m;
  mu64[j] = mu;
  sig64[j] = sg;
  mu_t[j] = (T)mu;
  isg_t[j] = (T)(1.0 / sg);
  if (isg64) {   // the context's copies of both types
    isg64[j] = 1.0 / sg;
    mu32[j] = (float)mu;
    isg32[j] = (float)(1.0 / sg);
  }
}

template <typename T>
hipError_t launch_colstats(const T* counters, const T* cycles, int64_t N, int32_t E, double* partial,
                           int32_t nchunks, double* mu64, double* sig64, T* mu_t, T* isg_t,
                           int32_t* status, hipStream_t s, double* lcyc, double* isg64, float* mu32, float* isg32) {
  if (N <= 0) return hipErrorInvalidValue;
  const int64_t per = (N + nchunks - 1) / nchunks;
  const int used = (int)((N + per - 1) / per);
  constexpr int VEC = 16 / sizeof(T);
  const bool vec = E % VEC == 0 && reinterpret_cast<uintptr_t>(counters) % 16 == 0;
  (void)hipGetLastError();  // report only this launch's status
  auto run = [&](auto vpl, auto vw) {
    hipLaunchKernelGGL((colstats_partial_kernel<T, decltype(vpl)::value, decltype(vw)::value>), dim3(used),
                       dim3(kStatThreads), 0, s, counters, cycles, N, (int)E, per, partial, lcyc, status);
  };
  using std::integral_constant;
  if (vec && E <= 64) run(integral_constant<int, 4>{}, integral_constant<int, VEC>{});
  else if (vec && E <= 128) run(integral_constant<int, 8>{}, integral_constant<int, VEC>{});
  else if (vec) run(integral_constant<int, 16>{}, integral_constant<int, VEC>{});
  else if (E <= 64) run(integral_constant<int, 4>{}, integral_constant<int, 1>{});
  else if (E <= 128) run(integral_constant<int, 8>{}, integral_constant<int, 1>{});
  else run(integral_constant<int, 16>{}, integral_constant<int, 1>{});
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(colstats_final_kernel<T>, dim3((E + 7) / 8), dim3(256), 0, s, counters, cycles,
                     N, (int)E, partial, used, mu64, sig64, mu_t, isg_t, isg64, mu32, isg32);
  return hipGetLastError();
}

// ---- standardised features in the plan dtype -----------------------------
template <typename T>
__global__ void standardize_kernel(const T* __restrict__ c, const T* __restrict__ cyc, int64_t N, int E,
                                   const T* __restrict__ mu, const T* __restrict__ isg, T* __restrict__ z,
                                   int32_t* status) {
  const int64_t total = N * E;
  bool bad = false;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < total;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t r = i / E;
    const int j = (int)(i - r * E);
    const T x = dlog<T>(c[i]) - dlog<T>(cyc[r]);
    bad |= !__builtin_isfinite(x);
    z[i] = (x - mu[j]) * isg[j];
  }
  if (__ballot(bad) != 0 && (threadIdx.x & 63) == 0) atomicOr(status, (int)kStatusBadCounter);
}

template <typename T>
hipError_t launch_standardize(const T* counters, const T* cycles, int64_t N, int32_t E, const T* mu,
                              const T* isg, T* z, int32_t* status, hipStream_t s) {
  const int64_t total = N * E;
  if (total <= 0) return hipSuccess;
  int64_t blocks = (total + 255) / 256;
  if (blocks > 8192) blocks = 8192;
  (void)hipGetLastError();  // report only this launch's status
  hipLaunchKernelGGL(standardize_kernel<T>, dim3((unsigned)blocks), dim3(256), 0, s, counters, cycles,
                     N, (int)E, mu, isg, z, status);
  return hipGetLastError();
}

// ---- standardised features of selected rows ------------------------------
// z[i][j] for row rows[i] (the baseline versions of a batch: rows = row_off),
// in the output type TO (the plan dtype, or BF16 for the surrogate's input):
// each 16-lane group takes one row at a time (ln of its cycle count once),
// its lanes striding over the columns; the value is (x - mu) * isg with
// x = ln c - ln cyc, rounded once to TO.
template <typename T, typename TO>
__global__ void standardize_rows_kernel(const T* __restrict__ c, const T* __restrict__ cyc,
                                        const int64_t* __restrict__ rows, int64_t nrows, int E,
                                        const T* __restrict__ mu, const T* __restrict__ isg, TO* __restrict__ z,
                                        int ldz, int32_t* status) {
  const int l16 = threadIdx.x & 15;
  const int64_t g0 = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 4, ng = ((int64_t)gridDim.x * blockDim.x) >> 4;
  bool bad = false;
  for (int64_t q = g0; q < nrows; q += ng) {
    const int64_t r = rows[q];
    const T lc = dlog<T>(cyc[r]);
    for (int j = l16; j < E; j += 16) {
      const T x = dlog<T>(c[r * E + j]) - lc;
      bad |= !__builtin_isfinite(x);
      z[q * ldz + j] = (TO)((x - mu[j]) * isg[j]);
    }
  }
  if (__ballot(bad) != 0 && (threadIdx.x & 63) == 0) atomicOr(status, (int)kStatusBadCounter);
}

template <typename T, typename TO>
hipError_t launch_standardize_rows_t(const T* counters, const T* cycles, const int64_t* rows, int64_t nrows, int32_t E,
                                     const T* mu, const T* isg, TO* z, int ldz, int32_t* status, hipStream_t s) {
  if (nrows <= 0 || E <= 0) return hipSuccess;
  int64_t blocks = (nrows + 15) / 16;   // 16 rows per workgroup of 256
  if (blocks > 16384) blocks = 16384;
  (void)hipGetLastError();  // report only this launch's status
  hipLaunchKernelGGL((standardize_rows_kernel<T, TO>), dim3((unsigned)blocks), dim3(256), 0, s, counters, cycles,
                     rows, nrows, (int)E, mu, isg, z, ldz, status);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_standardize_rows(const T* counters, const T* cycles, const int64_t* rows, int64_t nrows, int32_t E,
                                   const T* mu, const T* isg, T* z, int32_t* status, hipStream_t s) {
  return launch_standardize_rows_t<T, T>(counters, cycles, rows, nrows, E, mu, isg, z, E, status, s);
}

hipError_t launch_standardize_rows_bf16(const float* counters, const float* cycles, const int64_t* rows, int64_t nrows,
                                        int32_t E, const float* mu, const float* isg, __bf16* z, int32_t ldz,
                                        int32_t* status, hipStream_t s) {
  return launch_standardize_rows_t<float, __bf16>(counters, cycles, rows, nrows, E, mu, isg, z, ldz, status, s);
}

// ---- FP64 features for the regression ------------------------------------
template <typename T>
__global__ void zfeat64_kernel(const T* __restrict__ c, const T* __restrict__ cyc, int64_t N, int E,
                               const double* __restrict__ mu, const double* __restrict__ sig,
                               double* __restrict__ z, double* __restrict__ lcyc) {
  const int64_t total = N * E;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < total;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t r = i / E;
    const int j = (int)(i - r * E);
    const double lc = log((double)cyc[r]);
    const double x = log((double)c[i]) - lc;
    z[i] = (x - mu[j]) / sig[j];
    if (j == 0) lcyc[r] = lc;
  }
}

template <typename T>
hipError_t launch_zfeat64(const T* counters, const T* cycles, int64_t N, int32_t E, const double* mu64,
                          const double* sig64, double* z64, double* lcyc64, hipStream_t s) {
  const int64_t total = N * E;
  if (total <= 0) return hipSuccess;
  int64_t blocks = (total + 255) / 256;
  if (blocks > 16384) blocks = 16384;
  (void)hipGetLastError();  // report only this launch's status
  hipLaunchKernelGGL(zfeat64_kernel<T>, dim3((unsigned)blocks), dim3(256), 0, s, counters, cycles, N,
                     (int)E, mu64, sig64, z64, lcyc64);
  return hipGetLastError();
}

// ---- generic segmented Tier 3 ranking ------------------------------------
// One wave per segment: lanes stride over the segment keeping a best-first
// list each, then a butterfly of bitonic merges across the wave.
template <typename T, int KT>
__global__ void __launch_bounds__(256) rank_kernel(const T* __restrict__ scores,
                                                   const int64_t* __restrict__ seg_off, int nseg,
                                                   int skip, int n, T tau, int32_t* idx_out,
                                                   T* score_out, int32_t* count_out, int64_t seg_len) {
  const int lane = threadIdx.x & 63;
  const int seg = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  if (seg >= nseg) return;
  const int64_t b0 = seg_off ? seg_off[seg] : seg * seg_len, b1 = seg_off ? seg_off[seg + 1] : b0 + seg_len;
  const int64_t len = b1 - b0;
  Entry<T> lst[KT];
#pragma unroll
  for (int i = 0; i < KT; ++i) lst[i] = empty_entry<T>();
  for (int64_t p = skip + lane; p < len; p += kWave) {
    const T v = scores[b0 + p];
    if (v > tau) {
      Entry<T> e;
      e.v = v;
      e.s = (int32_t)p;
      list_insert<T, KT>(lst, e);
    }
  }
  group_merge<T, KT>(lst, kWave);
  if (lane == 0) write_list<T, KT>(lst, seg, n, idx_out, score_out, count_out);
}

template <typename T>
hipError_t launch_rank(const T* scores, const int64_t* seg_off, int32_t nseg, int32_t skip_head, int32_t n,
                       T tau, int32_t* idx_out, T* score_out, int32_t* count_out, hipStream_t s, int64_t seg_len) {
  if (nseg <= 0) return hipSuccess;
  const int blocks = (nseg + 3) / 4;
  (void)hipGetLastError();  // report only this launch's status
  if (n <= 4)
    hipLaunchKernelGGL((rank_kernel<T, 4>), dim3(blocks), dim3(256), 0, s, scores, seg_off, nseg, skip_head,
                       n, tau, idx_out, score_out, count_out, seg_len);
  else
    hipLaunchKernelGGL((rank_kernel<T, 8>), dim3(blocks), dim3(256), 0, s, scores, seg_off, nseg, skip_head,
                       n, tau, idx_out, score_out, count_out, seg_len);
  return hipGetLastError();
}

// Threshold band of a short suggestion list: for each segment whose top list
// (top_idx / top_count, as written by rank_kernel) holds fewer than n
// entries, the other entries p >= skip with score >= lo (compared in FP64),
// in ascending p, at most C of them; flag_out = 1 when there were more.  A
// full list has an empty band.  One wave per segment; the wave's ballot and
// prefix count place each taken entry, so the order is ascending.
template <typename T>
__global__ void __launch_bounds__(256) band_kernel(const T* __restrict__ scores,
                                                   const int64_t* __restrict__ seg_off, int nseg, int skip,
                                                   const int32_t* __restrict__ top_idx,
                                                   const int32_t* __restrict__ top_count, int n, double lo, int C,
                                                   int32_t* cand_out, T* ref_out, int32_t* flag_out) {
  const int lane = threadIdx.x & 63;
  const int seg = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  if (seg >= nseg) return;
  int32_t listed[kMaxSuggest];
  const int cnt = top_count[seg];
#pragma unroll
  for (int i = 0; i < kMaxSuggest; ++i) listed[i] = i < cnt && i < n ? top_idx[(int64_t)seg * n + i] : -1;
  int64_t total = 0;
  if (cnt < n) {
    const int64_t b0 = seg_off[seg], len = seg_off[seg + 1] - b0;
    for (int64_t base = skip; base < len; base += kWave) {   // uniform per wave
      const int64_t p = base + lane;
      bool take = false;
      T v = T(0);
      if (p < len) {
        v = scores[b0 + p];
        take = (double)v >= lo;
#pragma unroll
        for (int i = 0; i < kMaxSuggest; ++i) take = take && listed[i] != (int32_t)p;
      }
      const uint64_t m = __ballot(take);
      const int64_t pos = total + __popcll(m & ((1ull << lane) - 1ull));
      if (take && pos < C) {
        cand_out[(int64_t)seg * C + pos] = (int32_t)p;
        ref_out[(int64_t)seg * C + pos] = v;
      }
      total += __popcll(m);
    }
  }
  for (int64_t j = (total < C ? total : C) + lane; j < C; j += kWave) {
    cand_out[(int64_t)seg * C + j] = -1;
    ref_out[(int64_t)seg * C + j] = qnan<T>();
  }
  if (lane == 0) flag_out[seg] = total > C ? 1 : 0;
}

template <typename T>
hipError_t launch_band(const T* scores, const int64_t* seg_off, int32_t nseg, int32_t skip_head,
                       const int32_t* top_idx, const int32_t* top_count, int32_t n, double lo, int32_t C,
                       int32_t* cand_out, T* ref_out, int32_t* flag_out, hipStream_t s) {
  if (nseg <= 0) return hipSuccess;
  const int blocks = (nseg + 3) / 4;
  (void)hipGetLastError();  // report only this launch's status
  hipLaunchKernelGGL((band_kernel<T>), dim3(blocks), dim3(256), 0, s, scores, seg_off, nseg, skip_head, top_idx,
                     top_count, n, lo, C, cand_out, ref_out, flag_out);
  return hipGetLastError();
}

#define SUGG_INST(T)                                                                                     \
  template hipError_t launch_colstats<T>(const T*, const T*, int64_t, int32_t, double*, int32_t, double*, \
                                         double*, T*, T*, int32_t*, hipStream_t, double*, double*, float*, float*); \
  template hipError_t launch_standardize<T>(const T*, const T*, int64_t, int32_t, const T*, const T*, T*, \
                                            int32_t*, hipStream_t);                                       \
  template hipError_t launch_standardize_rows<T>(const T*, const T*, const int64_t*, int64_t, int32_t, const T*, \
                                                 const T*, T*, int32_t*, hipStream_t);                         \
  template hipError_t launch_zfeat64<T>(const T*, const T*, int64_t, int32_t, const double*,              \
                                        const double*, double*, double*, hipStream_t);                    \
  template hipError_t launch_rank<T>(const T*, const int64_t*, int32_t, int32_t, int32_t, T, int32_t*, T*, \
                                     int32_t*, hipStream_t, int64_t);                                     \
  template hipError_t launch_band<T>(const T*, const int64_t*, int32_t, int32_t, const int32_t*,         \
                                     const int32_t*, int32_t, double, int32_t, int32_t*, T*, int32_t*,    \
                                     hipStream_t);
SUGG_INST(float)
SUGG_INST(double)
#undef SUGG_INST

}  // namespace sugg
