// Prediction with M5P model trees (Section 3.4): per version row, Tier 1's
// standardised features, then for every optimisation the row needs a walk
// down that optimisation's tree and the leaf's smoothed linear model.
//
// A workgroup takes 16 versions of one kernel.  Sixteen lanes share a row
// (16-byte loads, the row arithmetic of the fused scoring kernel) and leave
// its features in LDS.  The tile's predictions are then walked one per
// thread, all at once (a walk is a chain of dependent loads, so the tile's
// critical path is one walk, not a row's several), and the leaf models are
// evaluated sixteen lanes per prediction with a DPP reduction.  Edge mode
// forms the predictions of the ascending chain only (row S predicts adding
// each b above its top bit: the one edge into every version S | 2^b); grid
// mode every b not in S.  Counters are read in the plan's dtype TI and every
// step computes in FP64 (features, tests, leaf models), so each walk takes
// the branch of the FP64 reference and FP32 plans differ from it only by the
// rounding of their outputs.
#include <hip/hip_runtime.h>

#include "kernels.hpp"
#include "m5p.hpp"
#include "path_impl.hpp"

namespace sugg {

constexpr int kM5pThreads = kM5pRows * kRowLanes;

// Lane l16's chunks of a row, columns (l16 + 16 ch) * VW + [0, VW), read in
// the plan dtype (1 past E), widened to FP64 where they are used.
template <typename TI, int NCH, int VW, typename TO>
__device__ __forceinline__ void m5p_load_row(const TI* rp, int E, int l16, TO (&c)[NCH][VW]) {
#pragma unroll
  for (int ch = 0; ch < NCH; ++ch) {
    const int c0 = (l16 + kRowLanes * ch) * VW;
    if (c0 + VW <= E) {
      const VecN<TI, VW> q = *reinterpret_cast<const VecN<TI, VW>*>(rp + c0);
#pragma unroll
      for (int v = 0; v < VW; ++v) c[ch][v] = (TO)q.v[v];
    } else {
#pragma unroll
      for (int v = 0; v < VW; ++v) c[ch][v] = c0 + v < E ? (TO)rp[c0 + v] : TO(1);
    }
  }
}

// row_features' check without the logarithms: those of a row are all finite
// where its counters and cycles are positive and finite (one class test each:
// positive normal or subnormal).
__device__ __forceinline__ bool m5p_ok(float v) { return __builtin_amdgcn_classf(v, 0x180); }
__device__ __forceinline__ bool m5p_ok(double v) { return __builtin_amdgcn_class(v, 0x180); }
template <typename TI, int NCH, int VW>
__device__ __forceinline__ bool m5p_bad(const TI (&c)[NCH][VW], TI cy) {
  bool bad = !m5p_ok(cy);
#pragma unroll
  for (int ch = 0; ch < NCH; ++ch)
#pragma unroll
    for (int v = 0; v < VW; ++v) bad |= !m5p_ok(c[ch][v]);
  return bad;
}

// Selections among a block's slots with constant indices (no dynamic
// indexing of register arrays).
template <typename V>
__device__ __forceinline__ V m5p_sel4(const V* v, int i) {
  const V lo = (i & 1) ? v[1] : v[0];
  const V hi = (i & 1) ? v[3] : v[2];
  return (i & 2) ? hi : lo;
}
template <typename V>
__device__ __forceinline__ V m5p_sel8(const V* v, int i) {
  const V lo = m5p_sel4(v, i & 3);
  const V hi = m5p_sel4(v + 4, i & 3);
  return (i & 4) ? hi : lo;
}
__device__ __forceinline__ int m5p_leaf_bits(float t) { return __float_as_int(t); }
__device__ __forceinline__ int m5p_leaf_bits(double t) { return (int)__double_as_longlong(t); }

// The leaf that a version with features zr (in LDS) reaches in the tree whose
// first block is blk.
template <typename T>
__device__ __forceinline__ int m5p_walk(const M5pBlock<T>* blocks, int blk, int max_blocks, const T* zr) {
  for (int it = 0; it < max_blocks; ++it) {   // a walk ends within max_blocks loads
    const M5pBlock<T> q = blocks[blk];         // three levels in one line
    int f = q.feat[0];
    T t = q.thr[0];
    if (f < 0) return m5p_leaf_bits(t);
    const int g0 = !(zr[f] <= t);
    f = g0 ? q.feat[2] : q.feat[1];
    t = g0 ? q.thr[2] : q.thr[1];
    if (f < 0) return m5p_leaf_bits(t);
    const int i2 = 2 * g0 + !(zr[f] <= t);
    f = m5p_sel4(q.feat + 3, i2);
    t = m5p_sel4(q.thr + 3, i2);
    if (f < 0) return m5p_leaf_bits(t);
    const int ex = m5p_sel8(q.exit, 2 * i2 + !(zr[f] <= t));
    if (ex < 0) return -1 - ex;
    blk = ex;
  }
  return 0;
}

// Predictions (edges) of the tile's row g = 0..15: edge mode every b above
// the top bit of S (all B bits for S = 0), grid mode every b not in S.
__device__ __forceinline__ int m5p_row_edges(int S, int B, bool grid) {
  if (S >= (1 << B)) return 0;
  return grid ? B - __popc((unsigned)S) : B - 1 - (S ? 31 - __clz(S) : -1);
}

template <typename TI, int VPL, int VW>
__global__ void __launch_bounds__(kM5pThreads) m5p_kernel(const M5pArgs<TI> a) {
  using T = double;
  constexpr int NCH = VPL / VW;
  constexpr int EP = kRowLanes * VPL;
  constexpr int kMaxEdges = kM5pRows * SUGG_MAX_OPTS;
  static_assert(kMaxEdges <= kM5pThreads, "one walk per thread");
  __shared__ __align__(32) T zl[kM5pRows][EP];
  __shared__ int32_t e_leaf[kMaxEdges];
  __shared__ int32_t e_gb[kMaxEdges];
  const int tid = threadIdx.x, g = tid / kRowLanes, l16 = tid % kRowLanes;
  const int k = a.tiles[2 * blockIdx.x];
  const int S0 = a.tiles[2 * blockIdx.x + 1];
  const int B = a.nopts[k];
  const int64_t r0 = a.row_off[k];
  const int32_t* ids = a.opt_ids + a.opt_off[k];
  const bool grid = a.grid != nullptr;
  // 1. rows: Tier 1 features into LDS of the versions that predict anything
  // (in edge mode those without the top optimisation, half of a kernel's
  // rows); the others' counters are only checked
  {
    const int S = S0 + g;
    const bool live = S < (1 << B), need = m5p_row_edges(S, B, grid) > 0;
    bool bad = false;
    if (live && !need) {
      TI c[NCH][VW];
      m5p_load_row<TI, NCH, VW>(a.counters + (r0 + S) * a.E, a.E, l16, c);
      bad = m5p_bad<TI, NCH, VW>(c, a.cycles[r0 + S]);
    }
    if (need) {
      T c[NCH][VW], s_r[NCH][VW], m_r[NCH][VW], z[NCH][VW];
      m5p_load_row<TI, NCH, VW>(a.counters + (r0 + S) * a.E, a.E, l16, c);
      const T cy = (T)a.cycles[r0 + S];
      column_constants<T, NCH, VW, false>(a.mu, a.isg, a.E, l16, s_r, m_r);
      const T chk = row_features<T, NCH, VW>(c, cy, s_r, m_r, z);
      bad = !__builtin_isfinite(chk);
#pragma unroll
      for (int ch = 0; ch < NCH; ++ch) {
        VecN<T, VW> q;
#pragma unroll
        for (int v = 0; v < VW; ++v) q.v[v] = z[ch][v];
        *reinterpret_cast<VecN<T, VW>*>(&zl[g][(l16 + kRowLanes * ch) * VW]) = q;
      }
    }
    if (__ballot(bad) != 0 && (tid % kWave) == 0) atomicOr(a.status, (int)kStatusBadCounter);
  }
  __syncthreads();
  // 2. walks: one thread per prediction of the tile, down its tree to a leaf
  int n_e = 0;
#pragma unroll
  for (int r = 0; r < kM5pRows; ++r) n_e += m5p_row_edges(S0 + r, B, grid);
  if (tid < n_e) {
    int rem = tid, r = 0;
    for (; r < kM5pRows; ++r) {
      const int cnt = m5p_row_edges(S0 + r, B, grid);
      if (rem < cnt) break;
      rem -= cnt;
    }
    const int S = S0 + r;
    int b;
    if (grid) {
      b = 0;
      for (int seen = -1;; ++b)
        if (!((S >> b) & 1) && ++seen == rem) break;
    } else {
      b = (S ? 31 - __clz(S) : -1) + 1 + rem;
    }
    e_leaf[tid] = m5p_walk<T>(a.blocks, a.root[ids[b]], a.max_blocks, zl[r]);
    e_gb[tid] = (r << 8) | b;
  }
  __syncthreads();
  // 3. leaf models: sixteen lanes per prediction, the row's features from LDS
  for (int e = g; e < n_e; e += kM5pRows) {
    const int r = e_gb[e] >> 8, b = e_gb[e] & 255, leaf = e_leaf[e];
    const T* wrow = a.lw + (int64_t)leaf * a.ldl;
    T part = T(0);
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch) {
      const int c0 = (l16 + kRowLanes * ch) * VW;
      const VecN<T, VW> zq = *reinterpret_cast<const VecN<T, VW>*>(&zl[r][c0]);
      const VecN<T, VW> w = *reinterpret_cast<const VecN<T, VW>*>(wrow + c0);
#pragma unroll
      for (int v = 0; v < VW; ++v) part = fma(zq.v[v], w.v[v], part);
    }
    const T p = row_sum16(part) + a.lb[leaf];
    if (l16 == 0) {
      const int S = S0 + r;
      if (grid) a.grid[(r0 + S) * a.Bmax + b] = (TI)p;
      // the chain edges in FP64 in both modes: the composition reads them
      if (!grid || b > (S ? 31 - __clz(S) : -1)) a.edges[r0 + (S | (1 << b))] = p;
    }
  }
}

// Batches of kernels of at most 2^MB versions (MB 4 to 7), chain edges only: one
// workgroup of 16 threads per version without the top optimisation, for one
// kernel.  The features of those rows (the edges start from them) into LDS,
// one row per 16-lane group; the other rows' counters are only checked.
// Then every chain edge walked at once (thread t takes version t + 1), the
// leaf models two per group with their weight rows in flight together, and
// Tier 3 by the first wave: the composition and the top n.  The arithmetic of
// an edge and of the composition is that of the tiled kernel and the separate
// composition, so both give the same bits.
//
// Bound by a chain of latencies (row addresses, rows, the walk's blocks, the
// leaf's weights) with the FP64 logarithms between: with 256 threads and the
// features of all 64 rows, 512 kernels of 64 versions and 128 FP32 events took
// 20.9 us, 9.9 of it features; now 15.4 (the whole call 22.1 -> 15.4, on counters
// that are not in a cache 24.5 -> 16.6; 300 of 128 versions by tiles and a separate
// composition 42, now 26; 1000 of 16 with 200 events 48 -> 16; 4096 of 64 145 ->
// 88).  Beyond 128 events the instance for 128 versions spills 4 to 8 registers.
template <typename TI, int VPL, int VW, int MB>
__global__ void __launch_bounds__(kRowLanes << (MB - 1)) m5p_small_kernel(const M5pArgs<TI> a, TI* table,
                                                                          int32_t* idx_out, TI* score_out,
                                                                          int32_t* count_out, int n, double tau) {
  using T = double;
  constexpr int NCH = VPL / VW;
  constexpr int EP = kRowLanes * VPL;
  constexpr int kV = 1 << MB, kRows = kV / 2;   // versions; rows that edges start from, one per group of 16 lanes
  constexpr int kPer = kV / kRows;              // edges of a group
  constexpr int kNv = kV > kWave ? kV / kWave : 1;   // versions of a lane of the first wave
  __shared__ __align__(32) T zl[kRows][EP];
  __shared__ T ev[kV];
  __shared__ int32_t e_leaf[kV];
  const int tid = threadIdx.x, g = tid / kRowLanes, l16 = tid % kRowLanes;
  const int k = blockIdx.x;
  const int B = a.nopts[k];
  const int V = 1 << B, half = V > 1 ? V / 2 : 1;
  const int64_t r0 = a.row_off[k];
  const int32_t* ids = a.opt_ids + a.opt_off[k];
  int root = 0;   // of this thread's walk
  if (tid + 1 < V) root = ids[31 - __clz(tid + 1)];
  {
    const bool own = g < half, more = half + g < V;   // uniform per group; for V >= 8 per wave
    T c[NCH][VW], cy = T(1);
    TI c2[NCH][VW], cy2 = TI(1);
    if (own) {
      m5p_load_row<TI, NCH, VW>(a.counters + (r0 + g) * a.E, a.E, l16, c);
      cy = (T)a.cycles[r0 + g];
    }
    if (more) {
      m5p_load_row<TI, NCH, VW>(a.counters + (r0 + half + g) * a.E, a.E, l16, c2);
      cy2 = a.cycles[r0 + half + g];
    }
    if (tid + 1 < V) root = a.root[root];
    T s_r[NCH][VW], m_r[NCH][VW];
    column_constants<T, NCH, VW, false>(a.mu, a.isg, a.E, l16, s_r, m_r);
    bool bad = false;
    if (own) {
      T z[NCH][VW];
      const T chk = row_features<T, NCH, VW>(c, cy, s_r, m_r, z);
      bad |= !__builtin_isfinite(chk);
#pragma unroll
      for (int ch = 0; ch < NCH; ++ch) {
        VecN<T, VW> q;
#pragma unroll
        for (int v = 0; v < VW; ++v) q.v[v] = z[ch][v];
        *reinterpret_cast<VecN<T, VW>*>(&zl[g][(l16 + kRowLanes * ch) * VW]) = q;
      }
    }
    if (more) bad |= m5p_bad<TI, NCH, VW>(c2, cy2);
    if (__ballot(bad) != 0 && (tid % kWave) == 0) atomicOr(a.status, (int)kStatusBadCounter);
  }
  __syncthreads();
  if (tid + 1 < V) {
    const int Sp = tid + 1, top = 31 - __clz(Sp);
    e_leaf[tid] = m5p_walk<T>(a.blocks, root, a.max_blocks, zl[Sp - (1 << top)]);
  }
  __syncthreads();
  {
    VecN<T, VW> w[kPer][NCH];
    T wb[kPer];
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const int e = g + kRows * i;
      const int leaf = e + 1 < V ? e_leaf[e] : 0;
      const T* wrow = a.lw + (int64_t)leaf * a.ldl;
#pragma unroll
      for (int ch = 0; ch < NCH; ++ch)
        w[i][ch] = *reinterpret_cast<const VecN<T, VW>*>(wrow + (l16 + kRowLanes * ch) * VW);
      wb[i] = a.lb[leaf];
    }
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const int e = g + kRows * i;
      if (e + 1 >= V) break;   // uniform per 16-lane group
      const int Sp = e + 1, top = 31 - __clz(Sp);
      const T* zr = zl[Sp - (1 << top)];
      T part = T(0);
#pragma unroll
      for (int ch = 0; ch < NCH; ++ch) {
        const VecN<T, VW> zq = *reinterpret_cast<const VecN<T, VW>*>(zr + (l16 + kRowLanes * ch) * VW);
#pragma unroll
        for (int v = 0; v < VW; ++v) part = fma(zq.v[v], w[i][ch].v[v], part);
      }
      const T p = row_sum16(part) + wb[i];
      if (l16 == 0) ev[Sp] = p;
    }
  }
  __syncthreads();
  if (tid < kWave) {
    const T none = -__builtin_huge_val();   // not above any threshold
    T v[kNv];
#pragma unroll
    for (int u = 0; u < kNv; ++u) {
      const int S = u * kWave + tid;
      v[u] = none;
      if (S < V) {
        T x = T(0);   // ascending, as L[S] = L[S without its top bit] + edge
        for (int b = 0; b < B; ++b)
          if ((S >> b) & 1) x += ev[S & ((2 << b) - 1)];
        if (table) table[r0 + S] = (TI)x;
        v[u] = S != 0 && x > tau ? x : none;
      }
    }
    if (idx_out) {
      // the best value, then the smallest version that has it, n times
      T bv = T(0);
      int bs = -1, cnt = 0;
      for (; cnt < n; ++cnt) {   // uniform
        T best = v[0];
#pragma unroll
        for (int u = 1; u < kNv; ++u) best = fmax(best, v[u]);
        best = group_max<T>(best, kWave, tid);
        if (!(lane_read(best, 0) > none)) break;
        int S = -1;
#pragma unroll
        for (int u = 0; u < kNv; ++u) {
          const uint64_t m = __ballot(v[u] == best);
          if (S < 0 && m) {   // uniform
            S = u * kWave + __builtin_ctzll(m);
            v[u] = u * kWave + tid == S ? none : v[u];
          }
        }
        bv = tid == cnt ? best : bv;
        bs = tid == cnt ? S : bs;
      }
      if (tid < n) {
        idx_out[(int64_t)k * n + tid] = bs;
        score_out[(int64_t)k * n + tid] = bs >= 0 ? (TI)bv : qnan<TI>();
      }
      if (tid == 0) count_out[k] = cnt;
    }
  }
}

template <typename TI, int VPL>
hipError_t launch_m5p_vpl(const M5pArgs<TI>& a, int n_tiles, hipStream_t s) {
  constexpr int VEC = 16 / sizeof(TI);
  const bool vec = (a.E % VEC) == 0 && (reinterpret_cast<uintptr_t>(a.counters) % 16) == 0;
  (void)hipGetLastError();
  if (vec) hipLaunchKernelGGL((m5p_kernel<TI, VPL, VEC>), dim3(n_tiles), dim3(kM5pThreads), 0, s, a);
  else hipLaunchKernelGGL((m5p_kernel<TI, VPL, 1>), dim3(n_tiles), dim3(kM5pThreads), 0, s, a);
  return hipGetLastError();
}

template <typename TI, int VPL, int MB>
hipError_t launch_m5p_small_mb(const M5pArgs<TI>& a, int K, TI* table, int32_t* idx, TI* score, int32_t* count,
                               int n, double tau, hipStream_t s) {
  constexpr int VEC = 16 / sizeof(TI);
  const bool vec = (a.E % VEC) == 0 && (reinterpret_cast<uintptr_t>(a.counters) % 16) == 0;
  (void)hipGetLastError();
  const dim3 grid(K), block(kRowLanes << (MB - 1));
  if (vec) hipLaunchKernelGGL((m5p_small_kernel<TI, VPL, VEC, MB>), grid, block, 0, s, a, table, idx, score, count, n, tau);
  else hipLaunchKernelGGL((m5p_small_kernel<TI, VPL, 1, MB>), grid, block, 0, s, a, table, idx, score, count, n, tau);
  return hipGetLastError();
}

template <typename TI, int VPL>
hipError_t launch_m5p_small_vpl(const M5pArgs<TI>& a, int K, TI* table, int32_t* idx, TI* score, int32_t* count,
                                int n, double tau, hipStream_t s) {
  if (a.Bmax <= 4) return launch_m5p_small_mb<TI, VPL, 4>(a, K, table, idx, score, count, n, tau, s);
  if (a.Bmax == 5) return launch_m5p_small_mb<TI, VPL, 5>(a, K, table, idx, score, count, n, tau, s);
  if (a.Bmax == 6) return launch_m5p_small_mb<TI, VPL, 6>(a, K, table, idx, score, count, n, tau, s);
  return launch_m5p_small_mb<TI, VPL, 7>(a, K, table, idx, score, count, n, tau, s);
}

template <typename TI>
hipError_t launch_m5p_small(const M5pArgs<TI>& a, int K, TI* table, int32_t* idx, TI* score, int32_t* count, int n,
                            double tau, hipStream_t s) {
  if (K <= 0) return hipSuccess;
  if (a.Bmax > kM5pSmallB) return hipErrorInvalidValue;
  if (a.E <= 16 * 4) return launch_m5p_small_vpl<TI, 4>(a, K, table, idx, score, count, n, tau, s);
  if (a.E <= 16 * 8) return launch_m5p_small_vpl<TI, 8>(a, K, table, idx, score, count, n, tau, s);
  return launch_m5p_small_vpl<TI, 16>(a, K, table, idx, score, count, n, tau, s);
}

template <typename TI>
hipError_t launch_m5p(const M5pArgs<TI>& a, int n_tiles, hipStream_t s) {
  if (n_tiles <= 0) return hipSuccess;
  if (a.E <= 16 * 4) return launch_m5p_vpl<TI, 4>(a, n_tiles, s);
  if (a.E <= 16 * 8) return launch_m5p_vpl<TI, 8>(a, n_tiles, s);
  return launch_m5p_vpl<TI, 16>(a, n_tiles, s);
}

template hipError_t launch_m5p<float>(const M5pArgs<float>&, int, hipStream_t);
template hipError_t launch_m5p<double>(const M5pArgs<double>&, int, hipStream_t);
template hipError_t launch_m5p_small<float>(const M5pArgs<float>&, int, float*, int32_t*, float*, int32_t*, int,
                                            double, hipStream_t);
template hipError_t launch_m5p_small<double>(const M5pArgs<double>&, int, double*, int32_t*, double*, int32_t*, int,
                                             double, hipStream_t);

}  // namespace sugg
