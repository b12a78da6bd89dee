// The scoring pass (Section 2, Tiers 1-3) in its streaming form, for ragged
// batches: each workgroup takes one chunk of consecutive whole kernels in
// memory order (of any mix of B, about a target number of rows; a larger
// kernel is a chunk alone), streams its rows (one contiguous read), forms
// Tier 1's features and Tier 2's chain edges into LDS, then composes the
// subset tables and takes Tier 3's top n of every kernel of the chunk.
//
// Unlike the persistent fused kernel, whose workgroups walk a work list of
// equal-B kernels and stop streaming at each item's composition, the chunks
// here are independent workgroups in memory order: the hardware dispatcher
// keeps every compute unit streaming while some of its workgroups compose,
// no work counter or item list is read, and a chunk's first rows need no
// metadata.  Row, edge and composition arithmetic are the fused kernel's
// (each edge, each table entry bit for bit); the ranking takes the same top
// n by (score descending, subset ascending).
#include <hip/hip_runtime.h>

#include "kernels.hpp"
#include "path_impl.hpp"

namespace sugg {

// Threads per workgroup: 256, or the wide form's 1024 (512 where a lane holds
// more than 32 bytes of a row, for its registers), which ends a large chunk
// sooner where there are too few chunks to fill the chip.
constexpr int kChunkThreads = 256;
template <typename T, int VPL>
constexpr int chunk_wide() { return sizeof(T) * VPL <= 32 ? 1024 : 512; }

// Lane 0's value of the row of 16 lanes, in every lane.
__device__ __forceinline__ float row_first(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x150, 0xF, 0xF, false));
}
__device__ __forceinline__ double row_first(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x150, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x150, 0xF, 0xF, false);
  return __hiloint2double(hi, lo);
}

struct ChunkSmem {
  int ep;
  size_t W, Wb, sm, e, L, kr, rk, total;
};

template <typename T>
__host__ __device__ inline ChunkSmem chunk_smem(int D, int E, int max_rows, int max_nk) {
  ChunkSmem s;
  s.ep = E <= 64 ? 64 : (E <= 128 ? 128 : 256);
  size_t o = 0;
  s.W = o;   o += sizeof(T) * (size_t)D * s.ep;
  s.Wb = o;  o += sizeof(T) * (size_t)D;
  o = align_up(o, 16);
  s.sm = o;  o += sizeof(T) * 2 * (size_t)s.ep;
  s.e = o;   o += sizeof(T) * (size_t)max_rows;
  s.L = o;   o += sizeof(T) * (size_t)max_rows;
  o = align_up(o, 16);
  s.kr = o;  o += sizeof(CRec) * (size_t)max_nk;
  s.rk = o;  o += sizeof(int16_t) * (size_t)max_rows;
  s.total = align_up(o, 16);
  return s;
}

size_t path_chunk_lds(size_t tsize, int D, int E, int max_rows, int max_nk) {
  return tsize == 4 ? chunk_smem<float>(D, E, max_rows, max_nk).total
                    : chunk_smem<double>(D, E, max_rows, max_nk).total;
}

// One 16-byte vector of the weight image in LDS (D rows of EP columns, zero
// past E): vector i of the row-major image.
template <typename T, bool FULL>
__device__ __forceinline__ VecN<T, 16 / sizeof(T)> weight_vec(const T* W, int ldw, int E, int EP, int i) {
  constexpr int VEC = 16 / sizeof(T);
  const int q = EP / VEC, o = i / q, j = (i - o * q) * VEC;
  VecN<T, VEC> r;
  if (FULL && sizeof(T) == 4) {   // rows of stride w32_ld(E): 16-byte aligned
    r = *reinterpret_cast<const VecN<T, VEC>*>(W + (int64_t)o * ldw + j);
  } else {
#pragma unroll
    for (int v = 0; v < VEC; ++v) r.v[v] = (FULL || j + v < E) ? W[(int64_t)o * ldw + j + v] : T(0);
  }
  return r;
}

// GRID: every optimisation a version lacks is predicted and the grid written
// (no ranking).  With kmask only selected kernels' rows are used and their
// outputs written; workgroup (j, segment) takes the j-th chunk with a selected
// kernel of 64 consecutive ones, so the workgroups with work come first and
// spread evenly over the chip, and the others end at once (28% of 4096 kernels
// of 1024 versions: 178 us with one workgroup per chunk and each row's flag
// read from memory, 174 with the packing, 132 with the flags in LDS too).
// Chunks of many small kernels (over 16, or 8 on average) stay one workgroup
// each: reading 64 chunks' flags would cost more than it evens out (250,000
// kernels of 8 versions, a quarter selected: 293 us packed, 212 not).
template <typename T, int VPL, int VW, int U, int KT, bool FULL, int TH, bool GRID>
__global__ void __launch_bounds__(TH) __attribute__((amdgpu_waves_per_eu(
    TH == 1024 && sizeof(T) == 4 ? 8 : 1)))   // two wide FP32 workgroups per compute unit
path_chunk_kernel(const ChunkArgs<T> a) {
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr int NCH = VPL / VW;
  constexpr int VEC = 16 / sizeof(T);
  constexpr int kGroups = TH / kRowLanes;
  constexpr int kWaves = TH / kWave;
  const int E = a.E, D = a.D;
  const int tid = threadIdx.x, g = tid / kRowLanes, l16 = tid % kRowLanes, lane = tid % kWave, wave = tid / kWave;
  const ChunkSmem ly = chunk_smem<T>(D, E, a.max_rows, a.max_nk);
  const int EP = ly.ep;
  T* Wl = reinterpret_cast<T*>(smem + ly.W);
  T* Wb = reinterpret_cast<T*>(smem + ly.Wb);
  T* sml = reinterpret_cast<T*>(smem + ly.sm);
  T* eb = reinterpret_cast<T*>(smem + ly.e);
  T* Lb = reinterpret_cast<T*>(smem + ly.L);
  CRec* kr = reinterpret_cast<CRec*>(smem + ly.kr);
  int16_t* rk = reinterpret_cast<int16_t*>(smem + ly.rk);

  // rows: step i covers chunk rows [kGroups U i, kGroups U (i + 1)); lane
  // group g takes rows kGroups U i + kGroups u + g.  Every load is issued
  // unconditionally (rows past the chunk re-read its last row and are never
  // used), so the loads in flight are the same on every path and a step
  // waits only for its own rows, not for the next step's.
  constexpr int step = kGroups * U;
  auto load = [&](const Chunk& c, int base, T (&cv)[U][NCH][VW], T (&cy)[U]) {
    const T* c0 = a.counters + c.row0 * E;
    const T* y0 = a.cycles + c.row0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      int r = base + kGroups * u + g;
      r = r < c.R ? r : c.R - 1;
      const uint32_t ro = (uint32_t)(r * E);   // below 2^20: a 32-bit offset from the chunk's uniform base
#pragma unroll
      for (int ch = 0; ch < NCH; ++ch) {
        const int cc = (l16 + kRowLanes * ch) * VW;
        if (FULL || cc < E) {
          const VecN<T, VW> q = *reinterpret_cast<const VecN<T, VW>*>(c0 + (ro + (uint32_t)cc));
#pragma unroll
          for (int v = 0; v < VW; ++v) cv[u][ch][v] = q.v[v];
        } else {
#pragma unroll
          for (int v = 0; v < VW; ++v) cv[u][ch][v] = T(1);
        }
      }
      cy[u] = y0[(uint32_t)r];
    }
  };
  const int4* recs = reinterpret_cast<const int4*>(a.recs);
  int4* krv = reinterpret_cast<int4*>(kr);
  int at = blockIdx.x;
  const bool packed = a.packed != 0;   // uniform
  if (packed) {
    const int nseg = (a.n_chunks + kWave - 1) / kWave, seg = at % nseg, i = seg * kWave + lane;
    int sel = 0;
    if (i < a.n_chunks) {
      const Chunk c = a.chunks[i];
      for (int j = 0; j < c.nk; ++j) sel |= a.kmask[c.k0 + j];
    }
    uint64_t live = __ballot(sel != 0);
    for (int j = at / nseg; j && live; --j) live &= live - 1;
    if (!live) return;   // uniform over the workgroup: every wave read the same flags
    at = seg * kWave + __builtin_ctzll(live);
  }
  const Chunk ck = a.chunks[at];
  const int R = ck.R, nk = ck.nk;
  if (a.kmask && !packed) {   // uniform
    // every wave reads all the flags: a vote of the workgroup would take LDS
    // beside the dynamic part, which may be all there is
    int sel = 0;
    for (int j = lane; j < nk; j += kWave) sel |= a.kmask[ck.k0 + j];
    if (!__any(sel)) return;
  }
  // loads in issue order: this chunk's kernel records and the model (small,
  // needed first), then the first two steps of rows; whatever would wait on
  // a load (a loop over a larger model or many kernels) comes before the rows
  // a kernel's record; its spare byte is nonzero where it is not selected
  auto chosen = [&](int j) {
    int4 q = recs[ck.k0 + j];
    if (a.kmask && !a.kmask[ck.k0 + j]) q.x |= 1 << 24;
    return q;
  };
  int4 rec = make_int4(0, 0, 0, 0);
  if (tid < nk) rec = chosen(tid);
  const int nwv = D * (EP / VEC);
  VecN<T, VEC> wv0, wv1;
  if (tid < nwv) wv0 = weight_vec<T, FULL>(a.W, a.ldw, E, EP, tid);
  if (tid + TH < nwv) wv1 = weight_vec<T, FULL>(a.W, a.ldw, E, EP, tid + TH);
  const T wb = tid < D ? a.W[(int64_t)tid * a.ldw + E] : T(0);
  T s0[NCH][VW], m0[NCH][VW];
  if (tid < kRowLanes) column_constants<T, NCH, VW, FULL>(a.mu, a.isg, E, l16, s0, m0);
  for (int i = tid + 2 * TH; i < nwv; i += TH)   // larger models
    *reinterpret_cast<VecN<T, VEC>*>(Wl + i * VEC) = weight_vec<T, FULL>(a.W, a.ldw, E, EP, i);
  for (int j = tid + TH; j < nk; j += TH) krv[j] = chosen(j);   // many small kernels
  T ca[U][NCH][VW], cb[U][NCH][VW];
  T cya[U], cyb[U];
  load(ck, 0, ca, cya);
  load(ck, step, cb, cyb);

  // model into LDS (once per workgroup)
  if (tid < nwv) *reinterpret_cast<VecN<T, VEC>*>(Wl + tid * VEC) = wv0;
  if (tid + TH < nwv) *reinterpret_cast<VecN<T, VEC>*>(Wl + (tid + TH) * VEC) = wv1;
  if (tid < D) Wb[tid] = wb;
  if (tid < kRowLanes) {
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch)
#pragma unroll
      for (int v = 0; v < VW; ++v) {
        sml[(l16 + kRowLanes * ch) * VW + v] = s0[ch][v];
        sml[EP + (l16 + kRowLanes * ch) * VW + v] = m0[ch][v];
      }
  }
  bool bad = false;
  if (tid < nk) krv[tid] = rec;
  __syncthreads();
  // each row's kernel: the last one starting at or before it; -1 for the rows
  // of a kernel that is not selected (from LDS: a load of the flag beside the
  // rows would wait for all the rows in flight)
  for (int r = tid; r < R; r += TH) {
    int lo = 0, hi = nk - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (kr[mid].rel <= r) lo = mid;
      else hi = mid - 1;
    }
    rk[r] = (int16_t)(kr[lo].skip ? -1 : lo);
  }
  __syncthreads();

  // ---- rows: Tier 1 features and Tier 2 chain edges into LDS -------------
  auto compute = [&](int base, const T (&c)[U][NCH][VW], const T (&cy)[U]) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int r = base + kGroups * u + g;
      if (r >= R) break;   // uniform per 16-lane group
      const int j = rk[r];
      if (j < 0) continue;   // uniform per 16-lane group
      const int B = kr[j].B;
      const int kb = kr[j].rel;
      const int S = r - kb;
      T z[NCH][VW], s_r[NCH][VW], m_r[NCH][VW];
#pragma unroll
      for (int ch = 0; ch < NCH; ++ch) {
        const VecN<T, VW> qs = *reinterpret_cast<const VecN<T, VW>*>(sml + (l16 + kRowLanes * ch) * VW);
        const VecN<T, VW> qm = *reinterpret_cast<const VecN<T, VW>*>(sml + EP + (l16 + kRowLanes * ch) * VW);
#pragma unroll
        for (int v = 0; v < VW; ++v) {
          s_r[ch][v] = qs.v[v];
          m_r[ch][v] = qm.v[v];
        }
      }
      const T chk = row_features<T, NCH, VW>(c[u], cy[u], s_r, m_r, z);
      bad |= !__builtin_isfinite(chk);
      const uint8_t* ops = kr[j].op;
      const int ms = msb((uint32_t)S);
      int b = GRID ? 0 : ms + 1;
      T mine = qnan<T>();   // GRID: this lane's column of the grid
      // two independent dot products at a time, each row_dot's arithmetic
      for (; b + 2 <= B; b += 2) {
        const int o0 = ops[b], o1 = ops[b + 1];
        const T p0 = row_dot<T, NCH, VW>(z, Wl + o0 * EP, l16) + Wb[o0];
        const T p1 = row_dot<T, NCH, VW>(z, Wl + o1 * EP, l16) + Wb[o1];
        if (GRID) {
          const T q0 = row_first(p0), q1 = row_first(p1);
          mine = l16 == b ? q0 : l16 == b + 1 ? q1 : mine;
        }
        if (l16 == 0) {
          if (!GRID || b > ms) eb[kb + (S | (1 << b))] = p0;
          if (!GRID || b + 1 > ms) eb[kb + (S | (2 << b))] = p1;
        }
      }
      if (b < B) {
        const int o0 = ops[b];
        const T p0 = row_dot<T, NCH, VW>(z, Wl + o0 * EP, l16) + Wb[o0];
        if (GRID) {
          const T q0 = row_first(p0);
          mine = l16 == b ? q0 : mine;
        }
        if (l16 == 0 && (!GRID || b > ms)) eb[kb + (S | (1 << b))] = p0;
      }
      if (GRID && l16 < a.grid_ld)
        a.grid[(ck.row0 + r) * a.grid_ld + l16] = ((S >> l16) & 1) ? qnan<T>() : mine;
    }
  };
  // pairs of steps, no exit inside (a step past the chunk computes nothing)
  const int pairs = (R + 2 * step - 1) / (2 * step);
  for (int i = 0, base = 0; i < pairs; ++i, base += 2 * step) {
    compute(base, ca, cya);
    load(ck, base + 2 * step, ca, cya);
    compute(base + step, cb, cyb);
    load(ck, base + 3 * step, cb, cyb);
  }
  if (__ballot(bad) != 0 && lane == 0) atomicOr(a.status, (int)kStatusBadCounter);
  __syncthreads();   // every edge of the chunk is in LDS

  // ---- compose: L(S) = sum over the bits b of S, ascending, of the edge
  // into S & (2^(b+1) - 1) (the fused kernel's order) ----------------------
  for (int r = tid; r < R; r += TH) {
    const int j = rk[r];
    if (j < 0) continue;
    const int kb = kr[j].rel;
    const uint32_t S = (uint32_t)(r - kb);
    const int B = kr[j].B;
    T L = T(0);
    for (int b = 0; b < B; ++b)
      if ((S >> b) & 1u) L += eb[kb + (int)(S & ((2u << b) - 1u))];
    Lb[r] = L;
    if (a.table) a.table[ck.row0 + r] = L;
  }

  // ---- Tier 3: per kernel, one wave: per-lane best-first lists, merged;
  // a chunk of one kernel of 256 versions or more: every wave a share of them,
  // the waves' lists merged by the first (the top n is unique either way) ----
  if (!GRID && a.idx_out) {
    __syncthreads();
    if (nk == 1 && R >= 256) {
      Entry<T> lst[KT];
#pragma unroll
      for (int i = 0; i < KT; ++i) lst[i] = empty_entry<T>();
      for (int S = tid; S < R; S += TH) {
        const T v = Lb[S];
        if (S != 0 && v > a.tau) {
          Entry<T> e;
          e.v = v;
          e.s = S;
          list_insert<T, KT>(lst, e);
        }
      }
      group_merge<T, KT>(lst, kWave);
      Entry<T>* xw = reinterpret_cast<Entry<T>*>(eb);   // the edges are no longer read
      static_assert(sizeof(Entry<T>) * KT * kWaves <= sizeof(T) * 256, "lists in the edges' space");
      if (lane == 0)
#pragma unroll
        for (int i = 0; i < KT; ++i) xw[wave * KT + i] = lst[i];
      __syncthreads();
      if (wave == 0) {
#pragma unroll
        for (int i = 0; i < KT; ++i) lst[i] = xw[(lane % kWaves) * KT + i];
        group_merge<T, KT>(lst, kWaves);
        if (lane == 0) write_list<T, KT>(lst, ck.k0, a.n, a.idx_out, a.score_out, a.count_out);
      }
      return;
    }
    for (int j = wave; j < nk; j += kWaves) {   // uniform per wave
      if (kr[j].skip) continue;
      const int kb = kr[j].rel;
      const int V = 1 << kr[j].B;
      Entry<T> lst[KT];
#pragma unroll
      for (int i = 0; i < KT; ++i) lst[i] = empty_entry<T>();
      for (int S = lane; S < V; S += kWave) {
        const T v = Lb[kb + S];
        if (S != 0 && v > a.tau) {
          Entry<T> e;
          e.v = v;
          e.s = S;
          list_insert<T, KT>(lst, e);
        }
      }
      group_merge<T, KT>(lst, kWave);
      if (lane == 0) write_list<T, KT>(lst, ck.k0 + j, a.n, a.idx_out, a.score_out, a.count_out);
    }
  }
}

template <typename T, int VPL, int VW, int U, int KT, bool FULL, int TH, bool GRID>
hipError_t launch_chunk_k(const ChunkArgs<T>& a, size_t smem, hipStream_t s) {
  auto kern = path_chunk_kernel<T, VPL, VW, U, KT, FULL, TH, GRID>;
  if (smem > 64 * 1024) {
    const hipError_t e =
        hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    if (e != hipSuccess) return e;
  }
  (void)hipGetLastError();  // report only this launch's status
  const int grid = a.packed ? (a.n_chunks + kWave - 1) / kWave * kWave : a.n_chunks;
  hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(TH), smem, s, a);
  return hipGetLastError();
}

template <typename T, int VPL, int U, int KT, int TH = kChunkThreads, bool GRID = false>
hipError_t launch_chunk_u(const ChunkArgs<T>& a, hipStream_t s) {
  constexpr int VEC = 16 / sizeof(T);
  constexpr int EP = kRowLanes * VPL;
  const size_t smem = chunk_smem<T>(a.D, a.E, a.max_rows, a.max_nk).total;
  const bool vec_ok = (a.E % VEC) == 0 && (reinterpret_cast<uintptr_t>(a.counters) % 16) == 0;
  if (vec_ok && a.E == EP) return launch_chunk_k<T, VPL, VEC, U, KT, true, TH, GRID>(a, smem, s);
  if (vec_ok) return launch_chunk_k<T, VPL, VEC, U, KT, false, TH, GRID>(a, smem, s);
  return launch_chunk_k<T, VPL, 1, U, KT, false, TH, GRID>(a, smem, s);
}

template <typename T, int VPL>
hipError_t launch_chunk_vpl(const ChunkArgs<T>& a, int unroll, hipStream_t s) {
  constexpr int WIDE = chunk_wide<T, VPL>();
  if (a.grid)
    return a.wide ? launch_chunk_u<T, VPL, 1, 4, WIDE, true>(a, s)
                  : launch_chunk_u<T, VPL, 1, 4, kChunkThreads, true>(a, s);
  if (a.wide) return a.n <= 4 ? launch_chunk_u<T, VPL, 1, 4, WIDE>(a, s) : launch_chunk_u<T, VPL, 1, 8, WIDE>(a, s);
  if (a.n <= 4) {
    if (unroll >= 4) return launch_chunk_u<T, VPL, 4, 4>(a, s);
    if (unroll == 2) return launch_chunk_u<T, VPL, 2, 4>(a, s);
    return launch_chunk_u<T, VPL, 1, 4>(a, s);
  }
  if (unroll >= 4) return launch_chunk_u<T, VPL, 4, 8>(a, s);
  if (unroll == 2) return launch_chunk_u<T, VPL, 2, 8>(a, s);
  return launch_chunk_u<T, VPL, 1, 8>(a, s);
}

template <typename T>
hipError_t launch_path_chunks(const ChunkArgs<T>& a, int unroll, hipStream_t s) {
  if (a.n_chunks <= 0) return hipSuccess;
  if (a.E <= 16 * 4) return launch_chunk_vpl<T, 4>(a, unroll, s);
  if (a.E <= 16 * 8) return launch_chunk_vpl<T, 8>(a, unroll, s);
  return launch_chunk_vpl<T, 16>(a, unroll, s);
}

template hipError_t launch_path_chunks<float>(const ChunkArgs<float>&, int, hipStream_t);
template hipError_t launch_path_chunks<double>(const ChunkArgs<double>&, int, hipStream_t);

}  // namespace sugg
