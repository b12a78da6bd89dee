// The serving query between the surrogate's tables and the plain pass: Tier 3
// on the surrogate's values, the threshold band of a short list, the plain
// values of both (the judge), and Tier 3's contract by the plain values, one
// wave per kernel.
//
// Bound by latency: a kernel reads its table (4 KB at 1024 versions, in L2
// since the network wrote it) and, for each listed subset, one counter row per
// optimisation in it (three subsets of five: 15 rows, 7.5 KB), cold and
// scattered.  The terms of all the subsets are therefore spread over the four
// groups of 16 lanes, up to sixteen rows requested together, and added in
// ascending order afterwards.  Separate launches for ranking, band, judge and
// contract took 15.9 + 6.0 + 35.7 + 5.9 us for 4096 kernels of 1024 versions
// (the judge ran a wave per place of a list of up to 3 + 16, each workgroup
// staging the weights); one takes 16 to 22 (by the subsets that are listed).
// A whole query of 64 kernels of 256 versions 53.9 -> 42.1, on counters that are
// not in a cache 55.3 -> 45.2; of 512 61.6 -> 44.8 and 64.2 -> 47.3.  Four waves a
// kernel: 26.2, with a sorted list per lane and merges for the ranking 38.6.
#include <hip/hip_runtime.h>

#include "kernels.hpp"
#include "path_impl.hpp"

namespace sugg {

constexpr int kTailJobs = kMaxSuggest + kMaxBand;   // listed and band subsets
constexpr int kTailTerms = kTailJobs * SUGG_MAX_OPTS;   // (subset, optimisation) pairs

template <int VPL, int VW>
__global__ void __launch_bounds__(kWave) serve_tail_kernel(const ServeTailArgs a) {
  constexpr int NCH = VPL / VW, kGroups = kWave / kRowLanes;
  constexpr int TU = VPL <= 8 ? 4 : 2;    // terms of a group in flight
  __shared__ int32_t job_S[kTailJobs];    // listed subsets, then the band's
  __shared__ float job_ref[kTailJobs];    // their surrogate values
  __shared__ float job_L[kTailJobs];      // their plain values
  __shared__ int16_t job_t[kTailJobs];    // their first terms
  __shared__ int16_t term[kTailTerms];    // job * 16 + bit
  __shared__ float pred[kTailTerms];      // each term's prediction
  __shared__ int32_t op[SUGG_MAX_OPTS];
  const int lane = threadIdx.x, l16 = lane & 15, g = lane / kRowLanes;
  const int k = blockIdx.x, V = 1 << a.B, n = a.n, E = a.E;
  const float* ys = a.ys + (int64_t)k * V;
  const int64_t r0 = a.row_off[k];
  if (lane < a.B) op[lane] = a.opt_ids[a.opt_off[k] + lane];
  int cnt = 0, nb = 0, flag = 0;   // uniform

  // ---- Tier 3 on the surrogate's values (or its list, already ranked) -------
  if (a.sc) {
    if (lane < n) {
      job_S[lane] = a.idx[(int64_t)k * n + lane];
      job_ref[lane] = a.sc[(int64_t)k * n + lane];
    }
    cnt = a.count[k];
  } else {
    // the best of up to 1024 values in registers (and of the winners so far,
    // lane i's cv / cs, all of smaller subsets), taken out one at a time: a
    // tenth of the instructions of a sorted list per lane and their merges
    constexpr int U = 16;
    const float none = -__builtin_huge_valf();   // not above any threshold
    float cv = none;
    int cs = -1;
    for (int p0 = 0; p0 < V; p0 += U * kWave) {   // uniform
      float v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int p = p0 + u * kWave + lane;
        v[u] = p < V ? ys[p] : none;
      }
#pragma unroll
      for (int u = 0; u < U; ++u) v[u] = (p0 + u * kWave + lane != 0) & (v[u] > a.tau) ? v[u] : none;
      float nv = none;
      int ns = -1;
      for (int i = 0; i < n; ++i) {   // uniform
        float best = cv;
#pragma unroll
        for (int u = 0; u < U; ++u) best = fmaxf(best, v[u]);
        best = group_max<float>(best, kWave, lane);
        if (!(lane_read(best, 0) > none)) break;
        // the smallest subset of that value
        uint64_t m = __ballot(cv == best);
        int S = 0;
        if (m) {
          const int l = __builtin_ctzll(m);
          S = __builtin_amdgcn_readlane(cs, l);
          cv = lane == l ? none : cv;
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (!m) {
            m = __ballot(v[u] == best);
            if (m) {
              const int l = __builtin_ctzll(m);
              S = p0 + u * kWave + l;
              v[u] = lane == l ? none : v[u];
            }
          }
        nv = lane == i ? best : nv;
        ns = lane == i ? S : ns;
      }
      cv = nv;
      cs = ns;
    }
    if (cs >= 0) {
      job_S[lane] = cs;
      job_ref[lane] = cv;
    }
    cnt = __popcll(__ballot(cs >= 0));
  }
  __syncthreads();

  // ---- the band of a short list (as band_kernel, C = cap) ---------------------
  if (cnt < n) {   // uniform
    int total = 0;
    for (int base = 1; base < V; base += kWave) {
      const int p = base + lane;
      bool take = false;
      float v = 0.0f;
      if (p < V) {
        v = ys[p];
        take = (double)v >= a.lo;
        for (int i = 0; i < cnt; ++i) take = take && job_S[i] != p;
      }
      const uint64_t m = __ballot(take);
      const int pos = total + __popcll(m & ((1ull << lane) - 1ull));
      if (take && pos < a.cap) {
        job_S[cnt + pos] = p;
        job_ref[cnt + pos] = v;
      }
      total += __popcll(m);
    }
    nb = total < a.cap ? total : a.cap;
    flag = total > a.cap;
    __syncthreads();
  }

  // ---- plain values: one group of 16 lanes per (subset, optimisation) ---------
  const int jobs = cnt + nb;
  int terms = 0;
  for (int j = 0; j < jobs; ++j) {   // uniform
    const uint32_t S = (uint32_t)job_S[j];
    if (lane < a.B && ((S >> lane) & 1u)) term[terms + __popc(S & ((1u << lane) - 1u))] = (int16_t)(j * 16 + lane);
    if (lane == 0) job_t[j] = (int16_t)terms;
    terms += __popc(S);
  }
  __syncthreads();
  float s_r[NCH][VW], m_r[NCH][VW];
  column_constants<float, NCH, VW, false>(a.mu, a.isg, E, l16, s_r, m_r);
  bool bad = false;
  for (int q0 = 0; q0 < terms; q0 += TU * kGroups) {   // uniform
    float c[TU][NCH][VW], cy[TU], wb[TU];
    VecN<float, VW> w[TU][NCH];
#pragma unroll
    for (int u = 0; u < TU; ++u) {
      const int q = q0 + u * kGroups + g;
      const int t = term[q < terms ? q : terms - 1], b = t & 15;   // (a surplus group repeats the last term)
      const int64_t row = r0 + (job_S[t >> 4] & ((1 << b) - 1));
      const float* rp = a.counters + row * E;
      const float* wp = a.W + (int64_t)op[b] * a.ldw;
#pragma unroll
      for (int ch = 0; ch < NCH; ++ch) {
        const int cc = (l16 + kRowLanes * ch) * VW;
        if (cc < E) {
          const VecN<float, VW> x = *reinterpret_cast<const VecN<float, VW>*>(rp + cc);
#pragma unroll
          for (int v = 0; v < VW; ++v) c[u][ch][v] = x.v[v];
          w[u][ch] = *reinterpret_cast<const VecN<float, VW>*>(wp + cc);
        } else {
#pragma unroll
          for (int v = 0; v < VW; ++v) {
            c[u][ch][v] = 1.0f;
            w[u][ch].v[v] = 0.0f;
          }
        }
      }
      cy[u] = a.cycles[row];
      wb[u] = wp[E];
    }
#pragma unroll
    for (int u = 0; u < TU; ++u) {
      const int q = q0 + u * kGroups + g;
      if (q >= terms) break;   // uniform per group
      float z[NCH][VW];
      const float chk = row_features<float, NCH, VW>(c[u], cy[u], s_r, m_r, z);
      bad |= !__builtin_isfinite(chk);
      float part = 0.0f;   // row_dot's order
#pragma unroll
      for (int ch = 0; ch < NCH; ++ch)
#pragma unroll
        for (int v = 0; v < VW; ++v) part = fma(z[ch][v], w[u][ch].v[v], part);
      const float p = row_sum16(part) + wb[u];
      if (l16 == 0) pred[q] = p;
    }
  }
  if (__ballot(bad) != 0 && lane == 0) atomicOr(a.status, (int)kStatusBadCounter);
  __syncthreads();

  // ---- contract: a plain value further than tol from the surrogate's, a
  // listed one not above tau or a band one above it flags the kernel ----------
  bool off = false;
  for (int j = lane; j < jobs; j += kWave) {
    const int nt = __popc((uint32_t)job_S[j]), t0 = job_t[j];
    float L = 0.0f;
    for (int i = 0; i < nt; ++i) L += pred[t0 + i];
    job_L[j] = L;
    off |= !(fabs((double)job_ref[j] - (double)L) <= a.tol) || (j < cnt ? !(L > a.tau) : L > a.tau);
  }
  flag |= __ballot(off) != 0;
  __syncthreads();
  if (lane < n) {
    // a kept list is sorted by its plain values (descending, then the smaller subset)
    const bool listed = lane < cnt;
    const int S = listed ? job_S[lane] : -1;
    const float L = listed ? job_L[lane] : qnan<float>();
    int pos = lane;
    if (listed && !flag) {
      pos = 0;
      for (int i = 0; i < cnt; ++i) pos += job_L[i] > L || (job_L[i] == L && job_S[i] < S);
    }
    a.idx[(int64_t)k * n + pos] = S;
    a.score[(int64_t)k * n + pos] = L;
  }
  if (lane == 0) {
    a.count[k] = cnt;
    a.flag[k] = flag;
  }
}

namespace {

template <int VPL>
void launch_tail_t(const ServeTailArgs& a, hipStream_t s) {
  if (a.E % 4 == 0 && reinterpret_cast<uintptr_t>(a.counters) % 16 == 0)
    hipLaunchKernelGGL((serve_tail_kernel<VPL, 4>), dim3((unsigned)a.K), dim3(kWave), 0, s, a);
  else
    hipLaunchKernelGGL((serve_tail_kernel<VPL, 1>), dim3((unsigned)a.K), dim3(kWave), 0, s, a);
}

}  // namespace

hipError_t launch_serve_tail(const ServeTailArgs& a, hipStream_t s) {
  if (a.K <= 0) return hipSuccess;
  if (a.B < 0 || a.B > SUGG_MAX_OPTS || a.n < 1 || a.n > kMaxSuggest || a.cap < 1 || a.cap > kMaxBand || a.E < 1 || a.E > 256)
    return hipErrorInvalidValue;
  (void)hipGetLastError();  // report only this launch's status
  if (a.E <= 64) launch_tail_t<4>(a, s);
  else if (a.E <= 128) launch_tail_t<8>(a, s);
  else launch_tail_t<16>(a, s);
  return hipGetLastError();
}

}  // namespace sugg
