// Tier 2 training (Section 2: before/after samples of each optimisation;
// Section 3.4: regression): per global optimisation o, the ridge normal
// equations
//   (X^T X + lambda diag(1,..,1,0)) w_o = X^T y,   X = [z(before), 1],
//   y = ln cyc(before) - ln cyc(after),
// over every pair (version S without o, version S with o) of the training
// kernels, accumulated and solved in FP64.
//
// gram_kernel         one workgroup per chunk of rows: Tier 1's features of a
//                     stage of rows go to LDS with the labels and a column of
//                     ones beside them, and the lower triangle of
//                     [Z | Y | 1]^T [Z | Y | 1] is accumulated by the FP64
//                     matrix cores; the partial goes to a workspace.
// gram_reduce_kernel  sums the chunks of every optimisation, in a fixed order.
// solve_kernel        one workgroup per optimisation: ridge term, Cholesky and
//                     two triangular solves.
#include <algorithm>

#include "kernels.hpp"
#include "path_impl.hpp"

namespace sugg {

typedef double doublex4 __attribute__((ext_vector_type(4)));

constexpr int kGramStage = 32;   // rows per stage

__device__ __forceinline__ int64_t insert_zero_bit(int64_t q, int b) {
  return ((q >> b) << (b + 1)) | (q & ((1ll << b) - 1));
}

// The rows of every segment, in order (built once per plan).
__global__ void __launch_bounds__(256) gram_rows_kernel(const GramSeg* __restrict__ segs, int nseg, int64_t n,
                                                        int pairs, const int32_t* __restrict__ klist,
                                                        const int64_t* __restrict__ row_off,
                                                        GramRow* __restrict__ out) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    int lo = 0, hi = nseg - 1;
    while (lo < hi) {   // last segment with base <= i
      const int mid = (lo + hi + 1) >> 1;
      if (segs[mid].base <= i) lo = mid;
      else hi = mid - 1;
    }
    const GramSeg g = segs[lo];
    const int64_t q = i - g.base;
    GramRow r;
    r.row = pairs ? row_off[g.first] + insert_zero_bit(q, g.sel) : row_off[klist[g.first + q]] + g.sel;
    r.bits = g.bits;
    out[i] = r;
  }
}

hipError_t launch_gram_rows(const GramSeg* segs, int nseg, int64_t n, bool pairs, const int32_t* klist,
                            const int64_t* row_off, GramRow* out, hipStream_t s) {
  if (n <= 0 || nseg <= 0) return hipSuccess;
  int64_t blocks = (n + 255) / 256;
  if (blocks > 8192) blocks = 8192;
  (void)hipGetLastError();  // report only this launch's status
  hipLaunchKernelGGL(gram_rows_kernel, dim3((unsigned)blocks), dim3(256), 0, s, segs, nseg, n, pairs ? 1 : 0, klist,
                     row_off, out);
  return hipGetLastError();
}

// Sixteen-column blocks of [Z | Y | 1]: E padded, and one block of 16 for the
// labels (columns 0..11, the row's optimisations in ascending id) and the
// ones (column kGramOnes).
constexpr int kGramOnes = 12;
static_assert(SUGG_MAX_OPTS <= kGramOnes, "label columns");
int gram_blocks(int E) { return E <= 64 ? 5 : E <= 128 ? 9 : 17; }
int64_t gram_stride(int E) { return (int64_t)gram_blocks(E) * (gram_blocks(E) + 1) / 2 * 256; }

// One work item: rows [begin, begin + n) of the row list, all of them before
// versions of the optimisations in `mask`.  A stage's rows are read from HBM
// (16 lanes a row), standardised and laid out in LDS as [row][column]; the
// block product of 16 columns by 16 columns over four rows is one
// v_mfma_f64_16x16x4_f64, whose A and B operands have the same lane layout
// (lane l: column l % 16 of row l / 16), so a 16-column operand serves as
// either.  The block rows of the lower triangle are dealt out to V waves from
// the longest down and back up, so each has about the same number of blocks
// (9 block columns: 12, 11, 11, 11 of 45); beyond 128 events two workgroups
// share an item's block rows.  The next stage's counters are in flight while
// the matrix cores work on this one, in the other half of the LDS.
//
// Bound by the FP64 matrix rate (73 TFLOP/s measured; the FP64 vector rate is
// the same, but there every 64 multiply-adds of an 8 x 8 register block cost
// 16 LDS reads) and the logarithms.  A row enters once, however many
// optimisations it is a before version of, where there are enough rows per
// set of optimisations (gram_classes): 4.8 M rows in place of 21.5 M pairs on
// the 16,384-kernel training set.  Features are formed here: their FP64 copy
// (4.9 GB there) was written once and read back 4.5 times.
// Measured on that set: 2.95 ms, where features and sums took 48.8 ms before;
// 512 kernels of 64 versions: 36 us, before 223 us.  Beyond 128 events 14 to 33 of
// the 256 registers spill (17 block columns of accumulators).
template <typename T, int NB, int VW>
__global__ void __launch_bounds__(NB <= 9 ? 256 : 512, 2) gram_kernel(const GramArgs a) {
  constexpr int W = NB <= 9 ? 4 : 8;            // waves per workgroup
  constexpr int V = NB <= 9 ? 4 : 16;           // waves that share an item's blocks (V / W workgroups)
  constexpr int LD = 16 * NB;                   // LDS row, doubles: NB odd, so two rows differ by 32 banks
  constexpr int NCH = (NB - 1) / VW;            // column chunks per lane
  constexpr int RP = W * 4;                     // rows per pass of the workgroup
  constexpr int NP = kGramStage / RP;           // passes per stage
  constexpr int N1 = NB > V ? NB - V : 0, N2 = NB > 2 * V ? NB - 2 * V : 0;
  static_assert(NB % 2 == 1 && (NB - 1) % VW == 0 && kGramStage % RP == 0, "stage shape");
  extern __shared__ __align__(16) unsigned char smem[];
  double* zs = reinterpret_cast<double*>(smem);            // [2][kGramStage][LD]
  double* cmu = zs + 2 * kGramStage * LD;                  // [16 (NB - 1)] column means, then 1 / sigma
  double* cis = cmu + 16 * (NB - 1);
  const int E = a.E;
  const GramWork w = a.work[blockIdx.x];
  const int tid = threadIdx.x, lane = tid & 63, l16 = tid & 15, rg = tid >> 4;
  const int v = blockIdx.y * W + (tid >> 6);               // which share of the block rows
  const int nids = __popcll(w.mask);
  for (int j = tid; j < 16 * (NB - 1); j += 64 * W) {
    cmu[j] = j < E ? a.mu[j] : 0.0;
    cis[j] = j < E ? 1.0 / a.sig[j] : 0.0;
  }
  const int nst = (w.n + kGramStage - 1) / kGramStage;
  const T* counters = reinterpret_cast<const T*>(a.counters);
  T cnt[NP][NCH][VW];
  double lc[NP], ly[NP];
  GramRow ent[NP];
  // list entries of a stage; past the item its last row is read again (and
  // enters as zeros)
  auto rows = [&](int st) {
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      const int r = st * kGramStage + p * RP + rg;
      ent[p] = a.rows[w.begin + (r < w.n ? r : w.n - 1)];
    }
  };
  auto load = [&]() {
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      const T* rp = counters + ent[p].row * E;
#pragma unroll
      for (int ch = 0; ch < NCH; ++ch) {
        const int c0 = (l16 + 16 * ch) * VW;
        if (c0 < E) {
          const VecN<T, VW> q = *reinterpret_cast<const VecN<T, VW>*>(rp + c0);
#pragma unroll
          for (int u = 0; u < VW; ++u) cnt[p][ch][u] = q.v[u];
        } else {
#pragma unroll
          for (int u = 0; u < VW; ++u) cnt[p][ch][u] = T(1);
        }
      }
      lc[p] = a.lcyc[ent[p].row];
      // lane j of the row: the after version of the row's j-th optimisation
      const int bit = (int)(ent[p].bits >> (4 * l16)) & 15;
      ly[p] = a.lcyc[ent[p].row + (l16 < nids ? (int64_t)1 << bit : 0)];
    }
  };
  auto store = [&](int st, double* buf) {
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      const int rr = p * RP + rg;
      const bool live = st * kGramStage + rr < w.n;
      double* zr = buf + rr * LD;
#pragma unroll
      for (int ch = 0; ch < NCH; ++ch) {
        const int c0 = (l16 + 16 * ch) * VW;
        VecN<double, VW> q;
#pragma unroll
        for (int u = 0; u < VW; ++u) {
          const double x = flog64((double)cnt[p][ch][u]) - lc[p];
          q.v[u] = live && c0 + u < E ? (x - cmu[c0 + u]) * cis[c0 + u] : 0.0;
        }
        *reinterpret_cast<VecN<double, VW>*>(zr + c0) = q;
      }
      zr[16 * (NB - 1) + l16] = !live ? 0.0 : l16 < nids ? lc[p] - ly[p] : l16 == kGramOnes ? 1.0 : 0.0;
    }
  };
  // this wave's block rows: NB-1-v, NB-2V+v and NB-1-2V-v, where they exist
  const int r0 = NB - 1 - v, r1 = NB - 2 * V + v;
  doublex4 acc0[NB], acc1[N1 > 0 ? N1 : 1], acc2[1];
#pragma unroll
  for (int j = 0; j < NB; ++j) acc0[j] = doublex4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int j = 0; j < (N1 > 0 ? N1 : 1); ++j) acc1[j] = doublex4{0.0, 0.0, 0.0, 0.0};
  acc2[0] = doublex4{0.0, 0.0, 0.0, 0.0};
  static_assert(N2 <= 1, "third block rows");

  rows(0);
  load();
  if (nst > 1) rows(1);
  __syncthreads();   // column constants
  store(0, zs);
  __syncthreads();
  for (int st = 0; st < nst; ++st) {
    const double* buf = zs + (st & 1) * kGramStage * LD;
    if (st + 1 < nst) {
      load();
      if (st + 2 < nst) rows(st + 2);
    }
#pragma unroll 2
    for (int k = 0; k < kGramStage; k += 4) {
      const double* zk = buf + (k + (lane >> 4)) * LD + l16;
      double b[NB];
#pragma unroll
      for (int j = 0; j < NB; ++j) b[j] = zk[16 * j];
      const double a0 = zk[16 * r0];
#pragma unroll
      for (int j = 0; j < NB; ++j)
        if (j <= r0) acc0[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, b[j], acc0[j], 0, 0, 0);
      if (N1 > 0 && r1 >= 0) {
        const double a1 = zk[16 * r1];
#pragma unroll
        for (int j = 0; j < N1; ++j)
          if (j <= r1) acc1[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b[j], acc1[j], 0, 0, 0);
      }
      if (N2 > 0 && v == 0) acc2[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(b[0], b[0], acc2[0], 0, 0, 0);
    }
    if (st + 1 < nst) store(st + 1, zs + ((st + 1) & 1) * kGramStage * LD);
    __syncthreads();
  }
  // element i of lane l: row 4 i + l / 16, column l % 16 of the block
  double* out = a.partial + (int64_t)blockIdx.x * (NB * (NB + 1) / 2 * 256);
  auto put = [&](int bi, int bj, const doublex4& c) {
    double* o = out + (bi * (bi + 1) / 2 + bj) * 256 + lane;
#pragma unroll
    for (int i = 0; i < 4; ++i) o[64 * i] = c[i];
  };
#pragma unroll
  for (int j = 0; j < NB; ++j)
    if (j <= r0) put(r0, j, acc0[j]);
  if (N1 > 0 && r1 >= 0) {
#pragma unroll
    for (int j = 0; j < N1; ++j)
      if (j <= r1) put(r1, j, acc1[j]);
  }
  if (N2 > 0 && v == 0) put(0, 0, acc2[0]);
}

template <typename T, int NB, int VW>
hipError_t launch_gram_t(const GramArgs& a, hipStream_t s) {
  constexpr int W = NB <= 9 ? 4 : 8, V = NB <= 9 ? 4 : 16;
  constexpr size_t smem = sizeof(double) * (2 * kGramStage * 16 * NB + 2 * 16 * (NB - 1));
  auto kern = gram_kernel<T, NB, VW>;
  if (smem > 64 * 1024) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(kern, dim3(a.n_work, V / W), dim3(64 * W), smem, s, a);
  return hipSuccess;
}

template <typename T>
hipError_t launch_gram(const GramArgs& a, hipStream_t s) {
  if (a.n_work <= 0) return hipSuccess;
  constexpr int VEC = 16 / sizeof(T);
  const bool vec = a.E % VEC == 0 && reinterpret_cast<uintptr_t>(a.counters) % 16 == 0;
  (void)hipGetLastError();  // report only this launch's status
  hipError_t e;
  switch (gram_blocks(a.E)) {
    case 5: e = vec ? launch_gram_t<T, 5, VEC>(a, s) : launch_gram_t<T, 5, 1>(a, s); break;
    case 9: e = vec ? launch_gram_t<T, 9, VEC>(a, s) : launch_gram_t<T, 9, 1>(a, s); break;
    default: e = vec ? launch_gram_t<T, 17, VEC>(a, s) : launch_gram_t<T, 17, 1>(a, s); break;
  }
  return e != hipSuccess ? e : hipGetLastError();
}
template hipError_t launch_gram<float>(const GramArgs&, hipStream_t);
template hipError_t launch_gram<double>(const GramArgs&, hipStream_t);

// Sums of the chunks' partials per optimisation, in two launches, each in a
// fixed order.  The first reads every partial once per 16 ids: a thread adds one
// element of every chunk of its slice to the accumulators of the optimisations in
// the chunk's mask (16 ids per workgroup; the mask is uniform).  The labels' rows
// are per chunk (the j-th id of its mask), so row 0 of the label blocks takes
// the row of the id it is summed for; rows other than that and the ones' are
// not used.
constexpr int kReduceIds = 16;
__global__ void __launch_bounds__(256) gram_reduce_kernel(const double* __restrict__ partial,
                                                          const GramWork* __restrict__ work, int n_work, int nb, int D,
                                                          double* __restrict__ out) {
  const int64_t stride = (int64_t)nb * (nb + 1) / 2 * 256;
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;   // stride is a multiple of 256
  const int t = blockIdx.x, G = gridDim.y, g = blockIdx.y, o0 = blockIdx.z * kReduceIds;
  const int tl = nb * (nb - 1) / 2;                    // first block of the labels' block row
  const int row = threadIdx.x >> 4, col = threadIdx.x & 15;
  const bool label = t >= tl && row == 0;
  // label blocks: element [j][col] of block t; in the diagonal one the ones'
  // column against label j
  double acc[kReduceIds];
#pragma unroll
  for (int o = 0; o < kReduceIds; ++o) acc[o] = 0.0;
  // eight chunks' elements in flight (two, as the compiler left it: 18.7 us for
  // 512 kernels of 64 versions, now 17.3)
  constexpr int U = 8;
  for (int q0 = g; q0 < n_work; q0 += U * G) {
    double v[U];
    uint64_t m[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int q = q0 + u * G;
      v[u] = partial[(q < n_work ? q : q0) * stride + i];
      m[u] = q < n_work ? work[q].mask : 0;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint64_t mask = m[u] >> o0, below = m[u] & ((1ull << o0) - 1ull);
      const double* p = partial + (q0 + u * G) * stride;
#pragma unroll
      for (int o = 0; o < kReduceIds; ++o)
        if ((mask >> o) & 1ull) {
          const int j = __popcll(below) + __popcll(mask & ((1ull << o) - 1ull));
          acc[o] += label ? p[(int64_t)t * 256 + j * 16 + col] : v[u];
        }
    }
  }
#pragma unroll
  for (int o = 0; o < kReduceIds; ++o)
    if (o0 + o < D) out[((int64_t)g * D + o0 + o) * stride + i] = acc[o];
}

__global__ void __launch_bounds__(256) gram_reduce2_kernel(const double* __restrict__ part, int G, int64_t n,
                                                           double* __restrict__ out) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;   // n is a multiple of 256
  double v = 0.0;
#pragma unroll 4
  for (int g = 0; g < G; ++g) v += part[g * n + i];
  out[i] = v;
}

// Slices of the first launch: about 16 chunks each, so that 45 blocks of
// elements (128 events) times the slices fill the chip; their sums at most 256
// MB (64 ids and 256 events: 12 slices of 20 MB in place of 32).
int gram_slices(int n_work, int D, int E) {
  const int most = (int)std::max<int64_t>(1, ((int64_t)1 << 25) / (std::max(D, 1) * gram_stride(E)));
  return std::max(1, std::min({32, n_work / 16, most}));
}

hipError_t launch_gram_reduce(const GramArgs& a, int D, double* slices, double* reduced, hipStream_t s) {
  if (D <= 0) return hipSuccess;
  const int nb = gram_blocks(a.E), G = gram_slices(a.n_work, D, a.E);
  const int64_t stride = gram_stride(a.E);
  (void)hipGetLastError();  // report only this launch's status
  hipLaunchKernelGGL(gram_reduce_kernel, dim3((unsigned)(stride / 256), G, (D + kReduceIds - 1) / kReduceIds), dim3(256),
                     0, s, a.partial, a.work, a.n_work, nb, D, slices);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(gram_reduce2_kernel, dim3((unsigned)(stride * D / 256)), dim3(256), 0, s, slices, G, stride * D,
                     reduced);
  return hipGetLastError();
}

// ---- the solve -----------------------------------------------------------------
// Lower triangle of 16 x 16 blocks (rows padded to 17 doubles, so that a
// column of a block spreads over the banks) of the system with its right-hand
// side as one more row: the features, the intercept (index E), the labels
// (index E + 1), then the identity.  The factorisation then leaves the forward
// solution in the labels' row.
constexpr int kSolveThreads = 512;
constexpr int kBlkLd = 17, kBlkSz = 16 * kBlkLd;
constexpr size_t kSolveLdsMax = 150 * 1024;
static int solve_blocks(int E) { return (E + 2 + 15) / 16; }
static size_t solve_matrix(int E) { return (size_t)solve_blocks(E) * (solve_blocks(E) + 1) / 2 * kBlkSz; }
static bool solve_in_lds(int E) { return sizeof(double) * (solve_matrix(E) + 32 * solve_blocks(E)) <= kSolveLdsMax; }
size_t solve_workspace(int E) { return solve_in_lds(E) ? 0 : solve_matrix(E); }

__device__ __forceinline__ double lane_value(double v, int l) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l),
                          __builtin_amdgcn_readlane(__double2loint(v), l));
}

// g = sqrt(d) and ih = 1 / sqrt(d), d > 0: Goldschmidt's iteration from the
// hardware's reciprocal square root, and one residual step for the root.
__device__ __forceinline__ void root_and_inverse(double d, double& g, double& ih) {
  const double y = __builtin_amdgcn_rsq(d);
  double h = 0.5 * y;
  g = d * y;
  double r = fma(-h, g, 0.5);
  g = fma(g, r, g);
  h = fma(h, r, h);
  r = fma(-h, g, 0.5);
  g = fma(g, r, g);
  h = fma(h, r, h);
  g = fma(fma(-g, g, d), h, g);
  ih = 2.0 * h;
}

// A = L L^T by block columns: one wave factorises the diagonal block in
// registers (a row per lane, pivots and multipliers by lane reads), a thread
// per row solves for the blocks below it, and the matrix cores update the
// rest, the next diagonal block first, so that its factorisation runs beside
// the others' updates.  Then L^T w = t, block by block from the last.
// A serial chain of E + 1 pivots bounds it: one column at a time, with three
// barriers each and two more per column and triangular solve, took 288 us at
// E = 128; in blocks 84, with the next diagonal block ahead 73 us.
__global__ void __launch_bounds__(kSolveThreads) solve_kernel(const SolveArgs a, const int use_lds) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int o = blockIdx.x;
  const int E = a.E, n1 = E + 1, M = (E + 2 + 15) / 16;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l16 = lane & 15, l4 = lane >> 4;
  const int nb = a.nb;
  const double* G = a.reduced + (int64_t)o * (nb * (nb + 1) / 2 * 256);   // this optimisation's summed partials
  const auto at = [&](int i, int j) -> double {   // element of the blocked lower triangle, i >= j
    const int bi = i >> 4, bj = j >> 4;
    return G[(bi * (bi + 1) / 2 + bj) * 256 + (i & 15) * 16 + (j & 15)];
  };
  const int one = 16 * (nb - 1) + kGramOnes, lab = 16 * (nb - 1);   // rows of the ones and of this label
  const double count = at(one, one);
  if (count == 0.0) {
    for (int j = tid; j < n1; j += kSolveThreads) {
      a.W64[(int64_t)o * n1 + j] = __builtin_nan("");
      a.W32[(int64_t)o * w32_ld(E) + j] = 0.0f;
    }
    return;
  }
  double* y = reinterpret_cast<double*>(smem);   // [16 M] the labels' row, then the solution
  double* inv = y + 16 * M;                      // [16 M] 1 / diagonal of L
  double* A = use_lds ? inv + 16 * M : a.A + (size_t)o * (M * (M + 1) / 2 * kBlkSz);
  const auto blk = [&](int bi, int bj) -> double* { return A + (bi * (bi + 1) / 2 + bj) * kBlkSz; };
  for (int idx = tid, bi = 0, bj = 0, t = 0; idx < M * (M + 1) / 2 * 256; idx += kSolveThreads) {
    for (; t < (idx >> 8); ++t)   // block t of the lower triangle, row by row
      if (++bj > bi) {
        bj = 0;
        ++bi;
      }
    const int r = (idx >> 4) & 15, c = idx & 15, i = bi * 16 + r, j = bj * 16 + c;
    double v = i == j ? 1.0 : 0.0;
    if (j <= i && j <= E) {
      if (i < E) v = at(i, j) + (i == j ? a.lambda : 0.0);
      else if (i == E) v = j < E ? at(one, j) : count;
      else if (i == E + 1) v = j < E ? at(lab, j) : G[(nb * (nb + 1) / 2 - 1) * 256 + kGramOnes];   // sum of the labels
    }
    A[(idx >> 8) * kBlkSz + r * kBlkLd + c] = v;
  }
  __syncthreads();
  bool bad = false;
  // block row bi, column bj of the trailing matrix, less the product of panel p
  const auto update = [&](int p, int bi, int bj) {
    const double* Li = blk(bi, p) + l16 * kBlkLd + l4;
    const double* Lj = blk(bj, p) + l16 * kBlkLd + l4;
    double* C = blk(bi, bj) + l4 * kBlkLd + l16;
    doublex4 c;
#pragma unroll
    for (int i = 0; i < 4; ++i) c[i] = C[4 * i * kBlkLd];
#pragma unroll
    for (int k = 0; k < 4; ++k) c = __builtin_amdgcn_mfma_f64_16x16x4f64(-Li[4 * k], Lj[4 * k], c, 0, 0, 0);
#pragma unroll
    for (int i = 0; i < 4; ++i) C[4 * i * kBlkLd] = c[i];
  };
  for (int p = -1; p < M; ++p) {
    if (p >= 0) {
      if (16 * p > E) break;
      for (int i = 16 * (p + 1) + tid; i < 16 * M; i += kSolveThreads) {
        const double* D = blk(p, p);
        double* X = blk(i >> 4, p) + (i & 15) * kBlkLd;
        double x[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) x[k] = X[k];
#pragma unroll
        for (int k = 0; k < 16; ++k) {
          x[k] *= inv[16 * p + k];
#pragma unroll
          for (int j = k + 1; j < 16; ++j) x[j] = fma(-x[k], D[j * kBlkLd + k], x[j]);
        }
#pragma unroll
        for (int k = 0; k < 16; ++k) X[k] = x[k];
      }
      __syncthreads();
    }
    if (wave == 0 && p + 1 < M) {   // the next diagonal block, while the others update the rest
      if (p >= 0) {
        update(p, p + 1, p + 1);
        __threadfence_block();   // its lanes exchange elements below
      }
      const int p1 = p + 1;
      double* D = blk(p1, p1);
      double row[16], iv = 1.0;
#pragma unroll
      for (int k = 0; k < 16; ++k) row[k] = D[l16 * kBlkLd + k];
#pragma unroll
      for (int k = 0; k < 16; ++k) {
        if (16 * p1 + k <= E) {   // the labels' row and the padding have no pivot
          double d = lane_value(row[k], k);
          if (!(d > 0.0)) {
            bad = true;
            d = 1.0;
          }
          double piv, ip;
          root_and_inverse(d, piv, ip);
          row[k] = l16 == k ? piv : row[k] * ip;
          iv = l16 == k ? ip : iv;
#pragma unroll
          for (int j = k + 1; j < 16; ++j) row[j] = fma(-row[k], lane_value(row[k], j), row[j]);
        }
      }
      if (lane < 16) {
#pragma unroll
        for (int k = 0; k < 16; ++k) D[l16 * kBlkLd + k] = row[k];   // above the diagonal: not used
        inv[16 * p1 + l16] = iv;
      }
    }
    if (wave != 0 && p >= 0) {
      int t = 0;
      for (int bi = p + 2; bi < M; ++bi)
        for (int bj = p + 1; bj <= bi; ++bj, ++t)
          if (t % (kSolveThreads / 64 - 1) == wave - 1) update(p, bi, bj);
    }
    __syncthreads();
  }
  for (int j = tid; j < 16 * M; j += kSolveThreads)
    y[j] = j <= E ? blk((E + 1) >> 4, j >> 4)[((E + 1) & 15) * kBlkLd + (j & 15)] : 0.0;
  __syncthreads();
  for (int p = E >> 4; p >= 0; --p) {
    if (wave == 0) {
      const double* D = blk(p, p);
      double col[16], t = y[16 * p + l16];
      const double iv = inv[16 * p + l16];
#pragma unroll
      for (int k = 0; k < 16; ++k) col[k] = D[k * kBlkLd + l16];
#pragma unroll
      for (int k = 15; k >= 0; --k)
        if (16 * p + k <= E) {
          const double wk = lane_value(t * iv, k);
          t = l16 == k ? wk : l16 < k ? fma(-col[k], wk, t) : t;
        }
      if (lane < 16) y[16 * p + l16] = t;
    }
    __syncthreads();
    for (int j = tid; j < 16 * p; j += kSolveThreads) {
      const double* L = blk(p, j >> 4) + (j & 15);
      double v = y[j];
#pragma unroll
      for (int k = 0; k < 16; ++k)
        if (16 * p + k <= E) v = fma(-L[k * kBlkLd], y[16 * p + k], v);
      y[j] = v;
    }
    __syncthreads();
  }
  for (int j = tid; j < n1; j += kSolveThreads) {
    a.W64[(int64_t)o * n1 + j] = y[j];
    a.W32[(int64_t)o * w32_ld(E) + j] = (float)y[j];
  }
  if (tid == 0 && bad) atomicOr(a.status, (int)kStatusSingular);
}

hipError_t launch_solve(const SolveArgs& a, hipStream_t s) {
  if (a.D <= 0) return hipSuccess;
  const int use_lds = solve_in_lds(a.E) ? 1 : 0;
  const size_t smem = sizeof(double) * (32 * solve_blocks(a.E) + (use_lds ? solve_matrix(a.E) : 0));
  if (smem > 64 * 1024) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(solve_kernel),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    if (e != hipSuccess) return e;
  }
  (void)hipGetLastError();  // report only this launch's status
  hipLaunchKernelGGL(solve_kernel, dim3(a.D), dim3(kSolveThreads), smem, s, a, use_lds);
  return hipGetLastError();
}

}  // namespace sugg
