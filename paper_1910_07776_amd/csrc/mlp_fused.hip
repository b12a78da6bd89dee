// Frozen inference of the surrogate in one launch, for large batches: a
// workgroup takes 64 rows through all three layers, the activations between
// them in LDS.
//
// Every output element is the sum the layer-by-layer GEMMs form: K ascending
// in steps of 16 of v_mfma_f32_32x32x16_bf16 with FP32 accumulation, bias,
// GELU and the rounding to BF16 as there (the same bits).  The operands trade
// places (weights A, activations B), so a lane holds four consecutive units of
// one row and writes them to LDS as 8 bytes.
//
// Weights come straight from L2 in operand order (mlp_frag_kernel: 1 KB per
// wave and step, each read once per workgroup), three steps ahead; activations
// are read from LDS.  Eight waves share the 512 hidden units, 64 each.
//
// Bound by the GELU's vector work (two transcendentals and about seventeen
// other operations on each of 1024 activations a row: 43 us for 65,536 rows at
// full rate) beside the matrix work (35 us at the rate of a large library
// product); two workgroups per compute unit overlap the two.  Layer by layer
// the rows also wrote and read 268 MB of activations: 65,536 kernels took 144
// us (features 23, GEMMs 98 and 27), now 84.  128 rows a workgroup, one per
// compute unit: 100 us (without the GELU 68, without the weights' reads 97).
// The ranking instances spill 3 registers of 128.
#include <hip/hip_runtime.h>

#include "mlp_math.hpp"
#include "path_impl.hpp"

namespace sugg {

constexpr int kHid = kFusedHidden, kHidSteps = kHid / 16;
constexpr int kFusedThreads = 512, kFusedWaves = 8;
constexpr int kActLd = kHid + 8;   // LDS row of activations, elements: 16-byte reads of 16 rows spread over the banks

typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

// ---- weights in operand order ---------------------------------------------------
// W [N x K] as tiles of 32 rows, steps of 16 columns: lane l holds columns (l /
// 32) * 8 + 0..7 of the step of row l % 32 (zero past K).
__global__ void __launch_bounds__(256) mlp_frag_kernel(const FragArgs a) {
  int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;   // lane slot over the three matrices
  int q = 0;
  while (q < 3 && i >= (int64_t)a.N[q] / 32 * a.steps[q] * 64) i -= (int64_t)a.N[q] / 32 * a.steps[q++] * 64;
  if (q == 3) return;
  const int lane = (int)(i & 63);
  const int64_t t = i >> 6;
  const int row = (int)(t / a.steps[q]) * 32 + (lane & 31), k0 = (int)(t % a.steps[q]) * 16 + (lane >> 5) * 8;
  const float* w = a.params + a.off[q] + (int64_t)row * a.K[q];
  bf16x8 v;
#pragma unroll
  for (int u = 0; u < 8; ++u) v[u] = k0 + u < a.K[q] ? to_bf16(w[k0 + u]) : (__bf16)0.0f;
  a.out[q][i] = v;
}

hipError_t launch_mlp_frag(const FragArgs& a, hipStream_t s) {
  int64_t n = 0;
  for (int q = 0; q < 3; ++q) n += (int64_t)a.N[q] / 32 * a.steps[q] * 64;
  (void)hipGetLastError();  // report only this launch's status
  hipLaunchKernelGGL(mlp_frag_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, a);
  return hipGetLastError();
}

// acc[c][r] += W tile c . activations tile r^T over `steps` steps: tiles of 32
// units and 32 rows; w: the first weight tile (tiles ws apart), x: LDS rows.
template <int C, int R, int LDX>
__device__ __forceinline__ void fused_product(floatx16 (&acc)[C][R], const bf16x8* __restrict__ w, int64_t ws,
                                              const __bf16* x, int ldx, int steps, int lane) {
  // steps of weights in flight; the next step's activations are read while
  // this one is multiplied.  The scheduling barriers keep it so (the loads of
  // several steps were otherwise moved together, to just before their use).
  constexpr int P = 3;
  const __bf16* xr = x + (lane & 31) * (LDX ? LDX : ldx) + (lane >> 5) * 8;
  bf16x8 q[P][C], b[2][R];
  auto fetch = [&](int slot, int k) {
    k = k < steps ? k : steps - 1;   // (surplus loads are not used)
#pragma unroll
    for (int c = 0; c < C; ++c) q[slot][c] = w[c * ws + (int64_t)k * 64 + lane];
  };
  auto read = [&](int slot, int k) {
    k = k < steps ? k : steps - 1;
#pragma unroll
    for (int r = 0; r < R; ++r) b[slot][r] = *reinterpret_cast<const bf16x8*>(xr + r * 32 * (LDX ? LDX : ldx) + k * 16);
  };
#pragma unroll
  for (int u = 0; u < P; ++u) fetch(u, u);
  read(0, 0);
  constexpr int N = 2 * P;   // a multiple of both buffers' depths
  for (int k0 = 0; k0 < steps; k0 += N) {
#pragma unroll
    for (int u = 0; u < N; ++u) {
      if (k0 + u >= steps) break;   // uniform
      read((u + 1) & 1, k0 + u + 1);
#pragma unroll
      for (int c = 0; c < C; ++c)
#pragma unroll
        for (int r = 0; r < R; ++r)
          acc[c][r] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(q[u % P][c], b[u & 1][r], acc[c][r], 0, 0, 0);
      fetch(u % P, k0 + u + P);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

template <int C, int R>
__device__ __forceinline__ void fused_zero(floatx16 (&acc)[C][R]) {
#pragma unroll
  for (int c = 0; c < C; ++c)
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[c][r][i] = 0.0f;
}

// The output layer: each wave takes C3 column tiles and R3 row tiles per pass.  FEAT: the input is Tier 1 of the
// rows listed in a.rows (as standardize_rows_kernel), else a.xb.  RANK: each
// row's top n (outputs of 64 or 128 columns).
template <int R3, int C3, bool FEAT, bool RANK>
__global__ void __launch_bounds__(kFusedThreads) __attribute__((amdgpu_waves_per_eu(4)))
mlp_fused_kernel(const FusedArgs a) {
  constexpr int RT = kFusedTile / 32;
  extern __shared__ __align__(16) unsigned char smem[];
  __bf16* act = reinterpret_cast<__bf16*>(smem);   // input rows, then the hidden activations, then the output tile
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int col = lane & 31, h4 = (lane >> 5) * 4;
  const int64_t m0 = (int64_t)blockIdx.x * (32 * RT);
  const int ksteps = (a.in + 15) / 16, ldx = 16 * ksteps + 8;

  // ---- the input rows in LDS (rows past M repeat the last one) -------------
  if (FEAT) {
    // 16 lanes a row, 128 columns of every row in flight together
    const int l16 = tid & 15;
    bool bad = false;
    int64_t row[RT];
    float cy[RT];
#pragma unroll
    for (int p = 0; p < RT; ++p) {
      const int64_t m = m0 + p * 32 + (tid >> 4);
      row[p] = a.rows[m < a.M ? m : a.M - 1];
    }
#pragma unroll
    for (int p = 0; p < RT; ++p) cy[p] = a.cycles[row[p]];
    for (int j0 = 4 * l16; j0 < 16 * ksteps; j0 += 128) {
      float4 c[RT][2];
#pragma unroll
      for (int p = 0; p < RT; ++p)
#pragma unroll
        for (int q = 0; q < 2; ++q)   // (columns past the row re-read its first; not used)
          c[p][q] = *reinterpret_cast<const float4*>(a.counters + row[p] * a.in + (j0 + 64 * q < a.in ? j0 + 64 * q : 0));
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const int j = j0 + 64 * q;
        if (j >= 16 * ksteps) break;
        const int jm = j < a.in ? j : 0;
        const float4 mu = *reinterpret_cast<const float4*>(a.mu + jm), is = *reinterpret_cast<const float4*>(a.isg + jm);
        const float muv[4] = {mu.x, mu.y, mu.z, mu.w}, isv[4] = {is.x, is.y, is.z, is.w};
#pragma unroll
        for (int p = 0; p < RT; ++p) {
          const float lc = dlog<float>(cy[p]);
          const float cv[4] = {c[p][q].x, c[p][q].y, c[p][q].z, c[p][q].w};
          bf16x4 o;
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const float x = dlog<float>(cv[u]) - lc;
            bad |= j < a.in && !__builtin_isfinite(x);
            o[u] = j < a.in ? (__bf16)((x - muv[u]) * isv[u]) : (__bf16)0.0f;
          }
          *reinterpret_cast<bf16x4*>(act + (p * 32 + (tid >> 4)) * ldx + j) = o;
        }
      }
    }
    if (__ballot(bad) != 0 && lane == 0) atomicOr(a.status, (int)kStatusBadCounter);
  } else {
    const int vec = 2 * ksteps;   // 8 elements each
    for (int i = tid; i < 32 * RT * vec; i += kFusedThreads) {
      const int r = i / vec, k = (i - r * vec) * 8;
      const int64_t m = m0 + r < a.M ? m0 + r : a.M - 1;
      bf16x8 v;
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = (__bf16)0.0f;
      if (k < a.in) v = *reinterpret_cast<const bf16x8*>(a.xb + m * a.in + k);   // in is a multiple of 8
      *reinterpret_cast<bf16x8*>(act + r * ldx + k) = v;
    }
  }
  __syncthreads();

  // ---- hidden layers: wave w computes units 64 w .. 64 w + 63 of every row --
  floatx16 acc[2][RT];
  auto activate = [&](const float* __restrict__ bias) {
    float4 b[2][4];
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int g = 0; g < 4; ++g) b[c][g] = *reinterpret_cast<const float4*>(bias + wave * 64 + c * 32 + g * 8 + h4);
    __syncthreads();   // every wave is done with the layer's input
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const float bv[4] = {b[c][g].x, b[c][g].y, b[c][g].z, b[c][g].w};
          bf16x4 o;
#pragma unroll
          for (int u = 0; u < 4; ++u) o[u] = to_bf16(gelu_f(acc[c][r][4 * g + u] + bv[u]));
          *reinterpret_cast<bf16x4*>(act + (r * 32 + col) * kActLd + wave * 64 + c * 32 + g * 8 + h4) = o;
        }
    __syncthreads();
  };
  fused_zero(acc);
  fused_product<2, RT, 0>(acc, a.w1 + (int64_t)(2 * wave) * ksteps * 64, (int64_t)ksteps * 64, act, ldx, ksteps, lane);
  activate(a.b1);
  fused_zero(acc);
  fused_product<2, RT, kActLd>(acc, a.w2 + (int64_t)(2 * wave) * kHidSteps * 64, (int64_t)kHidSteps * 64, act, kActLd,
                               kHidSteps, lane);
  activate(a.b2);

  // ---- output layer -----------------------------------------------------------
  constexpr int RG = RT / R3, CG = kFusedWaves / RG;   // row groups, column groups of waves
  const int rg = wave % RG, cg = wave / RG;
  const int tiles = a.out / 32;
  const int ldy = a.out + 1;
  float* Ty = reinterpret_cast<float*>(smem);          // RANK: the output tile, over the activations
  for (int t0 = 0; t0 < tiles; t0 += CG * C3) {        // uniform; one pass where RANK
    const int ct = t0 + cg * C3;
    const bool live = ct < tiles;                      // uniform per wave (tiles is a multiple of C3)
    floatx16 y[C3][R3];
    fused_zero(y);
    if (live)
      fused_product<C3, R3, kActLd>(y, a.w3 + (int64_t)ct * kHidSteps * 64, (int64_t)kHidSteps * 64,
                                    act + rg * R3 * 32 * kActLd, kActLd, kHidSteps, lane);
    if (RANK) __syncthreads();   // the activations are no longer read
    if (live)
#pragma unroll
      for (int c = 0; c < C3; ++c)
#pragma unroll
        for (int r = 0; r < R3; ++r) {
          const int tr = (rg * R3 + r) * 32 + col;
          const int64_t m = m0 + tr;
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            const int n0 = (ct + c) * 32 + g * 8 + h4;
            const float4 b = *reinterpret_cast<const float4*>(a.b3 + n0);
            float4 v;
            v.x = y[c][r][4 * g] + b.x;
            v.y = y[c][r][4 * g + 1] + b.y;
            v.z = y[c][r][4 * g + 2] + b.z;
            v.w = y[c][r][4 * g + 3] + b.w;
            if (a.y && m < a.M) *reinterpret_cast<float4*>(a.y + m * a.out + n0) = v;
            if (RANK) {
              float* t = Ty + tr * ldy + n0;
              t[0] = v.x;
              t[1] = v.y;
              t[2] = v.z;
              t[3] = v.w;
            }
          }
        }
  }
  if (RANK) {
    // TPR threads per row, each a best-first list of its share of the columns
    __syncthreads();
    constexpr int TPR = kFusedThreads / (32 * RT);
    const int r = tid / TPR, part = tid % TPR, w = a.out / TPR;
    auto rank = [&](auto kt) {
      constexpr int KT = decltype(kt)::value;
      Entry<float> lst[KT];
#pragma unroll
      for (int i = 0; i < KT; ++i) lst[i] = empty_entry<float>();
      for (int c = part * w; c < (part + 1) * w; ++c) {
        const float v = Ty[r * ldy + c];
        if (c >= a.skip && v > a.tau) {
          Entry<float> e;
          e.v = v;
          e.s = c;
          list_insert<float, KT>(lst, e);
        }
      }
      group_merge<float, KT>(lst, TPR);
      if (part == 0 && m0 + r < a.M) write_list<float, KT>(lst, (int)(m0 + r), a.n, a.idx_out, a.score_out, a.count_out);
    };
    if (a.n <= 4) rank(std::integral_constant<int, 4>{});
    else rank(std::integral_constant<int, kMaxSuggest>{});
  }
}

namespace {

template <int R3, int C3, bool FEAT, bool RANK>
hipError_t launch_fused_t(const FusedArgs& a, hipStream_t s) {
  constexpr int RT = kFusedTile / 32;
  const size_t act = sizeof(__bf16) * 32 * RT * (size_t)std::max(kActLd, (a.in + 15) / 16 * 16 + 8);
  const size_t ty = RANK ? sizeof(float) * 32 * RT * (size_t)(a.out + 1) : 0;
  const size_t lds = std::max(act, ty);
  auto kern = mlp_fused_kernel<R3, C3, FEAT, RANK>;
  if (lds > 64 * 1024) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(kern, dim3((unsigned)((a.M + 32 * RT - 1) / (32 * RT))), dim3(kFusedThreads), lds, s, a);
  return hipSuccess;
}

template <bool FEAT, bool RANK>
hipError_t launch_fused_f(const FusedArgs& a, hipStream_t s) {
  if (RANK || a.out <= 128) return launch_fused_t<1, 1, FEAT, RANK>(a, s);
  if (a.out >= 512 && a.out % 64 == 0) return launch_fused_t<2, 2, FEAT, false>(a, s);   // two column tiles per wave
  return launch_fused_t<2, 1, FEAT, false>(a, s);
}

}  // namespace

hipError_t launch_mlp_fused(const FusedArgs& a, hipStream_t s) {
  if (a.M <= 0) return hipSuccess;
  if (a.in < 8 || a.in % 8 || a.in > 512 || a.out < 32 || a.out % 32)
    return hipErrorInvalidValue;
  if (a.idx_out && ((a.out != 64 && a.out != 128) || a.n < 1 || a.n > kMaxSuggest || a.skip < 0))
    return hipErrorInvalidValue;
  (void)hipGetLastError();  // report only this launch's status
  hipError_t e;
  if (a.counters) e = a.idx_out ? launch_fused_f<true, true>(a, s) : launch_fused_f<true, false>(a, s);
  else e = a.idx_out ? launch_fused_f<false, true>(a, s) : launch_fused_f<false, false>(a, s);
  return e != hipSuccess ? e : hipGetLastError();
}

}  // namespace sugg
