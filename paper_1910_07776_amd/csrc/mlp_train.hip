// The training step's output layer and the backward through it in one launch,
// for the hidden width 512 and 64 or 128 outputs: a workgroup takes 32 rows
// through Y = H2 W3^T + b3, the squared error and dY, and half of dA2 = (dY
// W3) * gelu'(A2) (two workgroups form the same Y).
//
// Every sum is formed as by the separate products (K ascending in steps of 16
// of v_mfma_f32_32x32x16_bf16, the squared errors per 32 x 32 tile in the same
// lanes), so outputs and loss are the same bits.  Bound by latency: 256
// workgroups at the batch 4096, each a chain of loads, 32 dependent matrix
// instructions, the GELU's derivative and stores; everything the later phases
// read is therefore requested before the first.  As two launches (64
// workgroups of 64 rows, then the backward paired with dW3) it took 13.9 + 9.9
// us; with one workgroup for all of dA2 13.4, now 10.7, and dW3 shares dW1's launch.
#include <hip/hip_runtime.h>

#include "kernels.hpp"
#include "mlp_math.hpp"

namespace sugg {

constexpr int kOutRows = 32, kOutThreads = 512;
constexpr int kOutLd = kFusedHidden + 8;   // LDS row of 512 elements: 16-byte reads of 32 rows spread over the banks

template <int OUT>
__global__ void __launch_bounds__(kOutThreads) out_backward_kernel(const OutBackwardArgs a) {
  constexpr int H = kFusedHidden, DLD = OUT + 8, YW = OUT / 32;   // YW waves form Y, a 32 x 32 tile each
  constexpr int P = 8;                                            // steps of W3 in flight
  constexpr int HW = H / 2;                                       // hidden units of a workgroup, 32 a wave
  __shared__ __align__(16) __bf16 X[kOutRows * kOutLd];           // H2 rows, then dA2
  __shared__ __align__(16) __bf16 D[kOutRows * DLD];              // dY
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, col = lane & 31, hi = lane >> 5;
  const int m0 = blockIdx.x * kOutRows, h0 = blockIdx.y * HW;   // rows; hidden units of dA2
  const int mr = a.M - m0;   // valid rows from here (may be <= 0 in the last 64-row tile's second half)
  auto tile_row = [&](int r) { return (r >> 2) * 8 + hi * 4 + (r & 3); };
  auto clamped = [&](int tr) { return m0 + tr < a.M ? m0 + tr : a.M - 1; };

  // ---- requests, in the order of use (rows past M repeat the last one) ------
  bf16x8 x[4];
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int i = tid + kOutThreads * v;
    x[v] = *reinterpret_cast<const bf16x8*>(a.h2 + (int64_t)clamped(i / (H / 8)) * H + (i % (H / 8)) * 8);
  }
  const bool yw = wave < YW;   // uniform per wave
  const __bf16* w3 = a.w3 + (int64_t)((yw ? wave : 0) * 32 + col) * H + hi * 8;
  bf16x8 q[P];
  float t[16], b3 = 0.0f;
  if (yw) {
    int64_t src[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      src[r] = clamped(tile_row(r));
      if (a.trow) src[r] = a.trow[src[r]];
    }
#pragma unroll
    for (int u = 0; u < P; ++u) q[u] = *reinterpret_cast<const bf16x8*>(w3 + u * 16);
    b3 = a.b3[wave * 32 + col];
#pragma unroll
    for (int r = 0; r < 16; ++r) t[r] = a.target[src[r] * OUT + wave * 32 + col];
  }
  const int nl = wave * 32 + col;   // this lane's hidden unit, from h0
  float pre[16];
  bf16x8 wt[OUT / 16];
#pragma unroll
  for (int s = 0; s < OUT / 16; ++s)
    wt[s] = *reinterpret_cast<const bf16x8*>(a.w3t + (int64_t)(h0 + nl) * OUT + s * 16 + hi * 8);
#pragma unroll
  for (int r = 0; r < 16; ++r) pre[r] = a.a2[(int64_t)clamped(tile_row(r)) * H + h0 + nl];
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int i = tid + kOutThreads * v;
    *reinterpret_cast<bf16x8*>(X + (i / (H / 8)) * kOutLd + (i % (H / 8)) * 8) = x[v];
  }
  __syncthreads();

  // ---- Y, the squared errors, dY -----------------------------------------------
  if (yw) {
    floatx16 acc;
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = 0.0f;
#pragma unroll
    for (int s = 0; s < H / 16; ++s) {
      const bf16x8 f = *reinterpret_cast<const bf16x8*>(X + col * kOutLd + s * 16 + hi * 8);
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, q[s % P], acc, 0, 0, 0);
      if (s + P < H / 16) q[s % P] = *reinterpret_cast<const bf16x8*>(w3 + (s + P) * 16);
    }
    float sse = 0.0f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int tr = tile_row(r);
      const float y = acc[r] + b3;
      const float d = y - t[r];
      if (tr < mr) sse = fmaf(d, d, sse);
      D[tr * DLD + wave * 32 + col] = to_bf16(a.scale * d);
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) sse += __shfl_xor(sse, off, 64);
    // the four 32 x 32 parts of each 64 x 64 tile
    if (lane == 0 && h0 == 0)
      a.loss_part[((m0 / 64) * (OUT / 64) + wave / 2) * 4 + ((m0 / 32) & 1) * 2 + (wave & 1)] = sse;
  }
  __syncthreads();
  if (mr <= 0) return;   // uniform

  auto store = [&](const __bf16* T, int ld, int cols, __bf16* rowm, int ldr, __bf16* colm) {
    for (int v = tid; v < kOutRows * (cols / 8); v += kOutThreads) {
      const int r = v / (cols / 8), c = (v % (cols / 8)) * 8;
      if (r < mr)
        *reinterpret_cast<bf16x8*>(rowm + (int64_t)(m0 + r) * ldr + c) = *reinterpret_cast<const bf16x8*>(T + r * ld + c);
    }
    for (int v = tid; v < cols * (kOutRows / 8); v += kOutThreads) {
      const int c = v / (kOutRows / 8), r = (v % (kOutRows / 8)) * 8;
      __bf16* dst = colm + (int64_t)c * a.ldt + m0 + r;   // ldt and m0 + r: multiples of 8
      bf16x8 o;
#pragma unroll
      for (int i = 0; i < 8; ++i) o[i] = T[(r + i) * ld + c];
      if (r + 8 <= mr) *reinterpret_cast<bf16x8*>(dst) = o;
      else
#pragma unroll
        for (int i = 0; i < 8; ++i)
          if (r + i < mr) dst[i] = o[i];
    }
  };

  // ---- dA2 -----------------------------------------------------------------------
  floatx16 g;
#pragma unroll
  for (int i = 0; i < 16; ++i) g[i] = 0.0f;
#pragma unroll
  for (int s = 0; s < OUT / 16; ++s) {
    const bf16x8 f = *reinterpret_cast<const bf16x8*>(D + col * DLD + s * 16 + hi * 8);
    g = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, wt[s], g, 0, 0, 0);
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) X[tile_row(r) * kOutLd + nl] = to_bf16(g[r] * gelu_grad_f(pre[r]));
  if (h0 == 0) store(D, DLD, OUT, a.dy, OUT, a.dyt);
  __syncthreads();
  store(X, kOutLd, HW, a.da2 + h0, H, a.da2t + (int64_t)h0 * a.ldt);
}

hipError_t launch_out_backward(const OutBackwardArgs& a, int out, hipStream_t s) {
  if (a.M <= 0) return hipSuccess;
  if ((out != 64 && out != 128) || a.ldt % 8 || a.ldt < a.M) return hipErrorInvalidValue;
  const dim3 grid((a.M + 63) / 64 * 2, 2);   // every part of every 64-row tile's loss is written
  (void)hipGetLastError();  // report only this launch's status
  if (out == 64) hipLaunchKernelGGL(out_backward_kernel<64>, grid, dim3(kOutThreads), 0, s, a);
  else hipLaunchKernelGGL(out_backward_kernel<128>, grid, dim3(kOutThreads), 0, s, a);
  return hipGetLastError();
}

}  // namespace sugg
