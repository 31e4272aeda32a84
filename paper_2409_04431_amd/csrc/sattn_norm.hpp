// Hybrid-norm for gfx950: LayerNorm / RMSNorm (no learnable affine parameters) of the attention
// output over the concatenated heads, forward and backward (Section 5.5, Appendix G.6:
// x + norm(sigmoid-attention); the norm alone is computed here).
//
// Token (b, n) owns H*d features spread over the H head slices of a [B,H,N,d] tensor with
// arbitrary batch/head/token strides.  The work is one read and one write of the tensor (the
// backward reads two), i.e. HBM-bound: one wave per token keeps the whole row in registers
// (CPL 16-byte chunks per lane), so statistics and normalisation need no second pass over
// memory; the variance is the two-pass one (around the mean), in fp32.  A fused epilogue in
// the attention kernel is not possible: a workgroup there owns one head, the statistics span
// all heads.  Rows of up to 16 or 32 chunks share a wave four or two at a time.
// What it takes besides the bytes: every load of a token issued before the first is waited for, and
// non-temporal stores, which leave the inputs in the caches.  B8 H16 N4096 d128, forward + backward
// alternating: 126.0 -> 117.4 us (671 MB, 5.7 TB/s; a library's elementwise product over 1 GiB reaches
// 6.3, over a tensor of this size, which the caches hold, 7.5); H2 d128 of 30345 tokens, two to a wave,
// 26.5 -> 14.4.
// What the next kernel pays for non-temporal stores (us per chain, non-temporal / plain): write x, forward,
// residual 16 MiB 22.7 / 23.4, 64 MiB 72.0 / 72.2, 128 MiB 161 / 175, 512 MiB 689 / 682; write dy,
// backward, read dx 23.4 / 23.8, 84.2 / 84.0, 157 / 170, 726 / 722; equal up to 8 MiB.  Between attention and
// matrix products, forward and backward, 6 to 256 MiB: within 1 % either way.  They lose where x is
// in the caches already and nothing but the output is read next (128 MiB 95 / 88).
#pragma once
#include "sattn_common.hpp"

namespace sattn {

struct NormParams {
  TensorRef x, y;    // forward: input, output.  backward: x = forward input, y = dx
  TensorRef dy;      // backward only
  float* stats;      // [B, N, 2]: mean (0 for RMSNorm), 1/sqrt(var + eps); written by forward, read by backward
  int B, H, N, d;
  float eps;
};

// sum over groups of L consecutive lanes
template <int L>
__device__ __forceinline__ float group_sum(float v) {
#pragma unroll
  for (int m = L / 2; m >= 1; m >>= 1) v += __shfl_xor(v, m);
  return v;
}

// element pointer of 16-byte chunk c (8 bf16) of token (b, n)
__device__ __forceinline__ const __bf16* chunk_ptr(const TensorRef& t, int b, int n, int c, int cpr) {
  const int h = c / cpr, o = (c % cpr) * 8;
  return (const __bf16*)t.ptr + b * t.sb + h * t.sh + (int64_t)n * t.ss + o;
}

// L lanes per token, CPL chunks per lane (L * CPL chunks at least; L < 64 only with CPL = 1).
template <int CPL, int L, bool RMS, bool BACKWARD>
__global__ void __launch_bounds__(256)
headconcat_norm_kernel(const NormParams p) {
  const int lane = threadIdx.x & (L - 1);
  const int64_t token = (int64_t)blockIdx.x * (256 / L) + threadIdx.x / L;
  if (token >= (int64_t)p.B * p.N) return;  // whole group
  const int b = (int)(token / p.N), n = (int)(token % p.N);
  const int cpr = p.d / 8, nchunks = p.H * cpr;
  const float inv_f = 1.0f / (float)(p.H * p.d);

  // everything the token needs is requested before the first value is looked at
  u32x4 xr[CPL], gr[BACKWARD ? CPL : 1];
#pragma unroll
  for (int i = 0; i < CPL; ++i) {
    const int c = lane + L * i;
    xr[i] = u32x4{0, 0, 0, 0};
    if (BACKWARD) gr[i] = u32x4{0, 0, 0, 0};
    if (c < nchunks) {
      xr[i] = *(const u32x4*)chunk_ptr(p.x, b, n, c, cpr);
      if (BACKWARD) gr[i] = *(const u32x4*)chunk_ptr(p.dy, b, n, c, cpr);
    }
  }
  float xv[CPL][8];
#pragma unroll
  for (int i = 0; i < CPL; ++i) {
    const bf16x8 v = as_bf16x8(xr[i]);
#pragma unroll
    for (int e = 0; e < 8; ++e) xv[i][e] = (float)v[e];
  }

  float mean, rstd;
  if (!BACKWARD) {
    mean = 0.f;
    if (!RMS) {
      float s = 0.f;
#pragma unroll
      for (int i = 0; i < CPL; ++i)
#pragma unroll
        for (int e = 0; e < 8; ++e) s += xv[i][e];
      mean = group_sum<L>(s) * inv_f;
    }
    float q = 0.f;
#pragma unroll
    for (int i = 0; i < CPL; ++i)
      if (lane + L * i < nchunks) {
#pragma unroll
        for (int e = 0; e < 8; ++e) q = __builtin_fmaf(xv[i][e] - mean, xv[i][e] - mean, q);
      }
    // hardware reciprocal square root plus one Newton step (the statistics are kept for the
    // backward pass)
    const float a = group_sum<L>(q) * inv_f + p.eps;
    rstd = __builtin_amdgcn_rsqf(a);
    rstd = rstd * (1.5f - 0.5f * a * rstd * rstd);
    if (lane == 0) {
      p.stats[2 * token] = mean;
      p.stats[2 * token + 1] = rstd;
    }
#pragma unroll
    for (int i = 0; i < CPL; ++i) {
      const int c = lane + L * i;
      if (c < nchunks) {
        u32x4 w;
#pragma unroll
        for (int e = 0; e < 4; ++e)
          w[e] = pack_bf16((xv[i][2 * e] - mean) * rstd, (xv[i][2 * e + 1] - mean) * rstd);
        __builtin_nontemporal_store(w, (u32x4*)const_cast<__bf16*>(chunk_ptr(p.y, b, n, c, cpr)));
      }
    }
  } else {
    mean = p.stats[2 * token];
    rstd = p.stats[2 * token + 1];
    // dx = rstd * (dy - mean_f(dy) [LayerNorm only] - xhat * mean_f(dy * xhat))
    float gv[CPL][8];
    float sg = 0.f, sgy = 0.f;
#pragma unroll
    for (int i = 0; i < CPL; ++i) {
      const int c = lane + L * i;
      if (c < nchunks) {
        const bf16x8 v = as_bf16x8(gr[i]);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          gv[i][e] = (float)v[e];
          xv[i][e] = (xv[i][e] - mean) * rstd;  // xhat
          sg += gv[i][e];
          sgy = __builtin_fmaf(gv[i][e], xv[i][e], sgy);
        }
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) gv[i][e] = 0.f;
      }
    }
    const float mg = RMS ? 0.f : group_sum<L>(sg) * inv_f;
    const float mgy = group_sum<L>(sgy) * inv_f;
#pragma unroll
    for (int i = 0; i < CPL; ++i) {
      const int c = lane + L * i;
      if (c < nchunks) {
        u32x4 w;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float a0 = (gv[i][2 * e] - mg - xv[i][2 * e] * mgy) * rstd;
          const float a1 = (gv[i][2 * e + 1] - mg - xv[i][2 * e + 1] * mgy) * rstd;
          w[e] = pack_bf16(a0, a1);
        }
        __builtin_nontemporal_store(w, (u32x4*)const_cast<__bf16*>(chunk_ptr(p.y, b, n, c, cpr)));
      }
    }
  }
}

}  // namespace sattn
