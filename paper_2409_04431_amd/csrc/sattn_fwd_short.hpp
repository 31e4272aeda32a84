// Sigmoid-attention forward of sequences that one workgroup holds whole: up to 256 keys at d = 64, 128
// at d = 128 (bf16, no ALiBi).
//
// The kernels of sattn_fwd.hpp stream K and V through rings of 64-row tiles behind a three-stage
// pipeline, whose start and end a loop of one to four tiles does not repay.  Here K and V are in LDS
// once and for all, a wave owns 32 queries and goes through the keys without a barrier: S^T = K Q^T,
// P^T, O^T += V^T P^T in the order of those kernels, bit-equal to them.  No pipeline inside a wave
// keeps it at 84 to 100 registers (d = 64), so that four waves share a SIMD and hide each other's waits.
//
// What bounds it: up to 128 keys the memory (1024 heads of 64 tokens d 64: 67 MB in 6.7 us with the
// launch), at 250 vector issue and the first loads.  Measured (us, the choice among the kernels of sattn_fwd.hpp / this):
// d 64 1024 heads N64 10.4 / 7.2, N128 19.3 / 14.3, N250 37.9 / 36.6 (causal 32.8 / 29.0), 384 heads N128 8.9 / 7.5,
// N250 17.6 / 17.5 (causal 16.5 / 14.9), 16 heads N128 6.2 / 5.2; d 128 2048 heads N64 33.2 / 24.9, 1024 N100 26.8 / 23.3,
// 16 heads N128 8.3 / 6.6.
#pragma once
#include "sattn_bwd_short.hpp"
#include "sattn_fwd.hpp"

namespace sattn {

template <int D, int NW, bool CAUSAL>
__global__ void __launch_bounds__(64 * NW, D == 64 ? 4 : 2) attn_fwd_short_kernel(const FwdParams p) {
  constexpr int KD = D / 16, DT = D / 32, TILE = 64 * D * 2, SLOT = 2 * TILE;
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const uint32_t lds0 = (uint32_t)(uintptr_t)(SATTN_LDS(char)*)smem;
  ClockStart clk = clock_probe_begin(p.clock);
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  ShortHead hd;
  hd.b = blockIdx.x / p.H;
  hd.hd = blockIdx.x - hd.b * p.H;
  hd.N = p.N;
  hd.tok0 = 0;
  hd.nbias = p.nbias_log2;
  if (p.cu_seqlens) {
    hd.tok0 = p.cu_seqlens[hd.b];
    hd.N = min(p.cu_seqlens[hd.b + 1] - (int)hd.tok0, p.N);
    if (p.bias_vec) hd.nbias = -p.bias_vec[hd.b] * kLog2e;
    if (hd.N <= 0) return;
  }
  const int N = hd.N, n_tiles = (N + 63) / 64, n_chunks = (N + 31) / 32;
  {
    DmaStagerX<D, NW> sk, sv;
    sk.init(hd.of(p.k), p.k.ss, N, 0, wave, lane);
    sv.init(hd.of(p.v), p.v.ss, N, 0, wave, lane);
    for (int t = 0; t < n_tiles; ++t) {
      sk.issue(lds0 + t * SLOT, N, wave, lane);
      sv.issue(lds0 + t * SLOT + TILE, N, wave, lane);
    }
  }
  const int qblk = short_query_block<NW, CAUSAL>(wave, n_chunks), q0 = 32 * qblk, q_ld = min(q0 + l32, N - 1);
  const __bf16* qb = hd.of(p.q);
  bf16x8 x1[KD];
#pragma unroll
  for (int kk = 0; kk < KD; ++kk) x1[kk] = as_bf16x8(*(const u32x4*)(qb + (int64_t)q_ld * p.q.ss + 16 * kk + 8 * h));
  f32x16 o[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[dt][r] = 0.f;
  ShortLanes<D> at_lane;
  at_lane.init(lane);
  SATTN_WAIT_VMCNT(0);
  __syncthreads();
  clock_probe_mark(p.clock, clk, kMarkFirstProduct);
  if (n_tiles * 64 > N) {  // keys past the end weigh nothing
    short_pad<D, NW>(lds0 + (n_tiles - 1) * SLOT + TILE, n_tiles - 1, N, tid);
    __syncthreads();
  }
  const int c_hi = q0 < N ? (CAUSAL ? qblk + 1 : n_chunks) : 0;
  clk.steady_tiles = (c_hi + 1) / 2;
  clock_probe_mark(p.clock, clk, kMarkSteadyBegin);
#pragma nounroll
  for (int c = 0; c < c_hi; ++c) {
    const uint32_t at = lds0 + (c >> 1) * SLOT + (c & 1) * (32 * D * 2);
    f32x16 s;
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] = 0.f;
#pragma unroll
    for (int kk = 0; kk < KD; ++kk) s = mfma32(as_bf16x8(lds_read_b128(at + at_lane.row[kk])), x1[kk], s);
    float w[16];
#pragma unroll
    for (int r = 0; r < 16; ++r)
      w[r] = __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(__builtin_fmaf(s[r], p.nscale_log2, hd.nbias)));
    if (CAUSAL && c == qblk) {
#pragma unroll
      for (int r = 0; r < 16; ++r) w[r] = key_of_reg(r) + 8 * h <= l32 ? w[r] : 0.f;
    }
    const bf16x8 pb[2] = {pack8(w), pack8(w + 8)};
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
        const uint32_t off = at + TILE + ks * 16 * (D * 2);
        o[dt] = mfma32(join_tr(lds_read_tr16(off + at_lane.tr[dt][0]), lds_read_tr16(off + at_lane.tr[dt][1])), pb[ks], o[dt]);
      }
  }
  clock_probe_mark(p.clock, clk, kMarkSteadyEnd);
  __syncthreads();
  clock_probe_mark(p.clock, clk, kMarkStore);
  RowStore<D>::run(o, 1.0f, lds0 + wave * RowStore<D>::BYTES, lane, hd.of(p.o) + (int64_t)q0 * p.o.ss, p.o.ss, N - q0);
  clk.tiles = n_tiles;
  clock_probe_end(p.clock, clk, (int)blockIdx.x);
}

template <int D>
int launch_fwd_short(const FwdParams& p, int causal, hipStream_t st) {
  const dim3 grid(p.B * p.H);
  constexpr size_t per = 2 * 32 * D * 2;  // LDS of a wave's 32 keys
  static_assert(RowStore<D>::BYTES <= per, "outputs leave through the same LDS");
  if constexpr (D == 64) {
    if (p.N > 128)
      return causal ? launch(attn_fwd_short_kernel<D, 8, true>, grid, dim3(512), 8 * per, st, p)
                    : launch(attn_fwd_short_kernel<D, 8, false>, grid, dim3(512), 8 * per, st, p);
  }
  return causal ? launch(attn_fwd_short_kernel<D, 4, true>, grid, dim3(256), 4 * per, st, p)
                : launch(attn_fwd_short_kernel<D, 4, false>, grid, dim3(256), 4 * per, st, p);
}

}  // namespace sattn
