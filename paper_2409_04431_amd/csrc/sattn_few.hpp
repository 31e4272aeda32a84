// Sigmoid-attention forward for gfx950 when few queries meet many keys (new tokens at the end of a
// sequence whose keys and values are already there), bf16 operands, fp32 logits / sigmoid /
// accumulation; the arithmetic per pair is that of sattn_fwd.hpp.
//
// What bounds it: reading K and V once (one query per head makes 2 flops per byte).  The other
// forward kernels give a workgroup 128 or 256 query rows and walk the keys in one go, so a few
// queries make a few workgroups of one busy wave each.  Here a workgroup owns 32 query rows and
// its NW waves deal the 32-key chunks out among themselves; where heads are few, n_split
// workgroups share them as well.  Sigmoid attention has no normaliser, so partial outputs
// simply add: the waves' through LDS, the workgroups' through an fp32 workspace and
// few_partials_reduce_kernel, both in a fixed order (bit-reproducible).
//
// Every wave streams on its own, without barriers: K goes from memory straight into the A
// fragments of S^T = K Q^T, V as whole rows into registers and from there through the wave's
// private LDS to the transposing read that O^T += V^T P^T needs.  A register is refilled with the
// next chunk as soon as it has been consumed, so that a wave keeps up to a whole chunk (16 KB at
// d = 128) in flight.  MFMA use is wasteful with one query (one column of 32) and still takes
// less than a tenth of the time the chunk takes to arrive.
// Measured on one MI355X (us, the 128-row kernel -> this one with its reduction): one query, 4001
// keys, d 128, 128 heads with ALiBi 79 -> 50 (262 MB; 40 of it stream them, 6.6 TB/s), 16 heads 61 ->
// 14; one query, 32768 keys, 8 heads 468 -> 33; 64 queries, 8256 keys, 16 heads 125 -> 23; one
// query, 244 keys 7.0 -> 5.4.
#pragma once
#include "sattn_fwd.hpp"

namespace sattn {

// LDS of a workgroup: every wave's V chunk during the loop, the waves' fp32 partial outputs (rows
// padded by 16 bytes) at the end.
template <int D>
constexpr size_t few_lds_bytes(int nw) { return (size_t)nw * 32 * (D + 4) * sizeof(float); }

template <int D, bool CAUSAL, bool ALIBI, int NW>
__global__ void __launch_bounds__(64 * NW, 2)
attn_fwd_few_kernel(const FwdParams p) {
  constexpr int KD = D / 16, DT = D / 32, CPR = D / 8, RPI = 64 / CPR, NV = 32 / RPI, LDX = D + 4, NT = 64 * NW;
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  ClockStart clk = clock_probe_begin(p.clock);

  // place -> (head, key split, query block): the query blocks of a split run next to each other
  // on one XCD and share its keys
  const int place = xcd_remap(blockIdx.x, p.n_qblocks * p.n_split * p.B * p.H);
  const int qb = place % p.n_qblocks, sp = (place / p.n_qblocks) % p.n_split, bh = place / (p.n_qblocks * p.n_split);
  const int b = bh / p.H, hd = bh % p.H, hkv = hd / p.kv_group;
  const int N = p.N, Nk = p.Nk > 0 ? p.Nk : N;
  const int q0 = qb * 32, rows = N - q0 < 32 ? N - q0 : 32;
  const char* const kb = (const char*)((const __bf16*)p.k.ptr + b * p.k.sb + hkv * p.k.sh);
  const char* const vb = (const char*)((const __bf16*)p.v.ptr + b * p.v.sb + hkv * p.v.sh);
  const __bf16* const qbase = (const __bf16*)p.q.ptr + b * p.q.sb + hd * p.q.sh;

  int kv_len = Nk;
  if (CAUSAL) {  // keys visible to the block's last query
    const int kv = q0 + rows + p.qoff;
    kv_len = kv < 0 ? 0 : (kv < Nk ? kv : Nk);
  }
  const int n_chunks = (kv_len + 31) / 32, stride = NW * p.n_split;

  // per-lane byte offsets inside a head (the host checked that they fit 32 bits); rows past the
  // end re-read the last one (their weights are zero)
  const uint32_t ks = (uint32_t)p.k.ss * 2u, vs = (uint32_t)p.v.ss * 2u;
  const uint32_t klast = (uint32_t)(Nk - 1) * ks, vlast = (uint32_t)(Nk - 1) * vs;
  const int kap = kappa(l32), vrow = lane / CPR, vcol = lane % CPR;
  u32x4 kf[KD], vr[NV];
  auto load_k = [&](int c) {
    uint32_t o = (uint32_t)(32 * c + kap) * ks;
    o = (o < klast ? o : klast) + 16 * h;
#pragma unroll
    for (int kk = 0; kk < KD; ++kk) kf[kk] = *(const u32x4*)(kb + (size_t)(o + 32 * kk));
  };
  auto load_v = [&](int c) {
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      uint32_t o = (uint32_t)(32 * c + RPI * i + vrow) * vs;
      o = (o < vlast ? o : vlast) + 16 * vcol;
      vr[i] = *(const u32x4*)(vb + (size_t)o);
    }
  };
  int c = sp * NW + wave;
  if (c < n_chunks) { load_k(c); load_v(c); }

  bf16x8 qf[KD];
  {
    const int qi_ld = l32 < rows ? q0 + l32 : q0 + rows - 1;
#pragma unroll
    for (int kk = 0; kk < KD; ++kk) qf[kk] = as_bf16x8(*(const u32x4*)(qbase + (int64_t)qi_ld * p.q.ss + 16 * kk + 8 * h));
  }
  const uint32_t lds0 = (uint32_t)(uintptr_t)(SATTN_LDS(char)*)smem;
  const uint32_t vbuf = lds0 + wave * (32 * D * 2);
  uint32_t vw[NV], voff[DT];
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int r = RPI * i + vrow;
    vw[i] = vbuf + r * (D * 2) + ((vcol ^ Swz<D>::v(r)) << 4);
  }
  {
    const int i16 = lane & 15, blk1 = (lane >> 4) & 1, row = 8 * h + (i16 >> 2);
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
      const int cc = 4 * dt + 2 * blk1 + ((i16 & 3) >> 1);
      voff[dt] = vbuf + row * (D * 2) + ((cc ^ Swz<D>::v(row)) << 4) + ((i16 & 1) << 3);
    }
  }
  const int qpos = q0 + l32 + p.qoff;  // this lane's query's place on the key axis
  const float sl2 = ALIBI ? p.slopes[hd] * kLog2e : 0.f;
  f32x16 oacc[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int r = 0; r < 16; ++r) oacc[dt][r] = 0.f;

  clk.tiles = clk.steady_tiles = c < n_chunks ? (n_chunks - 1 - c) / stride + 1 : 0;  // (the wave's chunks)
  clock_probe_mark(p.clock, clk, kMarkFirstProduct);
  clock_probe_mark(p.clock, clk, kMarkSteadyBegin);
  for (; c < n_chunks; c += stride) {
    const int nxt = c + stride < n_chunks ? c + stride : c;
    f32x16 s;
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] = 0.f;
#pragma unroll
    for (int kk = 0; kk < KD; ++kk) s = mfma32(as_bf16x8(kf[kk]), qf[kk], s);
    __builtin_amdgcn_sched_barrier(0);
    load_k(nxt);
    // the reads of the previous chunk were consumed by its MFMAs; a wave's LDS accesses stay in order
#pragma unroll
    for (int i = 0; i < NV; ++i) lds_write_b128(vw[i], vr[i]);
    asm volatile("" ::: "memory");
    load_v(nxt);
    __builtin_amdgcn_sched_barrier(0);
    const int jl = 32 * c + 8 * h;  // key held by register 0 of this lane half
    const float dist0 = ALIBI ? (float)(qpos - jl) : 0.f;
    float pr[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      float w = p.nbias_log2;
      if (ALIBI) w = __builtin_fmaf(sl2, __builtin_fabsf(dist0 - (float)key_of_reg(r)), w);
      pr[r] = __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(__builtin_fmaf(s[r], p.nscale_log2, w)));
    }
    if (32 * c + 32 > Nk || (CAUSAL && 32 * c + 31 > q0 + p.qoff)) {  // wave-uniform
      int lim = Nk - 1 - jl;
      if (CAUSAL) lim = lim < qpos - jl ? lim : qpos - jl;
#pragma unroll
      for (int r = 0; r < 16; ++r) pr[r] = key_of_reg(r) <= lim ? pr[r] : 0.f;
    }
    bf16x8 pt[2];
#pragma unroll
    for (int ks2 = 0; ks2 < 2; ++ks2) {
      u32x4 w;
#pragma unroll
      for (int j = 0; j < 4; ++j) w[j] = pack_bf16(pr[8 * ks2 + 2 * j], pr[8 * ks2 + 2 * j + 1]);
      pt[ks2] = as_bf16x8(w);
    }
#pragma unroll
    for (int ks2 = 0; ks2 < 2; ++ks2)
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
        const uint32_t a = voff[dt] + ks2 * 16 * (D * 2);
        oacc[dt] = mfma32(join_tr(lds_read_tr16(a), lds_read_tr16(a + 4 * (D * 2))), pt[ks2], oacc[dt]);
      }
    asm volatile("" ::: "memory");
  }

  clock_probe_mark(p.clock, clk, kMarkSteadyEnd);
  // ---- partial outputs: register 4g+t of tile dt is O[q0 + l32][32dt + 8g + 4h + t]
  __syncthreads();
  float* const parts = (float*)smem;
  if (l32 < rows) {
    float* const row = parts + (wave * 32 + l32) * LDX + 4 * h;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int g = 0; g < 4; ++g)
        *(f32x4*)(row + 32 * dt + 8 * g) =
            f32x4{oacc[dt][4 * g], oacc[dt][4 * g + 1], oacc[dt][4 * g + 2], oacc[dt][4 * g + 3]};
  }
  __syncthreads();
  clock_probe_mark(p.clock, clk, kMarkStore);
  for (int idx = tid; idx < rows * (D / 8); idx += NT) {
    const int r = idx / (D / 8), cc = idx % (D / 8);
    f32x4 lo = {0.f, 0.f, 0.f, 0.f}, hi = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float* src = parts + (w * 32 + r) * LDX + 8 * cc;
      const f32x4 x = *(const f32x4*)src, y = *(const f32x4*)(src + 4);
#pragma unroll
      for (int e = 0; e < 4; ++e) { lo[e] += x[e]; hi[e] += y[e]; }
    }
    if (p.n_split > 1) {
      float* dst = p.part + (((int64_t)sp * p.B * p.H + bh) * N + q0 + r) * D + 8 * cc;
      *(f32x4*)dst = lo;
      *(f32x4*)(dst + 4) = hi;
    } else {
      u32x4 w;
      w[0] = pack_bf16(lo[0], lo[1]); w[1] = pack_bf16(lo[2], lo[3]);
      w[2] = pack_bf16(hi[0], hi[1]); w[3] = pack_bf16(hi[2], hi[3]);
      *(u32x4*)((__bf16*)p.o.ptr + b * p.o.sb + hd * p.o.sh + (int64_t)(q0 + r) * p.o.ss + 8 * cc) = w;
    }
  }
  clock_probe_end(p.clock, clk);
}

// O = sum of the splits' partial outputs, rounded to bf16 once.  One thread per four features.
template <int D>
__global__ void __launch_bounds__(256)
few_partials_reduce_kernel(const float* part, TensorRef o, int n_split, int B, int H, int N) {
  const int64_t slab = (int64_t)B * H * N * D, e0 = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
  if (e0 >= slab) return;
  f32x4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
  for (int s = 0; s < n_split; ++s) {
    const f32x4 x = *(const f32x4*)(part + (int64_t)s * slab + e0);
#pragma unroll
    for (int e = 0; e < 4; ++e) sum[e] += x[e];
  }
  const int64_t row = e0 / D;
  const int i = (int)(row % N), bh = (int)(row / N);
  u32x2 w;
  w[0] = pack_bf16(sum[0], sum[1]);
  w[1] = pack_bf16(sum[2], sum[3]);
  *(u32x2*)((__bf16*)o.ptr + (bh / H) * o.sb + (bh % H) * o.sh + (int64_t)i * o.ss + (int)(e0 % D)) = w;
}

}  // namespace sattn
