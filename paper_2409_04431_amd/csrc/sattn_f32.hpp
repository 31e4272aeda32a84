// fp32 sigmoid attention for gfx950: forward and the two backward passes in one template.
// Everything (operands, logits, sigmoid, accumulation, outputs) is fp32; the matrix
// products run on the fp32 MFMA (32x32x2), exp is the accurate one and the reciprocal is
// refined to full precision.  This is the precision path (agreement with the fp64 oracle to
// ~1e-6); the bf16 kernels are the throughput path.
//
// A workgroup owns 32 rows of the stationary side, kept in LDS, and its NW waves deal the
// 32-row chunks of the streamed side out among themselves (wave w takes chunks w, w+NW, ...):
//   FWD  : stationary Q          | stream K,V  : S^T = K Q^T, P^T, O^T += V^T P^T
//   DQ   : stationary Q, dO      | stream K,V  : S^T, dP^T = V dO^T, dS^T, dQ^T += K^T dS^T
//   DKDV : stationary K, V       | stream Q,dO : S = Q K^T, dP = dO V^T, dV^T += dO^T P, dK^T += Q^T dS
// (Algorithms 1 and 2 of the paper's Appendix F.1; the backward is split by output owner.)
// Sigmoid attention has no normaliser, so the waves' partial outputs simply add; they do so
// through LDS in a fixed order at the end (bit-reproducible).
//
// What bounds it: the fp32 matrix pipe.  An MFMA takes 64 cycles there and needs 4 bytes per lane
// of streamed operand, so a wave can fetch that operand from the L2 straight into registers, in
// the layouts the two products want, and needs no staging through LDS and no barrier in its
// loop.  Splitting the streamed side over the waves instead of giving each wave stationary rows
// of its own makes four (eight) times as many workgroups of a quarter (an eighth) of the length,
// which is what small problems and the causal triangle need.  Measured on one MI355X, us, forward + both
// backward passes, against a kernel whose four waves own 128 stationary rows and share 32-row
// tiles through LDS between two barriers (the passes as two launches):
//   B1 H2 N256 d64            35 + 106 -> 11 + 18        (latency: 16 and 32 workgroups)
//   B2 H8 N1000 d128 causal  216 + 627 -> 47 + 143
//   B4 H12 N1024 d64         206 + 700 -> 126 + 397
//   B1 H8 N2048 d128         421 + 1211 -> 144 + 465     (119 TFLOP/s forward, 129 over the seven
//                            backward products; a library product of two 4096^2 matrices runs at
//                            132 on this card, of two 8192^2 ones at 154)
//
// MFMA 32x32x2 fp32 fragment maps, lane l (l32 = l%32, h = l/32):
//   A (32x2): row l32, k = h;  B (2x32): col l32, k = h;  C: col l32, row 8*(r/4)+4h+r%4.
// With the streamed rows on C's rows, accumulator register r is directly the B operand
// (k-slot h <-> streamed row 8*(r/4)+4h+r%4) of the second product.  Both contractions may be
// permuted: the first products take feature 8g+4h+t in MFMA 4g+t, so that four MFMAs share one
// 16-byte load of a lane; the second products put feature DT*m+dt on row m of tile dt, so that
// the DT tiles of one MFMA step share one load of DT floats per lane, 32 lanes reading a whole row.
#pragma once
#include "sattn_common.hpp"

namespace sattn {

enum F32Mode { F32_FWD = 0, F32_DQ = 1, F32_DKDV = 2 };

struct F32Params {
  TensorRef q, k, v, dout;      // inputs (dout unused by FWD)
  TensorRef o, dq, dk, dv;      // outputs
  const float* slopes;
  int B, H, N;
  float scale;   // 1/sqrt(d)
  float bias;
  // DQ only, optional: row sums of dS, element (b, h, i) at b*db_sb + h*db_sh + i
  // (+ the sequence's first token in a variable-length call)
  float* db_rows;
  int64_t db_sb, db_sh;
  // The same extensions as the bf16 kernels' parameter blocks: packed sequences of different
  // lengths (cu_seqlens, optional bias per sequence), query head h reading K/V head
  // h / kv_group (>= 1; the dK/dV pass then runs per K/V head and sums over its query heads),
  // and a number of keys Nk that differs from the number of queries N (0: same; non-causal).
  const int* cu_seqlens;
  const float* bias_vec;
  int kv_group;
  int Nk;
  // position of query 0 on the key axis (Nk - N when the queries are the last N positions of the
  // key sequence, else 0; any value here): causal keeps key j for query i iff j <= i + qoff,
  // ALiBi measures |i + qoff - j|
  int qoff;
};

__device__ __forceinline__ f32x16 mfma_f32(float a, float b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

// Streamed operand groups of one chunk in order of use.  A group is four loads per lane; a group
// of rows (kRow1, kRow2: tensor 1, 2) feeds 16 MFMAs of a first product, a group of transposed
// operand (kTr1, kTr2) 4 * DT MFMAs of a second product.
enum F32Group { kRow1, kRow2, kTr1, kTr2 };
template <int D, int MODE>
struct F32Seq {
  static constexpr int DT = D / 32, NR = D / 32, NT = 4;
  static constexpr int NG = MODE == F32_FWD ? NR + NT : MODE == F32_DQ ? 2 * NR + NT : 2 * NR + 2 * NT;
  // groups in flight: enough that a load has about a thousand cycles of matrix work to land in,
  // few enough for two waves per SIMD (256 registers)
  static constexpr int RING = MODE == F32_FWD ? (D == 64 ? 3 : 4) : (MODE == F32_DKDV && D == 128) ? 2 : 4;
  static_assert(NG % RING == 0, "every group keeps its ring slot from chunk to chunk");
  static constexpr F32Group kind(int g) {
    if (g < NR) return kRow1;
    if (MODE == F32_FWD) return kTr2;
    if (g < 2 * NR) return kRow2;
    return (MODE == F32_DQ || g >= 2 * NR + NT) ? kTr1 : kTr2;
  }
  static constexpr int index(int g) {
    if (g < NR) return g;
    if (MODE == F32_FWD) return g - NR;
    return g < 2 * NR ? g - NR : (g - 2 * NR) % NT;
  }
};

// LDS of a workgroup: the stationary rows first, the waves' partial outputs afterwards, rows
// padded by 16 bytes (which spreads the 32 rows of an access over the banks).
template <int D>
constexpr size_t f32_lds_bytes(int nw) { return sizeof(float) * (nw * 32 * (D + 4) + nw * 32); }

// 1 / (1 + exp(-x)) with full fp32 precision.  The refinement needs a finite denominator with a normal
// reciprocal; above 2^126, infinity among it, the result (below the smallest normal number) is
// zero.  A NaN fails the comparison and comes out of the refinement as one.
__device__ __forceinline__ float f32_sigmoid(float x) {
  const float q = 1.0f + expf(-x);
  const float r = __builtin_amdgcn_rcpf(q);
  const float p = __builtin_fmaf(__builtin_fmaf(-q, r, 1.0f), r, r);
  return q > 0x1p126f ? 0.f : p;
}

// One block of 32 stationary rows: `bh` counts (batch, query head), in the dK/dV pass (batch, K/V
// head).
template <int D, int MODE, bool CAUSAL, bool ALIBI, int NW>
__device__ __forceinline__ void f32_block(const F32Params& p, const int bh, const int blk, float* smem) {
  using Seq = F32Seq<D, MODE>;
  constexpr int DT = D / 32, LDX = D + 4, NT = 64 * NW;
  constexpr bool TWO = MODE != F32_FWD;  // second stationary operand / dP product
  typedef float f32xt __attribute__((ext_vector_type(DT)));
  float* const x1s = smem;
  float* const x2s = smem + 32 * LDX;
  static_assert(NW >= 2, "the two stationary tiles fit where the partial outputs go");

  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int heads = MODE == F32_DKDV ? p.H / p.kv_group : p.H;
  const int b = bh / heads, hd = bh % heads;
  const int hkv = MODE == F32_DKDV ? hd : hd / p.kv_group;
  const int hq0 = MODE == F32_DKDV ? hd * p.kv_group : hd, n_hq = MODE == F32_DKDV ? p.kv_group : 1;
  int N = p.N;
  int64_t tok0 = 0;
  float bias = p.bias;
  if (p.cu_seqlens) {
    tok0 = p.cu_seqlens[b];
    const int len = p.cu_seqlens[b + 1] - (int)tok0;
    N = len < p.N ? len : p.N;  // never beyond the span the host checked
    if (p.bias_vec) bias = p.bias_vec[b];
    if (blk * 32 >= N) return;  // this sequence has no such block (whole workgroup)
  }
  // N counts the queries, Nk the keys; Ns / Nt are the row counts of this pass's stationary /
  // streamed side
  const int Nk = p.Nk > 0 ? p.Nk : N;
  const int Ns = MODE == F32_DKDV ? Nk : N, Nt = MODE == F32_DKDV ? N : Nk;

  const float* kb = (const float*)p.k.ptr + b * p.k.sb + hkv * p.k.sh + tok0 * p.k.ss;
  const float* vb = (const float*)p.v.ptr + b * p.v.sb + hkv * p.v.sh + tok0 * p.v.ss;
  auto qhead = [&](int hq) { return (const float*)p.q.ptr + b * p.q.sb + hq * p.q.sh + tok0 * p.q.ss; };
  auto dohead = [&](int hq) {
    return TWO ? (const float*)p.dout.ptr + b * p.dout.sb + hq * p.dout.sh + tok0 * p.dout.ss : nullptr;
  };

  // range of streamed chunks (32 rows each) this block meets
  const int a0 = blk * 32, a_hi = (a0 + 32 < Ns ? a0 + 32 : Ns) - 1;
  int t_lo = 0, t_hi = (Nt + 31) / 32;
  if (CAUSAL) {
    if (MODE == F32_DKDV) {  // queries before the first key's place on the query axis see nothing
      const int first = a0 - p.qoff;
      t_lo = (first > 0 ? first : 0) / 32;
    } else {                 // keys after the last query's place on the key axis are masked
      const int last = a_hi + p.qoff;
      t_hi = last < 0 ? 0 : (last < Nt ? last : Nt - 1) / 32 + 1;
    }
  }
  const int n_t = t_hi > t_lo ? t_hi - t_lo : 0, n_items = n_hq * n_t;

  // ---- streamed operands: per-lane byte offsets (32 bits; the host checked the span) from a
  // wave-uniform base.  Rows past the end re-read the last one (their weights are zero).
  const uint32_t ys1 = (uint32_t)(MODE == F32_DKDV ? p.q.ss : p.k.ss) * 4u;
  const uint32_t ys2 = (uint32_t)(MODE == F32_FWD || MODE == F32_DQ ? p.v.ss : p.dout.ss) * 4u;
  const uint32_t last1 = (uint32_t)(Nt - 1) * ys1, last2 = (uint32_t)(Nt - 1) * ys2;
  struct Src { const char *y1, *y2; int hq, b0; };
  auto source = [&](int item) {
    Src s;
    const int hi = n_hq == 1 ? 0 : item / (n_t > 0 ? n_t : 1);
    s.hq = hq0 + hi;
    s.b0 = (t_lo + item - hi * n_t) * 32;
    s.y1 = (const char*)(MODE == F32_DKDV ? qhead(s.hq) : kb);
    s.y2 = (const char*)(MODE == F32_DKDV ? dohead(s.hq) : vb);
    return s;
  };
  f32x4 ring[Seq::RING][4];
  auto load_group = [&](int g, const Src& s) {
    f32x4(&dst)[4] = ring[g % Seq::RING];
    const F32Group kind = Seq::kind(g);
    const int j = Seq::index(g);
    const bool first = kind == kRow1 || kind == kTr1;
    const char* base = first ? s.y1 : s.y2;
    const uint32_t ys = first ? ys1 : ys2, last = first ? last1 : last2;
    if (kind == kRow1 || kind == kRow2) {
      uint32_t o = (uint32_t)(s.b0 + l32) * ys;
      o = (o < last ? o : last) + h * 16;
#pragma unroll
      for (int i = 0; i < 4; ++i) dst[i] = *(const f32x4*)(base + (size_t)(o + (4 * j + i) * 32));
    } else {
      const uint32_t o0 = (uint32_t)(s.b0 + 8 * j + 4 * h) * ys;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        uint32_t o = o0 + i * ys;
        o = (o < last ? o : last) + l32 * (DT * 4);
        const f32xt v = *(const f32xt*)(base + (size_t)o);
#pragma unroll
        for (int e = 0; e < DT; ++e) dst[i][e] = v[e];
      }
    }
  };

  Src cur = source(wave < n_items ? wave : 0);
  if (wave < n_items) {
#pragma unroll
    for (int g = 0; g < Seq::RING; ++g) load_group(g, cur);
  }
  // ---- stationary rows into LDS
  {
    const float* x1 = MODE == F32_DKDV ? kb : qhead(hq0);
    const float* x2 = MODE == F32_DKDV ? vb : dohead(hq0);
    const int64_t x1s_ = MODE == F32_DKDV ? p.k.ss : p.q.ss, x2s_ = MODE == F32_DKDV ? p.v.ss : p.dout.ss;
#pragma unroll
    for (int idx = tid; idx < 32 * (D / 4); idx += NT) {
      const int r = idx / (D / 4), c = idx % (D / 4);
      const int row = a0 + r < Ns ? a0 + r : Ns - 1;
      *(f32x4*)(x1s + r * LDX + 4 * c) = *(const f32x4*)(x1 + (int64_t)row * x1s_ + 4 * c);
      if (TWO) *(f32x4*)(x2s + r * LDX + 4 * c) = *(const f32x4*)(x2 + (int64_t)row * x2s_ + 4 * c);
    }
  }
  f32x16 acc0[DT], acc1[MODE == F32_DKDV ? DT : 1];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      acc0[dt][r] = 0.f;
      if (MODE == F32_DKDV) acc1[dt][r] = 0.f;
    }
  float dbsum = 0.f;  // DQ: sum of this lane's dS elements
  __syncthreads();

  const int ai = a0 + l32;  // this lane's stationary row (query, or key for DKDV)
  const float* const xr1 = x1s + l32 * LDX + 4 * h;
  const float* const xr2 = x2s + l32 * LDX + 4 * h;
  for (int item = wave; item < n_items; item += NW) {
    const Src nxt = source(item + NW < n_items ? item + NW : item);  // (the last chunk is fetched again, into slots nobody reads)
    const float slope = ALIBI ? p.slopes[cur.hq] : 0.f;
    f32x16 s, dp;
#pragma unroll
    for (int r = 0; r < 16; ++r) { s[r] = 0.f; dp[r] = 0.f; }
#pragma unroll
    for (int g = 0; g < Seq::NG; ++g) {
      const F32Group kind = Seq::kind(g);
      const int j = Seq::index(g);
      const f32x4(&y)[4] = ring[g % Seq::RING];
      if (kind == kRow1 || kind == kRow2) {
        f32x4 x[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) x[i] = *(const f32x4*)((kind == kRow1 ? xr1 : xr2) + 8 * (4 * j + i));
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            if (kind == kRow1) s = mfma_f32(y[i][e], x[i][e], s);
            else dp = mfma_f32(y[i][e], x[i][e], dp);
          }
      } else {
        if (j == 0 && g == (MODE == F32_FWD ? 1 : 2) * Seq::NR) {
          // element (register r, this lane): streamed row bi = b0 + 8(r/4) + 4h + r%4, stationary row
          // ai; P replaces S and dS replaces dP in their registers
          const int bl = cur.b0 + 4 * h;
          float dist0 = 0.f;
          if (ALIBI) dist0 = (float)(MODE == F32_DKDV ? bl + p.qoff - ai : ai + p.qoff - bl);
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const float off = (float)(8 * (r >> 2) + (r & 3));
            float tt = s[r] * p.scale + bias;
            if (ALIBI) tt -= slope * __builtin_fabsf(MODE == F32_DKDV ? dist0 + off : dist0 - off);
            const float pv = f32_sigmoid(tt);
            s[r] = pv;
            if (TWO) dp[r] = pv * (1.0f - pv) * dp[r];
          }
          // only a chunk that crosses the diagonal or the end of the streamed side is masked
          bool edge = cur.b0 + 32 > Nt;
          if (CAUSAL) edge = edge || (MODE == F32_DKDV ? cur.b0 + p.qoff < a0 + 31 : cur.b0 + 31 > a0 + p.qoff);
          if (edge) {
            const int lim = Nt - bl, dgl = MODE == F32_DKDV ? ai - p.qoff - bl : ai + p.qoff - bl;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
              const int off = 8 * (r >> 2) + (r & 3);
              const bool keep = off < lim && (!CAUSAL || (MODE == F32_DKDV ? off >= dgl : off <= dgl));
              s[r] = keep ? s[r] : 0.f;
              if (TWO) dp[r] = keep ? dp[r] : 0.f;
            }
          }
          if (MODE == F32_DQ) {
#pragma unroll
            for (int r = 0; r < 16; ++r) dbsum += dp[r];
          }
        }
        // second products: acc^T[d][a] += Y^T[d][bi] * W[bi][a]
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int dt = 0; dt < DT; ++dt) {
            if (MODE == F32_FWD) acc0[dt] = mfma_f32(y[i][dt], s[4 * j + i], acc0[dt]);
            else if (kind == kTr1) acc0[dt] = mfma_f32(y[i][dt], dp[4 * j + i], acc0[dt]);
            else acc1[MODE == F32_DKDV ? dt : 0] = mfma_f32(y[i][dt], s[4 * j + i], acc1[MODE == F32_DKDV ? dt : 0]);
          }
      }
      load_group((g + Seq::RING) % Seq::NG, g + Seq::RING < Seq::NG ? cur : nxt);
      __builtin_amdgcn_sched_barrier(0);
    }
    cur = nxt;
  }

  // ---- the waves' partial sums meet in LDS, every wave adds up a part of them and stores rows
  float* const dbs = smem + NW * 32 * LDX;  // [NW][32]
  if (MODE == F32_DQ) {
    dbsum += __shfl_xor(dbsum, 32);  // the two halves of the wave: different keys of the same query row
    if (h == 0) dbs[wave * 32 + l32] = dbsum;
  }
#pragma unroll
  for (int out = 0; out < (MODE == F32_DKDV ? 2 : 1); ++out) {
    __syncthreads();  // the stationary rows (the previous output's partial sums) are no longer read
    const f32x16* const acc = out == 0 ? acc0 : acc1;
    float* const part = smem + (wave * 32 + l32) * LDX;
#pragma unroll
    for (int r = 0; r < 16; ++r) {  // row m = 8(r/4) + 4h + r%4 of tile dt is feature DT*m + dt
      f32xt w;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) w[dt] = acc[dt][r];
      *(f32xt*)(part + DT * (8 * (r >> 2) + 4 * h + (r & 3))) = w;
    }
    __syncthreads();
    const float osc = (MODE == F32_FWD || out == 1) ? 1.0f : p.scale;  // dQ, dK carry the 1/sqrt(d) of the logits
    const TensorRef& o = MODE == F32_FWD ? p.o : MODE == F32_DQ ? p.dq : out == 0 ? p.dk : p.dv;
    float* const ob = (float*)o.ptr + b * o.sb + hd * o.sh + (tok0 + a0) * o.ss;
#pragma unroll
    for (int idx = tid; idx < 32 * (D / 4); idx += NT) {
      const int r = idx / (D / 4), c = idx % (D / 4);
      f32x4 sum = *(const f32x4*)(smem + r * LDX + 4 * c);
#pragma unroll
      for (int w = 1; w < NW; ++w) {
        const f32x4 v = *(const f32x4*)(smem + (w * 32 + r) * LDX + 4 * c);
#pragma unroll
        for (int e = 0; e < 4; ++e) sum[e] += v[e];
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) sum[e] *= osc;
      if (a0 + r < Ns) *(f32x4*)(ob + (int64_t)r * o.ss + 4 * c) = sum;
    }
  }
  if (MODE == F32_DQ && p.db_rows && tid < 32 && a0 + tid < Ns) {
    float sum = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) sum += dbs[w * 32 + tid];
    p.db_rows[b * p.db_sb + hd * p.db_sh + tok0 + a0 + tid] = sum;
  }
}

// Workgroup id -> head and block.  Without the mask consecutive blocks of a head go to one XCD
// (xcd_remap).  Blocks of a causal head differ in length: they are dispatched longest first, one
// rank of all heads before the next, which spreads the lengths evenly over the XCDs (the hardware
// deals workgroups out round-robin) and keeps a head on one XCD where the number of heads is a
// multiple of 8.  Workgroups w and w + `cus` become neighbours on one compute unit (measured), so
// the second `cus` of them come in the opposite order, which puts long blocks next to short
// ones; whole rows of heads are mirrored there, so that a head stays on its XCD.
template <int MODE, bool CAUSAL>
__device__ __forceinline__ void f32_place(int wg, int n_blocks, int n_heads, int cus, int& bh, int& blk) {
  const int total = n_blocks * n_heads;
  if (!CAUSAL) {
    const int place = xcd_remap(wg, total);
    bh = place / n_blocks;
    blk = place - bh * n_blocks;
    return;
  }
  const int end = 2 * cus < total ? 2 * cus : total;
  const int i = (wg >= cus && wg < end) ? cus + end - 1 - wg : wg;
  const int rank = i / n_heads, row = rank * n_heads;
  bh = i - row;
  if (row >= cus && row + n_heads <= end) bh = n_heads - 1 - bh;
  blk = MODE != F32_DKDV ? n_blocks - 1 - rank : rank;
}

// One pass.  `first`: the number of the launch's first workgroup, where the grid takes several launches.
template <int D, int MODE, bool CAUSAL, bool ALIBI, int NW>
__global__ void __launch_bounds__(64 * NW, 2)
sigmoid_f32_kernel(const F32Params p, int n_blocks, int n_heads, int cus, int first) {
  extern __shared__ __attribute__((aligned(16))) float smem_f32[];
  int bh, blk;
  f32_place<MODE, CAUSAL>(first + (int)blockIdx.x, n_blocks, n_heads, cus, bh, blk);
  f32_block<D, MODE, CAUSAL, ALIBI, NW>(p, bh, blk, smem_f32);
}

// Both backward passes in one grid: first all dK/dV blocks, then all dQ blocks, which fill the
// compute units as the former run out.
template <int D, bool CAUSAL, bool ALIBI, int NW>
__global__ void __launch_bounds__(64 * NW, 2)
sigmoid_f32_bwd_kernel(const F32Params p, int nb_k, int nb_q, int cus, int first) {
  extern __shared__ __attribute__((aligned(16))) float smem_f32[];
  const int heads_k = p.B * (p.H / p.kv_group), heads_q = p.B * p.H, n_k = nb_k * heads_k, wg = first + (int)blockIdx.x;
  int bh, blk;
  if (wg < n_k) {
    f32_place<F32_DKDV, CAUSAL>(wg, nb_k, heads_k, cus, bh, blk);
    f32_block<D, F32_DKDV, CAUSAL, ALIBI, NW>(p, bh, blk, smem_f32);
  } else {
    f32_place<F32_DQ, CAUSAL>(wg - n_k, nb_q, heads_q, nb_q * heads_q, bh, blk);
    f32_block<D, F32_DQ, CAUSAL, ALIBI, NW>(p, bh, blk, smem_f32);
  }
}

}  // namespace sattn
