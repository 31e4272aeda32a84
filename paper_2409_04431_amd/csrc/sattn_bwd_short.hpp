// Sigmoid-attention backward of sequences that one workgroup holds whole: up to 256 keys at d = 64,
// 128 at d = 128 (bf16; ALiBi without a mask only: under it the passes add its terms in orders of their own).
//
// The two passes of sattn_bwd.hpp evaluate every logit, dP and sigmoid twice, because no workgroup
// holds all keys a dQ row has to be summed over.  Here one does.  A wave owns 32 keys (K, V
// fragments and the dK^T, dV^T accumulators in registers) and goes through the queries in
// chunks of 32: S = Q K^T, dP = dO V^T, dS, dV^T += dO^T P, dK^T += Q^T dS.  It leaves dS in LDS, keys by
// queries, and after every 128 queries the waves share out dQ^T = K^T dS^T by tiles of 32 queries x
// 32 features, each summed over all keys in ascending order: the additions of the dQ pass, so that results are
// the two passes' bit for bit.  Q, dO and K are in LDS once and for all, read by rows and transposed.
//
// Heads beyond whole rounds of the chip leave most of a last round empty; those take two
// workgroups, one for dK and dV and one for dQ (which then has to form S and dP again).
//
// What bounds it: 1350 cycles per 32 x 32 chunk and SIMD against 850 of its vector issue (the compiler's
// order, filled by the second wave of a SIMD; the next chunk's rows are read under the arithmetic of
// this one: N250 38.9 -> 36.5 us), and around it 4 to 5 us of first loads at the memory's rate, one
// workgroup's 160 KB of LDS leaving no room for another's.  Up to 128 keys two workgroups share a compute unit.
// Measured (us, the two passes / this): d64 384 heads N250 44.5 / 37.5 (causal 41.6 / 33.4), N128 19.4 / 14.7; 1024 heads
// N250 109 / 84 (103 / 74), N64 32.4 / 17.4; 16 heads N64 7.7 / 5.7; d128 512 heads N128 57.3 / 37.0, 1024 N100 101 /
// 66.7, 2048 N64 144 / 75.
#pragma once
#include <type_traits>

#include "sattn_bwd.hpp"

namespace sattn {

// LDS: Q and dO tiles of all queries, all keys, dS of 128 queries.
template <int D, int NW>
constexpr size_t short_lds_bytes() { return (size_t)NW * 32 * D * 2 * 3 + (size_t)NW * 32 * 128 * 2; }

// What a workgroup finds of its head.
struct ShortHead {
  int N;
  float nbias, sl2;  // bias and ALiBi slope in the exponent of two
  int64_t tok0;
  int b, hd;
  __device__ __forceinline__ __bf16* of(const TensorRef& t) const { return (__bf16*)t.ptr + b * t.sb + hd * t.sh + tok0 * t.ss; }
};

// Zeros in the rows from N on of a 64-row tile that starts at row 64 t.
template <int D, int NW>
__device__ __forceinline__ void short_pad(uint32_t tile, int t, int N, int tid) {
  for (int i = tid; i < (64 * (t + 1) - N) * (D / 8); i += 64 * NW)
    lds_write_b128(tile + ((N & 63) + i / (D / 8)) * (D * 2) + (i % (D / 8)) * 16, u32x4{0, 0, 0, 0});
}

// The 32 keys of a wave, or its 32 queries of `n` blocks in all (blocks from n on are past the end).  Under the mask
// the waves of a SIMD (w, w + 4) get blocks whose work adds up to the same, or to at most that of the longest block
// where there are fewer than eight: a key block's work falls with its place, a query block's rises (forward, d64 N192, 288
// heads, of the streaming kernel's time: 1.12 with query blocks dealt out like key blocks, 0.98 so).
template <int NW, bool CAUSAL>
__device__ __forceinline__ int short_key_block(int wave) { return (CAUSAL && NW == 8 && wave >= 4) ? 11 - wave : wave; }
template <int NW, bool CAUSAL>
__device__ __forceinline__ int short_query_block(int wave, int n) {
  return (CAUSAL && NW == 8) ? (wave < 4 ? n - 1 - wave : n - 4 + wave) & 7 : wave;
}

// Per-lane LDS offsets: rows of a 32-row chunk, transposed pairs of a 64-row tile.
template <int D>
struct ShortLanes {
  uint32_t row[D / 16], tr[D / 32][2];
  __device__ __forceinline__ void init(int lane) {
    const int l32 = lane & 31, h = lane >> 5, kap = kappa(l32), i16 = lane & 15, blk1 = (lane >> 4) & 1;
#pragma unroll
    for (int kk = 0; kk < D / 16; ++kk) row[kk] = kap * (D * 2) + (((2 * kk + h) ^ SwzX<D>::f(kap)) << 4);
#pragma unroll
    for (int rd = 0; rd < 2; ++rd) {
      const int r = 8 * h + 4 * rd + (i16 >> 2), c = 2 * blk1 + ((i16 & 3) >> 1);
#pragma unroll
      for (int dt = 0; dt < D / 32; ++dt) tr[dt][rd] = r * (D * 2) + (((4 * dt + c) ^ SwzX<D>::f(r)) << 4) + ((i16 & 1) << 3);
    }
  }
};

// dK, dV and, with DQ, dQ of a head.
template <int D, int NW, bool CAUSAL, bool ALIBI, bool DQ>
__device__ __forceinline__ void short_dkdv(const BwdParams& p, const ShortHead& hd, uint32_t lds0, ClockStart& clk) {
  constexpr int KD = D / 16, DT = D / 32, MAXN = 32 * NW, TILE = 64 * D * 2, SLOT = 2 * TILE;
  constexpr int N_SUB = 4 * DT / NW, SUB_STEP = NW / DT;  // dQ tiles (32 queries x 32 features) of a wave per 128 queries
  static_assert(NW % DT == 0 && N_SUB >= 1, "a wave keeps one tile of features");
  const uint32_t lds_k = lds0 + (MAXN / 64) * SLOT, lds_ds = lds_k + (MAXN / 64) * TILE;
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int N = hd.N;
  const float nbias = hd.nbias;
  const __bf16 *kb = hd.of(p.k), *vb = hd.of(p.v);

  // ---- K, the first 128 queries and this wave's V rows; the other queries follow while these are worked on
  const int n_tiles = (N + 63) / 64, n_chunks = (N + 31) / 32;
  DmaStagerX<D, NW> sq, sd;
  sq.init(hd.of(p.q), p.q.ss, N, 0, wave, lane);
  sd.init(hd.of(p.dout), p.dout.ss, N, 0, wave, lane);
  auto stage = [&](int t0, int t1) {
    for (int t = t0; t < t1; ++t) {
      sq.issue(lds0 + t * SLOT, N, wave, lane);
      sd.issue(lds0 + t * SLOT + TILE, N, wave, lane);
    }
  };
  {
    DmaStagerX<D, NW> sk;
    sk.init(kb, p.k.ss, N, 0, wave, lane);
    for (int t = 0; t < n_tiles; ++t) sk.issue(lds_k + t * TILE, N, wave, lane);
  }
  stage(0, min(n_tiles, 2));
  const int kblk = short_key_block<NW, CAUSAL>(wave);
  const int key0 = 32 * kblk, key = key0 + l32, key_ld = key < N ? key : N - 1;
  bf16x8 x1[KD], x2[KD];
#pragma unroll
  for (int kk = 0; kk < KD; ++kk) x2[kk] = as_bf16x8(*(const u32x4*)(vb + (int64_t)key_ld * p.v.ss + 16 * kk + 8 * h));
  f32x16 dk[DT], dv[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int r = 0; r < 16; ++r) dk[dt][r] = dv[dt][r] = 0.f;

  ShortLanes<D> at_lane;
  at_lane.init(lane);
  const auto& row = at_lane.row;
  const auto& tr = at_lane.tr;
  uint32_t ds_rd[2];  // transposed reads of dS (queries 32..63 of a row: bit 6 flipped)
#pragma unroll
  for (int rd = 0; rd < 2; ++rd) {
    const int i16 = lane & 15, r = 8 * h + 4 * rd + (i16 >> 2), c = 2 * ((lane >> 4) & 1) + ((i16 & 3) >> 1);
    ds_rd[rd] = r * 128 + ((c ^ SwzX<64>::f(r)) << 4) + ((i16 & 1) << 3);
  }
  const uint32_t ds_wr = lds_ds + key * 128 + ((h ^ SwzX<64>::f(key)) << 4);

  // Rows past the end repeat row N-1 in Q, K and V and are zeros in dO (where the repeated row would make an
  // infinite element of it a NaN in dV).  P and dS of queries there are zero by selection, and dS of keys there is
  // overwritten with zeros in LDS, whatever the logit and dP are.
  SATTN_WAIT_VMCNT(0);
  stage(2, n_tiles);
  __syncthreads();
  clock_probe_mark(p.clock, clk, kMarkFirstProduct);
  {
    const int at = key0 + l32;  // (rows of a wave past the end: whatever is there, nobody uses it)
#pragma unroll
    for (int kk = 0; kk < KD; ++kk) x1[kk] = as_bf16x8(lds_read_b128(lds_k + at * (D * 2) + (((2 * kk + h) ^ SwzX<D>::f(at)) << 4)));
  }
  if (n_tiles <= 2 && n_tiles * 64 > N) {
    short_pad<D, NW>(lds0 + (n_tiles - 1) * SLOT + TILE, n_tiles - 1, N, tid);
    __syncthreads();
  }

  bf16x8 f1[KD], f2[KD];  // row fragments of the next chunk
  auto rows_of = [&](int c) {
    const uint32_t at = lds0 + (c >> 1) * SLOT + (c & 1) * (32 * D * 2);
#pragma unroll
    for (int kk = 0; kk < KD; ++kk) {
      f1[kk] = as_bf16x8(lds_read_b128(at + row[kk]));
      f2[kk] = as_bf16x8(lds_read_b128(at + TILE + row[kk]));
    }
  };
  const int ragged = N & 31 ? N >> 5 : -1;
  // One chunk of 32 queries; `next`: the one whose rows are fetched under it.
  auto chunk = [&](int c, int next, auto masked) __attribute__((always_inline)) {
    const uint32_t at = lds0 + (c >> 1) * SLOT + (c & 1) * (32 * D * 2);
    f32x16 s, dp;
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] = dp[r] = 0.f;
#pragma unroll
    for (int kk = 0; kk < KD; ++kk) {
      s = mfma32(f1[kk], x1[kk], s);
      dp = mfma32(f2[kk], x2[kk], dp);
    }
    // (the transposed fragments of this chunk and the rows of the next one come in under the arithmetic)
    bf16x8 t1[2][DT], t2[2][DT];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
        const uint32_t off = at + ks * 16 * (D * 2);
        t2[ks][dt] = join_tr(lds_read_tr16(off + TILE + tr[dt][0]), lds_read_tr16(off + TILE + tr[dt][1]));
        t1[ks][dt] = join_tr(lds_read_tr16(off + tr[dt][0]), lds_read_tr16(off + tr[dt][1]));
      }
    rows_of(next);
    float pr[16], ds[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float w = ALIBI ? __builtin_fmaf(hd.sl2, __builtin_fabsf((float)(32 * c + 8 * h + key_of_reg(r) - key)), nbias) : nbias;
      const float e = __builtin_amdgcn_exp2f(__builtin_fmaf(s[r], p.nscale_log2, w));
      pr[r] = __builtin_amdgcn_rcpf(1.0f + e);
      ds[r] = __builtin_fmaf(-pr[r], pr[r], pr[r]) * dp[r];
    }
    if (decltype(masked)::value || (CAUSAL && (c == kblk || c == ragged))) {
      const int from = CAUSAL && c == kblk ? l32 : 0;
      // (a key past the end, l32 >= N & 31, may keep queries: its dK and dV are not stored, its dS leaves as zeros)
      const uint32_t span = (c == ragged ? N & 31 : 32) - from, first = 8 * h - from;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const bool keep = key_of_reg(r) + first < span;
        pr[r] = keep ? pr[r] : 0.f;
        ds[r] = keep ? ds[r] : 0.f;
      }
    }
    bf16x8 pb[2] = {pack8(pr), pack8(pr + 8)}, dsb[2] = {pack8(ds), pack8(ds + 8)};
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
        dv[dt] = mfma32(t2[ks][dt], pb[ks], dv[dt]);
        dk[dt] = mfma32(t1[ks][dt], dsb[ks], dk[dt]);
      }
    if constexpr (DQ) {
      // dS, keys by queries: rows of 64 queries of a key, two such tiles
      const uint32_t to = (ds_wr ^ ((c & 1) << 6)) + ((c >> 1) & 1) * (MAXN * 128);
      lds_write_b128(to, __builtin_bit_cast(u32x4, dsb[0]));
      lds_write_b128(to ^ 32, __builtin_bit_cast(u32x4, dsb[1]));
    }
  };
  const int rounds = (N + 127) / 128, c_end = key0 < N ? n_chunks : 0;  // (a wave past the end has no chunk)
  clk.steady_tiles = (c_end - (CAUSAL ? min(kblk, c_end) : 0) + 1) / 2;
  clock_probe_mark(p.clock, clk, kMarkSteadyBegin);
  for (int rnd = 0; rnd < rounds; ++rnd) {
    const int c_lo = CAUSAL ? max(4 * rnd, kblk) : 4 * rnd, c_hi = min(4 * rnd + 4, c_end);
    if (c_lo < c_hi) rows_of(c_lo);
    // The ragged last chunk is a copy of the body of its own: the selection as a branch inside the loop, also where
    // nothing is ragged, takes 2 to 9 % of the time (us: B64 H16 N128 d64 30.4 / 28.6, N64 18.8 / 17.3, B32 H16 N128 d128
    // 41.4 / 39.2).  Under the mask the loop has that branch anyway, and a third copy is slower to fetch than it saves
    // (N100, 384 heads: 13.1 / 13.8).
    const int plain = !CAUSAL && ragged >= 0 ? min(c_hi, ragged) : c_hi;
    int c = c_lo;
#pragma nounroll
    for (; c < plain; ++c) chunk(c, min(c + 1, c_hi - 1), std::false_type{});
    if (!CAUSAL && c < c_hi) chunk(c, c, std::true_type{});
    if (DQ && key >= N && key0 < N) {  // a row of dS, this lane's half: the writes of a wave are in order
#pragma unroll
      for (int i = 0; i < 8; ++i) lds_write_b128((ds_wr ^ ((i & 3) << 5)) + (i >> 2) * (MAXN * 128), u32x4{0, 0, 0, 0});
    }
    if (rnd == 0) SATTN_WAIT_VMCNT(0);  // the other queries have landed
    __syncthreads();
    if (rnd == 0 && n_tiles > 2 && n_tiles * 64 > N) short_pad<D, NW>(lds0 + (n_tiles - 1) * SLOT + TILE, n_tiles - 1, N, tid);
    if constexpr (DQ) {
      // dQ of these 128 queries: this wave's tile of features, all keys
      const int dt = wave % DT;
      const uint32_t kt0 = lds_k + tr[0][0], kt1 = lds_k + tr[0][1];
      const uint32_t flip = (uint32_t)(4 * dt) << 4;
#pragma unroll
      for (int i = 0; i < N_SUB; ++i) {
        const int sub = wave / DT + i * SUB_STEP, c = 4 * rnd + sub;
        if (c >= n_chunks) continue;
        const int n_kb = CAUSAL ? c + 1 : n_chunks;  // blocks of 32 keys
        const uint32_t from = lds_ds + (sub >> 1) * (MAXN * 128), half = (sub & 1) << 6;
        f32x16 dq;
#pragma unroll
        for (int r = 0; r < 16; ++r) dq[r] = 0.f;
        bf16x8 ka[2], wa[2];
        auto fetch = [&](int j) {
#pragma unroll
          for (int ks = 0; ks < 2; ++ks) {
            const uint32_t ko = (2 * j + ks) * 16 * (D * 2), so = from + (2 * j + ks) * 16 * 128;
            ka[ks] = join_tr(lds_read_tr16((kt0 ^ flip) + ko), lds_read_tr16((kt1 ^ flip) + ko));
            wa[ks] = join_tr(lds_read_tr16(so + (ds_rd[0] ^ half)), lds_read_tr16(so + (ds_rd[1] ^ half)));
          }
        };
        fetch(0);
#pragma nounroll
        for (int j = 0; j < n_kb; ++j) {
          const bf16x8 k0 = ka[0], k1 = ka[1], w0 = wa[0], w1 = wa[1];
          fetch(min(j + 1, n_kb - 1));
          dq = mfma32(k0, w0, dq);
          dq = mfma32(k1, w1, dq);
        }
        const int q = 32 * c + l32;
        if (q < N) {
          __bf16* out = hd.of(p.dq) + (int64_t)q * p.dq.ss + 32 * dt + 4 * h;
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            u32x2 w;
            w[0] = pack_bf16(dq[4 * g] * p.inv_sqrt_d, dq[4 * g + 1] * p.inv_sqrt_d);
            w[1] = pack_bf16(dq[4 * g + 2] * p.inv_sqrt_d, dq[4 * g + 3] * p.inv_sqrt_d);
            *(u32x2*)(out + 8 * g) = w;
          }
        }
      }
    }
    __syncthreads();
  }
  clock_probe_mark(p.clock, clk, kMarkSteadyEnd);
  clock_probe_mark(p.clock, clk, kMarkStore);
  const uint32_t obuf = lds0 + wave * (2 * RowStore<D>::BYTES);
  static_assert(NW * 2 * RowStore<D>::BYTES <= short_lds_bytes<D, NW>(), "outputs leave through the same LDS");
  RowStore<D>::run(dk, p.inv_sqrt_d, obuf, lane, hd.of(p.dk) + (int64_t)key0 * p.dk.ss, p.dk.ss, N - key0);
  RowStore<D>::run(dv, 1.0f, obuf + RowStore<D>::BYTES, lane, hd.of(p.dv) + (int64_t)key0 * p.dv.ss, p.dv.ss, N - key0);
  clk.tiles = n_tiles;
}

// dQ alone (DB: and the row sums of dS, in the order of the dQ pass): a wave owns 32 queries (Q, dO fragments, the
// dQ^T accumulators) and goes through the keys, whose rows P^T and dS^T have in registers: S^T = K Q^T, dP^T = V dO^T,
// dQ^T += K^T dS^T.
template <int D, int NW, bool CAUSAL, bool ALIBI, bool DB>
__device__ __forceinline__ void short_dq(const BwdParams& p, const ShortHead& hd, uint32_t lds0, ClockStart& clk) {
  constexpr int KD = D / 16, DT = D / 32, TILE = 64 * D * 2, SLOT = 2 * TILE;
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
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
  const __bf16 *qb = hd.of(p.q), *dob = hd.of(p.dout);
  bf16x8 x1[KD], x2[KD];
#pragma unroll
  for (int kk = 0; kk < KD; ++kk) {
    x1[kk] = as_bf16x8(*(const u32x4*)(qb + (int64_t)q_ld * p.q.ss + 16 * kk + 8 * h));
    x2[kk] = as_bf16x8(*(const u32x4*)(dob + (int64_t)q_ld * p.dout.ss + 16 * kk + 8 * h));
  }
  f32x16 dq[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int r = 0; r < 16; ++r) dq[dt][r] = 0.f;
  ShortLanes<D> at_lane;
  at_lane.init(lane);
  SATTN_WAIT_VMCNT(0);
  __syncthreads();
  clock_probe_mark(p.clock, clk, kMarkFirstProduct);
  float dbs[4] = {0.f, 0.f, 0.f, 0.f};
  const int c_hi = q0 < N ? (CAUSAL ? qblk + 1 : n_chunks) : 0;
  // Keys from N on repeat row N-1; their dS is zero by selection, whatever the logit and dP are (under the
  // mask no query has them).
  const int ragged = N & 31 ? N >> 5 : -1, keep = CAUSAL ? l32 + 1 : N & 31;
  bf16x8 f1[KD], f2[KD];
  auto rows_of = [&](int c) {
    const uint32_t at = lds0 + (c >> 1) * SLOT + (c & 1) * (32 * D * 2);
#pragma unroll
    for (int kk = 0; kk < KD; ++kk) {
      f1[kk] = as_bf16x8(lds_read_b128(at + at_lane.row[kk]));
      f2[kk] = as_bf16x8(lds_read_b128(at + TILE + at_lane.row[kk]));
    }
  };
  auto chunk = [&](int c, int next, auto masked) __attribute__((always_inline)) {
    const uint32_t at = lds0 + (c >> 1) * SLOT + (c & 1) * (32 * D * 2);
    f32x16 s, dp;
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] = dp[r] = 0.f;
#pragma unroll
    for (int kk = 0; kk < KD; ++kk) {
      s = mfma32(f1[kk], x1[kk], s);
      dp = mfma32(f2[kk], x2[kk], dp);
    }
    rows_of(next);
    float ds[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float a = ALIBI ? __builtin_fmaf(hd.sl2, __builtin_fabsf((float)(q0 + l32 - (32 * c + 8 * h + key_of_reg(r)))), hd.nbias) : hd.nbias;
      const float e = __builtin_amdgcn_exp2f(__builtin_fmaf(s[r], p.nscale_log2, a));
      const float w = __builtin_amdgcn_rcpf(1.0f + e);
      ds[r] = __builtin_fmaf(-w, w, w) * dp[r];
    }
    if constexpr (decltype(masked)::value) {
#pragma unroll
      for (int r = 0; r < 16; ++r) ds[r] = key_of_reg(r) + 8 * h < keep ? ds[r] : 0.f;
    }
    if constexpr (DB) {
#pragma clang fp contract(off)  // (dS is rounded before it is added, as in the dQ pass)
#pragma unroll
      for (int r = 0; r < 16; ++r) dbs[r & 3] += ds[r];
    }
    const bf16x8 dsb[2] = {pack8(ds), pack8(ds + 8)};
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
        const uint32_t off = at + ks * 16 * (D * 2);
        dq[dt] = mfma32(join_tr(lds_read_tr16(off + at_lane.tr[dt][0]), lds_read_tr16(off + at_lane.tr[dt][1])), dsb[ks], dq[dt]);
      }
  };
  if (c_hi > 0) rows_of(0);
  clk.steady_tiles = (c_hi + 1) / 2;
  clock_probe_mark(p.clock, clk, kMarkSteadyBegin);
  const int plain = CAUSAL ? c_hi - 1 : ragged >= 0 ? min(c_hi, ragged) : c_hi;  // (the last of them is on the diagonal)
  int c = 0;
#pragma nounroll
  for (; c < plain; ++c) chunk(c, min(c + 1, c_hi - 1), std::false_type{});
  if (c < c_hi) chunk(c, c, std::true_type{});
  clock_probe_mark(p.clock, clk, kMarkSteadyEnd);
  if constexpr (DB) {
    float rs = (dbs[0] + dbs[1]) + (dbs[2] + dbs[3]);
    rs += __shfl_xor(rs, 32);  // the two halves of the wave: different keys of the same query row
    if (h == 0 && q0 + l32 < N) p.db_rows[hd.b * p.db_sb + hd.hd * p.db_sh + hd.tok0 + q0 + l32] = rs;
  }
  __syncthreads();
  clock_probe_mark(p.clock, clk, kMarkStore);
  RowStore<D>::run(dq, p.inv_sqrt_d, lds0 + wave * RowStore<D>::BYTES, lane, hd.of(p.dq) + (int64_t)q0 * p.dq.ss, p.dq.ss, N - q0);
  clk.tiles = n_tiles;
}

// Heads below `whole` take a workgroup each, the others two: dK and dV first, then dQ.  The row sums of dS
// come with the latter (DB: whole = 0).
template <int D, int NW, bool CAUSAL, bool ALIBI = false, bool DB = false>
__global__ void __launch_bounds__(64 * NW, D == 64 ? 2 : 1) attn_bwd_short_kernel(const BwdParams p, const int whole) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const uint32_t lds0 = (uint32_t)(uintptr_t)(SATTN_LDS(char)*)smem;
  ClockStart clk = clock_probe_begin(p.clock);
  const int rest = p.B * p.H - whole, i = (int)blockIdx.x - whole;  // i < 0: a whole head
  const int bh = i < rest ? (int)blockIdx.x : whole + i - rest;
  ShortHead hd;
  hd.b = bh / p.H;
  hd.hd = bh - hd.b * p.H;
  hd.N = p.N;
  hd.tok0 = 0;
  hd.nbias = p.nbias_log2;
  hd.sl2 = ALIBI ? p.slopes[hd.hd] * kLog2e : 0.f;
  if (p.cu_seqlens) {
    hd.tok0 = p.cu_seqlens[hd.b];
    hd.N = min(p.cu_seqlens[hd.b + 1] - (int)hd.tok0, p.N);
    if (p.bias_vec) hd.nbias = -p.bias_vec[hd.b] * kLog2e;
    if (hd.N <= 0) return;
  }
  if (!DB && i < 0) short_dkdv<D, NW, CAUSAL, ALIBI, true>(p, hd, lds0, clk);
  else if (i < rest) short_dkdv<D, NW, CAUSAL, ALIBI, false>(p, hd, lds0, clk);
  else short_dq<D, NW, CAUSAL, ALIBI, DB>(p, hd, lds0, clk);
  clock_probe_end(p.clock, clk, (int)blockIdx.x);
}

}  // namespace sattn
