// C ABI of the sigmoid-attention library: argument validation and kernel dispatch.
// See include/sattn.h (product contract) and include/sattn_bench.h (measurement aids).
#include "../../include/sattn.h"
#include "../../include/sattn_bench.h"

#include <hip/hip_runtime.h>
#include <math.h>

#include <algorithm>
#include <atomic>
#include <mutex>
#include <map>
#include <utility>

#include "sattn_f32.hpp"
#include "sattn_launch.hpp"
#include "sattn_norm.hpp"

using namespace sattn;

namespace sattn {

bool ensure_dynamic_lds(const void* kernel, int dev, size_t lds) {
  static std::mutex mu;
  static std::map<std::pair<const void*, int>, size_t> granted;  // (kernel, device) -> largest size set so far
  const std::pair<const void*, int> key(kernel, dev);
  std::lock_guard<std::mutex> lock(mu);
  auto it = granted.find(key);
  if (it != granted.end() && it->second >= lds) return true;
  if (hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess) return false;
  granted[key] = lds;
  return true;
}

}  // namespace sattn

// Scratch of softmax_attn_bwd_noalloc: what softmax_attn_bwd takes as its workspace (two fp32
// per padded query row), held in the library's own device image so that the call allocates
// nothing.  Every GPU the library runs on holds its own copy until the process ends.
constexpr size_t kNoAllocRows = (size_t)1 << 20;  // padded query rows B*H*roundup(N, 64)
static __device__ __align__(256) float scratch[2 * kNoAllocRows];  // 8 MiB

namespace {

// Device address of `scratch` on the current device.  In host code the array's name is only
// a handle; the address kernels can use comes from the runtime, once per device.
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
float* g_scratch_ptr[kMaxDevices] = {};

int scratch_on_current_device(float** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) {
    (void)hipGetLastError();
    return SATTN_ERR_LAUNCH;
  }
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) {
      (void)hipGetLastError();
      return SATTN_ERR_LAUNCH;
    }
    g_scratch_ptr[dev] = (float*)ptr;
  }
  *out = g_scratch_ptr[dev];
  return SATTN_OK;
}

int elem_size(sattn_dtype t) { return t == SATTN_BF16 ? 2 : 4; }

// Register-resident MFMA loop of the matrix-rate probe: 4 accumulators, 8 MFMAs per iteration.
__global__ void __launch_bounds__(256) mfma_bf16_probe_kernel(float* sink, int iters) {
  f32x16 acc[4];
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[j][r] = 0.f;
  bf16x8 a, b;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    a[e] = (__bf16)(0.01f * (float)((threadIdx.x % 7) + e));
    b[e] = (__bf16)(0.02f * (float)((threadIdx.x % 5) + e));
  }
  for (int it = 0; it < iters; ++it) {
#pragma unroll
    for (int u = 0; u < 8; ++u) acc[u & 3] = mfma32(a, b, acc[u & 3]);
  }
  float s = 0.f;
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int r = 0; r < 16; ++r) s += acc[j][r];
  sink[(size_t)blockIdx.x * 256 + threadIdx.x] = s;
}

// out[bh] = sum over i < N of rows[b*sb + h*sh + i], in a fixed order (deterministic).
__global__ void __launch_bounds__(256)
rowsum_reduce_kernel(const float* rows, float* out, int H, int N, int64_t sb, int64_t sh) {
  __shared__ float part[256];
  const int bh = blockIdx.x, tid = threadIdx.x;
  const float* r = rows + (bh / H) * sb + (bh % H) * sh;
  float acc = 0.f;
  for (int i = tid; i < N; i += 256) acc += r[i];
  part[tid] = acc;
  __syncthreads();
#pragma unroll
  for (int m = 128; m >= 1; m >>= 1) {
    if (tid < m) part[tid] += part[tid + m];
    __syncthreads();
  }
  if (tid == 0) out[bh] = part[0];
}

// Packed sequences: out[b*H + h] = sum of rows[h*total + t] over the tokens t of sequence b that the
// backward pass covered (its first min(length, max_seqlen) tokens), in a fixed order.
__global__ void __launch_bounds__(256)
rowsum_reduce_varlen_kernel(const float* rows, float* out, const int* cu_seqlens, int H, int64_t total, int max_seqlen) {
  __shared__ float part[256];
  const int bh = blockIdx.x, tid = threadIdx.x, b = bh / H, h = bh % H;
  const int t0 = cu_seqlens[b], n = min(cu_seqlens[b + 1] - t0, max_seqlen);
  const float* r = rows + (int64_t)h * total + t0;
  float acc = 0.f;
  for (int i = tid; i < n; i += 256) acc += r[i];
  part[tid] = acc;
  __syncthreads();
#pragma unroll
  for (int m = 128; m >= 1; m >>= 1) {
    if (tid < m) part[tid] += part[tid + m];
    __syncthreads();
  }
  if (tid == 0) out[bh] = part[0];
}

// Validate one tensor and turn it into a TensorRef.  Strides are in elements.
int make_ref(const void* ptr, const sattn_strides* s, int H, int N, int d, sattn_dtype dt, TensorRef* out) {
  if (!ptr) return SATTN_ERR_NULL;
  const int64_t per16 = 16 / elem_size(dt);
  int64_t sb, sh, ss;
  if (s) {
    sb = s->batch; sh = s->head; ss = s->seq;
  } else {
    ss = d; sh = (int64_t)N * d; sb = (int64_t)H * N * d;
  }
  if (((uintptr_t)ptr & 15) != 0) return SATTN_ERR_ALIGN;
  if (sb % per16 || sh % per16 || ss % per16 || ss < d) return SATTN_ERR_ALIGN;
  // the kernels address the rows of one (batch, head) slice with 32-bit byte offsets
  if (((int64_t)N + 256) * ss * elem_size(dt) > 0xffffffffLL) return SATTN_ERR_SHAPE;
  out->ptr = const_cast<void*>(ptr);
  out->sb = sb; out->sh = sh; out->ss = ss;
  return SATTN_OK;
}

// Shape of a forward workgroup: waves (32 query rows each) and depth of the V ring.
// Head dimension 64: two 4-wave workgroups share a compute unit (their LDS rings both fit) and
// overlap each other's barriers, which measured faster than one 8-wave workgroup at every size.
// Head dimension 128: the 96 KB ring of the three-slot V ring admits one workgroup per compute
// unit, so 4 waves halve the occupancy; that only pays while the problem is too small to give
// every compute unit an 8-wave workgroup (causal problems a little longer: their workgroups run
// heavy-first, so a second, light round costs less than idle compute units in the first).  With a
// two-slot V ring (80 KB) two 4-wave workgroups fit again; they win while a workgroup's key loop
// is short (per-workgroup prologue, diagonal and barrier waits overlap with the neighbour) and
// lose a few percent on long loops, where V is staged only one tile ahead.
std::atomic<int> g_fwd_waves{0};   // 0: choose per problem; 4, 8, 64, 65, 66: forced; 32: choose among the 32-row shapes
std::atomic<int> g_fwd_vslots{0};  // 0: choose per problem; 2 or 3: forced (sattn_set_fwd_v_slots)
std::atomic<int> g_bwd_merged{0};  // 0: choose per problem; 1: one grid wherever that form exists; 2: never; 3: never, and single blocks (sattn_set_bwd_merged)
std::atomic<long long*> g_clock_out{nullptr};  // sattn_set_clock_probe
std::atomic<int> g_clock_cap{0};
ClockProbe clock_probe() { return ClockProbe{g_clock_out.load(std::memory_order_relaxed), g_clock_cap.load(std::memory_order_relaxed)}; }

int compute_units() {
  int dev = 0, n = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) {
    (void)hipGetLastError();
    return 256;
  }
  return n;
}

struct FwdShape { int waves, v_slots; };

// allow64 = false: the choice among the 32-row shapes only (the kernels that have no 64-row form)
FwdShape pick_fwd_shape(int B, int H, int N, int d, int causal, bool allow64 = true) {
  int forced_waves = g_fwd_waves.load(std::memory_order_relaxed);
  if (forced_waves == 32) { allow64 = false; forced_waves = 0; }
  FwdShape s{8, 3};
  if (d == 64) {
    s.waves = 4;
  } else {
    const int64_t wg4 = (int64_t)B * H * ((N + 127) / 128);
    const int64_t cus = compute_units();
    const int64_t avg_tiles = (causal ? (N + 1) / 2 : N) / 64;  // 64-key tiles a workgroup visits on average
    if (wg4 <= (causal ? cus + cus / 2 : cus)) s = FwdShape{4, 3};
    else if (avg_tiles < (causal ? 16 : 48)) s = FwdShape{4, 2};
    // Long key loops with at least one 256-row workgroup per compute unit: four waves of 64 query
    // rows, which read half as much K/V from LDS per MFMA (waves = 64).  From a sweep over B, N
    // and the mask (with the causal launches walking several heads abreast, head_and_rank): 3-12 %
    // faster than the best 32-row shape from 16 tiles per workgroup on average with the causal
    // mask (N >= 2048) and from 24 without (N >= 1536); slower below.
    const int64_t wg64 = (int64_t)B * H * ((N + 255) / 256);
    if (allow64 && wg64 >= cus && avg_tiles >= (causal ? 16 : 24)) s = FwdShape{64, 3};
  }
  const int forced_vslots = g_fwd_vslots.load(std::memory_order_relaxed);
  if (forced_waves) {
    if (forced_waves != s.waves) s.v_slots = 3;
    s.waves = forced_waves;
  }
  if (forced_vslots) s.v_slots = forced_vslots;
  if (s.waves >= 64 && (d != 128 || !allow64)) s = FwdShape{4, 3};  // (a forced 64 where no such kernel exists)
  if (s.waves != 4 || d != 128) s.v_slots = 3;  // the only shape with a two-slot V ring
  return s;
}

// The two passes of the sigmoid backward as one grid (where the launcher has that form: both
// passes asked for, self-attention, one K/V head per query head).  It pays
//  - while a pass alone cannot fill the chip: 10-28 % faster below two workgroups per pass and
//    compute unit under the causal mask; without it (equal workgroups) below three, where the one
//    grid takes fewer rounds than the two launches (per unit, d 128: 0.47 workgroups 18.7 -> 10.8 us,
//    but 1.83: 36.2 / 39.0, 1: 67.1 / 69.2, 2: 132 / 134);
//  - where two workgroups share a unit (d = 64, `two_per_cu`) up to six: B32 H12 N250 54.0 -> 48.9 us,
//    B24 H16 N384 82.9 -> 74.8, causal B6 H16 N1024 86.1 -> 70.1; from eight on two launches are 1-3 %
//    faster without the mask;
//  - where the causal launches, which deal blocks out in pairs, would leave more than 4 % of their
//    rounds of pairs empty (wgs / 2 not a multiple of the units): per unit 3 workgroups d 128 156 -> 133 us,
//    5: 237 -> 216, 9: 655 -> 630, 15: 1077 -> 1057; at multiples two launches are 4-6 % faster
//    (2: 85 / 90, 4: 170 / 176, 6: 250 / 264);
//  - for packed sequences, whose blocks differ in length, up to six per unit, nine at d = 64 (wgs
//    counts the longest length's blocks): B32 H12 50 .. 500 tokens causal d 128 206 -> 171 us, d 64
//    101 -> 89; 24 sequences of up to 1600 (9.75 per unit) d 64 259 / 273.
bool pick_bwd_merged(int B, int H, int N, int causal, bool two_per_cu, bool packed) {
  const int mode = g_bwd_merged.load(std::memory_order_relaxed);
  if (mode) return mode == 1;
  const int64_t nb = (N + 127) / 128, wgs = (int64_t)B * H * nb, cus = compute_units();
  if (packed) return wgs <= (two_per_cu ? 9 : 6) * cus;
  if (two_per_cu && wgs <= 6 * cus) return true;
  if (!causal || nb == 1) return wgs < 3 * cus && (2 * wgs + cus - 1) / cus < 2 * ((wgs + cus - 1) / cus);
  if (wgs < 2 * cus) return true;
  if (nb % 2 != 0 || nb < 4) return false;
  const int64_t pairs = wgs / 2, places = (pairs + cus - 1) / cus * cus;
  return (places - pairs) * 25 > places;
}

// The forward that holds a head whole (sattn_fwd_short.hpp).  Up to 128 keys always, but for a few causal
// heads of at most 48 tokens at d = 128 (one round of workgroups; us, streaming / this: N33 4 heads 5.4 / 5.8, N48
// 1.04 times as long, N64 0.96; of 257 to 512 heads N33 0.71).  Up to 256 keys at d = 64 from more heads than half the
// units on, where the two workgroups a head of the other kernels no longer each find a compute unit to
// themselves (N250 16 heads 7.8 / 8.9, 144 heads 10.9 / 9.5), but where unmasked heads of seven or eight
// blocks are one to one and a half a unit: some units hold two heads and some one, where the streaming kernel's
// smaller workgroups still share them out (N240 1.03 to 1.08 times as long with 257 to 383 heads, N208
// 1.00; 384 heads 0.99; causal 0.85 to 0.93).  Packed batches of one to one and a half heads a unit go 0.77 to
// 1.16 times as long, by how their lengths fall on the units, 0.95 on average.
bool pick_fwd_short(int64_t heads, int N, int d, int causal) {
  if (g_fwd_waves.load(std::memory_order_relaxed) != 0 || g_fwd_vslots.load(std::memory_order_relaxed) != 0) return false;
  if (heads > (1 << 21)) return false;
  const int cus = compute_units();
  if (N <= 128) return d == 64 || !causal || N > 48 || heads > cus;
  if (d != 64 || N > 256 || 2 * heads <= cus) return false;
  return causal || N <= 192 || heads <= cus || 2 * heads >= 3 * cus;
}

// The backward that holds a head whole (sattn_bwd_short.hpp), for every sequence short enough but where
// the two passes' four workgroups a head all find a place at once and nothing is masked (d64 N250 16 heads
// 12.5 us against 13.2, 64 heads 13.1 / 13.8; causal 0.85 of the passes' time with 72 heads, 0.97 with 64, but N256,
// where nothing is ragged and the passes run no step in its compiler-scheduled form, 1.05 to 1.07 up to 64
// heads and 0.87 with 72; N128: 9.3 / 7.2 us).  With the row sums of dS (`rows`) every head takes two workgroups,
// which pays up to 128 tokens (64 heads 9.3 / 7.3, 384: 18.1 / 15.3; d128 512 heads 54.7 / 50.3), not beyond (384 heads
// N250 43.5 / 44.3).  Not for ALiBi under the mask or with the row sums: the passes add its terms in orders of their own.
bool pick_bwd_short(int64_t heads, int N, int d, int causal, bool alibi, bool rows) {
  if (alibi && (causal || rows)) return false;
  if (g_bwd_merged.load(std::memory_order_relaxed) != 0 || N > (d == 64 && !rows ? 256 : 128)) return false;
  if (heads > (1 << 21)) return false;  // two workgroups a head of up to 512 work-items, which a launch counts in 32 bits
  if (d == 128 || N <= 128) return true;
  return causal ? N < 256 || 4 * heads > compute_units() : 2 * heads > compute_units();
}
// Its heads that take one workgroup.  What is left over after whole rounds of the chip takes two, one
// for dK and dV and one for dQ, where these still fit one round (us, one / two workgroups for
// the rest: 384 heads N250 d64 36.6 / 34.3, 16 heads 16.2 / 13.2; 384 heads N100 d128 30.6 / 28.6; where
// they do not fit: 144 heads N250 17.9 / 22.9).
int short_whole_heads(int64_t heads, int N, int d) {
  const int64_t places = (int64_t)compute_units() * (d == 64 && N <= 128 ? 2 : 1), rest = heads % places;
  return (int)(2 * rest <= places ? heads - rest : heads);
}

// Workgroups over which the dK/dV pass splits the query heads of one K/V head (a power of two
// that divides the group): one per K/V head and key block leaves compute units idle when there
// are few K/V heads -- with one K/V head, 8 sequences of 4096 tokens make 256 workgroups of
// unequal causal work -- so the group is split until the pass has two workgroups per compute
// unit under the causal mask (enough to deal the blocks out in pairs of equal work), one without.
// At d = 64, where two workgroups share a unit, it is split once more if that leaves some units with
// two (pairs of) workgroups and others with one: B7 H16 N5119 causal with one K/V head 1771 -> 1626 us,
// B3 H32 N3000 with four 578 -> 544; with one on each, a second one gains nothing (B4 H16 N2048 with one
// 166 / 168, B8 H32 N1024 with eight 187 / 190).
int pick_group_split(int B, int Hkv, int group, int N, int d, int causal) {
  const int64_t wgs = (int64_t)B * Hkv * ((N + 127) / 128), want = (int64_t)(causal ? 2 : 1) * compute_units();
  int s = 1;
  while (wgs * s < want && group % (2 * s) == 0) s *= 2;
  if (d == 64 && wgs * s > want && wgs * s < 2 * want && group % (2 * s) == 0) s *= 2;
  return s;
}

int check_shape(int B, int H, int N, int d, sattn_dtype dt) {
  if (dt != SATTN_BF16 && dt != SATTN_F32) return SATTN_ERR_UNSUPPORTED;
  if (d != 64 && d != 128) return SATTN_ERR_UNSUPPORTED;
  if (B <= 0 || H <= 0 || N <= 0) return SATTN_ERR_SHAPE;
  if ((int64_t)N > (1 << 24)) return SATTN_ERR_SHAPE;               // key distances are formed in fp32
  if ((int64_t)B * H * ((N + 31) / 32) > 0x7fffffffLL) return SATTN_ERR_SHAPE;  // 1-D grid of workgroups
  return SATTN_OK;
}

// ---------------------------------------------------------------- forward
// Waves of an fp32 workgroup.  Eight where that still leaves no compute unit with a second
// workgroup (half the chunks per wave), four otherwise (two workgroups per compute unit).
int f32_waves(int64_t wgs, int cus) { return wgs <= cus ? 8 : 4; }

// Runs `one(first workgroup, grid)` for a grid of `wgs` workgroups: the runtime counts the work-items
// of a launch in 32 bits, which packed batches with a large max_seqlen exceed (their workgroups
// beyond a sequence's end return at once).
template <typename Launch>
int launch_f32_grid(int64_t wgs, int threads, Launch one) {
  const int64_t most = ((int64_t)1 << 31) / threads;
  for (int64_t first = 0; first < wgs; first += most)
    if (int rc = one((int)first, dim3((unsigned)std::min(most, wgs - first)))) return rc;
  return SATTN_OK;
}

template <int D, int MODE>
int launch_f32_pass(const F32Params& p, int nb, int heads, int waves, int causal, bool alibi, hipStream_t st) {
  const int cus = compute_units();
  return launch_f32_grid((int64_t)nb * heads, 64 * waves, [&](int first, dim3 grid) {
    int rc = SATTN_OK;
    if (waves == 8)
      SATTN_DISPATCH2(causal, alibi, rc = launch(sigmoid_f32_kernel<D, MODE, A, B2, 8>, grid, dim3(512), f32_lds_bytes<D>(8),
                                                 st, p, nb, heads, cus, first));
    else
      SATTN_DISPATCH2(causal, alibi, rc = launch(sigmoid_f32_kernel<D, MODE, A, B2, 4>, grid, dim3(256), f32_lds_bytes<D>(4),
                                                 st, p, nb, heads, cus, first));
    return rc;
  });
}

template <int D>
int launch_fwd_f32(const F32Params& p, int causal, bool alibi, hipStream_t st) {
  const int nb = (p.N + 31) / 32, heads = p.B * p.H;
  return launch_f32_pass<D, F32_FWD>(p, nb, heads, f32_waves((int64_t)nb * heads, compute_units()), causal, alibi, st);
}

// The forward kernel for few queries (sattn_few.hpp: 32 query rows per workgroup, keys split over
// its eight waves and over n_split workgroups), or n_split = 0 for the kernels of 128 or 256 rows.
// It reads K and V from the L2 once per 32 rows, they once per 128, so it only pays while its
// blocks leave the chip unfilled.  Measured (us, the 128-row kernel / this one): up to one block
// per compute unit it wins -- one query, 4001 keys, d 128: 128 heads 63 / 50, 16 heads 61 / 14; 64
// queries, 8256 keys, 16 heads 125 / 23; 512 queries, 8704 keys, 8 heads (128 blocks) 139 / 48 --
// and at two blocks per unit it is at par for one query (512 heads, 1000 and 2000 keys 26 / 28,
// 48 / 48) and behind for more (256 queries, 4352 keys, 64 heads 75 / 103).
// Splits: as many as give every compute unit one workgroup and every wave a chunk; below 32 chunks
// the second kernel that adds the partial outputs up (3-4 us) costs what the split gains.
// From four keys per query on only: closer to the square every forward shape gives the same bits,
// which sums over the keys in another order would not.
// Without a workspace a single split has too few bytes in flight once a quarter of the units is
// busy with one block per head (128 heads: 63 / 69).
int few_splits(int B, int H, int N, int Nk, bool workspace) {
  const int64_t nb = (N + 31) / 32, blocks = (int64_t)B * H * nb, cus = compute_units();
  if (blocks > cus || (int64_t)Nk < 4 * (int64_t)N) return 0;
  const int64_t chunks = ((int64_t)Nk + 31) / 32;
  if (!workspace) return nb > 1 || blocks <= cus / 4 || chunks < 32 ? 1 : 0;
  return chunks < 32 ? 1 : (int)std::min(cus / blocks, chunks / 8);
}

struct FwdArgs {
  const void *q, *k, *v; void* o; float* lse;
  int B, H, N, d; sattn_dtype dtype; float bias; int causal; const float* slopes;
  const sattn_strides *sq, *sk, *sv, *so; void* stream;
  const int* cu_seqlens = nullptr; const float* bias_vec = nullptr;  // variable-length batches
  int Hkv = 0;                                                       // K/V heads (0: one per query head)
  int Nk = 0;                                                        // keys (0: as many as queries)
  bool end_aligned = false;                                          // queries = the last N positions of the key sequence
  bool split = false;                                                // few queries: the keys may be split over workgroups (workspace)
  void* workspace = nullptr; size_t workspace_bytes = 0;
};

// A key count that differs from the query count: sigmoid attention with one K/V head per query
// head.  Without `end_aligned` plain attention only (no mask, no ALiBi: positions undefined);
// with it the queries sit at the end of the key sequence, which defines both; the bf16 kernels
// then need the offset Nk - N to be a multiple of 32 under the causal mask (a wave's query rows
// and a key chunk must meet in one diagonal chunk), the fp32 kernel takes any.
template <typename Args>
int check_cross(const Args& a, bool softmax, bool pin, int Hkv, int* Nk) {
  *Nk = a.Nk > 0 ? a.Nk : a.N;
  if (*Nk == a.N) return SATTN_OK;
  if (softmax || !pin || a.cu_seqlens || Hkv != a.H) return SATTN_ERR_UNSUPPORTED;
  if (!a.end_aligned && (a.causal || a.slopes)) return SATTN_ERR_UNSUPPORTED;
  if (a.end_aligned && a.causal && a.dtype == SATTN_BF16 && (*Nk - a.N) % 32 != 0) return SATTN_ERR_UNSUPPORTED;
  return check_shape(a.B, a.H, *Nk, a.d, a.dtype);
}

template <bool SOFTMAX, bool PIN = true>
int fwd_impl(const FwdArgs& a) {
  int rc = check_shape(a.B, a.H, a.N, a.d, a.dtype);
  if (rc) return rc;
  const int Hkv = a.Hkv ? a.Hkv : a.H;
  if (Hkv <= 0 || a.H % Hkv) return SATTN_ERR_SHAPE;
  if (Hkv != a.H && (SOFTMAX || !PIN)) return SATTN_ERR_UNSUPPORTED;
  int Nk;
  if ((rc = check_cross(a, SOFTMAX, PIN, Hkv, &Nk))) return rc;
  TensorRef q, k, v, o;
  if ((rc = make_ref(a.q, a.sq, a.H, a.N, a.d, a.dtype, &q))) return rc;
  if ((rc = make_ref(a.k, a.sk, Hkv, Nk, a.d, a.dtype, &k))) return rc;
  if ((rc = make_ref(a.v, a.sv, Hkv, Nk, a.d, a.dtype, &v))) return rc;
  if ((rc = make_ref(a.o, a.so, a.H, a.N, a.d, a.dtype, &o))) return rc;
  if (SOFTMAX && !a.lse) return SATTN_ERR_NULL;
  hipStream_t st = (hipStream_t)a.stream;
  const bool alibi = a.slopes != nullptr;
  const float inv_sqrt_d = 1.0f / sqrtf((float)a.d);
  if (a.dtype == SATTN_F32) {
    if (SOFTMAX || !PIN) return SATTN_ERR_UNSUPPORTED;  // comparison kernels and twins: bf16 only
    F32Params p{};
    p.q = q; p.k = k; p.v = v; p.o = o;
    p.slopes = a.slopes; p.B = a.B; p.H = a.H; p.N = a.N;
    p.scale = inv_sqrt_d; p.bias = a.bias;
    p.cu_seqlens = a.cu_seqlens; p.bias_vec = a.bias_vec;
    p.kv_group = a.H / Hkv;
    p.Nk = Nk == a.N ? 0 : Nk;
    p.qoff = a.end_aligned ? Nk - a.N : 0;
    if (a.d == 128) return launch_fwd_f32<128>(p, a.causal, alibi, st);
    return launch_fwd_f32<64>(p, a.causal, alibi, st);
  }
  FwdParams p{};
  p.q = q; p.k = k; p.v = v; p.o = o;
  p.slopes = a.slopes; p.lse = a.lse;
  p.B = a.B; p.H = a.H; p.N = a.N;
  p.nscale_log2 = (SOFTMAX ? kLog2e : -kLog2e) * inv_sqrt_d;
  p.nbias_log2 = -a.bias * kLog2e;
  p.cu_seqlens = a.cu_seqlens; p.bias_vec = a.bias_vec;
  p.kv_group = a.H / Hkv;
  p.Nk = Nk == a.N ? 0 : Nk;
  p.qoff = a.end_aligned ? Nk - a.N : 0;
  p.clock = clock_probe();
  // the 64-row waves exist for the pinned sigmoid kernel at d = 128, ALiBi only in its causal form
  const bool has64 = !SOFTMAX && PIN && a.d == 128 && !(alibi && !a.causal);
  if (!SOFTMAX && PIN && Nk != a.N && g_fwd_waves.load(std::memory_order_relaxed) == 0) {
    p.n_split = few_splits(a.B, a.H, a.N, Nk, a.split);
    if (p.n_split > 1) {
      const size_t need = (size_t)p.n_split * a.B * a.H * a.N * a.d * sizeof(float);
      if (!a.workspace || a.workspace_bytes < need) return SATTN_ERR_WORKSPACE;
      if (((uintptr_t)a.workspace & 15) != 0) return SATTN_ERR_ALIGN;
      p.part = (float*)a.workspace;
    }
    if (p.n_split > 0)
      return a.d == 128 ? launch_fwd_few<128>(p, a.causal, alibi, st) : launch_fwd_few<64>(p, a.causal, alibi, st);
  }
  if (!SOFTMAX && PIN && Nk == a.N && Hkv == a.H && !alibi && pick_fwd_short((int64_t)a.B * a.H, a.N, a.d, a.causal))
    return a.d == 128 ? launch_fwd_short<128>(p, a.causal, st) : launch_fwd_short<64>(p, a.causal, st);
  const FwdShape shape = pick_fwd_shape(a.B, a.H, a.N, a.d, a.causal, has64);
  // The 64-row causal kernel deals a head's blocks out in pairs of equal work (longest with
  // shortest) where that still leaves a workgroup per compute unit.  Measured against single
  // blocks: 2-3.5 % faster from 16 blocks per head (N >= 4096), 3 % slower at 8 (B16 H16 N2048).
  // (66: single blocks, for that comparison.)
  const int nb64 = (a.N + 255) / 256;
  p.pair = shape.waves != 66 && a.causal && nb64 >= 16 && (int64_t)a.B * a.H * (nb64 / 2) >= compute_units();
  if (a.d == 128) return launch_fwd_bf16<128>(p, shape.waves, shape.v_slots, SOFTMAX, PIN, a.causal, alibi, st);
  return launch_fwd_bf16<64>(p, shape.waves, shape.v_slots, SOFTMAX, PIN, a.causal, alibi, st);
}

// ---------------------------------------------------------------- backward
template <int D>
int launch_bwd_f32(const F32Params& p, int causal, bool alibi, int parts, bool one_grid, hipStream_t st) {
  // the dQ pass runs one workgroup per query head and 32 queries, the dK/dV pass one per K/V
  // head and 32 keys; without `one_grid` after one another
  const int nb_q = (p.N + 31) / 32, nb_k = ((p.Nk > 0 ? p.Nk : p.N) + 31) / 32;
  const int heads_q = p.B * p.H, heads_k = p.B * (p.H / p.kv_group);
  const int64_t wgs = (int64_t)nb_q * heads_q + (int64_t)nb_k * heads_k;
  if (wgs > 0x7fffffffLL) return SATTN_ERR_SHAPE;
  const int cus = compute_units();
  const int waves = f32_waves(wgs, cus);  // the same for a pass alone: its sums then run in the same order
  if (parts == kBwdDkDv) return launch_f32_pass<D, F32_DKDV>(p, nb_k, heads_k, waves, causal, alibi, st);
  if (parts == kBwdDq) return launch_f32_pass<D, F32_DQ>(p, nb_q, heads_q, waves, causal, alibi, st);
  if (!one_grid) {
    const int rc = launch_f32_pass<D, F32_DKDV>(p, nb_k, heads_k, waves, causal, alibi, st);
    return rc == SATTN_OK ? launch_f32_pass<D, F32_DQ>(p, nb_q, heads_q, waves, causal, alibi, st) : rc;
  }
  return launch_f32_grid(wgs, 64 * waves, [&](int first, dim3 grid) {
    int rc = SATTN_OK;
    if (waves == 8)
      SATTN_DISPATCH2(causal, alibi, rc = launch(sigmoid_f32_bwd_kernel<D, A, B2, 8>, grid, dim3(512), f32_lds_bytes<D>(8), st,
                                                 p, nb_k, nb_q, cus, first));
    else
      SATTN_DISPATCH2(causal, alibi, rc = launch(sigmoid_f32_bwd_kernel<D, A, B2, 4>, grid, dim3(256), f32_lds_bytes<D>(4), st,
                                                 p, nb_k, nb_q, cus, first));
    return rc;
  });
}

struct BwdArgs {
  const void *q, *k, *v, *o; const float* lse; const void* dout; void *dq, *dk, *dv;
  int B, H, N, d; sattn_dtype dtype; float bias; int causal; const float* slopes;
  const sattn_strides *sq, *sk, *sv, *so, *sdout, *sdq, *sdk, *sdv;
  void* workspace; size_t workspace_bytes; int parts; void* stream;
  const int* cu_seqlens = nullptr; const float* bias_vec = nullptr;  // variable-length batches
  float* db_rows = nullptr; float* db = nullptr;                     // bias gradient (sigmoid only)
  int64_t db_tokens = 0;                                             // packed sequences: tokens in db_rows' [H, tokens]
  int Hkv = 0;                                                       // K/V heads (0: one per query head)
  int Nk = 0;                                                        // keys (0: as many as queries)
  bool end_aligned = false;                                          // queries = the last N positions of the key sequence
  bool group_split = false;                                          // shared K/V heads: split a group over workgroups (workspace)
};

// The bias gradient per head from the row sums of dS.
template <typename Params>
int reduce_rows(const BwdArgs& a, const Params& p, hipStream_t st) {
  if (a.cu_seqlens)
    return launch(rowsum_reduce_varlen_kernel, dim3(a.B * a.H), dim3(256), 0, st, (const float*)a.db_rows, a.db,
                  a.cu_seqlens, a.H, a.db_tokens, a.N);
  return launch(rowsum_reduce_kernel, dim3(a.B * a.H), dim3(256), 0, st, (const float*)a.db_rows, a.db, a.H, a.N,
                p.db_sb, p.db_sh);
}

template <bool SOFTMAX, bool PIN = true>
int bwd_impl(const BwdArgs& a) {
  int rc = check_shape(a.B, a.H, a.N, a.d, a.dtype);
  if (rc) return rc;
  const int Hkv = a.Hkv ? a.Hkv : a.H;
  if (Hkv <= 0 || a.H % Hkv) return SATTN_ERR_SHAPE;
  if (Hkv != a.H && (SOFTMAX || !PIN)) return SATTN_ERR_UNSUPPORTED;
  int Nk;
  if ((rc = check_cross(a, SOFTMAX, PIN, Hkv, &Nk))) return rc;
  if (Nk != a.N && a.db_rows) return SATTN_ERR_UNSUPPORTED;
  TensorRef q, k, v, dout, dq{}, dk{}, dv{}, o{};
  if ((rc = make_ref(a.q, a.sq, a.H, a.N, a.d, a.dtype, &q))) return rc;
  if ((rc = make_ref(a.k, a.sk, Hkv, Nk, a.d, a.dtype, &k))) return rc;
  if ((rc = make_ref(a.v, a.sv, Hkv, Nk, a.d, a.dtype, &v))) return rc;
  if ((rc = make_ref(a.dout, a.sdout, a.H, a.N, a.d, a.dtype, &dout))) return rc;
  if ((a.parts & kBwdDq) && (rc = make_ref(a.dq, a.sdq, a.H, a.N, a.d, a.dtype, &dq))) return rc;
  if ((a.parts & kBwdDkDv) && (rc = make_ref(a.dk, a.sdk, Hkv, Nk, a.d, a.dtype, &dk))) return rc;
  if ((a.parts & kBwdDkDv) && (rc = make_ref(a.dv, a.sdv, Hkv, Nk, a.d, a.dtype, &dv))) return rc;
  hipStream_t st = (hipStream_t)a.stream;
  const bool alibi = a.slopes != nullptr;
  const float inv_sqrt_d = 1.0f / sqrtf((float)a.d);
  // dQ may replace Q or dO: a workgroup of the dQ pass reads only its own rows of them, but the
  // dK/dV pass reads all rows and has to be through before
  const bool in_place = (a.parts & kBwdDq) && (a.dq == a.q || a.dq == a.dout);
  if (a.dtype == SATTN_F32) {
    if (SOFTMAX || !PIN) return SATTN_ERR_UNSUPPORTED;  // comparison kernels and twins: bf16 only
    F32Params p{};
    p.q = q; p.k = k; p.v = v; p.dout = dout; p.dq = dq; p.dk = dk; p.dv = dv;
    p.slopes = a.slopes; p.B = a.B; p.H = a.H; p.N = a.N;
    p.scale = inv_sqrt_d; p.bias = a.bias;
    p.cu_seqlens = a.cu_seqlens; p.bias_vec = a.bias_vec;
    p.kv_group = a.H / Hkv;
    p.Nk = Nk == a.N ? 0 : Nk;
    p.qoff = a.end_aligned ? Nk - a.N : 0;
    p.db_rows = a.db_rows; p.db_sb = (int64_t)a.H * a.N; p.db_sh = a.N;
    if (a.cu_seqlens && a.db_rows) { p.db_sb = 0; p.db_sh = a.db_tokens; }  // [H, tokens], as in the bf16 path
    if (a.d == 128) rc = launch_bwd_f32<128>(p, a.causal, alibi, a.parts, !in_place, st);
    else rc = launch_bwd_f32<64>(p, a.causal, alibi, a.parts, !in_place, st);
    if (rc == SATTN_OK && a.db) rc = reduce_rows(a, p, st);
    return rc;
  }
  BwdParams p{};
  p.q = q; p.k = k; p.v = v; p.dout = dout; p.dq = dq; p.dk = dk; p.dv = dv;
  p.slopes = a.slopes;
  p.B = a.B; p.H = a.H; p.N = a.N;
  p.inv_sqrt_d = inv_sqrt_d;
  p.nscale_log2 = -kLog2e * inv_sqrt_d;
  p.nbias_log2 = -a.bias * kLog2e;
  p.cu_seqlens = a.cu_seqlens; p.bias_vec = a.bias_vec;
  p.db_rows = a.db_rows; p.db_sb = (int64_t)a.H * a.N; p.db_sh = a.N;
  if (a.cu_seqlens && a.db_rows) { p.db_sb = 0; p.db_sh = a.db_tokens; }  // [H, tokens]: the kernel adds the sequence's first token
  p.kv_group = a.H / Hkv;
  p.Nk = Nk == a.N ? 0 : Nk;
  p.qoff = a.end_aligned ? Nk - a.N : 0;
  p.clock = clock_probe();
  if (SOFTMAX) {
    if (!a.lse) return SATTN_ERR_NULL;
    if ((rc = make_ref(a.o, a.so, a.H, a.N, a.d, a.dtype, &o))) return rc;
    const int npad = (a.N + 63) / 64 * 64;
    const int64_t prows = (int64_t)a.B * a.H * npad;
    const size_t need = 2 * (size_t)prows * sizeof(float);
    if (!a.workspace || a.workspace_bytes < need) return SATTN_ERR_WORKSPACE;
    if (((uintptr_t)a.workspace & 15) != 0) return SATTN_ERR_ALIGN;
    if ((prows + 15) / 16 > 0x7fffffffLL) return SATTN_ERR_SHAPE;
    float* nlse2 = (float*)a.workspace;
    float* dvec = nlse2 + prows;
    dim3 grid((unsigned)((prows + 15) / 16)), block(256);
    if (a.d == 128)
      rc = launch(softmax_bwd_prepass_kernel<128>, grid, block, 0, st, o, dout, a.lse, nlse2, dvec, a.B, a.H, a.N, npad);
    else
      rc = launch(softmax_bwd_prepass_kernel<64>, grid, block, 0, st, o, dout, a.lse, nlse2, dvec, a.B, a.H, a.N, npad);
    if (rc) return rc;
    p.nlse2 = nlse2; p.dvec = dvec; p.npad = npad;
  }
  if (!SOFTMAX && PIN && !in_place && Hkv == a.H && Nk == a.N && a.parts == (kBwdDkDv | kBwdDq) &&
      pick_bwd_short((int64_t)a.B * a.H, a.N, a.d, a.causal, alibi, a.db_rows != nullptr)) {
    const int whole = a.db_rows ? 0 : short_whole_heads((int64_t)a.B * a.H, a.N, a.d);
    rc = a.d == 128 ? launch_bwd_short<128>(p, a.causal, alibi, whole, st) : launch_bwd_short<64>(p, a.causal, alibi, whole, st);
    return rc == SATTN_OK && a.db ? reduce_rows(a, p, st) : rc;
  }
  const bool merged = !in_place && pick_bwd_merged(a.B, a.H, a.N, a.causal, a.d == 64 && !SOFTMAX, a.cu_seqlens != nullptr);
  int n_split = 1;
  if (a.group_split && !SOFTMAX && PIN && Hkv != a.H && !a.cu_seqlens && Nk == a.N && (a.parts & kBwdDkDv)) {
    n_split = pick_group_split(a.B, Hkv, a.H / Hkv, a.N, a.d, a.causal);
    if (n_split > 1) {
      const size_t one = 2 * (size_t)a.B * Hkv * a.N * a.d * sizeof(float);  // fp32 dK, dV of one split
      const bool room = a.workspace && a.workspace_bytes >= one * n_split, aligned = ((uintptr_t)a.workspace & 15) == 0;
      // The further split of d = 64 is taken only where the workspace serves it: what the rule of d = 128
      // asks for is enough, nothing where that does not split.
      const int fewer = pick_group_split(a.B, Hkv, a.H / Hkv, a.N, 128, a.causal);
      if (!room || !aligned) n_split = fewer;
      if (n_split > 1) {
        if (!a.workspace || a.workspace_bytes < one * n_split) return SATTN_ERR_WORKSPACE;
        if (!aligned) return SATTN_ERR_ALIGN;
        p.n_split = n_split;
        p.part = (float*)a.workspace;
      }
    }
  }
  // causal passes deal a head's blocks out in pairs of equal work (longest with shortest) where
  // a pair per compute unit remains (see the 64-row forward)
  p.pair = a.causal && PIN && g_bwd_merged.load(std::memory_order_relaxed) != 3 &&
           (int64_t)a.B * Hkv * n_split * ((std::min(a.N, Nk) + 127) / 128 / 2) >= compute_units();
  if (a.d == 128) rc = launch_bwd_bf16<128>(p, SOFTMAX, PIN, a.causal, alibi, a.parts, merged, st);
  else rc = launch_bwd_bf16<64>(p, SOFTMAX, PIN, a.causal, alibi, a.parts, merged, st);
  if (rc == SATTN_OK && a.db) rc = reduce_rows(a, p, st);
  return rc;
}

template <bool RMS, bool BACKWARD>
int launch_norm(const NormParams& p, hipStream_t st) {
  const int nchunks = p.H * (p.d / 8);
  const int64_t tokens = (int64_t)p.B * p.N;
  dim3 grid((unsigned)((tokens + 3) / 4)), grid2((unsigned)((tokens + 7) / 8)), grid4((unsigned)((tokens + 15) / 16)), block(256);
  if (nchunks <= 16) return launch(headconcat_norm_kernel<1, 16, RMS, BACKWARD>, grid4, block, 0, st, p);
  if (nchunks <= 32) return launch(headconcat_norm_kernel<1, 32, RMS, BACKWARD>, grid2, block, 0, st, p);
  if (nchunks <= 64) return launch(headconcat_norm_kernel<1, 64, RMS, BACKWARD>, grid, block, 0, st, p);
  if (nchunks <= 128) return launch(headconcat_norm_kernel<2, 64, RMS, BACKWARD>, grid, block, 0, st, p);
  if (nchunks <= 256) return launch(headconcat_norm_kernel<4, 64, RMS, BACKWARD>, grid, block, 0, st, p);
  if (nchunks <= 512) return launch(headconcat_norm_kernel<8, 64, RMS, BACKWARD>, grid, block, 0, st, p);
  return launch(headconcat_norm_kernel<16, 64, RMS, BACKWARD>, grid, block, 0, st, p);
}

int norm_impl(bool backward, const void* x, const void* dy, void* out, float* stats, int B, int H, int N, int d,
              sattn_dtype dtype, int kind, float eps, const sattn_strides* sx, const sattn_strides* sdy,
              const sattn_strides* sout, void* stream) {
  int rc = check_shape(B, H, N, d, dtype);
  if (rc) return rc;
  if (dtype != SATTN_BF16 || (kind != SATTN_NORM_LAYER && kind != SATTN_NORM_RMS)) return SATTN_ERR_UNSUPPORTED;
  if ((int64_t)H * d > 8192) return SATTN_ERR_SHAPE;  // a wave keeps one token's features in registers
  if (((int64_t)B * N + 3) / 4 > 0x7fffffffLL) return SATTN_ERR_SHAPE;  // 1-D grid, four tokens per workgroup
  if (!(eps >= 0.f)) return SATTN_ERR_SHAPE;
  if (!stats) return SATTN_ERR_NULL;
  if (((uintptr_t)stats & 7) != 0) return SATTN_ERR_ALIGN;
  NormParams p{};
  if ((rc = make_ref(x, sx, H, N, d, dtype, &p.x))) return rc;
  if ((rc = make_ref(out, sout, H, N, d, dtype, &p.y))) return rc;
  if (backward && (rc = make_ref(dy, sdy, H, N, d, dtype, &p.dy))) return rc;
  p.stats = stats; p.B = B; p.H = H; p.N = N; p.d = d; p.eps = eps;
  hipStream_t st = (hipStream_t)stream;
  if (kind == SATTN_NORM_RMS) return backward ? launch_norm<true, true>(p, st) : launch_norm<true, false>(p, st);
  return backward ? launch_norm<false, true>(p, st) : launch_norm<false, false>(p, st);
}

}  // namespace

extern "C" {

int sigmoid_attn_fwd(const void* q, const void* k, const void* v, void* o, int B, int H, int N, int d,
                     sattn_dtype dtype, float bias, int causal, const float* alibi_slopes, const sattn_strides* sq,
                     const sattn_strides* sk, const sattn_strides* sv, const sattn_strides* so, void* stream) {
  FwdArgs a{q, k, v, o, nullptr, B, H, N, d, dtype, bias, causal, alibi_slopes, sq, sk, sv, so, stream};
  return fwd_impl<false>(a);
}

int sigmoid_attn_bwd(const void* q, const void* k, const void* v, const void* dout, void* dq, void* dk, void* dv,
                     int B, int H, int N, int d, sattn_dtype dtype, float bias, int causal,
                     const float* alibi_slopes, const sattn_strides* sq, const sattn_strides* sk,
                     const sattn_strides* sv, const sattn_strides* sdout, const sattn_strides* sdq,
                     const sattn_strides* sdk, const sattn_strides* sdv, void* workspace, size_t workspace_bytes,
                     void* stream) {
  // the split by output owner needs no workspace
  BwdArgs a{q, k, v, nullptr, nullptr, dout, dq, dk, dv, B, H, N, d, dtype, bias, causal, alibi_slopes,
            sq, sk, sv, nullptr, sdout, sdq, sdk, sdv, workspace, workspace_bytes, kBwdDkDv | kBwdDq, stream};
  return bwd_impl<false>(a);
}

int sigmoid_attn_bwd_dkdv(const void* q, const void* k, const void* v, const void* dout, void* dk, void* dv,
                          int B, int H, int N, int d, sattn_dtype dtype, float bias, int causal,
                          const float* alibi_slopes, const sattn_strides* sq, const sattn_strides* sk,
                          const sattn_strides* sv, const sattn_strides* sdout, const sattn_strides* sdk,
                          const sattn_strides* sdv, void* stream) {
  BwdArgs a{q, k, v, nullptr, nullptr, dout, nullptr, dk, dv, B, H, N, d, dtype, bias, causal, alibi_slopes,
            sq, sk, sv, nullptr, sdout, nullptr, sdk, sdv, nullptr, 0, kBwdDkDv, stream};
  return bwd_impl<false>(a);
}

int sigmoid_attn_bwd_dq(const void* q, const void* k, const void* v, const void* dout, void* dq, int B, int H,
                        int N, int d, sattn_dtype dtype, float bias, int causal, const float* alibi_slopes,
                        const sattn_strides* sq, const sattn_strides* sk, const sattn_strides* sv,
                        const sattn_strides* sdout, const sattn_strides* sdq, void* stream) {
  BwdArgs a{q, k, v, nullptr, nullptr, dout, dq, nullptr, nullptr, B, H, N, d, dtype, bias, causal, alibi_slopes,
            sq, sk, sv, nullptr, sdout, sdq, nullptr, nullptr, nullptr, 0, kBwdDq, stream};
  return bwd_impl<false>(a);
}

int sigmoid_attn_bwd_bias_grad(const void* q, const void* k, const void* v, const void* dout, void* dq, void* dk,
                               void* dv, float* db_rows, float* db, int B, int H, int N, int d, sattn_dtype dtype,
                               float bias, int causal, const float* alibi_slopes, const sattn_strides* sq,
                               const sattn_strides* sk, const sattn_strides* sv, const sattn_strides* sdout,
                               const sattn_strides* sdq, const sattn_strides* sdk, const sattn_strides* sdv,
                               void* stream) {
  if (!db_rows) return SATTN_ERR_NULL;
  if (((uintptr_t)db_rows & 3) != 0 || ((uintptr_t)db & 3) != 0) return SATTN_ERR_ALIGN;
  BwdArgs a{q, k, v, nullptr, nullptr, dout, dq, dk, dv, B, H, N, d, dtype, bias, causal, alibi_slopes,
            sq, sk, sv, nullptr, sdout, sdq, sdk, sdv, nullptr, 0, kBwdDkDv | kBwdDq, stream};
  a.db_rows = db_rows; a.db = db;
  return bwd_impl<false>(a);
}

size_t sigmoid_attn_bwd_workspace_bytes(int, int, int, int, sattn_dtype) { return 0; }

int sigmoid_attn_fwd_compiler_scheduled(const void* q, const void* k, const void* v, void* o, int B, int H, int N,
                                        int d, sattn_dtype dtype, float bias, int causal, const float* alibi_slopes,
                                        const sattn_strides* sq, const sattn_strides* sk, const sattn_strides* sv,
                                        const sattn_strides* so, void* stream) {
  FwdArgs a{q, k, v, o, nullptr, B, H, N, d, dtype, bias, causal, alibi_slopes, sq, sk, sv, so, stream};
  return fwd_impl<false, false>(a);
}

int sigmoid_attn_bwd_compiler_scheduled(const void* q, const void* k, const void* v, const void* dout, void* dq,
                                        void* dk, void* dv, int B, int H, int N, int d, sattn_dtype dtype, float bias,
                                        int causal, const float* alibi_slopes, const sattn_strides* sq,
                                        const sattn_strides* sk, const sattn_strides* sv, const sattn_strides* sdout,
                                        const sattn_strides* sdq, const sattn_strides* sdk, const sattn_strides* sdv,
                                        void* workspace, size_t workspace_bytes, void* stream) {
  BwdArgs a{q, k, v, nullptr, nullptr, dout, dq, dk, dv, B, H, N, d, dtype, bias, causal, alibi_slopes,
            sq, sk, sv, nullptr, sdout, sdq, sdk, sdv, workspace, workspace_bytes, kBwdDkDv | kBwdDq, stream};
  return bwd_impl<false, false>(a);
}

int softmax_attn_fwd(const void* q, const void* k, const void* v, void* o, float* lse, int B, int H, int N, int d,
                     sattn_dtype dtype, int causal, const float* alibi_slopes, const sattn_strides* sq,
                     const sattn_strides* sk, const sattn_strides* sv, const sattn_strides* so, void* stream) {
  FwdArgs a{q, k, v, o, lse, B, H, N, d, dtype, 0.0f, causal, alibi_slopes, sq, sk, sv, so, stream};
  return fwd_impl<true>(a);
}

int softmax_attn_fwd_compiler_scheduled(const void* q, const void* k, const void* v, void* o, float* lse, int B, int H,
                                        int N, int d, sattn_dtype dtype, int causal, const float* alibi_slopes,
                                        const sattn_strides* sq, const sattn_strides* sk, const sattn_strides* sv,
                                        const sattn_strides* so, void* stream) {
  FwdArgs a{q, k, v, o, lse, B, H, N, d, dtype, 0.0f, causal, alibi_slopes, sq, sk, sv, so, stream};
  return fwd_impl<true, false>(a);
}

int softmax_attn_bwd(const void* q, const void* k, const void* v, const void* o, const float* lse, const void* dout,
                     void* dq, void* dk, void* dv, int B, int H, int N, int d, sattn_dtype dtype, int causal,
                     const float* alibi_slopes, const sattn_strides* sq, const sattn_strides* sk,
                     const sattn_strides* sv, const sattn_strides* so, const sattn_strides* sdout,
                     const sattn_strides* sdq, const sattn_strides* sdk, const sattn_strides* sdv, void* workspace,
                     size_t workspace_bytes, void* stream) {
  BwdArgs a{q, k, v, o, lse, dout, dq, dk, dv, B, H, N, d, dtype, 0.0f, causal, alibi_slopes,
            sq, sk, sv, so, sdout, sdq, sdk, sdv, workspace, workspace_bytes, kBwdDkDv | kBwdDq, stream};
  return bwd_impl<true>(a);
}

int softmax_attn_bwd_compiler_scheduled(const void* q, const void* k, const void* v, const void* o, const float* lse,
                                        const void* dout, void* dq, void* dk, void* dv, int B, int H, int N, int d,
                                        sattn_dtype dtype, int causal, const float* alibi_slopes,
                                        const sattn_strides* sq, const sattn_strides* sk, const sattn_strides* sv,
                                        const sattn_strides* so, const sattn_strides* sdout, const sattn_strides* sdq,
                                        const sattn_strides* sdk, const sattn_strides* sdv, void* workspace,
                                        size_t workspace_bytes, void* stream) {
  BwdArgs a{q, k, v, o, lse, dout, dq, dk, dv, B, H, N, d, dtype, 0.0f, causal, alibi_slopes,
            sq, sk, sv, so, sdout, sdq, sdk, sdv, workspace, workspace_bytes, kBwdDkDv | kBwdDq, stream};
  return bwd_impl<true, false>(a);
}

size_t softmax_attn_bwd_workspace_bytes(int B, int H, int N, int d, sattn_dtype dtype) {
  if (check_shape(B, H, N, d, dtype) != SATTN_OK) return 0;
  // rowsum(dO o O) and the rescaled log-sum-exp: two fp32 per query row, rows padded to 64
  return 2 * (size_t)B * H * ((N + 63) / 64 * 64) * sizeof(float);
}

size_t softmax_attn_bwd_noalloc_max_rows(void) { return kNoAllocRows; }

int softmax_attn_bwd_noalloc(const void* q, const void* k, const void* v, const void* o, const float* lse,
                             const void* dout, void* dq, void* dk, void* dv, int B, int H, int N, int d,
                             sattn_dtype dtype, int causal, const float* alibi_slopes, const sattn_strides* sq,
                             const sattn_strides* sk, const sattn_strides* sv, const sattn_strides* so,
                             const sattn_strides* sdout, const sattn_strides* sdq, const sattn_strides* sdk,
                             const sattn_strides* sdv, void* stream) {
  int rc = check_shape(B, H, N, d, dtype);
  if (rc) return rc;
  // the pre-pass writes every padded row it later reads, so the last call's contents need no clearing
  const size_t rows = (size_t)B * H * ((size_t)(N + 63) / 64 * 64);
  if (rows > kNoAllocRows) return SATTN_ERR_TOO_LARGE;
  float* ws = nullptr;
  if ((rc = scratch_on_current_device(&ws))) return rc;
  BwdArgs a{q, k, v, o, lse, dout, dq, dk, dv, B, H, N, d, dtype, 0.0f, causal, alibi_slopes,
            sq, sk, sv, so, sdout, sdq, sdk, sdv, ws, 2 * kNoAllocRows * sizeof(float), kBwdDkDv | kBwdDq, stream};
  return bwd_impl<true>(a);
}

const char* sattn_strerror(int code) {
  switch (code) {
    case SATTN_OK: return "success";
    case SATTN_ERR_NULL: return "a required pointer is NULL";
    case SATTN_ERR_SHAPE: return "B, H and N must be positive and within the supported range";
    case SATTN_ERR_UNSUPPORTED: return "unsupported head dimension or dtype (d must be 64 or 128; softmax is bf16 only)";
    case SATTN_ERR_ALIGN: return "pointers and strides must keep rows 16-byte aligned";
    case SATTN_ERR_WORKSPACE: return "workspace missing or too small";
    case SATTN_ERR_LAUNCH: return "the HIP runtime rejected the kernel launch";
    case SATTN_ERR_TOO_LARGE: return "problem exceeds the fixed scratch of the allocation-free entry point";
    default: return "unknown error code";
  }
}

// Packed [tokens, H, d] strides for a variable-length call: batch stride 0; head and token
// strides from the caller, or contiguous.
static sattn_strides varlen_strides(const sattn_strides* s, int H, int d) {
  sattn_strides r;
  r.batch = 0;
  r.head = s ? s->head : d;
  r.seq = s ? s->seq : (int64_t)H * d;
  return r;
}

int sigmoid_attn_varlen_fwd(const void* q, const void* k, const void* v, void* o, const int32_t* cu_seqlens,
                            const float* bias_per_seq, int B, int H, int max_seqlen, int d, sattn_dtype dtype,
                            float bias, int causal, const float* alibi_slopes, const sattn_strides* sq,
                            const sattn_strides* sk, const sattn_strides* sv, const sattn_strides* so,
                            void* stream) {
  if (!cu_seqlens) return SATTN_ERR_NULL;
  const sattn_strides tq = varlen_strides(sq, H, d), tk = varlen_strides(sk, H, d), tv = varlen_strides(sv, H, d),
                      to = varlen_strides(so, H, d);
  FwdArgs a{q, k, v, o, nullptr, B, H, max_seqlen, d, dtype, bias, causal, alibi_slopes, &tq, &tk, &tv, &to, stream};
  a.cu_seqlens = cu_seqlens; a.bias_vec = bias_per_seq;
  return fwd_impl<false>(a);
}

int sigmoid_attn_varlen_bwd(const void* q, const void* k, const void* v, const void* dout, void* dq, void* dk,
                            void* dv, const int32_t* cu_seqlens, const float* bias_per_seq, int B, int H,
                            int max_seqlen, int d, sattn_dtype dtype, float bias, int causal,
                            const float* alibi_slopes, const sattn_strides* sq, const sattn_strides* sk,
                            const sattn_strides* sv, const sattn_strides* sdout, const sattn_strides* sdq,
                            const sattn_strides* sdk, const sattn_strides* sdv, void* stream) {
  if (!cu_seqlens) return SATTN_ERR_NULL;
  const sattn_strides tq = varlen_strides(sq, H, d), tk = varlen_strides(sk, H, d), tv = varlen_strides(sv, H, d),
                      tdo = varlen_strides(sdout, H, d), tdq = varlen_strides(sdq, H, d),
                      tdk = varlen_strides(sdk, H, d), tdv = varlen_strides(sdv, H, d);
  BwdArgs a{q, k, v, nullptr, nullptr, dout, dq, dk, dv, B, H, max_seqlen, d, dtype, bias, causal, alibi_slopes,
            &tq, &tk, &tv, nullptr, &tdo, &tdq, &tdk, &tdv, nullptr, 0, kBwdDkDv | kBwdDq, stream};
  a.cu_seqlens = cu_seqlens; a.bias_vec = bias_per_seq;
  return bwd_impl<false>(a);
}

int sigmoid_attn_varlen_bwd_bias_grad(const void* q, const void* k, const void* v, const void* dout, void* dq,
                                      void* dk, void* dv, float* db_rows, float* db, const int32_t* cu_seqlens,
                                      const float* bias_per_seq, int B, int H, int max_seqlen, int64_t total_tokens,
                                      int d, sattn_dtype dtype, float bias, int causal, const float* alibi_slopes,
                                      const sattn_strides* sq, const sattn_strides* sk, const sattn_strides* sv,
                                      const sattn_strides* sdout, const sattn_strides* sdq, const sattn_strides* sdk,
                                      const sattn_strides* sdv, void* stream) {
  if (!cu_seqlens || !db_rows) return SATTN_ERR_NULL;
  if (((uintptr_t)db_rows & 3) != 0 || ((uintptr_t)db & 3) != 0) return SATTN_ERR_ALIGN;
  if (total_tokens <= 0) return SATTN_ERR_SHAPE;
  const sattn_strides tq = varlen_strides(sq, H, d), tk = varlen_strides(sk, H, d), tv = varlen_strides(sv, H, d),
                      tdo = varlen_strides(sdout, H, d), tdq = varlen_strides(sdq, H, d),
                      tdk = varlen_strides(sdk, H, d), tdv = varlen_strides(sdv, H, d);
  BwdArgs a{q, k, v, nullptr, nullptr, dout, dq, dk, dv, B, H, max_seqlen, d, dtype, bias, causal, alibi_slopes,
            &tq, &tk, &tv, nullptr, &tdo, &tdq, &tdk, &tdv, nullptr, 0, kBwdDkDv | kBwdDq, stream};
  a.cu_seqlens = cu_seqlens; a.bias_vec = bias_per_seq;
  a.db_rows = db_rows; a.db = db; a.db_tokens = total_tokens;
  return bwd_impl<false>(a);
}

int sigmoid_attn_mqa_fwd(const void* q, const void* k, const void* v, void* o, int B, int H, int Hkv, int N, int d,
                         sattn_dtype dtype, float bias, int causal, const float* alibi_slopes,
                         const sattn_strides* sq, const sattn_strides* sk, const sattn_strides* sv,
                         const sattn_strides* so, void* stream) {
  if (Hkv <= 0) return SATTN_ERR_SHAPE;
  FwdArgs a{q, k, v, o, nullptr, B, H, N, d, dtype, bias, causal, alibi_slopes, sq, sk, sv, so, stream};
  a.Hkv = Hkv;
  return fwd_impl<false>(a);
}

int sigmoid_attn_mqa_bwd(const void* q, const void* k, const void* v, const void* dout, void* dq, void* dk,
                         void* dv, int B, int H, int Hkv, int N, int d, sattn_dtype dtype, float bias, int causal,
                         const float* alibi_slopes, const sattn_strides* sq, const sattn_strides* sk,
                         const sattn_strides* sv, const sattn_strides* sdout, const sattn_strides* sdq,
                         const sattn_strides* sdk, const sattn_strides* sdv, void* stream) {
  if (Hkv <= 0) return SATTN_ERR_SHAPE;
  BwdArgs a{q, k, v, nullptr, nullptr, dout, dq, dk, dv, B, H, N, d, dtype, bias, causal, alibi_slopes,
            sq, sk, sv, nullptr, sdout, sdq, sdk, sdv, nullptr, 0, kBwdDkDv | kBwdDq, stream};
  a.Hkv = Hkv;
  return bwd_impl<false>(a);
}

size_t sigmoid_attn_mqa_bwd_workspace_bytes(int B, int H, int Hkv, int N, int d, sattn_dtype dtype, int causal) {
  if (check_shape(B, H, N, d, dtype) != SATTN_OK || Hkv <= 0 || H % Hkv || Hkv == H || dtype != SATTN_BF16) return 0;
  const int s = pick_group_split(B, Hkv, H / Hkv, N, d, causal);
  return s > 1 ? 2 * (size_t)s * B * Hkv * N * d * sizeof(float) : 0;
}

int sigmoid_attn_mqa_bwd_split(const void* q, const void* k, const void* v, const void* dout, void* dq, void* dk,
                               void* dv, int B, int H, int Hkv, int N, int d, sattn_dtype dtype, float bias,
                               int causal, const float* alibi_slopes, const sattn_strides* sq,
                               const sattn_strides* sk, const sattn_strides* sv, const sattn_strides* sdout,
                               const sattn_strides* sdq, const sattn_strides* sdk, const sattn_strides* sdv,
                               void* workspace, size_t workspace_bytes, void* stream) {
  if (Hkv <= 0) return SATTN_ERR_SHAPE;
  BwdArgs a{q, k, v, nullptr, nullptr, dout, dq, dk, dv, B, H, N, d, dtype, bias, causal, alibi_slopes,
            sq, sk, sv, nullptr, sdout, sdq, sdk, sdv, workspace, workspace_bytes, kBwdDkDv | kBwdDq, stream};
  a.Hkv = Hkv;
  a.group_split = true;
  return bwd_impl<false>(a);
}

int sigmoid_attn_cross_fwd(const void* q, const void* k, const void* v, void* o, int B, int H, int Nq, int Nk, int d,
                           sattn_dtype dtype, float bias, const sattn_strides* sq, const sattn_strides* sk,
                           const sattn_strides* sv, const sattn_strides* so, void* stream) {
  if (Nk <= 0) return SATTN_ERR_SHAPE;
  FwdArgs a{q, k, v, o, nullptr, B, H, Nq, d, dtype, bias, 0, nullptr, sq, sk, sv, so, stream};
  a.Nk = Nk;
  return fwd_impl<false>(a);
}

int sigmoid_attn_cross_bwd(const void* q, const void* k, const void* v, const void* dout, void* dq, void* dk,
                           void* dv, int B, int H, int Nq, int Nk, int d, sattn_dtype dtype, float bias,
                           const sattn_strides* sq, const sattn_strides* sk, const sattn_strides* sv,
                           const sattn_strides* sdout, const sattn_strides* sdq, const sattn_strides* sdk,
                           const sattn_strides* sdv, void* stream) {
  if (Nk <= 0) return SATTN_ERR_SHAPE;
  BwdArgs a{q, k, v, nullptr, nullptr, dout, dq, dk, dv, B, H, Nq, d, dtype, bias, 0, nullptr,
            sq, sk, sv, nullptr, sdout, sdq, sdk, sdv, nullptr, 0, kBwdDkDv | kBwdDq, stream};
  a.Nk = Nk;
  return bwd_impl<false>(a);
}

int sigmoid_attn_cross_aligned_fwd(const void* q, const void* k, const void* v, void* o, int B, int H, int Nq, int Nk,
                                   int d, sattn_dtype dtype, float bias, int causal, const float* alibi_slopes,
                                   const sattn_strides* sq, const sattn_strides* sk, const sattn_strides* sv,
                                   const sattn_strides* so, void* stream) {
  if (Nk <= 0) return SATTN_ERR_SHAPE;
  FwdArgs a{q, k, v, o, nullptr, B, H, Nq, d, dtype, bias, causal, alibi_slopes, sq, sk, sv, so, stream};
  a.Nk = Nk;
  a.end_aligned = true;
  return fwd_impl<false>(a);
}

size_t sigmoid_attn_cross_aligned_fwd_workspace_bytes(int B, int H, int Nq, int Nk, int d, sattn_dtype dtype) {
  if (check_shape(B, H, Nq, d, dtype) != SATTN_OK || check_shape(B, H, Nk, d, dtype) != SATTN_OK || Nq == Nk ||
      dtype != SATTN_BF16)
    return 0;
  const int s = few_splits(B, H, Nq, Nk, true);
  return s > 1 ? (size_t)s * B * H * Nq * d * sizeof(float) : 0;
}

int sigmoid_attn_cross_aligned_fwd_split(const void* q, const void* k, const void* v, void* o, int B, int H, int Nq,
                                         int Nk, int d, sattn_dtype dtype, float bias, int causal,
                                         const float* alibi_slopes, const sattn_strides* sq, const sattn_strides* sk,
                                         const sattn_strides* sv, const sattn_strides* so, void* workspace,
                                         size_t workspace_bytes, void* stream) {
  if (Nk <= 0) return SATTN_ERR_SHAPE;
  FwdArgs a{q, k, v, o, nullptr, B, H, Nq, d, dtype, bias, causal, alibi_slopes, sq, sk, sv, so, stream};
  a.Nk = Nk;
  a.end_aligned = true;
  a.split = true;
  a.workspace = workspace; a.workspace_bytes = workspace_bytes;
  return fwd_impl<false>(a);
}

int sigmoid_attn_cross_aligned_bwd(const void* q, const void* k, const void* v, const void* dout, void* dq, void* dk,
                                   void* dv, int B, int H, int Nq, int Nk, int d, sattn_dtype dtype, float bias,
                                   int causal, const float* alibi_slopes, const sattn_strides* sq,
                                   const sattn_strides* sk, const sattn_strides* sv, const sattn_strides* sdout,
                                   const sattn_strides* sdq, const sattn_strides* sdk, const sattn_strides* sdv,
                                   void* stream) {
  if (Nk <= 0) return SATTN_ERR_SHAPE;
  BwdArgs a{q, k, v, nullptr, nullptr, dout, dq, dk, dv, B, H, Nq, d, dtype, bias, causal, alibi_slopes,
            sq, sk, sv, nullptr, sdout, sdq, sdk, sdv, nullptr, 0, kBwdDkDv | kBwdDq, stream};
  a.Nk = Nk;
  a.end_aligned = true;
  return bwd_impl<false>(a);
}

int sattn_mfma_bf16_probe(int blocks, int iters, float* sink, void* stream) {
  if (!sink) return SATTN_ERR_NULL;
  if (blocks <= 0 || iters <= 0) return SATTN_ERR_SHAPE;
  return launch(mfma_bf16_probe_kernel, dim3(blocks), dim3(256), 0, (hipStream_t)stream, sink, iters);
}

int sattn_headconcat_norm_fwd(const void* x, void* y, float* stats, int B, int H, int N, int d, sattn_dtype dtype,
                              int kind, float eps, const sattn_strides* sx, const sattn_strides* sy, void* stream) {
  return norm_impl(false, x, nullptr, y, stats, B, H, N, d, dtype, kind, eps, sx, nullptr, sy, stream);
}

int sattn_headconcat_norm_bwd(const void* x, const void* dy, const float* stats, void* dx, int B, int H, int N, int d,
                              sattn_dtype dtype, int kind, const sattn_strides* sx, const sattn_strides* sdy,
                              const sattn_strides* sdx, void* stream) {
  return norm_impl(true, x, dy, dx, const_cast<float*>(stats), B, H, N, d, dtype, kind, 0.f, sx, sdy, sdx, stream);
}

int sattn_set_fwd_waves(int waves) {
  if (waves != 0 && waves != 4 && waves != 8 && waves != 32 && (waves < 64 || waves > 66)) return SATTN_ERR_UNSUPPORTED;
  g_fwd_waves.store(waves, std::memory_order_relaxed);
  return SATTN_OK;
}

int sattn_bwd_one_grid(int B, int H, int N, int d, int causal, int packed) {
  if (B <= 0 || H <= 0 || N <= 0) return SATTN_ERR_SHAPE;
  if (d != 64 && d != 128) return SATTN_ERR_UNSUPPORTED;
  return pick_bwd_merged(B, H, N, causal, d == 64, packed != 0) ? 1 : 0;
}

int sattn_bwd_short(int B, int H, int N, int d, int causal, int alibi, int bias_grad) {
  if (B <= 0 || H <= 0 || N <= 0) return SATTN_ERR_SHAPE;
  if (d != 64 && d != 128) return SATTN_ERR_UNSUPPORTED;
  const int64_t heads = (int64_t)B * H;
  if (!pick_bwd_short(heads, N, d, causal, alibi != 0, bias_grad != 0)) return 0;
  return (int)(2 * heads) - (bias_grad ? 0 : short_whole_heads(heads, N, d));
}
int sattn_fwd_short(int B, int H, int N, int d, int causal) {
  if (B <= 0 || H <= 0 || N <= 0) return SATTN_ERR_SHAPE;
  if (d != 64 && d != 128) return SATTN_ERR_UNSUPPORTED;
  return pick_fwd_short((int64_t)B * H, N, d, causal) ? (N > 128 ? 8 : 4) : 0;
}
int sattn_bwd_merged(int B, int H, int N, int causal) { return sattn_bwd_one_grid(B, H, N, 128, causal, 0); }

int sattn_set_bwd_merged(int mode) {
  if (mode < 0 || mode > 3) return SATTN_ERR_UNSUPPORTED;
  g_bwd_merged.store(mode, std::memory_order_relaxed);
  return SATTN_OK;
}

int sattn_set_fwd_v_slots(int v_slots) {
  if (v_slots != 0 && v_slots != 2 && v_slots != 3) return SATTN_ERR_UNSUPPORTED;
  g_fwd_vslots.store(v_slots, std::memory_order_relaxed);
  return SATTN_OK;
}

int sattn_set_clock_probe(void* device_buffer, int capacity) {
  if (capacity < 0 || (device_buffer && ((uintptr_t)device_buffer & 7) != 0)) return SATTN_ERR_ALIGN;
  g_clock_cap.store(device_buffer ? capacity : 0, std::memory_order_relaxed);
  g_clock_out.store((long long*)device_buffer, std::memory_order_relaxed);
  return SATTN_OK;
}

int sattn_fwd_waves(int B, int H, int N, int d, int causal) {
  if (B <= 0 || H <= 0 || N <= 0) return SATTN_ERR_SHAPE;
  if (d != 64 && d != 128) return SATTN_ERR_UNSUPPORTED;
  return pick_fwd_shape(B, H, N, d, causal).waves;
}

int sattn_fwd_v_slots(int B, int H, int N, int d, int causal) {
  if (B <= 0 || H <= 0 || N <= 0) return SATTN_ERR_SHAPE;
  if (d != 64 && d != 128) return SATTN_ERR_UNSUPPORTED;
  return pick_fwd_shape(B, H, N, d, causal).v_slots;
}

int sattn_device_info(int* compute_units, int* clock_khz) {
  if (!compute_units || !clock_khz) return SATTN_ERR_NULL;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(compute_units, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      hipDeviceGetAttribute(clock_khz, hipDeviceAttributeClockRate, dev) != hipSuccess) {
    (void)hipGetLastError();
    return SATTN_ERR_LAUNCH;
  }
  return SATTN_OK;
}

int sattn_wall_clock_khz(void) {
  int dev = 0, khz = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, dev) != hipSuccess || khz <= 0) {
    (void)hipGetLastError();
    return SATTN_ERR_LAUNCH;
  }
  return khz;
}

int sattn_version(void) { return 102; }

}  // extern "C"
