// V-norm weighting (Eq. 3 / Eq. 4) and per-KV-head selection "top h of the non-recent segment plus
// the recent window" (Sec. 3.1), batched over layers that share one C.
//
//   score kernel : S[l, kv, j] = C[kv, j] * ||V[l, kv, j, :]||_2.  Pure HBM stream over V: one 16-lane
//                  group per row, 16-byte loads (4 rows in flight per group), fp32 sum of squares,
//                  fixed-order lane reduction.
//   select kernel: one workgroup per (layer, KV head).  The h-th largest value is found exactly on the
//                  order-preserving integer image of the fp32 scores by an MSB-first radix select (rows of up to
//                  32768 scores stay in registers and are read from memory once; longer rows re-read L2 in
//                  every pass; where a head's V rows are 128 KB or less, the kernel forms the scores itself: one
//                  launch); an ordered pass then emits, ascending, every
//                  index above it plus the lowest-index ties.  Integer work only: the result is the one a
//                  stable full sort would give.
#include <mutex>

#include "common.h"

namespace purekv {
namespace {

constexpr int SEL_THREADS = 1024;

// Order-preserving map from fp32 to uint32 (-0.0 first folded onto +0.0).
__device__ __forceinline__ uint32_t sort_key(float s) {
  const uint32_t u = __float_as_uint(s + 0.0f);
  return u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u);
}

// One lane's share (16 bytes) of a V row's sum of squares, and the sum over the row's LPR lanes, in each of them, on the DPP path
// (lane ^ 1, lane ^ 2, then mirrors of 8 and 16, where all lanes of a quad or half row already agree: the partners, and with
// them the sums bit for bit, of a butterfly of shuffles, which goes through the LDS crossbar).
__device__ __forceinline__ float piece_norm2(u32x4 x) {
  float ss = 0.f;
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    const float lo = bf16_lo(x[w]), hi = bf16_hi(x[w]);
    ss += lo * lo + hi * hi;
  }
  return ss;
}
template <int CTRL>
__device__ __forceinline__ float dpp_partner(float x) {
  return __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(x), CTRL, 0xf, 0xf, false));
}
template <int LPR>
__device__ __forceinline__ float row_norm2(float ss) {
  static_assert(LPR == 8 || LPR == 16);
  ss += dpp_partner<0xB1>(ss);
  ss += dpp_partner<0x4E>(ss);
  ss += dpp_partner<0x141>(ss);
  if (LPR == 16) ss += dpp_partner<0x140>(ss);
  return ss;
}

// Cross-lane primitives on the DPP path of the vector ALU (a few cycles each; the generic shuffles go through
// the LDS crossbar, ~100 cycles a step with 16 wavefronts on the CU).
// row_shr:n = 0x110 + n moves a value n lanes up within a row of 16 lanes; row_bcast:15 (0x142) hands lane 15 of
// each row to the next row, row_bcast:31 (0x143) lane 31 to rows 2 and 3.  Lanes without a source receive `ident`.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ uint32_t dpp_move(uint32_t ident, uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)ident, (int)v, CTRL, ROW_MASK, 0xf, false);
}
// Inclusive prefix sum over the 64 lanes of a wavefront.
__device__ __forceinline__ uint32_t wave_scan_add(uint32_t v) {
  v += dpp_move<0x111, 0xf>(0u, v);
  v += dpp_move<0x112, 0xf>(0u, v);
  v += dpp_move<0x114, 0xf>(0u, v);
  v += dpp_move<0x118, 0xf>(0u, v);
  v += dpp_move<0x142, 0xa>(0u, v);
  v += dpp_move<0x143, 0xc>(0u, v);
  return v;
}
// Minimum / maximum over the wavefront, valid in lane 63 (the scans run upwards); over each row of 16 lanes, in its last one.
__device__ __forceinline__ uint32_t row_scan_min(uint32_t v) {
  v = min(v, dpp_move<0x111, 0xf>(0xffffffffu, v));
  v = min(v, dpp_move<0x112, 0xf>(0xffffffffu, v));
  v = min(v, dpp_move<0x114, 0xf>(0xffffffffu, v));
  return min(v, dpp_move<0x118, 0xf>(0xffffffffu, v));
}
__device__ __forceinline__ uint32_t row_scan_max(uint32_t v) {
  v = max(v, dpp_move<0x111, 0xf>(0u, v));
  v = max(v, dpp_move<0x112, 0xf>(0u, v));
  v = max(v, dpp_move<0x114, 0xf>(0u, v));
  return max(v, dpp_move<0x118, 0xf>(0u, v));
}
__device__ __forceinline__ uint32_t wave_scan_min(uint32_t v) {
  v = row_scan_min(v);
  v = min(v, dpp_move<0x142, 0xa>(0xffffffffu, v));
  return min(v, dpp_move<0x143, 0xc>(0xffffffffu, v));
}
__device__ __forceinline__ uint32_t wave_scan_max(uint32_t v) {
  v = row_scan_max(v);
  v = max(v, dpp_move<0x142, 0xa>(0u, v));
  return max(v, dpp_move<0x143, 0xc>(0u, v));
}

// grid = (row blocks, layers * Hkv): a workgroup streams 256 / LPR * SCORE_UNROLL consecutive rows of one (layer, KV head).
// Rows in flight per lane: four, with twice the workgroups of eight.  One layer of 4608 x 8 rows of 128 5.5 -> 4.7 us, 16384 x 4 6.6 -> 5.8,
// 8192 x 104 36.0 -> 34.1 (kernel trace).  With two, the last and its compaction together take 73.7 instead of 70.9.
constexpr int SCORE_UNROLL = 4;
template <int D>
__global__ __launch_bounds__(256) void score_kernel(const float* __restrict__ c, const uint16_t* __restrict__ v,
                                                    int64_t v_layer_stride, int64_t v_head_stride,
                                                    int64_t v_tok_stride, float* __restrict__ s_out,
                                                    int32_t n_keys, int32_t Hkv) {
  constexpr int LPR = D / 8;         // lanes per row
  constexpr int RPB = 256 / LPR;     // rows per pass of the workgroup
  const int sub = threadIdx.x % LPR, rslot = threadIdx.x / LPR;
  const int lk = blockIdx.y, layer = lk / Hkv, kvh = lk - layer * Hkv;
  const uint16_t* vh = v + (int64_t)layer * v_layer_stride + (int64_t)kvh * v_head_stride;
  const int j0 = blockIdx.x * (RPB * SCORE_UNROLL) + rslot;
  u32x4 x[SCORE_UNROLL];
#pragma unroll
  for (int u = 0; u < SCORE_UNROLL; ++u) {
    const int j = min(j0 + u * RPB, n_keys - 1);
    x[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(vh + (int64_t)j * v_tok_stride + sub * 8));
  }
#pragma unroll
  for (int u = 0; u < SCORE_UNROLL; ++u) {
    const float ss = row_norm2<LPR>(piece_norm2(x[u]));
    const int j = j0 + u * RPB;
    if (sub == 0 && j < n_keys) s_out[(int64_t)lk * n_keys + j] = c[(int64_t)kvh * n_keys + j] * __builtin_sqrtf(ss);
  }
}

// Squared norms of all V rows of one layer, as a pass of its own (same access pattern as the score kernel).
template <int D>
__global__ __launch_bounds__(256) void vnorm2_kernel(const uint16_t* __restrict__ v, int64_t v_head_stride,
                                                     int64_t v_tok_stride, float* __restrict__ n2_out, int32_t N,
                                                     int32_t kvh0) {
  constexpr int LPR = D / 8, RPB = 256 / LPR;
  const int sub = threadIdx.x % LPR, rslot = threadIdx.x / LPR;
  const int kvh = kvh0 + blockIdx.y;
  const uint16_t* vh = v + (int64_t)kvh * v_head_stride;
  const int j0 = blockIdx.x * (RPB * SCORE_UNROLL) + rslot;
  u32x4 x[SCORE_UNROLL];
#pragma unroll
  for (int u = 0; u < SCORE_UNROLL; ++u) {
    const int j = min(j0 + u * RPB, N - 1);
    x[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(vh + (int64_t)j * v_tok_stride + sub * 8));
  }
#pragma unroll
  for (int u = 0; u < SCORE_UNROLL; ++u) {
    const float ss = row_norm2<LPR>(piece_norm2(x[u]));
    const int j = j0 + u * RPB;
    if (sub == 0 && j < N) n2_out[(int64_t)kvh * N + j] = ss;
  }
}

// The same scores from squared norms that already exist (the prefill kernel emits them while the V tiles are in
// LDS): S[l, kv, j] = C[kv, j] * sqrt(n2[l, kv, j]).  4 bytes per key instead of a V row.
__global__ __launch_bounds__(256) void score_from_norms_kernel(const float* __restrict__ c, const float* __restrict__ n2,
                                                               int64_t n2_layer_stride, float* __restrict__ s_out,
                                                               int32_t N, int32_t n_keys, int32_t Hkv) {
  const int lk = blockIdx.y, layer = lk / Hkv, kvh = lk - layer * Hkv;
  const int j = blockIdx.x * 256 + threadIdx.x;
  if (j >= n_keys) return;
  const float x = n2[(int64_t)layer * n2_layer_stride + (int64_t)kvh * N + j];
  s_out[(int64_t)lk * n_keys + j] = c[(int64_t)kvh * n_keys + j] * __builtin_sqrtf(x);
}

// Block-wide exclusive scan of two counters (1024 threads = 16 wavefronts).
__device__ __forceinline__ void block_scan2(uint32_t& a, uint32_t& b, uint32_t* lds /* 34 words */) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t ia = wave_scan_add(a), ib = wave_scan_add(b);
  if (lane == 63) {
    lds[wave] = ia;
    lds[16 + wave] = ib;
  }
  __syncthreads();
  // lanes 0..15 scan the 16 wavefront totals of a, lanes 16..31 those of b (one row of 16 lanes each)
  uint32_t tot = lane < 32 ? lds[lane] : 0u, inc = tot;
  inc += dpp_move<0x111, 0xf>(0u, inc);
  inc += dpp_move<0x112, 0xf>(0u, inc);
  inc += dpp_move<0x114, 0xf>(0u, inc);
  inc += dpp_move<0x118, 0xf>(0u, inc);
  const uint32_t excl = inc - tot;
  const uint32_t oa = __builtin_amdgcn_readlane(excl, wave), ob = __builtin_amdgcn_readlane(excl, 16 + wave);
  a = oa + ia - a;
  b = ob + ib - b;
  __syncthreads();
}

// EPT = scores per thread: element e of thread t is score e * 1024 + t, so loads are whole cache lines, the scores are read
// from memory once (their integer images stay in registers) and a wavefront's elements of one e are 64 consecutive indices.
//
// MSB-first radix select on the keys' distances from the smallest one, 12 bits a pass, LDS histogram of 4096 bins: a row's range
// is some 14 octaves, so a bin of the first pass holds a 64th of an octave or so and the h-th largest key shares it with a
// few dozen others.  SEL_LIST or fewer are ranked directly, one candidate a wavefront at a time; more are looked at again from
// the smallest of them on (a pass over the bin's own range would leave keys that are all equal, or nearly, together).
//
// A row is one workgroup's chain of barriers and LDS round trips and its 16 wavefronts' vector instructions on one CU; what
// counts is how few of both there are.  The histogram has two buffers, the idle one is cleared behind the scan; ballots count
// the kept keys of every 64 consecutive indices, and each wavefront scans the table of those counts by itself; a row without a
// tie at the threshold needs one comparison a key for that, not two.  One histogram means that keys of one bin are added one
// after the other, so crowded bins are counted apart.  us, 4 rows, calls one after the other, with digits of 8 bits and 16
// copies of their histogram, with 4096 bins and nothing for crowds, now:
//   scores              log-normal         nine in ten are 0    four values        all but one alike   three in ten are 0
//   4199                6.7, 5.1, 4.8      8.0, 15.2, 5.6       7.8, 9.5, 5.7      7.8, 13.4, 7.3      6.7, 5.8, 5.5
//   8192                7.5, 5.8, 5.3      9.2, 24.9, 6.6       8.6, 14.0, 7.4     8.7, 21.6, 8.7      7.6, 8.2, 7.9
//   16384               11.7, 8.3, 7.7     14.3, 45.5, 9.8      13.0, 24.0, 12.0   13.3, 38.9, 13.4    11.2, 12.6, 11.5
//   17000               15.8, 11.5, 10.5   19.5, 49.2, 14.7     18.3, 27.2, 15.6   18.6, 42.5, 20.0    15.9, 15.9, 16.4
// (Histogram in two copies of 2048 bins: log-normal 16384 0.6 more.  Lists of 128: no change.)
constexpr uint32_t SEL_LIST = 64;
constexpr int CROWD = 6;   // of 64 lanes: 64 p^2 share a bin with lane ^ 1 where a fraction p of the keys is in one (12: "three in ten" 0.5 to 1.3 us more)
// A layer's V of up to 128 KB per KV head (eight loads of 16 bytes per thread, all in flight together) is read by the selecting
// workgroup itself: one round trip to memory instead of a launch, its drain and the scores' way through memory.  256 keys of 64:
// 3.8 + 5.1 us in two launches, 4.0 in one.  Beyond that a single CU pulls the rows in slower than the chip does: at the line both
// take the same for few rows (4 KV heads of 128, 512 keys in one launch 6.6 us, 520 in two 6.4), one launch less for many (26 layers
// of 8 KV heads 9.2, 11.1).
constexpr int kFusedBytes = 128 * 1024;
struct ScoreArgs {   // what the scores are formed from: arguments of purekv_topk_select
  const float* c;
  const uint16_t* v;
  int64_t v_layer_stride, v_head_stride, v_tok_stride;
  float* s_out;      // or null
  int32_t Hkv;
};
// D != 0: the scores are not read but formed here, from C and V (rows of D elements; at most kFusedBytes of them).
template <int EPT, int D>
__global__ __launch_bounds__(SEL_THREADS) void select_kernel(const float* __restrict__ s, const ScoreArgs sa,
                                                             int32_t* __restrict__ idx_out, int32_t N, int32_t w, int32_t h) {
  // Histogram: 4096 bins.  Bin b sits at word b + 4 (b / 64): the scan's lanes, 64 bins each, then read 16 bytes a lane from
  // different banks.
  constexpr int WAVES = SEL_THREADS / 64, HBITS = 12, HWORDS = 4096 + 4 * 64;
  constexpr int TPL = (EPT * WAVES + 63) / 64;   // entries of the table of counts per lane
  constexpr int FULL = EPT == 1 ? 0 : EPT == 2 ? 1 : EPT == 4 ? 2 : EPT == 6 ? 4 : EPT == 8 ? 6 : EPT / 2;   // elements that every thread has (the next smaller width)
  static_assert(WAVES % TPL == 0, "entry e * WAVES + w is entry w % TPL of its lane");
  __shared__ __attribute__((aligned(16))) uint32_t hist[2][HWORDS];
  __shared__ __attribute__((aligned(16))) uint32_t counts[64 * TPL];   // [e][wavefront] kept keys: above | equal << 16
  __shared__ uint32_t ext[2][WAVES];      // per-wavefront minimum and maximum key
  __shared__ uint32_t list[SEL_LIST];
  __shared__ uint32_t list_n;
  __shared__ uint32_t sel[3];             // chosen digit, remaining count, keys with that digit
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n_keys = N - w;
  int32_t* out = idx_out + (size_t)blockIdx.x * (h + w);

  if (h == 0 && (D == 0 || sa.s_out == nullptr)) {
    for (int t = tid; t < w; t += SEL_THREADS) out[t] = N - w + t;
    return;
  }
  float raw[EPT];
  auto clear = [&]() {
    for (int t = tid; t < w; t += SEL_THREADS) out[h + t] = N - w + t;
    for (int i = tid; i < HWORDS; i += SEL_THREADS) hist[0][i] = 0;
    if (tid == 0) list_n = 0;
  };
  if constexpr (D == 0) {
    const float* sv = s + (size_t)blockIdx.x * n_keys;
#pragma unroll
    for (int e = 0; e < EPT; ++e) raw[e] = sv[min(e * SEL_THREADS + tid, n_keys - 1)];
    clear();
  } else {
    constexpr int LPR = D / 8, RPB = SEL_THREADS / LPR, UNROLL = kFusedBytes / (SEL_THREADS * 16);
    static_assert(UNROLL * RPB <= EPT * SEL_THREADS && UNROLL * RPB <= HWORDS, "rows, and their scores in the idle histogram");
    float* const sc = reinterpret_cast<float*>(hist[1]);
    const int layer = blockIdx.x / sa.Hkv, kvh = blockIdx.x - layer * sa.Hkv, sub = tid % LPR, row = tid / LPR;
    const uint16_t* vh = sa.v + (int64_t)layer * sa.v_layer_stride + (int64_t)kvh * sa.v_head_stride + sub * 8;
    u32x4 x[UNROLL];
    float cj[UNROLL];
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
      if (u * RPB >= n_keys) break;
      const int j = min(u * RPB + row, n_keys - 1);
      x[u] = *reinterpret_cast<const u32x4*>(vh + (int64_t)j * sa.v_tok_stride);
      cj[u] = sa.c[(int64_t)kvh * n_keys + j];
    }
    clear();
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
      if (u * RPB >= n_keys) break;
      const float score = cj[u] * __builtin_sqrtf(row_norm2<LPR>(piece_norm2(x[u])));
      const int j = u * RPB + row;
      if (sub == 0 && j < n_keys) {
        sc[j] = score;
        if (sa.s_out != nullptr) sa.s_out[(int64_t)blockIdx.x * n_keys + j] = score;
      }
    }
    if (h == 0) return;
    __syncthreads();
#pragma unroll
    for (int e = 0; e < EPT; ++e) raw[e] = sc[min(e * SEL_THREADS + tid, n_keys - 1)];
  }
  // Keys are the scores' images.  Elements past the end of the row (they were loaded as its last one) become key 0, below every
  // score's: they are never among the h <= n_keys largest.
  uint32_t key[EPT];
  uint32_t kmin = 0xffffffffu, kmax = 0u;
#pragma unroll
  for (int e = 0; e < EPT; ++e) {
    key[e] = max(sort_key(raw[e]), 1u);
    kmin = min(kmin, key[e]);
    kmax = max(kmax, key[e]);
  }
  kmin = wave_scan_min(kmin);
  kmax = wave_scan_max(kmax);
  if (lane == 63) {
    ext[0][wave] = kmin;
    ext[1][wave] = kmax;
  }
  __syncthreads();
  static_assert(WAVES == 16, "a row of 16 lanes holds the wavefronts'");
  // Candidates for the h-th largest: the keys of [base, base + range], `remaining` of them are among the kept ones.
  uint32_t base = __builtin_amdgcn_readlane(row_scan_min(ext[0][lane & 15]), 15);
  uint32_t range = __builtin_amdgcn_readlane(row_scan_max(ext[1][lane & 15]), 15) - base;
#pragma unroll
  for (int e = FULL; e < EPT; ++e)
    if ((e + 1) * SEL_THREADS > n_keys) key[e] = e * SEL_THREADS + tid < n_keys ? key[e] : 0u;
  uint32_t remaining = (uint32_t)h, n_cand = (uint32_t)n_keys;
  bool first_pass = true;
  int buf = 0;
  auto word_of = [](uint32_t bin) { return bin + 4u * (bin >> 6); };
  auto chosen = [&](int i) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)sel[i]); };   // uniform: so are the branches on it
  while (range != 0u) {
    // digit = the highest HBITS bits of the distance from `base`
    const int shift = max(32 - HBITS - __clz((int)range), 0);
    uint32_t* const my_hist = hist[buf];
    // Keys crowded into one or two bins (weights that are exactly 0, few distinct values, one key far from all others): additions
    // of a wavefront to one address are served a lane at a time, 130 cycles for 64 lanes.  Where many lanes share the bin of
    // lane ^ 1, the bins of the first two that differ are counted in scalar registers.
    const uint32_t bin0 = key[0] - base <= range ? (key[0] - base) >> shift : 0x10000u + (uint32_t)lane;
    const uint64_t shared = __ballot(bin0 == (uint32_t)__builtin_amdgcn_update_dpp(0, (int)bin0, 0xB1, 0xf, 0xf, false));
    // (opaque: what the loops below have in common, and all that is the same in every pass, would be formed ahead of them for
    // every element and kept in scalar registers that are not there)
    uint32_t from = base;
    int n_here = n_keys;
    asm volatile("" : "+s"(from), "+s"(n_here));
    if (EPT > 1 && __builtin_expect(__popcll(shared) >= CROWD, 0)) {
      const uint32_t c0 = __builtin_amdgcn_readlane(bin0, __ffsll((unsigned long long)shared) - 1);
      const uint64_t others = shared & __ballot(bin0 != c0);
      const uint32_t c1 = others != 0 ? __builtin_amdgcn_readlane(bin0, __ffsll((unsigned long long)others) - 1) : c0;
      uint32_t n0 = 0, n1 = 0;
#pragma unroll
      for (int e = 0; e < EPT; ++e) {
        const uint32_t at = key[e] - from, bin = at >> shift;
        const uint64_t in = __builtin_amdgcn_ballot_w64(at <= range), in0 = in & __builtin_amdgcn_ballot_w64(bin == c0),
                       in1 = in & __builtin_amdgcn_ballot_w64(bin == c1);
        n0 += (uint32_t)__popcll(in0);
        n1 += (uint32_t)__popcll(in1);
        asm volatile("" : "+s"(n0), "+s"(n1));   // (counted here: the masks of all elements do not fit the scalar registers)
        if ((in & ~(in0 | in1)) >> lane & 1u) atomicAdd(&my_hist[word_of(bin)], 1u);
      }
      if (lane == 0) atomicAdd(&my_hist[word_of(c0)], n0);
      if (lane == 1 && c1 != c0) atomicAdd(&my_hist[word_of(c1)], n1);
    } else if (first_pass) {   // every score is a candidate
#pragma unroll
      for (int e = 0; e < EPT; ++e) {
        const uint32_t at = key[e] - from;
        if (e < FULL || (e + 1) * SEL_THREADS <= n_here || at <= range) atomicAdd(&my_hist[word_of(at >> shift)], 1u);
      }
    } else {
#pragma unroll
      for (int e = 0; e < EPT; ++e) {
        const uint32_t at = key[e] - from;
        if (at <= range) atomicAdd(&my_hist[word_of(at >> shift)], 1u);
      }
    }
    first_pass = false;
    __syncthreads();
    if (wave == 0) {
      // lane t owns digits 4095 - 64 t .. 4032 - 64 t; find where the count from the top reaches `remaining`: first the lane,
      // then, its 64 bins over the lanes, the digit
      const uint32_t* const mine_h = hist[buf] + 68 * (63 - lane);
      u32x4 c4 = {0u, 0u, 0u, 0u};
#pragma unroll
      for (int i = 0; i < 16; ++i) c4 += *reinterpret_cast<const u32x4*>(mine_h + 4 * i);
      const uint32_t tot = (c4[0] + c4[1]) + (c4[2] + c4[3]);
      const uint32_t inc = wave_scan_add(tot);
      const int at = __ffsll((unsigned long long)__ballot(inc >= remaining)) - 1;   // (the last lane's is at least `remaining`)
      const uint32_t before = __builtin_amdgcn_readlane(inc, at) - __builtin_amdgcn_readlane(tot, at);
      const uint32_t count = hist[buf][68 * (63 - at) + (63 - lane)];
      const uint32_t upto = before + wave_scan_add(count);
      const int in = __ffsll((unsigned long long)__ballot(upto >= remaining)) - 1;
      if (lane == in) {
        sel[0] = 4095 - 64 * at - in;
        sel[1] = remaining - (upto - count);
        sel[2] = count;
      }
    } else {
      for (int i = tid - 64; i < HWORDS; i += SEL_THREADS - 64) hist[buf ^ 1][i] = 0;
    }
    __syncthreads();
    const uint32_t below = chosen(0) << shift;
    base += below;
    range = min(range - below, (1u << shift) - 1u);
    remaining = chosen(1);
    n_cand = chosen(2);
    buf ^= 1;
    if (range == 0u) break;
    if (n_cand <= SEL_LIST) {
      // few keys share the digits: gather them (in any order) and rank them, a candidate a wavefront at a time
#pragma unroll
      for (int e = 0; e < EPT; ++e)
        if (key[e] - base <= range) list[atomicAdd(&list_n, 1u)] = key[e];   // n_cand of them
      __syncthreads();
      const uint32_t other = lane < (int)n_cand ? list[lane] : 0u;   // (below every candidate)
      for (int i = wave; i < (int)n_cand; i += WAVES) {
        const uint32_t cand = __builtin_amdgcn_readlane(other, i);
        const uint32_t above = (uint32_t)__popcll(__ballot(other > cand)), upto = (uint32_t)__popcll(__ballot(other >= cand));
        if (above < remaining && remaining <= upto && lane == 0) {   // (equal candidates write the same)
          sel[0] = cand;
          sel[1] = remaining - above;
          sel[2] = upto - above;
        }
      }
      __syncthreads();
      base = chosen(0);
      remaining = chosen(1);
      n_cand = chosen(2);
      break;
    }
    // Many keys share them: their own range, which is 0 for a row of few distinct values, instead of the bin's.
    uint32_t cmin = 0xffffffffu, cmax = 0u;
#pragma unroll
    for (int e = 0; e < EPT; ++e)
      if (key[e] - base <= range) {
        cmin = min(cmin, key[e]);
        cmax = max(cmax, key[e]);
      }
    cmin = wave_scan_min(cmin);
    cmax = wave_scan_max(cmax);
    if (lane == 63) {
      ext[0][wave] = cmin;
      ext[1][wave] = cmax;
    }
    __syncthreads();
    base = __builtin_amdgcn_readlane(row_scan_min(ext[0][lane & 15]), 15);
    range = __builtin_amdgcn_readlane(row_scan_max(ext[1][lane & 15]), 15) - base;
  }
  // base = key of the h-th largest score; `remaining` of the n_cand keys equal to it are kept (lowest indices)
  const uint32_t tau = base, need = remaining;
  const bool all_ties = remaining == n_cand;   // every one of them is
  // With no tie to break (nearly always), a kept key is one that is not less than tau: one comparison, one rank.
  uint32_t mine = 0;   // lane e: counts of this wavefront's element e
  if (all_ties) {
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
      const uint32_t ge = (uint32_t)__popcll(__ballot(key[e] >= tau));
      mine = lane == e ? ge : mine;
    }
  } else {
#pragma unroll
    for (int e = 0; e < EPT; ++e) {   // sums stay below 2^16 (above, at most h - 1) and within 2^16 (equal)
      const uint32_t gt = (uint32_t)__popcll(__ballot(key[e] > tau)), eq = (uint32_t)__popcll(__ballot(key[e] == tau));
      mine = lane == e ? (gt | eq << 16) : mine;
    }
  }
  if (lane < EPT) counts[lane * WAVES + wave] = mine;
  if (EPT * WAVES % 64 != 0 && tid >= EPT * WAVES && tid < 64 * TPL) counts[tid] = 0;
  __syncthreads();
  // exclusive scan of the table (in order of the index), TPL entries per lane; of those, entry wave % TPL is the one this
  // wavefront asks some lane for
  uint32_t ent[TPL], tot = 0;
#pragma unroll
  for (int i = 0; i < TPL; ++i) {
    ent[i] = counts[lane * TPL + i];
    tot += ent[i];
  }
  uint32_t ahead = wave_scan_add(tot) - tot;
#pragma unroll
  for (int i = 0; i < TPL - 1; ++i) ahead += i < wave % TPL ? ent[i] : 0u;
  auto rank = [](uint64_t m, uint32_t before) {   // of the lane among those of m
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, before));
  };
  if (all_ties) {
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
      if (e >= FULL && e * SEL_THREADS >= n_keys) break;
      const uint32_t b = __builtin_amdgcn_readlane(ahead, (e * WAVES + wave) / TPL);
      const bool kept = key[e] >= tau;
      const uint32_t at = rank(__ballot(kept), b);
      if (kept) out[at] = e * SEL_THREADS + tid;
    }
  } else {
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
      if (e >= FULL && e * SEL_THREADS >= n_keys) break;
      const uint32_t b = __builtin_amdgcn_readlane(ahead, (e * WAVES + wave) / TPL);
      const bool is_gt = key[e] > tau, is_eq = key[e] == tau;
      const uint32_t gt = rank(__ballot(is_gt), b & 0xffffu), eq = rank(__ballot(is_eq), b >> 16);
      if (is_gt || (is_eq && eq < need)) out[gt + min(eq, need)] = e * SEL_THREADS + tid;
    }
  }
}

// Any length: the scores are re-read from memory (L2) in every pass.
__global__ __launch_bounds__(SEL_THREADS) void select_kernel_stream(const float* __restrict__ s,
                                                                    int32_t* __restrict__ idx_out, int32_t N,
                                                                    int32_t w, int32_t h) {
  __shared__ uint32_t hist[256];
  __shared__ uint32_t scan_lds[34];
  __shared__ uint32_t sel[2];  // chosen digit, remaining count
  const int tid = threadIdx.x, lane = tid & 63;
  const int n_keys = N - w;
  const float* sv = s + (size_t)blockIdx.x * n_keys;
  int32_t* out = idx_out + (size_t)blockIdx.x * (h + w);

  for (int t = tid; t < w; t += SEL_THREADS) out[h + t] = N - w + t;
  if (h == 0) return;

  uint32_t prefix = 0, mask = 0, remaining = (uint32_t)h;
  for (int pass = 0; pass < 4; ++pass) {
    const int shift = 24 - 8 * pass;
    if (tid < 256) hist[tid] = 0;
    __syncthreads();
    for (int j0 = 0; j0 < n_keys; j0 += SEL_THREADS) {
      const int j = j0 + tid;
      const bool in = j < n_keys;
      const uint32_t u = in ? sort_key(sv[j]) : 0u;
      const bool cand = in && ((u & mask) == prefix);
      const uint32_t dgt = (u >> shift) & 255u;
      // wave-uniform digits (the common case for the exponent byte) cost one atomic per wavefront
      const uint64_t votes = __ballot(cand);
      if (votes != 0) {
        const int leader = __ffsll((unsigned long long)votes) - 1;
        const uint32_t d0 = __shfl(dgt, leader, 64);
        const bool uniform = __all(!cand || dgt == d0);
        if (uniform) {
          if (lane == leader) atomicAdd(&hist[d0], (uint32_t)__popcll(votes));
        } else if (cand) {
          atomicAdd(&hist[dgt], 1u);
        }
      }
    }
    __syncthreads();
    if (tid < 64) {
      // lane t owns digits 255-4t .. 252-4t (descending); find where the count from the top reaches `remaining`
      uint32_t cnt[4], tot = 0;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        cnt[r] = hist[255 - 4 * tid - r];
        tot += cnt[r];
      }
      uint32_t inc = tot;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const uint32_t tv = __shfl_up(inc, o, 64);
        if (tid >= o) inc += tv;
      }
      const uint32_t before = inc - tot;  // elements with larger digits than this lane's
      if (before < remaining && remaining <= inc) {
        uint32_t run = before;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          if (run < remaining && remaining <= run + cnt[r]) {
            sel[0] = 255 - 4 * tid - r;
            sel[1] = remaining - run;
          }
          run += cnt[r];
        }
      }
    }
    __syncthreads();
    prefix |= sel[0] << shift;
    mask |= 255u << shift;
    remaining = sel[1];
    __syncthreads();
  }
  // prefix = key of the h-th largest score; `remaining` of the keys equal to it are kept (lowest indices)
  const uint32_t tau = prefix, need = remaining;
  const int chunk = (n_keys + SEL_THREADS - 1) / SEL_THREADS;
  const int jb = tid * chunk, je = min(jb + chunk, n_keys);
  uint32_t gt = 0, eq = 0;
  for (int j = jb; j < je; ++j) {
    const uint32_t u = sort_key(sv[j]);
    gt += u > tau;
    eq += u == tau;
  }
  block_scan2(gt, eq, scan_lds);
  for (int j = jb; j < je; ++j) {
    const uint32_t u = sort_key(sv[j]);
    if (u > tau) {
      out[gt + min(eq, need)] = j;
      ++gt;
    } else if (u == tau) {
      if (eq < need) out[gt + eq] = j;
      ++eq;
    }
  }
}

// Score buffer of purekv_topk_select_static: device memory that exists from the moment the library is loaded
// on a GPU until the process ends, so that the call needs no workspace from its caller and no allocation.  Host
// code never uses the array's name as an address (in host code the name is only a handle for the symbol look-up):
// static_score_buffer() asks the runtime once per device for the array's device address and hands that out.
constexpr size_t kStaticScoreFloats = (size_t)1 << 20;   // 4 MiB
static __device__ __align__(256) float scratch[kStaticScoreFloats];

}  // namespace

size_t topk_static_capacity_floats() { return kStaticScoreFloats; }

int static_score_buffer(int device, float** out) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static float* ptrs[kMaxDevices] = {};
  if (device < 0 || device >= kMaxDevices) return PUREKV_EINVAL;
  std::lock_guard<std::mutex> lock(mu);
  if (ptrs[device] == nullptr) {
    int cur = -1;
    PUREKV_HIP_TRY(hipGetDevice(&cur));
    if (cur != device) return PUREKV_EINVAL;   // every GPU has its own copy of the array: look it up on its own device
    void* p = nullptr;
    PUREKV_HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (p == nullptr) return PUREKV_EHIP;
    ptrs[device] = static_cast<float*>(p);
  }
  *out = ptrs[device];
  return PUREKV_OK;
}

size_t topk_ws_bytes(const purekv_plan& p, int32_t n_layers, int32_t w) {
  // scores, when the caller does not ask for them
  const int64_t n_keys = (int64_t)p.g.N - w;
  return n_keys > 0 ? (size_t)n_layers * p.g.Hkv * n_keys * sizeof(float) : 0;
}

static int launch_select(const purekv_plan& p, const float* scores, int32_t n_layers, int32_t w, int32_t h,
                         int32_t* idx_out, hipStream_t st);

int launch_vnorm2(const purekv_plan& p, const void* v, float* vnorm2, hipStream_t st) {
  const int rows_per_block = (256 / (p.g.d / 8)) * SCORE_UNROLL;
  const unsigned gx = (unsigned)((p.g.N + rows_per_block - 1) / rows_per_block);
  auto launch = [&](int kvh0, int count) {
    const dim3 grid(gx, (unsigned)count);
    if (p.g.d == 128)
      hipLaunchKernelGGL(vnorm2_kernel<128>, grid, dim3(256), 0, st, static_cast<const uint16_t*>(v), p.g.kv_sh,
                         p.g.kv_st, vnorm2, p.g.N, kvh0);
    else
      hipLaunchKernelGGL(vnorm2_kernel<64>, grid, dim3(256), 0, st, static_cast<const uint16_t*>(v), p.g.kv_sh,
                         p.g.kv_st, vnorm2, p.g.N, kvh0);
  };
  if (p.head_sel.empty()) {
    launch(0, p.g.Hkv);
  } else {   // a plan over a head subset: only the KV heads it reads
    for (int kvh = 0; kvh < p.g.Hkv; ++kvh) {
      bool any = false;
      for (int gq = 0; gq < p.g.G; ++gq) any |= p.head_sel[(size_t)kvh * p.g.G + gq] != 0;
      if (any) launch(kvh, 1);
    }
  }
  PUREKV_HIP_TRY(hipGetLastError());
  return PUREKV_OK;
}

int launch_topk_norms(const purekv_plan& p, const float* c, const float* vnorm2, int64_t vn_layer_stride,
                      int32_t n_layers, int32_t w, int32_t h, int32_t* idx_out, float* s_out, void* ws, hipStream_t st) {
  const int32_t n_keys = p.g.N - w;
  const float* scores = c;
  if (n_keys > 0) {
    float* sbuf = s_out ? s_out : static_cast<float*>(ws);
    const dim3 grid((unsigned)((n_keys + 255) / 256), (unsigned)(n_layers * p.g.Hkv));
    hipLaunchKernelGGL(score_from_norms_kernel, grid, dim3(256), 0, st, c, vnorm2, vn_layer_stride, sbuf, p.g.N, n_keys,
                       p.g.Hkv);
    scores = sbuf;
  }
  return launch_select(p, scores, n_layers, w, h, idx_out, st);
}

int launch_topk(const purekv_plan& p, const float* c, const void* v, int64_t v_layer_stride, int32_t n_layers,
                int32_t w, int32_t h, int32_t* idx_out, float* s_out, void* ws, hipStream_t st) {
  const int32_t n_keys = p.g.N - w;
  const float* scores = c;
  if (v != nullptr && n_keys > 0 && (int64_t)n_keys * p.g.d * 2 <= kFusedBytes) {
    const ScoreArgs sa{c, static_cast<const uint16_t*>(v), v_layer_stride, p.g.kv_sh, p.g.kv_st, s_out, p.g.Hkv};
    const dim3 grid((unsigned)(n_layers * p.g.Hkv));
    const float* none = nullptr;
    if (p.g.d == 128)
      hipLaunchKernelGGL((select_kernel<1, 128>), grid, dim3(SEL_THREADS), 0, st, none, sa, idx_out, p.g.N, w, h);
    else
      hipLaunchKernelGGL((select_kernel<1, 64>), grid, dim3(SEL_THREADS), 0, st, none, sa, idx_out, p.g.N, w, h);
    PUREKV_HIP_TRY(hipGetLastError());
    return PUREKV_OK;
  }
  if (v != nullptr && n_keys > 0) {
    float* sbuf = s_out ? s_out : static_cast<float*>(ws);
    const int rows_per_block = (256 / (p.g.d / 8)) * SCORE_UNROLL;
    const dim3 grid((unsigned)((n_keys + rows_per_block - 1) / rows_per_block), (unsigned)(n_layers * p.g.Hkv));
    if (p.g.d == 128)
      hipLaunchKernelGGL(score_kernel<128>, grid, dim3(256), 0, st, c, static_cast<const uint16_t*>(v),
                         v_layer_stride, p.g.kv_sh, p.g.kv_st, sbuf, n_keys, p.g.Hkv);
    else
      hipLaunchKernelGGL(score_kernel<64>, grid, dim3(256), 0, st, c, static_cast<const uint16_t*>(v),
                         v_layer_stride, p.g.kv_sh, p.g.kv_st, sbuf, n_keys, p.g.Hkv);
    scores = sbuf;
  } else if (s_out != nullptr && n_keys > 0) {
    PUREKV_HIP_TRY(hipMemcpyAsync(s_out, c, (size_t)p.g.Hkv * n_keys * sizeof(float), hipMemcpyDeviceToDevice, st));
  }
  return launch_select(p, scores, n_layers, w, h, idx_out, st);
}

static int launch_select(const purekv_plan& p, const float* scores, int32_t n_layers, int32_t w, int32_t h,
                         int32_t* idx_out, hipStream_t st) {
  const int32_t n_keys = p.g.N - w;
  const dim3 sgrid((unsigned)(n_layers * p.g.Hkv)), sblock(SEL_THREADS);
  const int per_thread = (n_keys + SEL_THREADS - 1) / SEL_THREADS;
  auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, sgrid, sblock, 0, st, scores, ScoreArgs{}, idx_out, p.g.N, w, h); };
  // A row takes little less than the longest one of its width: 4199 and 6144 log-normal scores 4.8 and 4.9 us, 8192 5.3; 9000 and
  // 16384 6.9 and 7.7; 17000 and 32768 10.5 and 12.2 (so widths between the last three would save rows just above 8192 and 16384
  // a us or two; there are none).
  if (per_thread <= 1)
    launch(select_kernel<1, 0>);
  else if (per_thread <= 2)
    launch(select_kernel<2, 0>);
  else if (per_thread <= 4)
    launch(select_kernel<4, 0>);
  else if (per_thread <= 6)
    launch(select_kernel<6, 0>);
  else if (per_thread <= 8)
    launch(select_kernel<8, 0>);
  else if (per_thread <= 16)
    launch(select_kernel<16, 0>);
  else if (per_thread <= 32)
    launch(select_kernel<32, 0>);
  else
    hipLaunchKernelGGL(select_kernel_stream, sgrid, sblock, 0, st, scores, idx_out, p.g.N, w, h);
  PUREKV_HIP_TRY(hipGetLastError());
  return PUREKV_OK;
}

}  // namespace purekv
