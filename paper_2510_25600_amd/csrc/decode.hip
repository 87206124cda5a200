// Decode attention of one new token against the compact cache (the decode stage of the paper's
// inference-speed table), optionally fused with the append of that token's key and value.  Latency bound: a few MB of
// cache, one query row per head.  ONE launch does everything:
//   * the kept keys are cut into chunks of 128, 256 or 512, one workgroup (8 wavefronts x 16, 32 or 64 keys) per (chunk,
//     KV head, block of 16 query heads of the group); every K/V row is read once and used for all heads of the block;
//   * scores S^T = K Q^T on the matrix pipe (v_mfma_f32_16x16x32_bf16: 16 keys x 16 heads per instruction; the K rows
//     and the query rows are the operands as they lie in memory, 16 bytes per lane), softmax over the keys in fp32
//     (a lane holds 4 keys of one head: in-lane reduction plus two cross-lane steps), probabilities rounded to bf16 and
//     O^T = V^T P^T with v_mfma_f32_16x16x16_bf16, whose B operand is the probabilities exactly as the score product
//     left them and whose result is four columns of one head per lane; V rows pass through LDS once and come back
//     through the transposing read ds_read_b64_tr_b16;
//   * every load of a wavefront (query, K rows, V rows) is issued before the first is used;
//   * the wavefronts are merged through LDS, the chunks through a workspace in global memory: a workgroup leaves its
//     (max, sum, unnormalised output) there, and a GATHERING workgroup per query head, placed behind all chunks in the
//     grid, adds them up in a fixed order and writes the result.
// How the partial results are handed over.  Every word of the workspace is 0 between calls and no partial result holds a
// 0 word (+0 is stored as -0), so a word that is not 0 has been written by this call: a gathering workgroup looks at the
// (max, sum) pairs of its head until half of them are there, then asks for pairs and outputs together until all are, and
// leaves zeros.  It looks a bounded number of times; one that gives up leaves its head to whoever of the chunks' and the
// gathering workgroups counts itself in last at the (KV head, head block)'s counter, by when everything is in memory.  So
// no wait is without end, whatever order the workgroups run in, and only the head that gave up is added up late.
// What that rests on: a word is stored and loaded whole (a 16-byte piece may arrive in parts, so each of its words is looked at);
// device-scope (sc1) stores go through to memory, and device-scope loads are not served from an L2's older copy; the zeros that a
// gathering workgroup leaves are such stores, and a launch on the stream begins when the one before has ended, stores and all.
// What bounds it is the chain of memory round trips behind the launch.  Counting in and letting the workgroup that arrived
// last add everything up had four of them behind the chunk's own (stores acknowledged, arrival counted, partial results
// in, output out) and one compute unit that pulled in all heads of the group; asking for the data itself leaves two and
// spreads them over as many compute units as there are heads.  (Three where a head has more than 48 chunks with heads of 128, 32 of
// 64: this compiler puts a wait for the others ahead of a lane's last load.)  5491 keys x 4 KV heads x 7 query heads 9.9 -> 7.6 us a call,
// 6900 keys 11.2 -> 8.8 (28 caches in turn), 1690 keys 8.7 -> 7.0, 10 000 keys x 8 KV heads x 4 17.8 -> 12.5.  (All eight
// wavefronts asking for pairs and outputs from the start got in the way of the stores they were waiting for: 8.5.  4000
// keys x 4 x 7, waiting for half of the pairs, all of them, three quarters: 7.64, 7.76, 7.63.)
// With k_new/v_new given, row n_cached - 1 of the cache is taken from them instead of the cache and the workgroup
// that owns that key also stores it there (append and attention in one pass over the cache).
#include <algorithm>

#include "common.h"

namespace purekv {
namespace {

constexpr int DEC_WAVES = 8;     // wavefronts per workgroup
constexpr int DEC_NT = 64 * DEC_WAVES;
constexpr int DEC_HB = 16;       // query heads per workgroup

typedef short shortx4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) shortx4* LdsShortx4;

// Keys of a chunk are 128 x the tiles (of 16 keys) per wavefront.
constexpr int chunk_keys(int tiles) { return 16 * tiles * DEC_WAVES; }
inline int splits_of(int n, int tiles) { return (n + chunk_keys(tiles) - 1) / chunk_keys(tiles); }

struct DecodeArgs {
  const uint16_t* q;
  const uint16_t* k_new;   // [Hkv, D] or null
  const uint16_t* v_new;
  uint16_t* kc;
  uint16_t* vc;
  uint16_t* out;
  float* ws_o;         // [n_splits, Hq, D] unnormalised partial outputs, zero on entry and on exit
  float* ws_ml;        // [Hq, max_splits, 2] running maximum (log2 domain) and sum, likewise
  uint64_t* counters;  // [Hkv * head_blocks]: workgroups that have arrived | heads that are gathered << 32, likewise
  int32_t Hq, G, n_cached, cap, n_splits, max_splits, head_blocks;
  int32_t looks;       // of a gathering workgroup, before it gives up
  float scale_log2;
};

// Rows of 16 lanes on the DPP path of the vector ALU (lane ^ 1, lane ^ 2, mirror of 8, mirror of 16), rows and halves by
// v_permlane16_swap and v_permlane32_swap.
template <int CTRL>
__device__ __forceinline__ float dpp_f32(float x) {
  return __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(x), CTRL, 0xf, 0xf, false));
}
struct LanePair {
  float a, b;
};
__device__ __forceinline__ LanePair swap16(float x) {   // {even row's, odd row's} value of each pair of rows of 16 lanes
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return {__uint_as_float(r[0]), __uint_as_float(r[1])};
}
__device__ __forceinline__ LanePair swap32(float x) {   // {lower half's, upper half's} value
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return {__uint_as_float(r[0]), __uint_as_float(r[1])};
}
__device__ __forceinline__ float wave_max(float x) {   // over the wavefront, result in every lane
  x = fmaxf(x, dpp_f32<0xB1>(x));
  x = fmaxf(x, dpp_f32<0x4E>(x));
  x = fmaxf(x, dpp_f32<0x141>(x));
  x = fmaxf(x, dpp_f32<0x140>(x));
  const LanePair p = swap16(x);
  const LanePair q = swap32(fmaxf(p.a, p.b));
  return fmaxf(q.a, q.b);
}
__device__ __forceinline__ float wave_sum(float x) {
  x += dpp_f32<0xB1>(x);
  x += dpp_f32<0x4E>(x);
  x += dpp_f32<0x141>(x);
  x += dpp_f32<0x140>(x);
  const LanePair p = swap16(x);
  const LanePair q = swap32(p.a + p.b);
  return q.a + q.b;
}

// A word of a partial result as it is stored: never 0, which is what an unwritten word holds (+0 becomes -0).
__device__ __forceinline__ float mark_written(float x) {
  const uint32_t u = __float_as_uint(x);
  return __uint_as_float(u == 0u ? 0x80000000u : u);
}

// One lane counts its workgroup in at (KV head, head block), `gathered` being the heads it has finished.  Whoever is the
// last of the n_splits chunks and ng gatherings resets the counter and receives the heads that nobody has finished (their
// partial results are in memory: every chunk's stores were acknowledged before it counted itself in), everybody else 0.
__device__ __forceinline__ void count_in(const DecodeArgs& a, int kvh, int hb, int ng, uint32_t gathered, uint32_t& lds_rest) {
  uint64_t* const counter = a.counters + kvh * a.head_blocks + hb;
  const uint64_t add = 1u | (uint64_t)gathered << 32;
  const uint64_t now = __hip_atomic_fetch_add(counter, add, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + add;
  const bool last = (uint32_t)now == (uint32_t)(a.n_splits + ng);
  if (last) __hip_atomic_store(counter, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // ready for the next call
  lds_rest = last ? ~(uint32_t)(now >> 32) & ((1u << ng) - 1u) : 0u;
}

// Adds up the partial results of head i of the block and writes its output; whole workgroup.  A group of LPR lanes takes the
// four-column pieces of every NG-th chunk; a wavefront holds the (max, sum) pairs of 64 chunks, one a lane, and turns them
// into weights with cross-lane steps.  With `counts` it is this workgroup's first gathering: it looks a.looks times at
// most, counts itself in and returns what count_in leaves it; without, everything is in memory.
template <int D, int BYTES>
__device__ __forceinline__ uint32_t gather_head(const DecodeArgs& a, int kvh, int hb, int ng, int i, bool counts,
                                                uint8_t (&smem)[DEC_WAVES][BYTES], uint32_t& lds_rest) {
  constexpr int LPR = D / 4;            // lanes per row of four-column pieces
  constexpr int NG = DEC_NT / LPR;      // groups of LPR lanes
  constexpr int U = 64 / NG;            // chunks per group and pass of 64
  static_assert(BYTES >= (D + 1) * 4, "the wavefronts' sums and flags fit");
  float* const red = reinterpret_cast<float*>(&smem[0][0]);   // [DEC_WAVES][D]
  int* const failed = reinterpret_cast<int*>(red + DEC_WAVES * D);   // [DEC_WAVES]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int li = tid % LPR, gi = tid / LPR;
  const int hq = kvh * a.G + hb * DEC_HB + i;
  const uint32_t o_stride = (uint32_t)a.Hq * D * 4u;
  const BufferRsrc mlb = make_rsrc(a.ws_ml + (size_t)hq * a.max_splits * 2);
  float run_m = -INFINITY, run_l = 0.f;
  floatx4 acc = {0.f, 0.f, 0.f, 0.f};
  int looks = counts ? a.looks : kDecodeLooks;
  for (int s0 = 0; s0 < a.n_splits; s0 += 64) {
    const int nsb = min(64, a.n_splits - s0);
    const BufferRsrc ob = make_rsrc(a.ws_o + (size_t)s0 * a.Hq * D);
    floatx2 ml;
    floatx4 ov[U];
    // What does not exist counts as there: weight 0 of -0.
    auto load_pairs = [&]() {
      ml = floatx2{-INFINITY, -0.f};
      if (lane < nsb) ml = load_device_8(mlb, (uint32_t)(s0 + lane) * 8u);
    };
    auto pair_there = [&]() { return __float_as_uint(ml[0]) != 0u && __float_as_uint(ml[1]) != 0u; };
    // The loads of a look are ordinary ones to the compiler, of addresses that do not change: without a barrier ahead of each look
    // it may load once and look at the same registers until the looks are used up.
    auto memory_has_changed = []() { asm volatile("" ::: "memory"); };
    for (;;) {
      memory_has_changed();
      load_pairs();
      if (__popcll(__ballot(pair_there())) >= 64 - nsb / 2 || --looks <= 0) break;
      __builtin_amdgcn_s_sleep(1);
    }
    while (looks > 0) {
      memory_has_changed();
      load_pairs();
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int c = gi + u * NG;
        ov[u] = floatx4{-0.f, -0.f, -0.f, -0.f};
        if (c < nsb) ov[u] = load_device_16(ob, (uint32_t)c * o_stride + (uint32_t)(hq * D + 4 * li) * 4u);
      }
      bool there = pair_there();
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int k = 0; k < 4; ++k) there &= __float_as_uint(ov[u][k]) != 0u;
      if (__all(there)) break;
      --looks;
    }
    if (looks <= 0) break;
    const float mnew = fmaxf(run_m, wave_max(ml[0]));
    const float mref = (mnew == -INFINITY) ? 0.f : mnew;   // every score so far is -inf: weights 0, not NaN
    const float f = __builtin_amdgcn_exp2f(ml[0] - mref);
    const float lsum = wave_sum(ml[1] * f);
    const float fo = __builtin_amdgcn_exp2f(run_m - mref);   // first pass: 2^(-inf) = 0
    acc *= fo;
    run_l = run_l * fo + lsum;
    run_m = mnew;
#pragma unroll
    for (int u = 0; u < U; ++u) acc += ov[u] * __shfl(f, gi + u * NG, 64);
  }
  // the groups of a wavefront, then the wavefronts, in order
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    if (LPR == 16) {
      const LanePair p = swap16(acc[k]);
      acc[k] = p.a + p.b;
    }
    const LanePair p = swap32(acc[k]);
    acc[k] = p.a + p.b;
  }
  if (lane < LPR) *reinterpret_cast<floatx4*>(red + wave * D + 4 * li) = acc;
  if (lane == 0) failed[wave] = looks <= 0;
  __syncthreads();
  int bad = 0;
#pragma unroll
  for (int wv = 0; wv < DEC_WAVES; ++wv) bad |= failed[wv];
  bad = __builtin_amdgcn_readfirstlane(bad);
  if (counts && tid == DEC_NT - 64) count_in(a, kvh, hb, ng, bad ? 0u : 1u << i, lds_rest);   // beside the output
  if (!bad) {
    if (tid < LPR) {
      floatx4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int wv = 0; wv < DEC_WAVES; ++wv) sum += *reinterpret_cast<const floatx4*>(red + wv * D + 4 * li);
      *reinterpret_cast<u32x2*>(a.out + (size_t)hq * D + 4 * li) =
          u32x2{pack_bf16(sum[0] / run_l, sum[1] / run_l), pack_bf16(sum[2] / run_l, sum[3] / run_l)};
    }
    // nobody reads the partial results again: back to 0
    for (int s0 = 0; s0 < a.n_splits; s0 += 64) {
      const int nsb = min(64, a.n_splits - s0);
      const BufferRsrc ob = make_rsrc(a.ws_o + (size_t)s0 * a.Hq * D);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int c = gi + u * NG;
        if (c < nsb) store_device_16(ob, (uint32_t)c * o_stride + (uint32_t)(hq * D + 4 * li) * 4u, floatx4{0.f, 0.f, 0.f, 0.f});
      }
      if (wave == 1 && lane < nsb) store_device_8(mlb, (uint32_t)(s0 + lane) * 8u, floatx2{0.f, 0.f});
    }
  }
  __syncthreads();
  const uint32_t rest = counts ? lds_rest : 0u;
  asm volatile("" ::: "memory");
  return rest;
}

// LDS bytes per wavefront: V rows, then the outputs (rows of both padded: consecutive rows start 8 or 4 banks apart).
template <int D, int KT>
constexpr int kDecodeSmem = std::max(16 * KT * (D * 2 + 32), DEC_HB * (D + 4) * 4);

// One chunk of keys of one KV head and head block; returns what count_in leaves this workgroup.
template <int D, int KT>
__device__ __forceinline__ uint32_t attend_chunk(const DecodeArgs& a, int kvh, int hb, uint8_t (&smem)[DEC_WAVES][kDecodeSmem<D, KT>],
                                                 float (&lds_ml)[DEC_WAVES][DEC_HB][2], uint32_t& lds_rest) {
  constexpr int KEYS = 16 * KT;         // keys per wavefront
  constexpr int KS = D / 32;            // k-steps of the score product
  constexpr int NC = D / 16;            // 16-column blocks of the output
  constexpr int CPR = D / 8;            // 16-byte pieces per row
  constexpr int NV = KEYS * CPR / 64;   // V pieces per lane
  constexpr int VROW = D * 2 + 32;      // bytes per V row in LDS
  constexpr int OROW = D + 4;           // floats per head of a wavefront's output block
  constexpr int LPR = D / 4;            // lanes per row of four-column pieces in the merges
  constexpr int NG = DEC_NT / LPR;      // groups of LPR lanes
  static_assert(KEYS * VROW <= kDecodeSmem<D, KT> && DEC_HB * OROW * 4 <= kDecodeSmem<D, KT>);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n = lane & 15, kg = lane >> 4;
  const int split = blockIdx.x, g0 = hb * DEC_HB;
  const int ng = min(DEC_HB, a.G - g0);
  const int key0 = (split * DEC_WAVES + wave) * KEYS;
  const int last = a.n_cached - 1;
  const int j_new = a.k_new != nullptr ? last : -1;   // the key that comes from k_new / v_new

  // ---- every load of this wavefront, before any use ----
  bf16x8 qf[KS], kf[KT][KS];
  {
    const uint16_t* qr = a.q + (size_t)(kvh * a.G + g0 + min(n, ng - 1)) * D + 8 * kg;
#pragma unroll
    for (int s = 0; s < KS; ++s) qf[s] = *reinterpret_cast<const bf16x8*>(qr + 32 * s);
  }
  const size_t head_base = (size_t)kvh * a.cap * D;
#pragma unroll
  for (int t = 0; t < KT; ++t) {
    const int j = min(key0 + 16 * t + n, last);   // rows past the end repeat the last key (masked below)
    const uint16_t* kr = (j == j_new ? a.k_new + (size_t)kvh * D : a.kc + head_base + (size_t)j * D) + 8 * kg;
#pragma unroll
    for (int s = 0; s < KS; ++s) kf[t][s] = *reinterpret_cast<const bf16x8*>(kr + 32 * s);
  }
  u32x4 vreg[NV];
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int p = i * 64 + lane, r = p / CPR, c = p % CPR;
    const int j = min(key0 + r, last);
    const uint16_t* vr = j == j_new ? a.v_new + (size_t)kvh * D : a.vc + head_base + (size_t)j * D;
    vreg[i] = *reinterpret_cast<const u32x4*>(vr + c * 8);
  }

  // ---- scores: lane (n, kg) holds keys 16 t + 4 kg + i of head n ----
  // At most two tiles share a reference: its key has a probability that bf16 holds exactly, and with one for four tiles the
  // outputs are 3-4 % further (2-norm) from a 64-bit evaluation.
  constexpr int NR = (KT + 1) / 2, TR = KT / NR;   // references, tiles of each
  const int n_valid = a.n_cached - key0;   // keys of this wavefront that exist (may be <= 0 or > KEYS)
  float m[NR], l[NR];
  shortx4 pa[KT];
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    float sc[TR][4];
    m[r] = -INFINITY;
#pragma unroll
    for (int t = 0; t < TR; ++t) {
      floatx4 sacc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < KS; ++s) sacc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[TR * r + t][s], qf[s], sacc, 0, 0, 0);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        sc[t][i] = (16 * (TR * r + t) + 4 * kg + i < n_valid) ? sacc[i] * a.scale_log2 : -INFINITY;
        m[r] = fmaxf(m[r], sc[t][i]);
      }
    }
    {
      const LanePair p = swap16(m[r]);
      const LanePair q = swap32(fmaxf(p.a, p.b));
      m[r] = fmaxf(q.a, q.b);
    }
    const float mu = (m[r] == -INFINITY) ? 0.f : m[r];
    l[r] = 0.f;
#pragma unroll
    for (int t = 0; t < TR; ++t) {
      const uint32_t w0 = pack_bf16(__builtin_amdgcn_exp2f(sc[t][0] - mu), __builtin_amdgcn_exp2f(sc[t][1] - mu));
      const uint32_t w1 = pack_bf16(__builtin_amdgcn_exp2f(sc[t][2] - mu), __builtin_amdgcn_exp2f(sc[t][3] - mu));
      l[r] += (bf16_lo(w0) + bf16_hi(w0)) + (bf16_lo(w1) + bf16_hi(w1));   // the sum of what is multiplied with V
      pa[TR * r + t] = __builtin_bit_cast(shortx4, u32x2{w0, w1});
    }
    {
      const LanePair p = swap16(l[r]);
      const LanePair q = swap32(p.a + p.b);
      l[r] = q.a + q.b;
    }
  }
  float fr[NR];   // weights of the references' partial outputs
  if constexpr (NR == 2) {
    const float mw = fmaxf(m[0], m[1]), mu = (mw == -INFINITY) ? 0.f : mw;
    fr[0] = __builtin_amdgcn_exp2f(m[0] - mu);
    fr[1] = __builtin_amdgcn_exp2f(m[1] - mu);
    m[0] = mw;
    l[0] = l[0] * fr[0] + l[1] * fr[1];
  }
  if (kg == 0) {
    lds_ml[wave][n][0] = m[0];
    lds_ml[wave][n][1] = l[0];
  }

  // ---- V rows to LDS (this wavefront's own area: no barrier, a wavefront's LDS accesses stay in order) ----
  uint8_t* vs = smem[wave];
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int p = i * 64 + lane, r = p / CPR, c = p % CPR;
    *reinterpret_cast<u32x4*>(vs + r * VROW + c * 16) = vreg[i];
  }
  asm volatile("" ::: "memory");

  // ---- O^T = V^T P^T: lane (n, kg) receives head n, columns 16 c + 4 kg .. + 3 ----
  // transposing read: in a 16-lane group lane s gives the address of row s / 4, columns 4 (s % 4) .. + 3 and lane j
  // receives column j of those four rows: the A operand (keys 4 kg .. + 3 of column n) of the 16x16x16 product.
  floatx4 o[NC];
  {
    const uint8_t* vb = vs + (4 * kg + (n >> 2)) * VROW + 8 * (n & 3);
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      floatx4 part[NR];
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        part[r] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = TR * r; t < TR * (r + 1); ++t) {
          const shortx4 vfrag = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LdsShortx4)(vb + 16 * t * VROW + 32 * c));
          part[r] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(vfrag, pa[t], part[r], 0, 0, 0);
        }
      }
      o[c] = part[0];
      if constexpr (NR == 2) o[c] = part[0] * fr[0] + part[1] * fr[1];
    }
  }
  // ---- the wavefront's block [heads][D] fp32 replaces its V rows in LDS ----
  asm volatile("" ::: "memory");
  {
    float* ow = reinterpret_cast<float*>(vs) + n * OROW + 4 * kg;
    if (n < ng) {
#pragma unroll
      for (int c = 0; c < NC; ++c) *reinterpret_cast<floatx4*>(ow + 16 * c) = o[c];
    }
  }

  // ---- append: the wavefront that owns key j_new stores it (head block 0 only) ----
  if (j_new >= 0 && hb == 0 && j_new >= key0 && j_new < key0 + KEYS) {
#pragma unroll
    for (int t = 0; t < KT; ++t) {
      if (key0 + 16 * t + n == j_new) {
        uint16_t* kw = a.kc + head_base + (size_t)j_new * D + 8 * kg;
#pragma unroll
        for (int s = 0; s < KS; ++s) *reinterpret_cast<bf16x8*>(kw + 32 * s) = kf[t][s];
      }
    }
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int p = i * 64 + lane, r = p / CPR, c = p % CPR;
      if (key0 + r == j_new) *reinterpret_cast<u32x4*>(a.vc + head_base + (size_t)j_new * D + c * 8) = vreg[i];
    }
  }
  __syncthreads();

  // ---- merge the wavefronts: a thread takes four columns of one head ----
  const int li = tid % LPR, gi = tid / LPR;   // lane within its group of LPR lanes, group
  const bool single = a.n_splits == 1;
  const BufferRsrc ws_o = make_rsrc(a.ws_o + (size_t)split * a.Hq * D);
  for (int g = gi; g < ng; g += NG) {
    float mw[DEC_WAVES], mn = -INFINITY;
#pragma unroll
    for (int wv = 0; wv < DEC_WAVES; ++wv) {
      mw[wv] = lds_ml[wv][g][0];
      mn = fmaxf(mn, mw[wv]);
    }
    const float mref = (mn == -INFINITY) ? 0.f : mn;
    floatx4 acc = {0.f, 0.f, 0.f, 0.f};
    float ls = 0.f;
#pragma unroll
    for (int wv = 0; wv < DEC_WAVES; ++wv) {
      const float f = __builtin_amdgcn_exp2f(mw[wv] - mref);
      acc += *reinterpret_cast<const floatx4*>(reinterpret_cast<const float*>(smem[wv]) + g * OROW + 4 * li) * f;
      ls += lds_ml[wv][g][1] * f;
    }
    const int hq = kvh * a.G + g0 + g;
    if (single) {
      u32x2 w;
      w[0] = f32_to_bf16(acc[0] / ls) | (f32_to_bf16(acc[1] / ls) << 16);
      w[1] = f32_to_bf16(acc[2] / ls) | (f32_to_bf16(acc[3] / ls) << 16);
      *reinterpret_cast<u32x2*>(a.out + (size_t)hq * D + 4 * li) = w;
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[i] = mark_written(acc[i]);
      store_device_16(ws_o, (uint32_t)(hq * D + 4 * li) * 4u, acc);
      if (li == 0)
        store_device_8(make_rsrc(a.ws_ml + (size_t)(kvh * a.G + g0) * a.max_splits * 2), (uint32_t)(g * a.max_splits + split) * 8u,
                       floatx2{mark_written(mn), mark_written(ls)});
    }
  }
  if (single) return 0u;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this thread's stores have completed
  __syncthreads();
  if (tid == 0) count_in(a, kvh, hb, ng, 0u, lds_rest);
  __syncthreads();
  const uint32_t rest = lds_rest;
  asm volatile("" ::: "memory");
  return rest;
}

// grid = (chunks, KV heads, head blocks, and behind them as many planes as the gathering workgroups need)
template <int D, int KT>
__global__ __launch_bounds__(DEC_NT) void decode_kernel(const DecodeArgs a) {
  __shared__ __attribute__((aligned(16))) uint8_t smem[DEC_WAVES][kDecodeSmem<D, KT>];
  __shared__ float lds_ml[DEC_WAVES][DEC_HB][2];
  __shared__ uint32_t lds_rest;
  int kvh = blockIdx.y, hb = blockIdx.z;
  bool gathers = hb >= a.head_blocks;
  uint32_t todo;   // heads of the block that this workgroup adds up
  if (gathers) {
    const int hq = ((hb - a.head_blocks) * (int)gridDim.y + kvh) * a.n_splits + (int)blockIdx.x;
    if (hq >= a.Hq) return;
    kvh = hq / a.G;
    const int g = hq - kvh * a.G;
    hb = g / DEC_HB;
    todo = 1u << (g - hb * DEC_HB);
  } else {
    todo = attend_chunk<D, KT>(a, kvh, hb, smem, lds_ml, lds_rest);
  }
  const int ng = min(DEC_HB, a.G - hb * DEC_HB);
  while (todo != 0u) {
    const int i = __builtin_ctz(todo);
    todo &= todo - 1u;
    const uint32_t rest = gather_head<D>(a, kvh, hb, ng, i, gathers, smem, lds_rest);
    if (gathers) todo = rest;
    gathers = false;
  }
}

}  // namespace

// Workspace: [arrival counters, padded to 256 bytes][partial outputs][their (max, sum)].
static int decode_head_blocks(const purekv_plan& p) { return (p.g.G + DEC_HB - 1) / DEC_HB; }
static size_t decode_counter_bytes(const purekv_plan& p) {
  return ((size_t)p.g.Hkv * decode_head_blocks(p) * sizeof(uint64_t) + 255) / 256 * 256;
}

// Tiles per wavefront: the fewest with which the workgroups, the gathering ones among them, have a compute unit each, else
// four; caches of one chunk of 256 keys are not cut.  256 compute units, us a call with 1, 2, 4 tiles (the old kernel, two):
//   28 query heads on 4 KV heads of 128, keys 1690: 7.0, 8.1, 10.5 (8.7); 6900 (244 workgroups with one tile): 9.0, 9.5,
//   12.0 (11.2); 8100 (284, 156 with two): 10.4, 9.3, 11.8 (11.7); 16000 (280 with two): 15.4, 12.7, 12.6 (15.8)
//   32 on 8 of 128, keys 2500 (192): 7.9, 8.9, 11.8 (9.9); 4000 (288, 160): 9.6, 9.1, 11.7 (10.6); 10000 (352 with two): 18.1, 13.7,
//   12.7 (17.8);  200 keys, 28 on 4: 6.9, 5.1 (5.1)
// With more workgroups than compute units the second one of a unit starts its loads behind the first one's.
// A gathering workgroup takes 64 chunks at a time, each time another round trip or two, so few KV heads are not cut into as many
// chunks as there is room for: with one tile into 64, with two into 64 with heads of 64, 192 of 128 (four tiles are 147 KB of LDS
// to fill there).  us, without that limit -> with it (the old kernel): 2 query heads on 1 KV head of 64, 16000 keys 7.6 -> 6.5 (8.0),
// 31000 11.5 -> 8.0 (10.2), 50000 10.8 -> 9.3 (13.8); 2 on 1 of 128, 16000 9.5 -> 8.4 (9.6), 31000 13.7 -> 10.3 (11.2), 50000 13.7 ->
// 12.5 (14.2); 4 on 2 of 128, 16000 10.8 -> 9.0 (10.4).  Heads of 128 with two tiles in up to 64 chunks, else four: 18000 keys 10.5
// instead of 9.6, 33000 12.0 instead of 11.1.
static int decode_room(const purekv_plan& p) { return (p.n_cu - p.g.Hq) / (p.g.Hkv * decode_head_blocks(p)); }   // chunks per KV head
static int decode_limit(const purekv_plan& p, int tiles) { return std::min(decode_room(p), tiles == 2 && p.g.d == 128 ? 192 : 64); }
static int decode_tiles(const purekv_plan& p, int n) {
  if (n <= chunk_keys(1)) return 1;
  if (n <= chunk_keys(2)) return 2;
  return splits_of(n, 1) <= decode_limit(p, 1) ? 1 : splits_of(n, 2) <= decode_limit(p, 2) ? 2 : 4;
}
// Chunks of any n <= cap.
static int decode_max_splits(const purekv_plan& p, int cap) {
  return std::max({1, std::min(splits_of(cap, 1), decode_limit(p, 1)), std::min(splits_of(cap, 2), decode_limit(p, 2)), splits_of(cap, 4)});
}

size_t decode_ws_bytes(const purekv_plan& p, int32_t cap) {
  return decode_counter_bytes(p) + (size_t)decode_max_splits(p, cap) * p.g.Hq * (p.g.d + 2) * sizeof(float);
}

namespace {
__global__ void clear_decode_workspace_kernel(uint32_t* ws, size_t n) {   // a kernel, not a memset: callers may be capturing
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) ws[i] = 0u;
}
}  // namespace

int launch_decode_ws_init(void* ws, size_t bytes, hipStream_t st) {
  const size_t n = bytes / 4;
  const unsigned grid = (unsigned)std::min<size_t>((n + 255) / 256, 4096);
  hipLaunchKernelGGL(clear_decode_workspace_kernel, dim3(grid), dim3(256), 0, st, static_cast<uint32_t*>(ws), n);
  PUREKV_HIP_TRY(hipGetLastError());
  return PUREKV_OK;
}

int launch_decode(const purekv_plan& p, const void* q_new, const void* k_new, const void* v_new, void* kc, void* vc,
                  int32_t n_cached, int32_t cap, void* out, void* ws, int32_t looks, hipStream_t st) {
  DecodeArgs a;
  a.q = static_cast<const uint16_t*>(q_new);
  a.k_new = static_cast<const uint16_t*>(k_new);
  a.v_new = static_cast<const uint16_t*>(v_new);
  a.kc = static_cast<uint16_t*>(kc);
  a.vc = static_cast<uint16_t*>(vc);
  a.out = static_cast<uint16_t*>(out);
  const int tiles = decode_tiles(p, n_cached);
  a.head_blocks = decode_head_blocks(p);
  a.n_splits = splits_of(n_cached, tiles);
  a.max_splits = decode_max_splits(p, cap);
  a.looks = looks;
  a.counters = static_cast<uint64_t*>(ws);
  a.ws_o = reinterpret_cast<float*>(static_cast<char*>(ws) + decode_counter_bytes(p));
  a.ws_ml = a.ws_o + (size_t)a.max_splits * p.g.Hq * p.g.d;
  a.Hq = p.g.Hq;
  a.G = p.g.G;
  a.n_cached = n_cached;
  a.cap = cap;
  a.scale_log2 = p.g.scale * kLog2e;
  const int64_t per_plane = (int64_t)a.n_splits * p.g.Hkv;
  const int gather_planes = a.n_splits > 1 ? (int)((p.g.Hq + per_plane - 1) / per_plane) : 0;
  const dim3 grid((unsigned)a.n_splits, (unsigned)p.g.Hkv, (unsigned)(a.head_blocks + gather_planes));
  auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, dim3(DEC_NT), 0, st, a); };
  if (p.g.d == 128)
    tiles == 1 ? launch(decode_kernel<128, 1>) : tiles == 2 ? launch(decode_kernel<128, 2>) : launch(decode_kernel<128, 4>);
  else
    tiles == 1 ? launch(decode_kernel<64, 1>) : tiles == 2 ? launch(decode_kernel<64, 2>) : launch(decode_kernel<64, 4>);
  PUREKV_HIP_TRY(hipGetLastError());
  return PUREKV_OK;
}

}  // namespace purekv
