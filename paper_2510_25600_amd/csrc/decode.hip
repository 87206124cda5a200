// Decode attention of one new token against the compact cache (the decode stage of the paper's
// inference-speed table), optionally fused with the append of that token's key and value.  Latency bound: a few MB of
// cache, one query row per head.  ONE launch does everything:
//   * the kept keys are cut into chunks of 256, one workgroup (8 wavefronts x 32 keys) per (chunk, KV head, block of
//     16 query heads of the group); every K/V row is read once and used for all heads of the block;
//   * scores S^T = K Q^T on the matrix pipe (v_mfma_f32_16x16x32_bf16: 16 keys x 16 heads per instruction; the K rows
//     and the query rows are the operands as they lie in memory, 16 bytes per lane), softmax over the keys in fp32
//     (a lane holds 4 keys of one head: in-lane reduction plus two cross-lane steps), probabilities rounded to bf16 and
//     O^T = V^T P^T with v_mfma_f32_16x16x16_bf16, whose B operand is the probabilities exactly as the score product
//     left them and whose result is four columns of one head per lane; V rows pass through LDS once and come back
//     through the transposing read ds_read_b64_tr_b16;
//   * every load of a wavefront (query, 32 K rows, 32 V rows) is issued before the first is used;
//   * the wavefronts are merged through LDS, the chunks through a workspace in global memory: each workgroup
//     writes its (max, sum, unnormalised output), and the workgroup that arrives last at a per-(KV head, head block)
//     counter merges all chunks in a fixed order and writes the result.  Nobody waits for anybody: a workgroup that is
//     not the last simply ends.  The counters lead the caller's workspace and are zero between calls (the last
//     workgroup resets its counter): calls on different workspaces are independent of each other.
// What bounds it is the chain of memory round trips behind the launch, in time stamps of one call on 5491 keys x 4 KV
// heads x 7 query heads (88 workgroups, ~9.2 us): K rows there 2.5 us, V rows 2.9, products done 3.6, wavefronts merged
// 4.5, stores acknowledged 4.9, arrival counted 5.7, chunk maxima and sums there 7.4, chunks added up 8.3, output stored
// 9.2.  The final merge therefore has one round trip and one barrier: with the maxima, sums and outputs fetched one after
// the other and reduced through LDS with seven barriers it took 7.6 us of 14 (13.9 -> 9.9 us per call, 15.5 -> 11.1 on
// 6900 keys).
// With k_new/v_new given, row n_cached - 1 of the cache is taken from them instead of the cache and the workgroup
// that owns that key also stores it there (append and attention in one pass over the cache).
#include "common.h"

namespace purekv {
namespace {

constexpr int DEC_WAVES = 8;     // wavefronts per workgroup
constexpr int DEC_NT = 64 * DEC_WAVES;
constexpr int DEC_HB = 16;       // query heads per workgroup
// 16-key tiles per wavefront.  5491 keys x 4 KV heads, one call: 11.5 us with one tile (twice the chunks to merge), 9.9
// with two, 10.4 with three, 11.5 with four (fewer CUs pull the cache in).
constexpr int DEC_TILES = 2;
constexpr int DEC_CHUNK = 16 * DEC_TILES * DEC_WAVES;   // keys per workgroup

typedef short shortx4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) shortx4* LdsShortx4;

inline int decode_splits(int n) { return n <= 0 ? 1 : (n + DEC_CHUNK - 1) / DEC_CHUNK; }

struct DecodeArgs {
  const uint16_t* q;
  const uint16_t* k_new;   // [Hkv, D] or null
  const uint16_t* v_new;
  uint16_t* kc;
  uint16_t* vc;
  uint16_t* out;
  float* ws_o;        // [n_splits, Hq, D] unnormalised partial outputs
  float* ws_ml;       // [n_splits, Hq, 2] running maximum (log2 domain) and sum
  int32_t* counters;  // [Hkv * n_head_blocks], zero on entry and on exit
  int32_t Hq, G, n_cached, cap, n_splits;
  float scale_log2;
};

// Maximum / sum over groups of W lanes (16 or 32), result in every lane: rows of 16 on the DPP path of the vector ALU
// (lane ^ 1, lane ^ 2, mirror of 8, mirror of 16), two rows by v_permlane16_swap.
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
template <int W>
__device__ __forceinline__ float group_max(float x) {
  x = fmaxf(x, dpp_f32<0xB1>(x));
  x = fmaxf(x, dpp_f32<0x4E>(x));
  x = fmaxf(x, dpp_f32<0x141>(x));
  x = fmaxf(x, dpp_f32<0x140>(x));
  if constexpr (W == 32) {
    const LanePair p = swap16(x);
    x = fmaxf(p.a, p.b);
  }
  return x;
}
template <int W>
__device__ __forceinline__ float group_sum(float x) {
  x += dpp_f32<0xB1>(x);
  x += dpp_f32<0x4E>(x);
  x += dpp_f32<0x141>(x);
  x += dpp_f32<0x140>(x);
  if constexpr (W == 32) {
    const LanePair p = swap16(x);
    x = p.a + p.b;
  }
  return x;
}

template <int D>
__global__ __launch_bounds__(DEC_NT) void decode_kernel(const DecodeArgs a) {
  constexpr int KT = DEC_TILES;
  constexpr int KEYS = 16 * KT;         // keys per wavefront
  constexpr int KS = D / 32;            // k-steps of the score product
  constexpr int NC = D / 16;            // 16-column blocks of the output
  constexpr int CPR = D / 8;            // 16-byte pieces per row
  constexpr int NV = KEYS * CPR / 64;   // V pieces per lane
  constexpr int VROW = D * 2 + 32;      // bytes per V row in LDS (padded: consecutive rows start 8 banks apart)
  constexpr int OROW = D + 4;           // floats per head of a wavefront's output block (padded likewise)
  constexpr int LPR = D / 4;            // lanes per row of four-column pieces in the merges
  constexpr int NG = DEC_NT / LPR;      // groups of LPR lanes
  constexpr int SB = 4 * LPR;           // chunks per pass of the final merge (four per lane)
  constexpr int U = 16;                 // partial outputs in flight per lane in the final merge
  constexpr int kVBytes = KEYS * VROW, kOBytes = DEC_HB * OROW * 4;
  __shared__ __attribute__((aligned(16))) uint8_t smem[DEC_WAVES][kVBytes > kOBytes ? kVBytes : kOBytes];
  __shared__ float lds_ml[DEC_WAVES][DEC_HB][2];
  __shared__ int lds_last;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n = lane & 15, kg = lane >> 4;
  const int split = blockIdx.x, kvh = blockIdx.y, g0 = blockIdx.z * DEC_HB;
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
  const int n_valid = a.n_cached - key0;   // keys of this wavefront that exist (may be <= 0 or > KEYS)
  float sc[KT][4];
  float m = -INFINITY;
#pragma unroll
  for (int t = 0; t < KT; ++t) {
    floatx4 sacc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < KS; ++s) sacc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[t][s], qf[s], sacc, 0, 0, 0);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      sc[t][i] = (16 * t + 4 * kg + i < n_valid) ? sacc[i] * a.scale_log2 : -INFINITY;
      m = fmaxf(m, sc[t][i]);
    }
  }
  {
    const LanePair p = swap16(m);
    const LanePair q = swap32(fmaxf(p.a, p.b));
    m = fmaxf(q.a, q.b);
  }
  const float mu = (m == -INFINITY) ? 0.f : m;
  float l = 0.f;
  shortx4 pa[KT];
#pragma unroll
  for (int t = 0; t < KT; ++t) {
    const uint32_t w0 = pack_bf16(__builtin_amdgcn_exp2f(sc[t][0] - mu), __builtin_amdgcn_exp2f(sc[t][1] - mu));
    const uint32_t w1 = pack_bf16(__builtin_amdgcn_exp2f(sc[t][2] - mu), __builtin_amdgcn_exp2f(sc[t][3] - mu));
    l += (bf16_lo(w0) + bf16_hi(w0)) + (bf16_lo(w1) + bf16_hi(w1));   // the sum of what is multiplied with V
    pa[t] = __builtin_bit_cast(shortx4, u32x2{w0, w1});
  }
  {
    const LanePair p = swap16(l);
    const LanePair q = swap32(p.a + p.b);
    l = q.a + q.b;
  }
  if (kg == 0) {
    lds_ml[wave][n][0] = m;
    lds_ml[wave][n][1] = l;
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
      o[c] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int t = 0; t < KT; ++t) {
        const shortx4 vfrag = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LdsShortx4)(vb + 16 * t * VROW + 32 * c));
        o[c] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(vfrag, pa[t], o[c], 0, 0, 0);
      }
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
  if (j_new >= 0 && blockIdx.z == 0 && j_new >= key0 && j_new < key0 + KEYS) {
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
  const BufferRsrc ws_ml = make_rsrc(a.ws_ml + (size_t)split * a.Hq * 2);
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
      store_device_16(ws_o, (uint32_t)(hq * D + 4 * li) * 4u, acc);
      if (li == 0) store_device_8(ws_ml, (uint32_t)hq * 8u, floatx2{mn, ls});
    }
  }
  if (single) return;

  // ---- the workgroup that arrives last merges the chunks ----
  // Partial results travel through device-scope stores and loads only (they pass through the L2 of the XCD that
  // issues them, so the eight L2s need no write-back or invalidation); the arrival is counted once every store of
  // the workgroup has completed.
  int32_t* counter = a.counters + kvh * gridDim.z + blockIdx.z;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this thread's stores have completed
  __syncthreads();
  if (tid == 0) lds_last = __hip_atomic_fetch_add(counter, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == a.n_splits - 1;
  __syncthreads();
  if (!lds_last) return;
  asm volatile("" ::: "memory");

  // What this costs is round trips to memory, so there is one: a group of LPR lanes takes one head (its four-column
  // pieces side by side) and every n_parts-th chunk, requests the (max, sum) pairs of ALL chunks of its head (chunk c on
  // lane c % LPR) and its first U partial outputs together, turns the pairs into weights with cross-lane steps and a table
  // of its own in LDS -- no barrier -- and adds up.  Then the parts of a head are added through LDS, in order.
  const int n_parts = NG / ng, part = gi / ng, g = gi - part * ng;   // ng <= NG
  const bool work = part < n_parts;
  const int hq = kvh * a.G + g0 + g;
  const uint32_t o_stride = (uint32_t)a.Hq * D * 4u, ml_stride = (uint32_t)a.Hq * 8u;
  float* const wl = reinterpret_cast<float*>(&smem[0][0]) + gi * SB;   // [SB] weights of this pass' chunks
  static_assert(NG * SB * 4 + DEC_NT * 16 <= (int)sizeof(smem), "weight tables and the parts' sums fit");
  float* const ps = reinterpret_cast<float*>(&smem[0][0]) + NG * SB;   // [DEC_NT][4] sums of the parts
  float run_m = -INFINITY, run_l = 0.f;
  floatx4 acc = {0.f, 0.f, 0.f, 0.f};
  if (work) {
    for (int s0 = 0; s0 < a.n_splits; s0 += SB) {
      const int nsb = min(SB, a.n_splits - s0);
      // (32-bit offsets from the pass' own base)
      const BufferRsrc mlb = make_rsrc(a.ws_ml + (size_t)s0 * a.Hq * 2), ob = make_rsrc(a.ws_o + (size_t)s0 * a.Hq * D);
      floatx2 ml[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        ml[r] = floatx2{-INFINITY, 0.f};
        if (li + r * LPR < nsb) ml[r] = load_device_8(mlb, (uint32_t)(li + r * LPR) * ml_stride + (uint32_t)hq * 8u);
      }
      floatx4 ov[U];
      auto load_batch = [&](int c0) {   // only what exists is requested
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int c = c0 + u * n_parts;
          ov[u] = floatx4{0.f, 0.f, 0.f, 0.f};
          if (c < nsb) ov[u] = load_device_16(ob, (uint32_t)c * o_stride + (uint32_t)(hq * D + 4 * li) * 4u);
        }
      };
      load_batch(part);
      float pm = fmaxf(fmaxf(ml[0][0], ml[1][0]), fmaxf(ml[2][0], ml[3][0]));
      pm = group_max<LPR>(pm);
      const float mnew = fmaxf(run_m, pm);
      const float mref = (mnew == -INFINITY) ? 0.f : mnew;   // every score so far is -inf: weights 0, not NaN
      float lsum = 0.f;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float f = __builtin_amdgcn_exp2f(ml[r][0] - mref);
        lsum += ml[r][1] * f;
        wl[li + r * LPR] = f;
      }
      lsum = group_sum<LPR>(lsum);
      const float fo = __builtin_amdgcn_exp2f(run_m - mref);   // first pass: 2^(-inf) = 0
      acc *= fo;
      run_l = run_l * fo + lsum;
      run_m = mnew;
      asm volatile("" ::: "memory");   // the table is read by other lanes of the wavefront that wrote it
      for (int c0 = part;;) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int c = c0 + u * n_parts;
          if (c < nsb) acc += ov[u] * wl[c];
        }
        c0 += U * n_parts;
        if (c0 >= nsb) break;
        load_batch(c0);
      }
      asm volatile("" ::: "memory");
    }
  }
  if (n_parts > 1) {
    *reinterpret_cast<floatx4*>(ps + 4 * tid) = acc;
    __syncthreads();
    if (work && part == 0)
      for (int p = 1; p < n_parts; ++p) acc += *reinterpret_cast<const floatx4*>(ps + 4 * (tid + p * ng * LPR));
  }
  if (work && part == 0) {
    u32x2 w;
    w[0] = f32_to_bf16(acc[0] / run_l) | (f32_to_bf16(acc[1] / run_l) << 16);
    w[1] = f32_to_bf16(acc[2] / run_l) | (f32_to_bf16(acc[3] / run_l) << 16);
    *reinterpret_cast<u32x2*>(a.out + (size_t)hq * D + 4 * li) = w;
  }
  if (tid == 0) __hip_atomic_store(counter, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // ready for the next call
}

}  // namespace

// Workspace: [arrival counters, padded to 256 bytes][partial outputs][their (max, sum)].
static int decode_counter_count(const purekv_plan& p) { return p.g.Hkv * ((p.g.G + DEC_HB - 1) / DEC_HB); }
static size_t decode_counter_bytes(const purekv_plan& p) {
  return ((size_t)decode_counter_count(p) * sizeof(int32_t) + 255) / 256 * 256;
}

size_t decode_ws_bytes(const purekv_plan& p, int32_t cap) {
  return decode_counter_bytes(p) + (size_t)decode_splits(cap) * p.g.Hq * (p.g.d + 2) * sizeof(float);
}

namespace {
__global__ void clear_decode_counters_kernel(int32_t* c, int n) {   // a kernel, not a memset: callers may be capturing
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) c[i] = 0;
}
}  // namespace

int launch_decode_ws_init(const purekv_plan& p, void* ws, hipStream_t st) {
  const int n = decode_counter_count(p);
  hipLaunchKernelGGL(clear_decode_counters_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st,
                     static_cast<int32_t*>(ws), n);
  PUREKV_HIP_TRY(hipGetLastError());
  return PUREKV_OK;
}

int launch_decode(const purekv_plan& p, const void* q_new, const void* k_new, const void* v_new, void* kc, void* vc,
                  int32_t n_cached, int32_t cap, void* out, void* ws, hipStream_t st) {
  DecodeArgs a;
  a.q = static_cast<const uint16_t*>(q_new);
  a.k_new = static_cast<const uint16_t*>(k_new);
  a.v_new = static_cast<const uint16_t*>(v_new);
  a.kc = static_cast<uint16_t*>(kc);
  a.vc = static_cast<uint16_t*>(vc);
  a.out = static_cast<uint16_t*>(out);
  const int head_blocks = (p.g.G + DEC_HB - 1) / DEC_HB;
  a.n_splits = decode_splits(n_cached);
  a.counters = static_cast<int32_t*>(ws);
  a.ws_o = reinterpret_cast<float*>(static_cast<char*>(ws) + decode_counter_bytes(p));
  a.ws_ml = a.ws_o + (size_t)decode_splits(cap) * p.g.Hq * p.g.d;
  a.Hq = p.g.Hq;
  a.G = p.g.G;
  a.n_cached = n_cached;
  a.cap = cap;
  a.scale_log2 = p.g.scale * kLog2e;
  const dim3 grid((unsigned)a.n_splits, (unsigned)p.g.Hkv, (unsigned)head_blocks);
  auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, dim3(DEC_NT), 0, st, a); };
  if (p.g.d == 128)
    launch(decode_kernel<128>);
  else
    launch(decode_kernel<64>);
  PUREKV_HIP_TRY(hipGetLastError());
  return PUREKV_OK;
}

}  // namespace purekv
