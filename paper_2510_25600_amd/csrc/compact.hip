// KV-cache compaction: gather of the kept rows (selection rule of Sec. 3.1) into a compact cache, and the
// append of one decoded token.  Pure byte movement: one 16-lane group (8 for head_dim 64) moves one
// row of K and one of V with 16-byte loads and stores; indices ascend, so reads walk HBM forwards.
#include <algorithm>

#include "common.h"

namespace purekv {
namespace {

// grid = (row blocks, layers * Hkv).  Bound by two dependent trips to memory (index, rows) for one layer, by HBM for a stack.
// (One axis over all rows took two 64-bit divisions per row ahead of them: 2.96 against 1.80 us for 57 rows of 64, 5.5 against
// 5.3 for 1689 x 4 of 128, 31.4 against 31.0 for 26 layers of those.  Two rows in flight per lane and twice the workgroups of four:
// 29.5 for the 26 layers; one: 29.0, but 2.1 for the 57 rows.)
template <int D>
__global__ __launch_bounds__(256) void compact_kernel(const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
                                                      int64_t layer_stride, int64_t head_stride, int64_t tok_stride,
                                                      const int32_t* __restrict__ idx,
                                                      uint16_t* __restrict__ kc, uint16_t* __restrict__ vc, int32_t N,
                                                      int32_t Hkv, int32_t n_keep, int32_t cap) {
  constexpr int LPR = D / 8, RPB = 256 / LPR, UNROLL = 2;
  const int sub = threadIdx.x % LPR, rslot = threadIdx.x / LPR;
  const int lk = blockIdx.y, layer = lk / Hkv, kvh = lk - layer * Hkv;
  const int64_t src0 = layer * layer_stride + kvh * head_stride + sub * 8;
  const int64_t dst0 = (int64_t)lk * cap * D + sub * 8;
  const int32_t* const rows = idx + (int64_t)lk * n_keep;
  const int pos0 = blockIdx.x * (RPB * UNROLL) + rslot;
  int32_t j[UNROLL];
#pragma unroll
  for (int u = 0; u < UNROLL; ++u) j[u] = rows[min(pos0 + u * RPB, n_keep - 1)];
  u32x4 xk[UNROLL], xv[UNROLL];
#pragma unroll
  for (int u = 0; u < UNROLL; ++u) {
    const int64_t src = src0 + min(max(j[u], 0), N - 1) * tok_stride;
    xk[u] = *reinterpret_cast<const u32x4*>(k + src);
    xv[u] = *reinterpret_cast<const u32x4*>(v + src);
  }
#pragma unroll
  for (int u = 0; u < UNROLL; ++u) {
    const int pos = pos0 + u * RPB;
    if (pos < n_keep) {
      // (non-temporal: the compact cache is written once here and read by a later launch: 0.97 of the time of plain stores for
      // the 26-layer batch of the 32-frame shape; the same hint on the gathered loads costs 8 %)
      const int64_t dst = dst0 + (int64_t)pos * D;
      __builtin_nontemporal_store(xk[u], reinterpret_cast<u32x4*>(kc + dst));
      __builtin_nontemporal_store(xv[u], reinterpret_cast<u32x4*>(vc + dst));
    }
  }
}

__global__ void append_kernel(const uint16_t* __restrict__ k_new, const uint16_t* __restrict__ v_new,
                              uint16_t* __restrict__ kc, uint16_t* __restrict__ vc, int32_t Hkv, int32_t d,
                              int32_t n_cached, int32_t cap) {
  const int chunks = d / 8;
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= Hkv * chunks) return;
  const int kvh = t / chunks, c = t % chunks;
  const size_t dst = ((size_t)kvh * cap + n_cached) * d + c * 8, src = (size_t)kvh * d + c * 8;
  *reinterpret_cast<u32x4*>(kc + dst) = *reinterpret_cast<const u32x4*>(k_new + src);
  *reinterpret_cast<u32x4*>(vc + dst) = *reinterpret_cast<const u32x4*>(v_new + src);
}

}  // namespace

int launch_compact(const purekv_plan& p, const void* k, const void* v, int64_t kv_layer_stride, int32_t n_layers,
                   const int32_t* idx, int32_t n_keep, void* kc, void* vc, int32_t cap, hipStream_t st) {
  if (n_keep == 0) return PUREKV_OK;
  const int rows_per_block = (256 / (p.g.d / 8)) * 2;
  const unsigned gx = (unsigned)((n_keep + rows_per_block - 1) / rows_per_block);
  // (a grid has 65535 blocks on its second axis: more heads than that go layer by layer, in as many launches as it takes)
  const int32_t layers_per_launch = std::max(1, 65535 / p.g.Hkv);
  for (int32_t l0 = 0; l0 < n_layers; l0 += layers_per_launch) {
    const dim3 grid(gx, (unsigned)(std::min(layers_per_launch, n_layers - l0) * p.g.Hkv));
    const int64_t src = l0 * kv_layer_stride, rows = (int64_t)l0 * p.g.Hkv;
    const uint16_t *ks = static_cast<const uint16_t*>(k) + src, *vs = static_cast<const uint16_t*>(v) + src;
    uint16_t *kd = static_cast<uint16_t*>(kc) + rows * cap * p.g.d, *vd = static_cast<uint16_t*>(vc) + rows * cap * p.g.d;
    auto launch = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, grid, dim3(256), 0, st, ks, vs, kv_layer_stride, p.g.kv_sh, p.g.kv_st, idx + rows * n_keep, kd, vd,
                         p.g.N, p.g.Hkv, n_keep, cap);
    };
    if (p.g.d == 128) launch(compact_kernel<128>);
    else launch(compact_kernel<64>);
  }
  PUREKV_HIP_TRY(hipGetLastError());
  return PUREKV_OK;
}

int launch_append(const purekv_plan& p, const void* k_new, const void* v_new, void* kc, void* vc, int32_t n_cached,
                  int32_t cap, hipStream_t st) {
  const int total = p.g.Hkv * (p.g.d / 8);
  hipLaunchKernelGGL(append_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st,
                     static_cast<const uint16_t*>(k_new), static_cast<const uint16_t*>(v_new),
                     static_cast<uint16_t*>(kc), static_cast<uint16_t*>(vc), p.g.Hkv, p.g.d, n_cached, cap);
  PUREKV_HIP_TRY(hipGetLastError());
  return PUREKV_OK;
}

}  // namespace purekv
