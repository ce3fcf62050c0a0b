// Accumulators on their way out: groups of four consecutive dims, and the layout of partial results (of calls whose
// keys or rows are split over workgroups) together with the kernel that adds them up.
#pragma once
#include "mfma_common.h"

namespace oomb {

constexpr int PART_ROWS = 128;  // rows of a row tile / keys of a unit: four blocks of 32
// blocks of 32 keys in a dK / dV unit: 128 keys, or (one list per query page) one page
__host__ __device__ __forceinline__ int part_key_blocks(const Params& p) { return !p.qp ? PART_ROWS / 32 : p.P <= 32 ? 1 : p.P / 32; }

// the accumulator in groups of four consecutive dims: f(dim, a, b, c, d) for D / 8 groups per lane
template <typename T, int D, typename F>
__device__ __forceinline__ void part_emit(const f32x16 (&acc)[D / 32], int hh, F&& f) {
  if constexpr (sizeof(T) == 2) {
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
      for (int a = 0; a < 4; ++a)
        f(32 * db + 8 * a + 4 * hh, acc[db][4 * a], acc[db][4 * a + 1], acc[db][4 * a + 2], acc[db][4 * a + 3]);
  } else if constexpr (D == 128) {
#pragma unroll
    for (int x = 0; x < 16; ++x) f(4 * (8 * (x >> 2) + 4 * hh + (x & 3)), acc[0][x], acc[1][x], acc[2][x], acc[3][x]);
  } else {
#pragma unroll
    for (int x = 0; x < 16; x += 2)
      f(2 * (8 * (x >> 2) + 4 * hh + (x & 3)), acc[0][x], acc[1][x], acc[0][x + 1], acc[1][x + 1]);
  }
}
// Partial results keep the register order -- float4 [block of 32 rows][group of part_emit][lane] -- so that every store and
// load of a wave is one contiguous KiB
template <typename T, int D>
__device__ __forceinline__ void part_store(float* part, int64_t block, int lane, const f32x16 (&acc)[D / 32], float scale) {
  float4* dst = reinterpret_cast<float4*>(part) + block * (D / 8) * 64 + lane;
  int k = 0;
  part_emit<T, D>(acc, lane >> 5, [&](int, float a, float b, float c, float d) __attribute__((always_inline)) {
    dst[64 * k++] = make_float4(a * scale, b * scale, c * scale, d * scale);
  });
}
// the first dim of group k of a lane
template <typename T, int D> __device__ __forceinline__ int part_group_dim(int k, int hh) {
  if (sizeof(T) == 2) return 32 * (k >> 2) + 8 * (k & 3) + 4 * hh;
  const int x = D == 128 ? k : 2 * k;
  return (D / 32) * (8 * (x >> 2) + 4 * hh + (x & 3));
}
template <typename T> __device__ __forceinline__ void part_store4(T* p, float a, float b, float c, float d);
template <> __device__ __forceinline__ void part_store4<float>(float* p, float a, float b, float c, float d) {
  *reinterpret_cast<float4*>(p) = make_float4(a, b, c, d);
}
template <> __device__ __forceinline__ void part_store4<bf16_t>(bf16_t* p, float a, float b, float c, float d) {
  *reinterpret_cast<uint2*>(p) = make_uint2(pack2_bf16(a, b), pack2_bf16(c, d));
}
template <typename T> __device__ __forceinline__ float4 part_load4(const T* p);
template <> __device__ __forceinline__ float4 part_load4<float>(const float* p) { return *reinterpret_cast<const float4*>(p); }
template <> __device__ __forceinline__ float4 part_load4<bf16_t>(const bf16_t* p) {
  const uint2 v = *reinterpret_cast<const uint2*>(p);
  return make_float4(__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xffff0000u), __uint_as_float(v.y << 16), __uint_as_float(v.y & 0xffff0000u));
}
template <typename T> __device__ __forceinline__ void part_add4(T* p, float a, float b, float c, float d) {
  const float4 v = part_load4<T>(p);
  part_store4<T>(p, v.x + a, v.y + b, v.z + c, v.w + d);
}

// What is left of a backward with splits, in one launch (attn_generic.hip): the dQ partials of `dq_split` key ranges
// (1: none) and, with kv_units > 0, the slices of that many dK / dV units per KV head.  Slot of slice sp of unit u and KV
// head g: (u kv_split + sp) Hkv + g, or as the work table says with one list per query page; a slot holds the blocks of
// 32 keys x D of a unit (part_key_blocks): dK, then dV.
hipError_t launch_bwd_finish(const Params& p, bool is_bf16, int32_t dq_split, const float* dq_part, int32_t kv_units, int32_t kv_split,
                             const float* kv_part, hipStream_t st);

}  // namespace oomb
