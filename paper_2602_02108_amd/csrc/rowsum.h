// Sequential fp32 row sums with 16-byte loads, shared by the page scorer and the paged manager
// (paper Sec. 4.2: a key page is represented by the mean of its keys).  The additions stay in
// token order with one rounding each, so every user produces the same bits.
#pragma once
#include "common.h"

#pragma clang fp contract(off)

namespace oomb {

template <typename T> struct Vec16;  // one 16-byte load worth of elements
template <> struct Vec16<float> {
  static constexpr int N = 4;
  static __device__ __forceinline__ void unpack(const uint4& r, float* f) {
    f[0] = __uint_as_float(r.x); f[1] = __uint_as_float(r.y);
    f[2] = __uint_as_float(r.z); f[3] = __uint_as_float(r.w);
  }
};
template <> struct Vec16<bf16_t> {
  static constexpr int N = 8;
  static __device__ __forceinline__ void unpack(const uint4& r, float* f) {
    f[0] = __uint_as_float(r.x << 16); f[1] = __uint_as_float(r.x & 0xffff0000u);
    f[2] = __uint_as_float(r.y << 16); f[3] = __uint_as_float(r.y & 0xffff0000u);
    f[4] = __uint_as_float(r.z << 16); f[5] = __uint_as_float(r.z & 0xffff0000u);
    f[6] = __uint_as_float(r.w << 16); f[7] = __uint_as_float(r.w & 0xffff0000u);
  }
};

// 16 bytes, optionally with a non-temporal load
template <bool STREAM> __device__ __forceinline__ uint4 load16(const void* ptr) {
  typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
  if (STREAM) {
    const u32x4_t v = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(ptr));
    return make_uint4(v.x, v.y, v.z, v.w);
  }
  return *reinterpret_cast<const uint4*>(ptr);
}

// four floats of a workspace, which need not be aligned beyond a float (one load all the same)
__device__ __forceinline__ float4 load_floats(const float* ptr) {
  typedef float f32x4_t __attribute__((ext_vector_type(4), aligned(4)));
  const f32x4_t v = *reinterpret_cast<const f32x4_t*>(ptr);
  return make_float4(v.x, v.y, v.z, v.w);
}

// Left-to-right sum of `count` rows (row stride `stride` elements) of the VEC
// elements this lane owns.  Loads are issued U at a time, adds stay in order.
// STREAM: the rows are read once and not again soon (the whole key history behind the page scorer):
// non-temporal loads, which neither displace what the next kernels need from the caches nor wait for
// an allocation there (page scoring at the 1M-token benchmark shape: 5.0 -> 6.2 TB/s).
template <typename T, int U, bool STREAM = false>
__device__ __forceinline__ void seq_row_sum(const T* base, int64_t stride, int count, float* acc) {
  constexpr int VEC = Vec16<T>::N;
#pragma unroll
  for (int v = 0; v < VEC; ++v) acc[v] = 0.0f;
  int t = 0;
  for (; t + U <= count; t += U) {
    uint4 r[U];
#pragma unroll
    for (int u = 0; u < U; ++u) r[u] = load16<STREAM>(base + (int64_t)(t + u) * stride);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float f[VEC];
      Vec16<T>::unpack(r[u], f);
#pragma unroll
      for (int v = 0; v < VEC; ++v) acc[v] = __fadd_rn(acc[v], f[v]);
    }
  }
  for (; t < count; ++t) {
    const uint4 r = load16<STREAM>(base + (int64_t)t * stride);
    float f[VEC];
    Vec16<T>::unpack(r, f);
#pragma unroll
    for (int v = 0; v < VEC; ++v) acc[v] = __fadd_rn(acc[v], f[v]);
  }
}

// <q, k> over D dims held four per lane by D / 4 consecutive lanes: one product per dim, then a tree of strides D / 2 .. 1
// (valid in the first of the lanes)
template <int D> __device__ __forceinline__ float score_tree(const float4& q, const float4& k) {
  float x[4] = {__fmul_rn(q.x, k.x), __fmul_rn(q.y, k.y), __fmul_rn(q.z, k.z), __fmul_rn(q.w, k.w)};
#pragma unroll
  for (int s = D / 2; s >= 4; s >>= 1) {
#pragma unroll
    for (int v = 0; v < 4; ++v) x[v] = __fadd_rn(x[v], __shfl_xor(x[v], s / 4, 64));
  }
  x[0] = __fadd_rn(x[0], x[2]);
  x[1] = __fadd_rn(x[1], x[3]);
  return __fadd_rn(x[0], x[1]);
}

// Sum of `count` rows of D elements by one workgroup, in the same order: the tile is brought into LDS with all its loads in
// flight at once (a chain of additions that waits for its own loads, 32 in flight, takes 8 us for 128 rows; this 3 to
// 4), then a thread owns one dim (fp32) or two (bf16) and walks the rows.
// lds: count * D elements, 16-byte aligned; out(d, sum) gets the sums.
template <typename T, int D, typename O>
__device__ __forceinline__ void lds_row_sum(int count, const unsigned char* lds, O&& out) {
  const int tid = threadIdx.x;
  constexpr int DPT = 4 / sizeof(T), RW = D / DPT;   // dims per thread, words per row
  if (tid >= RW) return;
  const uint32_t* w = reinterpret_cast<const uint32_t*>(lds) + tid;
  float a = 0.0f, b = 0.0f;
  auto add = [&](uint32_t x) __attribute__((always_inline)) {
    if (sizeof(T) == 4) {
      a = __fadd_rn(a, __uint_as_float(x));
    } else {
      a = __fadd_rn(a, __uint_as_float(x << 16));
      b = __fadd_rn(b, __uint_as_float(x & 0xffff0000u));
    }
  };
  int t = 0;
  for (; t + 16 <= count; t += 16) {
    uint32_t x[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) x[u] = w[(t + u) * RW];
#pragma unroll
    for (int u = 0; u < 16; ++u) add(x[u]);
  }
  for (; t < count; ++t) add(w[t * RW]);
  out(DPT * tid, a);
  if (sizeof(T) == 2) out(DPT * tid + 1, b);
}
template <typename T, int D, typename O>
__device__ __forceinline__ void tile_row_sum(const T* base, int64_t stride, int count, unsigned char* lds, O&& out) {
  constexpr int VEC = Vec16<T>::N, GPR = D / VEC, U = 8;
  const int tid = threadIdx.x, n = blockDim.x, total = count * GPR;
  for (int e0 = tid; e0 < total; e0 += U * n) {
    uint4 v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int e = e0 + u * n < total ? e0 + u * n : e0;
      v[u] = *reinterpret_cast<const uint4*>(base + (int64_t)(e / GPR) * stride + (e % GPR) * VEC);
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (e0 + u * n < total) reinterpret_cast<uint4*>(lds)[e0 + u * n] = v[u];
  }
  __syncthreads();
  lds_row_sum<T, D>(count, lds, out);
}

// Dims of a 128-byte line, and whether a page's tile is cut into slices of that width, a workgroup each.  What bounds a short call is how fast one
// compute unit takes in its tile (32 KiB: 3 us of a launch of 5 to 6), so more of them take less each; the 64 KiB of an fp32 page also left two
// workgroups to a compute unit.  Per launch, whole -> in slices: 28 query heads, one page of 128 in bf16 6.1 -> 5.1 us, the append of 4 KV heads with
// means 7.1 -> 6.1; fp32, 4 query pages and 124 past ones 14.7 -> 10.3 us (608 tiles).  Where the tiles fill the chip by themselves
// nothing changes (896 bf16 tiles: 9.1, 9.2).  Tiles below 16 KiB hold a few loads per thread as they are.
template <typename T> constexpr int LINE_DIMS = 128 / (int)sizeof(T);
template <typename T> static inline bool page_in_slices(const Params& p) { return p.D > LINE_DIMS<T> && (size_t)p.P * p.D * sizeof(T) >= 16384; }

}  // namespace oomb
