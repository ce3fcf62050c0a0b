// Paged-manager steps either side of the attention path (paper Sec. 4.1: the KV cache grows chunk
// by chunk in pages; Sec. 4.2: page means represent the pages, local-attention layers retrieve the
// most recent pages):
//   kv_append          the chunk's K / V -> its m local pages in the pools
//   page_means         mean of each page of a range -> cache [logical page][KV head][D] (fp32)
//   page_score_cached  scores from the cached means instead of streaming the keys
//   local_page_list    the page list of a local-attention layer
// The means and scores use the fixed fp32 operation order of the streaming scorer
// (score_topk.hip), so both paths give the same bits.
#include "common.h"
#include "launch.h"
#include "rowsum.h"

#pragma clang fp contract(off)

namespace oomb {

// chunk K / V [C][Hkv][D] (contiguous) -> pool page page_table[n_past + page of the chunk], one workgroup per (page, KV head, slice of DW dims), and (cache given) the
// page's mean while its keys are in LDS: one launch for both.  32 + 1 pages x 4 heads: 36 -> 6 us with the means, which used to
// walk the pool once more, one thread per dim.
template <typename T, int D, int DW>
__global__ __launch_bounds__(256) void kv_append_kernel(Params p, const T* __restrict__ kc, const T* __restrict__ vc, T* __restrict__ k_pool,
                                                        T* __restrict__ v_pool, float inv_p, float* __restrict__ cache) {
  extern __shared__ __align__(16) unsigned char lds[];
  constexpr int VEC = Vec16<T>::N, GPR = DW / VEC, NS = D / DW;
  const int b = blockIdx.x / NS, d0 = (blockIdx.x - b * NS) * DW, tau = b / p.Hkv, g = b - tau * p.Hkv, tid = threadIdx.x;
  const int64_t l = p.n_past + tau;
  const int64_t src = ((int64_t)tau * p.P * p.Hkv + g) * D + d0, stride = (int64_t)p.Hkv * D;
  const int64_t dst = (int64_t)p.page_table[l] * p.pool_page_stride + (int64_t)g * p.pool_head_stride + d0;
  const int total = p.P * GPR;
  for (int e0 = tid; e0 < total; e0 += 8 * 256) {   // (the loads of K and V are all in flight before the first store)
    uint4 a[8], b[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int e = e0 + u * 256 < total ? e0 + u * 256 : e0;
      const int64_t at = src + (int64_t)(e / GPR) * stride + (e % GPR) * VEC;
      a[u] = *reinterpret_cast<const uint4*>(kc + at);
      b[u] = *reinterpret_cast<const uint4*>(vc + at);
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int e = e0 + u * 256;
      if (e >= total) break;
      const int64_t at = dst + (int64_t)(e / GPR) * p.pool_tok_stride + (e % GPR) * VEC;
      *reinterpret_cast<uint4*>(k_pool + at) = a[u];
      *reinterpret_cast<uint4*>(v_pool + at) = b[u];
      if (cache) reinterpret_cast<uint4*>(lds)[e] = a[u];
    }
  }
  if (!cache) return;
  __syncthreads();
  float* out = cache + ((int64_t)l * p.Hkv + g) * D + d0;
  lds_row_sum<T, DW>(p.P, lds, [&](int d, float sum) __attribute__((always_inline)) { out[d] = __fmul_rn(sum, inv_p); });
}

// mean of logical pages [first, first + count) with 16-byte loads: a group of LPR lanes walks one (page, KV head)
// tile token by token; this is the kernel that streams a whole history when the means are not cached.
template <typename T, int D>
__global__ __launch_bounds__(256) void page_means_vec_kernel(Params p, int64_t first, int64_t count, float inv_p,
                                                             float* __restrict__ cache) {
  constexpr int VEC = Vec16<T>::N, LPR = D / VEC, PPB = 256 / LPR;
  const int g = blockIdx.y;
  const int lr = threadIdx.x % LPR;
  const int64_t k = (int64_t)blockIdx.x * PPB + threadIdx.x / LPR;
  if (k >= count) return;
  const int64_t l = first + k;
  const T* base = (const T*)p.k_pool + (int64_t)p.page_table[l] * p.pool_page_stride +
                  (int64_t)g * p.pool_head_stride + lr * VEC;
  float x[VEC];
  seq_row_sum<T, 8, true>(base, p.pool_tok_stride, p.P, x);
  float* out = cache + ((int64_t)l * p.Hkv + g) * D + lr * VEC;
#pragma unroll
  for (int v = 0; v < VEC; ++v) out[v] = __fmul_rn(x[v], inv_p);
}

// score[g][l] = tree sum over d of qbar[g][d] * cache[l][g][d] (stride-halving tree, strides D/2 .. 1):
// a group of D / 4 lanes per (head, page), four floats per lane
template <int D>
__global__ __launch_bounds__(256) void page_score_cached_kernel(Params p, const float* __restrict__ qbar,
                                                                const float* __restrict__ cache,
                                                                float* __restrict__ scores) {
  constexpr int VEC = 4, LPR = D / VEC, PPB = 256 / LPR;
  const int g = blockIdx.y;
  const int lr = threadIdx.x % LPR;
  const int64_t l = (int64_t)blockIdx.x * PPB + threadIdx.x / LPR;
  const bool active = l < p.n_past;
  const int64_t lc = active ? l : 0;
  const float4 kb = load_floats(cache + ((int64_t)lc * p.Hkv + g) * D + lr * VEC);
  const float4 qb = load_floats(qbar + g * D + lr * VEC);
  const float s = score_tree<D>(qb, kb);
  if (active && lr == 0) scores[(int64_t)g * p.n_past + l] = s;
}

__global__ void local_page_list_kernel(int64_t n_past, int64_t n, int32_t window, int32_t stride,
                                       int32_t* __restrict__ sel, int32_t* __restrict__ sel_count) {
  const int g = blockIdx.x;
  const int64_t w = window < n_past ? window : n_past;
  const int32_t cnt = (int32_t)(w + (n - n_past));
  for (int32_t j = threadIdx.x; j < stride; j += blockDim.x)
    sel[(int64_t)g * stride + j] = j < cnt ? (int32_t)(n_past - w + j) : -1;
  if (threadIdx.x == 0) sel_count[g] = cnt;
}

template <typename T, int D, int DW>
static hipError_t append(const Params& p, const void* kc, const void* vc, void* k_pool, void* v_pool, float* cache, hipStream_t st) {
  ProfScope prof_("kv_append", st);
  const size_t lds = cache ? (size_t)p.P * DW * sizeof(T) : 0;   // (at most 16 KiB)
  kv_append_kernel<T, D, DW><<<dim3((unsigned)p.m * p.Hkv * (D / DW)), dim3(256), lds, st>>>(p, (const T*)kc, (const T*)vc, (T*)k_pool, (T*)v_pool,
                                                                                             1.0f / (float)p.P, cache);
  return hipGetLastError();
}
template <typename T, int D>
static hipError_t append(const Params& p, const void* kc, const void* vc, void* k_pool, void* v_pool, float* cache, hipStream_t st) {
  return page_in_slices<T>(p) ? append<T, D, LINE_DIMS<T>>(p, kc, vc, k_pool, v_pool, cache, st) : append<T, D, D>(p, kc, vc, k_pool, v_pool, cache, st);
}
hipError_t launch_kv_append(const Params& p, bool is_bf16, const void* kc, const void* vc, void* k_pool, void* v_pool,
                            float* cache, hipStream_t st) {
  if (is_bf16) return p.D == 128 ? append<bf16_t, 128>(p, kc, vc, k_pool, v_pool, cache, st) : append<bf16_t, 64>(p, kc, vc, k_pool, v_pool, cache, st);
  return p.D == 128 ? append<float, 128>(p, kc, vc, k_pool, v_pool, cache, st) : append<float, 64>(p, kc, vc, k_pool, v_pool, cache, st);
}

hipError_t launch_page_means(const Params& p, bool is_bf16, int64_t first, int64_t count, float* cache, hipStream_t st) {
  if (count <= 0) return hipSuccess;
  const float inv_p = 1.0f / (float)p.P;
  ProfScope prof_("page_means", st);
  const int lpr = is_bf16 ? p.D / 8 : p.D / 4, ppb = 256 / lpr;
  dim3 grid((unsigned)((count + ppb - 1) / ppb), (unsigned)p.Hkv);
  if (is_bf16 && p.D == 128) page_means_vec_kernel<bf16_t, 128><<<grid, dim3(256), 0, st>>>(p, first, count, inv_p, cache);
  else if (is_bf16) page_means_vec_kernel<bf16_t, 64><<<grid, dim3(256), 0, st>>>(p, first, count, inv_p, cache);
  else if (p.D == 128) page_means_vec_kernel<float, 128><<<grid, dim3(256), 0, st>>>(p, first, count, inv_p, cache);
  else page_means_vec_kernel<float, 64><<<grid, dim3(256), 0, st>>>(p, first, count, inv_p, cache);
  return hipGetLastError();
}

hipError_t launch_page_score_cached(const Params& p, const float* qbar, const float* cache, float* scores, hipStream_t st) {
  if (p.n_past <= 0) return hipSuccess;
  ProfScope prof_("page_score_cached", st);
  if (p.D == 128) {
    dim3 grid((unsigned)((p.n_past + 7) / 8), p.Hkv);
    page_score_cached_kernel<128><<<grid, dim3(256), 0, st>>>(p, qbar, cache, scores);
  } else {
    dim3 grid((unsigned)((p.n_past + 15) / 16), p.Hkv);
    page_score_cached_kernel<64><<<grid, dim3(256), 0, st>>>(p, qbar, cache, scores);
  }
  return hipGetLastError();
}

hipError_t launch_local_page_list(const Params& p, int32_t window, int32_t* sel, int32_t* sel_count, hipStream_t st) {
  ProfScope prof_("local_page_list", st);
  local_page_list_kernel<<<dim3(p.Hkv), dim3(256), 0, st>>>(p.n_past, p.n, window, window + p.m, sel, sel_count);
  return hipGetLastError();
}

}  // namespace oomb
