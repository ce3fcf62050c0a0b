// Page scoring and top-k page selection (paper Sec. 4.2): the mean of each key
// page is scored against the mean-pooled chunk query of its KV head and the
// top-K past pages are kept, plus the chunk's own pages.
//
// The fp32 operation order is fixed so that scores are reproducible bit for bit:
//   token sums left to right; qbar sums query pages (outer) then heads (inner);
//   dot product as a stride-halving tree over d.  No fused multiply-add.
// The page-mean kernel is HBM-bound: it streams every past key once.
#include <mutex>

#include "common.h"
#include "launch.h"
#include "rowsum.h"

#pragma clang fp contract(off)

namespace oomb {

// Step S1a: A[h][tau][d] = sum over the P tokens of query page tau of Q, one workgroup per (query page, head, slice of DW dims); with
// means != nullptr the workgroups past those compute S2 for one (past page, KV head, slice) each, means[l][g][d] as the paged
// manager caches them (short histories, whose pages are too few to fill the chip page by page).
template <typename T, int D, int DW>
__global__ __launch_bounds__(256) void qpool_partial_kernel(Params p, float* __restrict__ A, float* __restrict__ means, float inv_p) {
  extern __shared__ __align__(16) unsigned char lds[];
  constexpr int NS = D / DW;
  const int b = blockIdx.x / NS, d0 = (blockIdx.x - b * NS) * DW, n_q = p.Hq * p.m;
  if (b < n_q) {
    const int tau = b / p.Hq, h = b - tau * p.Hq;
    float* out = A + ((int64_t)h * p.m + tau) * D + d0;
    tile_row_sum<T, DW>((const T*)p.q + (int64_t)tau * p.P * p.q_tok_stride + (int64_t)h * p.q_head_stride + d0, p.q_tok_stride, p.P, lds,
                        [&](int d, float sum) __attribute__((always_inline)) { out[d] = sum; });
  } else {
    const int l = (b - n_q) / p.Hkv, g = (b - n_q) - l * p.Hkv;
    float* out = means + ((int64_t)l * p.Hkv + g) * D + d0;
    tile_row_sum<T, DW>((const T*)p.k_pool + (int64_t)p.page_table[l] * p.pool_page_stride + (int64_t)g * p.pool_head_stride + d0, p.pool_tok_stride, p.P, lds,
                        [&](int d, float sum) __attribute__((always_inline)) { out[d] = __fmul_rn(sum, inv_p); });
  }
}
template <typename T, int D, int DW> static void run_qpool_partial(const Params& p, float* A, float* means, float inv_p, hipStream_t st) {
  const int64_t tiles = (int64_t)p.Hq * p.m + (means ? p.n_past * p.Hkv : 0);
  qpool_partial_kernel<T, D, DW><<<dim3((unsigned)(tiles * (D / DW))), dim3(256), (size_t)p.P * DW * sizeof(T), st>>>(p, A, means, inv_p);
}

// Step S1b: qbar[g][d] = (sum over tau (outer), heads of g (inner) of A) * r.  The sum of a (g, d) is one sequential chain
// over the m G terms k = tau * G + (h - g G); a workgroup of NT threads brings the terms of its DW dims into LDS at once
// (FLOATS / DW rows at a time), then a thread per dim walks its chain, 16 reads ahead of the additions.
static inline size_t final_lds_bytes(const Params& p, int dims, int floats) {
  const size_t all = (size_t)p.m * p.G * dims;
  return 4 * ((all < (size_t)floats ? all : (size_t)floats) + 32 * dims);   // (32 rows for the reads ahead)
}
// thread x < DW returns qbar[g][d0 + x]
template <int DW, int NT, int FLOATS>
__device__ __forceinline__ float qpool_final(const Params& p, const float* __restrict__ A, float r, int g, int d0, float* rows) {
  constexpr int GPR = DW / 4, PASS = FLOATS / DW;   // float4 of a row, rows per pass
  const int tid = threadIdx.x, n = p.m * p.G;
  float acc = 0.0f;
  for (int k0 = 0; k0 < n; k0 += PASS) {
    const int cnt = n - k0 < PASS ? n - k0 : PASS, total = cnt * GPR;
    for (int e0 = tid; e0 < total; e0 += 8 * NT) {   // (eight loads per thread in flight)
      float4 v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int e = e0 + u * NT < total ? e0 + u * NT : e0, k = k0 + e / GPR;
        const int tau = (int)div_g(p, (uint32_t)k), h = g * p.G + (k - tau * p.G);
        v[u] = load_floats(A + ((int64_t)h * p.m + tau) * p.D + d0 + 4 * (e % GPR));
      }
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (e0 + u * NT < total) reinterpret_cast<float4*>(rows)[e0 + u * NT] = v[u];
    }
    __syncthreads();
    if (tid < DW) {
      // (what a batch reads past the last row is inside the allocation and not added)
      float a[16], b[16];
      const float* at = rows + tid;
      auto read = [&](float (&x)[16]) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < 16; ++u) x[u] = at[u * DW];
        at += 16 * DW;
      };
      int left = cnt;
      auto add = [&](const float (&x)[16]) __attribute__((always_inline)) {
        if (left >= 16) {
#pragma unroll
          for (int u = 0; u < 16; ++u) acc = __fadd_rn(acc, x[u]);
        } else {
#pragma unroll
          for (int u = 0; u < 16; ++u) acc = u < left ? __fadd_rn(acc, x[u]) : acc;
        }
        left -= 16;
      };
      read(a);
      while (left > 0) {
        read(b);
        add(a);
        if (left <= 0) break;
        read(a);
        add(b);
      }
    }
    __syncthreads();
  }
  return __fmul_rn(acc, r);
}
// One workgroup per KV head and 16 dims: one compute unit takes about 10 bytes per ns of lines that another one wrote, so few of
// them are slow (224 rows of 128 floats: 9.1 us with one workgroup per head, 5.7 so; 448 rows: 16.5, 8.6).
constexpr int FINAL_DIMS = 16, FINAL_THREADS = 256, FINAL_FLOATS = 16384;   // (floats of a pass in LDS)
__global__ __launch_bounds__(FINAL_THREADS) void qpool_final_kernel(Params p, const float* __restrict__ A, float* __restrict__ qbar, float r) {
  extern __shared__ __align__(16) float rows[];
  const int g = blockIdx.x, d0 = blockIdx.y * FINAL_DIMS;
  const float v = qpool_final<FINAL_DIMS, FINAL_THREADS, FINAL_FLOATS>(p, A, r, g, d0, rows);
  if ((int)threadIdx.x < FINAL_DIMS) qbar[g * p.D + d0 + threadIdx.x] = v;
}

// Steps S2 + S3: one group of LPR lanes walks one (KV head, logical page) tile
// of the K pool token by token; a wave covers 64 / LPR pages at once.
template <typename T, int D>
__global__ __launch_bounds__(256) void page_score_kernel(Params p, const float* __restrict__ qbar,
                                                         float* __restrict__ scores, float inv_p) {
  constexpr int VEC = Vec16<T>::N, LPR = D / VEC, PPB = 256 / LPR;
  const int g = blockIdx.y;
  const int lr = threadIdx.x % LPR;
  const int64_t l = (int64_t)blockIdx.x * PPB + threadIdx.x / LPR;
  const bool active = l < p.n_past;
  const int64_t lc = active ? l : 0;
  const T* base = (const T*)p.k_pool + (int64_t)p.page_table[lc] * p.pool_page_stride +
                  (int64_t)g * p.pool_head_stride + lr * VEC;
  float x[VEC];
  seq_row_sum<T, 16, true>(base, p.pool_tok_stride, p.P, x);
  const float* qb = qbar + g * D + lr * VEC;
#pragma unroll
  for (int v = 0; v < VEC; ++v) x[v] = __fmul_rn(qb[v], __fmul_rn(x[v], inv_p));
  // tree over d: strides D/2 .. VEC cross lanes, then VEC/2 .. 1 inside the lane
#pragma unroll
  for (int s = D / 2; s >= VEC; s >>= 1) {
#pragma unroll
    for (int v = 0; v < VEC; ++v) x[v] = __fadd_rn(x[v], __shfl_xor(x[v], s / VEC, 64));
  }
#pragma unroll
  for (int s = VEC / 2; s >= 1; s >>= 1) {
#pragma unroll
    for (int v = 0; v < VEC; ++v)
      if (v < s) x[v] = __fadd_rn(x[v], x[v + s]);
  }
  if (active && lr == 0) scores[(int64_t)g * p.n_past + l] = x[0];
}

// Order-preserving map float -> uint32 (larger float = larger key); -0 maps with +0.
__device__ __forceinline__ uint32_t order_key(float s) {
  uint32_t b = __float_as_uint(s);
  if ((b << 1) == 0u) b = 0u;
  return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

constexpr int SELECT_THREADS = 1024;

// block-wide sum of a 64-bit value (used for three 21-bit counters packed in one word)
__device__ __forceinline__ unsigned long long block_sum64(unsigned long long v, unsigned long long* smem /*[16]*/) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
  __syncthreads();  // protects smem reuse across calls
  if ((threadIdx.x & 63) == 0) smem[threadIdx.x >> 6] = v;
  __syncthreads();
  unsigned long long tot = 0;
#pragma unroll
  for (int w = 0; w < SELECT_THREADS / 64; ++w) tot += smem[w];
  return tot;
}

// Step S4.  One workgroup per list: per KV head, or (per_qp) per KV head and query page tau =
// blockIdx.x % m, whose list ends with the tau + 1 local pages its rows can see.  The k-th largest
// key is found by bisection over its 32 bits (count of keys >= candidate), then the list is
// emitted in ascending logical id: all keys above the threshold, the lowest-id
// keys equal to it, and the local pages.
__global__ __launch_bounds__(SELECT_THREADS) void topk_select_kernel(
    const float* __restrict__ scores, int64_t n_past, int32_t m, int32_t top_k,
    int32_t* __restrict__ sel, int32_t* __restrict__ sel_count, int32_t lds_cap, int32_t per_qp) {
  extern __shared__ uint32_t keys[];  // first min(n_past, lds_cap) keys cached
  __shared__ unsigned long long red[SELECT_THREADS / 64];
  const int g = blockIdx.x, tid = threadIdx.x;
  const int32_t n_loc = per_qp ? (int32_t)(blockIdx.x % m) + 1 : m;
  const float* sc = scores + (int64_t)g * n_past;
  const int32_t stride = top_k + m;
  int32_t* out = sel + (int64_t)g * stride;
  const int32_t k_eff = (int32_t)(top_k < n_past ? top_k : n_past);
  const int64_t cached = n_past < lds_cap ? n_past : lds_cap;

  for (int64_t l = tid; l < cached; l += SELECT_THREADS) keys[l] = order_key(sc[l]);
  __syncthreads();
  auto key_at = [&](int64_t l) -> uint32_t { return l < cached ? keys[l] : order_key(sc[l]); };

  // T = the k_eff-th largest key = the largest T with #(key >= T) >= k_eff, found two bits at
  // a time: the counts for the three candidates T | (1..3 << b) travel in one 64-bit sum
  // (21 bits each; n_past <= 2^20).
  uint32_t T = 0;
  int take_eq = 0;
  if (k_eff > 0) {
    for (int b = 30; b >= 0; b -= 2) {
      const uint32_t c1 = T | (1u << b), c2 = T | (2u << b), c3 = T | (3u << b);
      unsigned long long c = 0;
      for (int64_t l = tid; l < n_past; l += SELECT_THREADS) {
        const uint32_t k = key_at(l);
        c += (unsigned long long)(k >= c1) | ((unsigned long long)(k >= c2) << 21) | ((unsigned long long)(k >= c3) << 42);
      }
      const unsigned long long tot = block_sum64(c, red);
      const int n1 = (int)(tot & 0x1fffff), n2 = (int)((tot >> 21) & 0x1fffff), n3 = (int)((tot >> 42) & 0x1fffff);
      if (n3 >= k_eff) T = c3;
      else if (n2 >= k_eff) T = c2;
      else if (n1 >= k_eff) T = c1;
    }
    unsigned long long c = 0;
    for (int64_t l = tid; l < n_past; l += SELECT_THREADS) c += key_at(l) > T;
    take_eq = k_eff - (int)block_sum64(c, red);  // how many keys equal to T are kept (lowest ids)
  }

  // ordered emission: thread t owns the contiguous id range [t*per, (t+1)*per)
  const int64_t per = (n_past + SELECT_THREADS - 1) / SELECT_THREADS;
  const int64_t lo = (int64_t)tid * per, hi = (lo + per < n_past) ? lo + per : n_past;
  int n_eq = 0, n_gt = 0;
  if (k_eff > 0)
    for (int64_t l = lo; l < hi; ++l) {
      const uint32_t k = key_at(l);
      n_eq += k == T;
      n_gt += k > T;
    }
  // exclusive scans of (n_eq, n_gt) over threads, packed in one 64-bit add
  unsigned long long v = ((unsigned long long)(uint32_t)n_eq << 32) | (uint32_t)n_gt;
  unsigned long long incl = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    unsigned long long nb = __shfl_up(incl, o, 64);
    if ((tid & 63) >= o) incl += nb;
  }
  __shared__ unsigned long long wave_tot[SELECT_THREADS / 64];
  if ((tid & 63) == 63) wave_tot[tid >> 6] = incl;
  __syncthreads();
  unsigned long long base = 0;
  for (int w = 0; w < (tid >> 6); ++w) base += wave_tot[w];
  const unsigned long long excl = base + incl - v;
  int eq_before = (int)(excl >> 32);
  int gt_before = (int)(excl & 0xffffffffu);
  if (k_eff > 0) {
    // position = kept keys with lower id = gt_before + min(eq_before, take_eq)
    int pos = gt_before + (eq_before < take_eq ? eq_before : take_eq);
    for (int64_t l = lo; l < hi; ++l) {
      const uint32_t k = key_at(l);
      if (k > T) {
        out[pos++] = (int32_t)l;
      } else if (k == T) {
        if (eq_before < take_eq) out[pos++] = (int32_t)l;
        ++eq_before;
      }
    }
  }
  for (int32_t j = tid; j < n_loc; j += SELECT_THREADS) out[k_eff + j] = (int32_t)(n_past + j);
  for (int32_t j = k_eff + n_loc + tid; j < stride; j += SELECT_THREADS) out[j] = -1;
  if (tid == 0) sel_count[g] = k_eff + n_loc;
}

// Step S4 for lists of at most PER * SELECT_THREADS candidates: the same selection with the keys held in
// registers, thread t's i-th that of page 1024 i + t (a run of pages per thread makes every load touch as many cache lines
// as it has lanes: 32700 candidates 31 us, 23 now).  The
// k_eff-th largest key is found by a radix select, eleven bits per pass from the top (sign, exponent, two bits of the
// fraction): the keys that still match the prefix are counted into a histogram in LDS (integer additions: the
// order does not matter), which is scanned from the top, and the bin where the count crosses what is still wanted
// extends the prefix.  Once FEW keys or less match, mostly after the first pass, they move to LDS and each is ranked by
// comparing it with the others.  The ordered emission counts per wave and row of pages and scans those counts.  Such a kernel is all
// barriers and LDS round trips; eight bits per pass, four passes: 1023 candidates 6.9 us, 8160 14.0, 32700 38; now 4.8, 9.3 and 23.
struct SelectLds {
  static constexpr int WAVES = SELECT_THREADS / 64, BITS = 11, BINS = 1 << BITS, COPIES = 2, FEW = SELECT_THREADS / 4;
  uint32_t hist[COPIES][BINS];   // (even and odd waves)
  __align__(16) uint32_t few[FEW];
  uint32_t n_few;
  uint32_t scan_tot[WAVES];
  uint32_t picked[3];  // {bin, how many keys of that bin are still wanted, how many it holds}
  uint32_t before[32 * WAVES], wave_tot[8];   // {equal, above} kept keys in 16 bits each (at most 32768 of either)
};
// list `g` (its row of sel and sel_count), ending with n_loc local pages; load(l): score of past page l
template <int PER, typename F>
__device__ __forceinline__ void select_reg(SelectLds& lds, F&& load, int g, int64_t n_past, int32_t m, int32_t n_loc, int32_t top_k,
                                           int32_t* __restrict__ sel, int32_t* __restrict__ sel_count) {
  typedef SelectLds S;
  auto& picked = lds.picked;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int32_t stride = top_k + m;
  int32_t* out = sel + (int64_t)g * stride;
  const int32_t k_eff = (int32_t)(top_k < n_past ? top_k : n_past);
  const int32_t np = (int32_t)n_past;

  uint32_t key[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) key[i] = 0u;
  if (np > 0) {
    float f[PER];   // (no load waits for another)
#pragma unroll
    for (int i = 0; i < PER; ++i) f[i] = load(i * SELECT_THREADS + tid < np ? i * SELECT_THREADS + tid : 0);
#pragma unroll
    for (int i = 0; i < PER; ++i) key[i] = i * SELECT_THREADS + tid < np ? order_key(f[i]) : 0u;
  }

  uint32_t T = 0;
  int take_eq = 0;
  if (k_eff > 0) {
    uint32_t want = (uint32_t)k_eff;  // keys still wanted among those that match the prefix
    if (tid == 0) lds.n_few = 0u;
    if (tid < S::FEW) lds.few[tid] = 0u;
    int shift = 32;   // bits not yet decided
    while (shift > 0) {
      const int above = shift;
      shift = shift > S::BITS ? shift - S::BITS : 0;
      for (int e = tid; e < S::COPIES * S::BINS; e += SELECT_THREADS) (&lds.hist[0][0])[e] = 0u;
      __syncthreads();
#pragma unroll
      for (int i = 0; i < PER; ++i) {
        const bool match = i * SELECT_THREADS + tid < np && (above == 32 || (key[i] >> (above & 31)) == (T >> (above & 31)));
        if (match) atomicAdd(&lds.hist[wave & 1][(key[i] >> shift) & (S::BINS - 1)], 1u);
      }
      __syncthreads();
      // thread t takes bins BINS - 1 - 2 t and the one below: an inclusive scan over t counts the keys in bins >= its own
      const int b0 = S::BINS - 1 - 2 * tid;
      const uint32_t v0 = lds.hist[0][b0] + lds.hist[1][b0], v1 = lds.hist[0][b0 - 1] + lds.hist[1][b0 - 1];
      uint32_t inc = v0 + v1;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const uint32_t nb = __shfl_up(inc, o, 64);
        if (lane >= o) inc += nb;
      }
      if (lane == 63) lds.scan_tot[wave] = inc;
      __syncthreads();
#pragma unroll
      for (int w = 0; w < S::WAVES; ++w) inc += w < wave ? lds.scan_tot[w] : 0u;
      const uint32_t higher = inc - v0 - v1;  // keys in bins above b0
      if (higher < want && inc >= want) {
        const bool first = higher + v0 >= want;
        picked[0] = (uint32_t)(first ? b0 : b0 - 1);
        picked[1] = want - higher - (first ? 0u : v0);
        picked[2] = first ? v0 : v1;
      }
      __syncthreads();
      T |= picked[0] << shift;
      want = picked[1];
      if (picked[2] <= S::FEW) break;
    }
    if (shift > 0) {   // (else the prefix is the key)
#pragma unroll
      for (int i = 0; i < PER; ++i)
        if (i * SELECT_THREADS + tid < np && (key[i] >> shift) == (T >> shift)) lds.few[atomicAdd(&lds.n_few, 1u)] = key[i];
      __syncthreads();
      // four threads to a candidate count the keys above it and those not below it (the slots past n count for neither: 0
      // is above nothing, and equal only to a key of 0, which is the last one anyway)
      const int n = (int)lds.n_few, x = tid >> 2;
      const uint32_t mine = lds.few[x];
      uint32_t cnt = 0;   // {not below, above}
      for (int j = 4 * (tid & 3); j < n; j += 16) {
        const uint4 k = *reinterpret_cast<const uint4*>(lds.few + j);
        cnt += (k.x > mine) + (k.y > mine) + (k.z > mine) + (k.w > mine);
        cnt += ((k.x >= mine) + (k.y >= mine) + (k.z >= mine) + (k.w >= mine)) << 16;
      }
      cnt += __shfl_xor(cnt, 1, 64);
      cnt += __shfl_xor(cnt, 2, 64);
      if (x < n && (cnt & 0xffffu) < want && (cnt >> 16) >= want) {   // (equal candidates write the same)
        picked[0] = mine;
        picked[1] = want - (cnt & 0xffffu);
      }
      __syncthreads();
      T = picked[0];
      want = picked[1];
    }
    take_eq = (int)want;  // how many keys equal to T are kept (lowest ids)
  }

  if (k_eff > 0) {
    constexpr int ROWS = PER * S::WAVES;
    uint32_t mine = 0;
#pragma unroll
    for (int i = 0; i < PER; ++i) {   // (pages past the end have key 0: below T, or equal to a T of 0 and then behind every page)
      const uint32_t n_gt = (uint32_t)__builtin_popcountll(__ballot(key[i] > T)), n_eq = (uint32_t)__builtin_popcountll(__ballot(key[i] == T));
      if (lane == i) mine = n_eq << 16 | n_gt;
    }
    if (lane < PER) lds.before[lane * S::WAVES + wave] = mine;
    __syncthreads();
    // exclusive scan over the rows of 64 pages
    uint32_t v = tid < ROWS ? lds.before[tid] : 0u, inc = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t nb = __shfl_up(inc, o, 64);
      if (lane >= o) inc += nb;
    }
    if (lane == 63 && wave < 8) lds.wave_tot[wave] = inc;
    __syncthreads();
    if (tid < ROWS) {
      for (int w = 0; w < wave; ++w) inc += lds.wave_tot[w];
      lds.before[tid] = inc - v;
    }
    __syncthreads();
    const uint64_t lower = (1ull << lane) - 1ull;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      // position = kept keys with lower id = those above T + those equal to T, of which the first take_eq are kept
      const uint32_t at = lds.before[i * S::WAVES + wave];
      const int gt = (int)(at & 0xffffu) + __builtin_popcountll(__ballot(key[i] > T) & lower);
      const int eq = (int)(at >> 16) + __builtin_popcountll(__ballot(key[i] == T) & lower);
      const bool kept = key[i] > T || (key[i] == T && eq < take_eq);
      if (kept && i * SELECT_THREADS + tid < np) out[gt + (eq < take_eq ? eq : take_eq)] = i * SELECT_THREADS + tid;
    }
  }
  for (int32_t j = tid; j < n_loc; j += SELECT_THREADS) out[k_eff + j] = (int32_t)(n_past + j);
  for (int32_t j = k_eff + n_loc + tid; j < stride; j += SELECT_THREADS) out[j] = -1;
  if (tid == 0) sel_count[g] = k_eff + n_loc;
}
template <int PER>
__global__ __launch_bounds__(SELECT_THREADS) void topk_select_reg_kernel(
    const float* __restrict__ scores, int64_t n_past, int32_t m, int32_t top_k,
    int32_t* __restrict__ sel, int32_t* __restrict__ sel_count, int32_t per_qp) {
  __shared__ SelectLds lds;
  const float* sc = scores + (int64_t)blockIdx.x * n_past;
  select_reg<PER>(lds, [&](int32_t l) { return sc[l]; }, blockIdx.x, n_past, m, per_qp ? (int32_t)(blockIdx.x % m) + 1 : m, top_k, sel, sel_count);
}

// Steps S1b, S3 and S4 of a KV head in one workgroup, from page means, for short histories and chunks: three kernels
// that do next to nothing (56 pages: 16 us and two launches more than the 4.6 of one).  The means are under way while the
// query is pooled; so few keys are ranked by comparing each with all others, no histograms.  One compute unit takes in
// about 10 bytes per ns here, so the kernel ends where pages + rows to pool are SMALL_ROWS rows of D floats: about 15 us.
constexpr int SMALL_PAGES = 192, SMALL_ROWS = 192;
template <int D>
__global__ __launch_bounds__(SELECT_THREADS) void select_small_kernel(Params p, const float* __restrict__ A, float r, const float* __restrict__ means,
                                                                      float* __restrict__ scores, int32_t top_k, int32_t* __restrict__ sel,
                                                                      int32_t* __restrict__ sel_count) {
  extern __shared__ __align__(16) float rows[];
  __shared__ __align__(16) float qb[D];
  __shared__ __align__(16) uint32_t keys[SMALL_PAGES];
  __shared__ uint32_t ranks[SELECT_THREADS / SMALL_PAGES][SMALL_PAGES];
  __shared__ int32_t kept[SMALL_PAGES / 64];
  constexpr int VEC = 4, LPR = D / VEC, GROUPS = SELECT_THREADS / LPR, PER = SMALL_PAGES / GROUPS;   // pages per group
  const int g = blockIdx.x, tid = threadIdx.x, lr = tid % LPR, grp = tid / LPR;
  const int32_t np = (int32_t)p.n_past;
  float4 kb[PER];
#pragma unroll
  for (int u = 0; u < PER; ++u)
    if (grp + u * GROUPS < np) kb[u] = load_floats(means + ((int64_t)(grp + u * GROUPS) * p.Hkv + g) * D + lr * VEC);
  if (tid < SMALL_PAGES) keys[tid] = 0u;
  const float v = qpool_final<D, SELECT_THREADS, SMALL_ROWS * D>(p, A, r, g, 0, rows);
  if (tid < D) qb[tid] = v;
  __syncthreads();
  const float4 q4 = *reinterpret_cast<const float4*>(qb + lr * VEC);
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const int32_t l = grp + u * GROUPS;
    if (l >= np) break;   // (the same for all lanes of a group)
    const float s = score_tree<D>(q4, kb[u]);
    if (lr == 0) {
      keys[l] = order_key(s);
      scores[(int64_t)g * p.n_past + l] = s;
    }
  }
  __syncthreads();
  // rank of page tid: keys above its own, and equal ones of lower pages (real keys are above 0).  TPP threads, of
  // different waves, count a part of the pages each.
  const int32_t k_eff = top_k < np ? top_k : np, stride = top_k + p.m;
  constexpr int TPP = SELECT_THREADS / SMALL_PAGES, CHUNK = (SMALL_PAGES / TPP + 3) & ~3;
  const int part = tid / SMALL_PAGES, page = tid - part * SMALL_PAGES;
  if (part < TPP) {
    const uint32_t mine = keys[page];
    const int32_t first = __builtin_amdgcn_readfirstlane(page & ~63), end = (part + 1) * CHUNK < np ? (part + 1) * CHUNK : np;   // (a wave's pages: first .. first + 63)
    uint32_t r = 0;
    for (int32_t j = part * CHUNK; j < end; j += 4) {
      const uint4 k = *reinterpret_cast<const uint4*>(keys + j);
      if (j + 4 <= first) r += (k.x >= mine) + (k.y >= mine) + (k.z >= mine) + (k.w >= mine);
      else if (j >= first + 64) r += (k.x > mine) + (k.y > mine) + (k.z > mine) + (k.w > mine);
      else {
        const int32_t d = page - j;
        r += (k.x > mine || (k.x == mine && d > 0)) + (k.y > mine || (k.y == mine && d > 1)) + (k.z > mine || (k.z == mine && d > 2)) +
             (k.w > mine || (k.w == mine && d > 3));
      }
    }
    ranks[part][page] = r;
  }
  __syncthreads();
  int32_t rank = 0;
  if (tid < SMALL_PAGES) {
#pragma unroll
    for (int u = 0; u < TPP; ++u) rank += (int32_t)ranks[u][tid];
  }
  const bool keep = tid < np && rank < k_eff;
  const uint64_t votes = __ballot(keep);
  if (tid < SMALL_PAGES && (tid & 63) == 0) kept[tid >> 6] = __builtin_popcountll(votes);
  __syncthreads();
  int32_t* out = sel + (int64_t)g * stride;
  if (keep) {
    int32_t pos = __builtin_popcountll(votes & ((1ull << (tid & 63)) - 1ull));
    for (int w = 0; w < (tid >> 6); ++w) pos += kept[w];
    out[pos] = tid;
  }
  for (int32_t j = tid; j < stride - k_eff; j += SELECT_THREADS) out[k_eff + j] = j < p.m ? np + j : -1;
  if (tid == 0) sel_count[g] = k_eff + p.m;
}

// Steps S1b and S3 in one kernel, from page means, for few rows to pool: a group of D / 4 lanes per page, as page_score_cached_kernel has, whose
// lanes walk the chains of their own four dims, eight rows in flight, while the means are under way.
constexpr int POOLED_PAGES = 2;   // pages per group
template <int D>
__global__ __launch_bounds__(256) void page_score_pooled_kernel(Params p, const float* __restrict__ A, float r, const float* __restrict__ means, float* __restrict__ scores) {
  constexpr int VEC = 4, LPR = D / VEC, GROUPS = 256 / LPR;
  const int g = blockIdx.y, lr = threadIdx.x % LPR, n = p.m * p.G;
  const int64_t l0 = (int64_t)blockIdx.x * (GROUPS * POOLED_PAGES) + threadIdx.x / LPR;
  float4 kb[POOLED_PAGES];
#pragma unroll
  for (int u = 0; u < POOLED_PAGES; ++u) {
    const int64_t l = l0 + u * GROUPS;
    kb[u] = load_floats(means + ((l < p.n_past ? l : 0) * p.Hkv + g) * D + lr * VEC);
  }
  const float* at = A + lr * VEC;
  auto read = [&](const int k0, float4 (&v)[8]) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int k = k0 + u < n ? k0 + u : n - 1, tau = (int)div_g(p, (uint32_t)k), h = g * p.G + (k - tau * p.G);
      v[u] = load_floats(at + ((int64_t)h * p.m + tau) * D);
    }
  };
  float4 q = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int k0 = 0; k0 < n; k0 += 8) {
    float4 v[8];
    read(k0, v);
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const bool row = k0 + u < n;
      q.x = row ? __fadd_rn(q.x, v[u].x) : q.x;
      q.y = row ? __fadd_rn(q.y, v[u].y) : q.y;
      q.z = row ? __fadd_rn(q.z, v[u].z) : q.z;
      q.w = row ? __fadd_rn(q.w, v[u].w) : q.w;
    }
  }
  q = make_float4(__fmul_rn(q.x, r), __fmul_rn(q.y, r), __fmul_rn(q.z, r), __fmul_rn(q.w, r));
#pragma unroll
  for (int u = 0; u < POOLED_PAGES; ++u) {
    const int64_t l = l0 + u * GROUPS;
    const float s = score_tree<D>(q, kb[u]);
    if (l < p.n_past && lr == 0) scores[(int64_t)g * p.n_past + l] = s;
  }
}

static hipError_t launch_topk_select(const Params& p, const float* scores, int32_t top_k, int32_t* sel, int32_t* sel_count,
                                     int per_qp, hipStream_t st) {
  const dim3 grid((unsigned)(per_qp ? p.Hkv * p.m : p.Hkv)), block(SELECT_THREADS);
  const int64_t per = (p.n_past + SELECT_THREADS - 1) / SELECT_THREADS;
  if (per <= 32) {  // the keys of a list fit the registers of one workgroup
    ProfScope prof_("topk_select", st);
#define OOMB_TOPK_REG(PER) topk_select_reg_kernel<PER><<<grid, block, 0, st>>>(scores, p.n_past, p.m, top_k, sel, sel_count, per_qp)
    if (per <= 2) OOMB_TOPK_REG(2);
    else if (per <= 4) OOMB_TOPK_REG(4);
    else if (per <= 8) OOMB_TOPK_REG(8);
    else if (per <= 12) OOMB_TOPK_REG(12);
    else if (per <= 16) OOMB_TOPK_REG(16);
    else if (per <= 24) OOMB_TOPK_REG(24);
    else OOMB_TOPK_REG(32);
#undef OOMB_TOPK_REG
    return hipGetLastError();
  }
  constexpr int WANT = 144 * 1024;
  static DeviceOnce lds_once;
  if (hipError_t e = ensure_max_dynamic_lds(lds_once, (const void*)topk_select_kernel, WANT); e != hipSuccess) return e;
  const int64_t cap = WANT / 4;
  const int64_t cached = p.n_past < cap ? p.n_past : cap;
  ProfScope prof_("topk_select", st);
  topk_select_kernel<<<grid, block, (size_t)cached * 4, st>>>(
      scores, p.n_past, p.m, top_k, sel, sel_count, (int32_t)cap, per_qp);
  return hipGetLastError();
}

// Layout of the scoring workspace.  Page means of a short history get a place of their own behind the rest, if all of
// it fits the built-in scratch array (callers without a workspace take the same kernels): with as many workgroups as tiles they
// are there in 6 us more, where the kernel that walks a page per group of lanes takes 18 for 512 x 2 pages of 128 tokens (13 of 64; pages
// of 16 and 32 are short chains there).  From MEANS_TILES tiles on that one has groups enough to be as fast.
constexpr int64_t MEANS_TILES = 2048;
// Few rows to pool: pooled by the scoring kernel itself, in every group of lanes anew, which saves a launch.  The selection before and so, us: 7 rows, 4092
// (head, page) pairs 12.4 and 10.4; 16 rows, 8184 pairs 13.3 and 11.7, 32760 pairs 16.7 and 16.6; 28 rows, 4092 pairs 12.4 and 12.4, 64000 pairs 26.1 and 33.5; 56
// rows, 4092 pairs 13.0 and 14.2.
constexpr int64_t POOLED_ROWS = 16, POOLED_TILES = 32768;
struct ScoreLayout {
  size_t off_qbar, off_scores, off_means, bytes;   // (means at the end: a call works without them)
  bool means, small;   // scores from means; one workgroup per KV head for what follows them
};
static ScoreLayout score_layout(const Params& p, bool cached, size_t ws_bytes) {
  auto up = [](size_t x) { return (x + 255) & ~(size_t)255; };
  ScoreLayout L{};
  L.off_qbar = up((size_t)p.Hq * p.m * p.D * sizeof(float));
  L.off_scores = L.off_qbar + up((size_t)p.Hkv * p.D * sizeof(float));
  L.bytes = L.off_means = L.off_scores + up((size_t)p.Hkv * (size_t)(p.n_past > 0 ? p.n_past : 1) * sizeof(float));
  const size_t means = up((size_t)p.n_past * p.Hkv * p.D * sizeof(float));
  const bool few = p.n_past <= SMALL_PAGES && p.n_past + (int64_t)p.m * p.G <= SMALL_ROWS;
  L.means = cached || ((few || (p.P >= 64 && p.n_past * p.Hkv <= MEANS_TILES)) && L.bytes + means <= (size_t)OOMB_NOALLOC_SCRATCH_BYTES && L.bytes + means <= ws_bytes);
  L.small = few && L.means;
  if (L.means && !cached) L.bytes += means;
  return L;
}
size_t score_workspace_bytes(const Params& p) { return score_layout(p, false, SIZE_MAX).bytes; }
// what a call cannot do without: a workspace sized for a longer history (which has no place for means) serves shorter ones
size_t score_workspace_min_bytes(const Params& p) { return score_layout(p, false, 0).bytes; }

// kbar_cache != nullptr: the page means come from the cache instead of the keys
template <typename T, int D>
static hipError_t launch_scoring(const Params& p, int32_t top_k, int32_t* sel, int32_t* sel_count, float* scores_out, unsigned char* ws,
                                 size_t ws_bytes, const float* kbar_cache, hipStream_t st) {
  constexpr int VEC = Vec16<T>::N, LPR = D / VEC, PER_BLOCK = 256 / LPR;
  const ScoreLayout L = score_layout(p, kbar_cache != nullptr, ws_bytes);
  float* A = (float*)ws;
  float* qbar = (float*)(ws + L.off_qbar);
  float* scores = scores_out ? scores_out : (float*)(ws + L.off_scores);
  float* means = L.means && !kbar_cache ? (float*)(ws + L.off_means) : nullptr;
  const float inv_p = 1.0f / (float)p.P, r = 1.0f / (float)((int64_t)p.C * p.G);
  {
    ProfScope prof_("qpool_partial", st);
    if (page_in_slices<T>(p)) run_qpool_partial<T, D, LINE_DIMS<T>>(p, A, means, inv_p, st);
    else run_qpool_partial<T, D, D>(p, A, means, inv_p, st);
  }
  if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  if (L.small) {
    static DeviceOnce lds_once;
    if (hipError_t e = ensure_max_dynamic_lds(lds_once, (const void*)select_small_kernel<D>, (SMALL_ROWS + 32) * D * 4); e != hipSuccess) return e;
    ProfScope prof_("select_small", st);
    select_small_kernel<D><<<dim3(p.Hkv), dim3(SELECT_THREADS), final_lds_bytes(p, D, SMALL_ROWS * D), st>>>(p, A, r, kbar_cache ? kbar_cache : means, scores, top_k, sel,
                                                                                         sel_count);
    return hipGetLastError();
  }
  if (L.means && p.n_past > 0 && (int64_t)p.m * p.G <= POOLED_ROWS && p.n_past * p.Hkv <= POOLED_TILES) {
    ProfScope prof_("page_score_pooled", st);
    constexpr int PAGES = POOLED_PAGES * 256 / (D / 4);   // of a workgroup
    page_score_pooled_kernel<D><<<dim3((unsigned)((p.n_past + PAGES - 1) / PAGES), p.Hkv), dim3(256), 0, st>>>(p, A, r, kbar_cache ? kbar_cache : means, scores);
    if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
    return launch_topk_select(p, scores, top_k, sel, sel_count, 0, st);
  }
  {
    static DeviceOnce lds_once;   // (16 dims of 1024 rows and the rows read ahead: 66 KiB)
    if (hipError_t e = ensure_max_dynamic_lds(lds_once, (const void*)qpool_final_kernel, 4 * (FINAL_FLOATS + 32 * FINAL_DIMS)); e != hipSuccess) return e;
    ProfScope prof_("qpool_final", st);
    qpool_final_kernel<<<dim3(p.Hkv, D / FINAL_DIMS), dim3(FINAL_THREADS), final_lds_bytes(p, FINAL_DIMS, FINAL_FLOATS), st>>>(p, A, qbar, r);
  }
  if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  if (L.means) {
    if (hipError_t e = launch_page_score_cached(p, qbar, kbar_cache ? kbar_cache : means, scores, st); e != hipSuccess) return e;
  } else if (p.n_past > 0) {   // (a first chunk has nothing to score: a grid of no workgroups is a launch error)
    dim3 grid((unsigned)((p.n_past + PER_BLOCK - 1) / PER_BLOCK), p.Hkv);
    { ProfScope prof_("page_score", st); page_score_kernel<T, D><<<grid, dim3(256), 0, st>>>(p, qbar, scores, inv_p); }
    if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  }
  return launch_topk_select(p, scores, top_k, sel, sel_count, 0, st);
}

// Returns hipSuccess or the launch error.  dtype_is_bf16 picks the element type.
hipError_t launch_score_topk(const Params& p, bool is_bf16, int32_t top_k, int32_t* sel,
                             int32_t* sel_count, float* scores_out, void* ws, size_t ws_bytes, const float* kbar_cache,
                             hipStream_t st) {
  unsigned char* w = (unsigned char*)ws;
  if (is_bf16)
    return p.D == 128 ? launch_scoring<bf16_t, 128>(p, top_k, sel, sel_count, scores_out, w, ws_bytes, kbar_cache, st)
                      : launch_scoring<bf16_t, 64>(p, top_k, sel, sel_count, scores_out, w, ws_bytes, kbar_cache, st);
  return p.D == 128 ? launch_scoring<float, 128>(p, top_k, sel, sel_count, scores_out, w, ws_bytes, kbar_cache, st)
                    : launch_scoring<float, 64>(p, top_k, sel, sel_count, scores_out, w, ws_bytes, kbar_cache, st);
}

// Built-in scratch memory of oomb_page_score_topk_noalloc: the scoring workspace (query-page sums, pooled
// queries, scores) for callers that cannot hand one over.  Every device the library runs on holds its own
// copy of the array until the process ends.  In host code the array's name is only a stand-in; the address
// on the current device comes from hipGetSymbolAddress, once per device.
static __device__ __align__(256) unsigned char scratch[OOMB_NOALLOC_SCRATCH_BYTES];

hipError_t score_scratch_ptr(void** out) {
  constexpr int MAX_DEVICES = 64;
  static std::mutex mu;
  static void* ptrs[MAX_DEVICES] = {};
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= MAX_DEVICES) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lk(mu);
  if (!ptrs[dev]) {
    void* ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!ptr) return hipErrorInvalidSymbol;
    ptrs[dev] = ptr;
  }
  *out = ptrs[dev];
  return hipSuccess;
}

// votes [Hkv][m][n_past] -> one list per (KV head, query page), sel [Hkv][m][top_k + m]
hipError_t launch_topk_select_qp(const Params& p, const float* votes, int32_t top_k, int32_t* sel, int32_t* sel_count,
                                 hipStream_t st) {
  return launch_topk_select(p, votes, top_k, sel, sel_count, 1, st);
}

}  // namespace oomb
