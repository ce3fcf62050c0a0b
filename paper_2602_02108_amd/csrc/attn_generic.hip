// Paged attention for the (element type, head dim, page size) combinations without a kernel of
// their own: fp32 tensors, head dim 64, pages of 16 .. 64 tokens.  Forward: Sec. 4.1 operator;
// backward: Sec. 3 Eq. 3 accumulation into the paged gradient pool, no atomics.
//
// All three kernels are the same matrix-core loop: one side stays in registers (32 rows or keys per
// wave), the other side streams through LDS in row tiles that are copied straight from the pools
// (or from Q / dO) with direct global -> LDS loads, two buffers, one tile ahead:
//   forward  Q rows stay,   K / V stream:  S^T = K Q^T, O^T += V^T P^T
//   dQ       Q, dO stay,    K / V stream:  S^T, dP^T = V dO^T, dQ^T += K^T dS^T
//   dK / dV  K, V stay,     Q / dO stream: S = Q K^T, dP = dO V^T, dV^T += dO^T P, dK^T += Q^T dS
// With 32 x 32 accumulators a lane owns one column of the staying side, so softmax statistics are
// per-lane scalars (forward, dQ) and the accumulator feeds the second product from registers.
// bf16: v_mfma_f32_32x32x16_bf16, the transposed operand by transposing LDS reads.  fp32:
// v_mfma_f32_32x32x2_f32 (fp32 products and sums); an operand is one dword per lane, so any
// order of the contraction index that both operands share will do, and four instructions
// take one 16-byte read.
//
// Page sizes disappear in "list-token space": the tokens of a page list in list order.  The list is
// ascending, so what a row sees is a prefix of that sequence: one number per row.  Row space of a
// KV head: r = token * G + head in group, so a tile's rows are consecutive tokens of all G heads,
// and the rows of a query page are contiguous for every page size.
//
// What bounds them: fp32 the matrix pipe itself (256 flops per cycle and compute unit, 157 TFLOP/s);
// bf16 the exposed vector work and LDS latency of one or two waves per SIMD; short calls the number
// of workgroups, which is why the streamed side is cut into splits whose partial sums a second
// kernel combines in a fixed order.  Measured against one wave per query row (per key in dK / dV)
// with plain fp32 arithmetic: 28 / 4 heads fp32, chunk 512, 16 + 4 pages of 128: 41.5 -> 0.84 ms
// (59 GFLOP); 8 / 2 heads bf16, chunk 1088, 24 + 17 pages of 64: 18.4 -> 0.13 ms (32 GFLOP).
#include "mfma_common.h"
#include "launch.h"

namespace oomb {

constexpr int GN_WAVES = 4;
constexpr int GN_THREADS = GN_WAVES * 64;
constexpr int GN_ROWS = GN_WAVES * 32;  // rows of a tile (forward, dQ) / keys of a unit (dK / dV)
constexpr int GN_BUF = 32768;           // one LDS buffer: two row tiles of at most 16 KiB
constexpr int GN_STAT = 2 * GN_BUF;     // dK / dV: {lse2, delta} of the streamed rows, two buffers
constexpr int GN_LDS = GN_STAT + 2 * 2 * 64 * 4;

// Geometry of a row tile: RB bytes per row, NG granules of 16 bytes, granule c of row r at position
// c ^ swz(r).  The swizzle frees both access patterns of bank conflicts: 16 rows at one granule, and
// the second product's (bf16: 4 rows x 64 bytes of a transposing read; fp32: whole rows).
template <typename T, int D> struct Gn {
  static constexpr bool BF = sizeof(T) == 2;
  static constexpr int ES = sizeof(T), RB = D * ES, NG = RB / 16;
  static constexpr int NJ = NG / 2;                // k-steps of the first product (one granule per lane each)
  static constexpr int DB = D / 32;                // accumulator blocks of the second product
  static constexpr int KT = RB == 512 ? 32 : 64;   // rows of a tile
  static constexpr int TILE = KT * RB;
  static constexpr int RPI = 1024 / RB;            // rows per copy instruction of a wave
  static constexpr int NI = TILE / 1024 / GN_WAVES;  // copy instructions per wave and tile
  static constexpr int RW = NI * RPI;              // rows a wave copies: 8 or 16, so they lie in one page
  static __device__ __forceinline__ constexpr uint32_t swz(uint32_t r) {
    return !BF ? (r & 15) : RB == 256 ? row_tile_f(r) : ((((r >> 1) & 1) << 2) | ((r >> 2) & 3));
  }
};

// C += A B over one granule pair: A, B hold 16 bytes per lane (granule 2 j + lane / 32 of the lane's row)
template <typename T> __device__ __forceinline__ void gn_mma(const uint4& a, const uint4& b, f32x16& c) {
  if constexpr (sizeof(T) == 2) {
    c = mfma32(as_bf16x8(a), as_bf16x8(b), c);
  } else {
    c = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.x), __uint_as_float(b.x), c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.y), __uint_as_float(b.y), c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.z), __uint_as_float(b.z), c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.w), __uint_as_float(b.w), c, 0, 0, 0);
  }
}

template <int N> __device__ __forceinline__ void gn_zero(f32x16 (&v)[N]) {
#pragma unroll
  for (int k = 0; k < N; ++k)
#pragma unroll
    for (int x = 0; x < 16; ++x) v[k][x] = 0.f;
}

// first product: 32 rows of the tile at `base` (LDS byte offset of row 32 u) against the staying fragments
template <typename T, int D>
__device__ __forceinline__ f32x16 gn_chain(const unsigned char* smem, uint32_t base, uint32_t lane_row, const uint4 (&st)[Gn<T, D>::NJ]) {
  f32x16 c;
#pragma unroll
  for (int x = 0; x < 16; ++x) c[x] = 0.f;
#pragma unroll
  for (int j = 0; j < Gn<T, D>::NJ; ++j)
    gn_mma<T>(*reinterpret_cast<const uint4*>(smem + (base + (lane_row ^ (uint32_t)(j << 5)))), st[j], c);
  return c;
}

__device__ __forceinline__ uint4 gn_pack8(const f32x16& v, int base) {
  return make_uint4(pack2_bf16(v[base + 0], v[base + 1]), pack2_bf16(v[base + 2], v[base + 3]),
                    pack2_bf16(v[base + 4], v[base + 5]), pack2_bf16(v[base + 6], v[base + 7]));
}

// second product: acc += tile^T s, s in accumulator layout (register x = tile row 8 (x / 4) + 4 hh + x % 4).
// bf16: acc[db] row m is dim 32 db + m.  fp32: acc[e] row m is dim DB m + e (a lane reads DB consecutive dims).
template <typename T, int D>
__device__ __forceinline__ void gn_tprod(const unsigned char* smem, uint32_t base, int lane, const f32x16& s, f32x16 (&acc)[Gn<T, D>::DB]) {
  typedef Gn<T, D> X;
  if constexpr (X::BF) {
    const uint32_t L = lane & 15, gq = lane >> 4, row = 4 * (gq >> 1) + (L >> 2);
    const uint32_t t = row * X::RB + (((2 * (gq & 1) + ((L & 3) >> 1)) ^ X::swz(row)) << 4) + 8 * (L & 1);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const bf16x8 b = as_bf16x8(gn_pack8(s, 8 * u));
#pragma unroll
      for (int db = 0; db < X::DB; ++db) {
        const uint32_t a0 = base + (t ^ (uint32_t)(db << 6)) + 16 * u * X::RB;
        const uint32_t a1 = base + (t ^ (uint32_t)(db << 6) ^ 32u) + (16 * u + 8) * X::RB;   // rows + 8: the swizzle changes by 2
        const u32x2_t lo = __builtin_bit_cast(u32x2_t, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (__attribute__((address_space(3))) s16x4_t*)(smem + a0)));
        const u32x2_t hi = __builtin_bit_cast(u32x2_t, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (__attribute__((address_space(3))) s16x4_t*)(smem + a1)));
        acc[db] = mfma32(__builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3)), b, acc[db]);
      }
    }
  } else {
    const uint32_t lq = lane & 31, hh = lane >> 5;
    const uint32_t gran = D == 128 ? lq : lq >> 1, sub = D == 128 ? 0 : 8 * (lq & 1);
    const uint32_t t = 4 * hh * X::RB + ((gran ^ (4 * hh)) << 4) + sub;
#pragma unroll
    for (int x = 0; x < 16; ++x) {
      const int r = 8 * (x >> 2) + (x & 3);
      const unsigned char* at = smem + (base + (t ^ (uint32_t)((r & 15) << 4)) + r * X::RB);
      if constexpr (D == 128) {
        const float4 a = *reinterpret_cast<const float4*>(at);
        acc[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a.x, s[x], acc[0], 0, 0, 0);
        acc[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a.y, s[x], acc[1], 0, 0, 0);
        acc[2] = __builtin_amdgcn_mfma_f32_32x32x2f32(a.z, s[x], acc[2], 0, 0, 0);
        acc[3] = __builtin_amdgcn_mfma_f32_32x32x2f32(a.w, s[x], acc[3], 0, 0, 0);
      } else {
        const float2 a = *reinterpret_cast<const float2*>(at);
        acc[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a.x, s[x], acc[0], 0, 0, 0);
        acc[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a.y, s[x], acc[1], 0, 0, 0);
      }
    }
  }
}

// the accumulator in groups of four consecutive dims: f(dim, a, b, c, d) for D / 8 groups per lane
template <typename T, int D, typename F>
__device__ __forceinline__ void gn_emit(const f32x16 (&acc)[Gn<T, D>::DB], int hh, F&& f) {
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
template <typename T> __device__ __forceinline__ void gn_store4(T* p, float a, float b, float c, float d);
template <> __device__ __forceinline__ void gn_store4<float>(float* p, float a, float b, float c, float d) {
  *reinterpret_cast<float4*>(p) = make_float4(a, b, c, d);
}
template <> __device__ __forceinline__ void gn_store4<bf16_t>(bf16_t* p, float a, float b, float c, float d) {
  *reinterpret_cast<uint2*>(p) = make_uint2(pack2_bf16(a, b), pack2_bf16(c, d));
}
template <typename T> __device__ __forceinline__ void gn_add4(T* p, float a, float b, float c, float d);
template <> __device__ __forceinline__ void gn_add4<float>(float* p, float a, float b, float c, float d) {
  const float4 v = *reinterpret_cast<const float4*>(p);
  *reinterpret_cast<float4*>(p) = make_float4(v.x + a, v.y + b, v.z + c, v.w + d);
}
template <> __device__ __forceinline__ void gn_add4<bf16_t>(bf16_t* p, float a, float b, float c, float d) {
  const uint2 v = *reinterpret_cast<const uint2*>(p);
  gn_store4<bf16_t>(p, __uint_as_float(v.x << 16) + a, __uint_as_float(v.x & 0xffff0000u) + b, __uint_as_float(v.y << 16) + c,
                    __uint_as_float(v.y & 0xffff0000u) + d);
}

// One copy instruction of a wave: lane l moves 16 bytes from its own address to LDS byte dst + 16 l.
__device__ __forceinline__ void gn_copy16(const unsigned char* src, uint32_t dst) {
  asm volatile(
      "s_mov_b32 m0, %0\n\t"
      "s_nop 0\n\t"
      "global_load_lds_dwordx4 %1, off\n\t" ::"s"(dst), "v"(src) : "memory", "m0");
}

// ---- rows and page lists of a tile (forward, dQ) -------------------------------------------------
// Tiles partition the rows of a KV head (one list per head) or the rows of each query page.
__host__ __device__ __forceinline__ int32_t gn_tiles(int32_t C, int32_t G, int32_t P, int32_t m, int qp) {
  return qp ? m * ((P * G + GN_ROWS - 1) / GN_ROWS) : (int32_t)(((int64_t)C * G + GN_ROWS - 1) / GN_ROWS);
}

struct GnTile {
  int lid;
  int32_t r, i, h;        // this lane's row (clamped to the tile's last), its chunk token and query head
  bool valid, active;     // the lane owns a row; the wave owns at least one
  int32_t T_ent;          // list entries that some row of the tile sees
  int32_t V, V_last;      // list tokens this lane's row / the tile's last row sees
};

__device__ __forceinline__ GnTile gn_tile(const Params& p, int g, int32_t tile, int wave, int lane, int lp) {
  GnTile t;
  int32_t base, end;
  if (!p.qp) {
    base = tile * GN_ROWS;
    end = p.C * p.G;
    t.lid = g;
  } else {
    const int32_t rpq = p.P * p.G, tpq = (rpq + GN_ROWS - 1) / GN_ROWS, tau = tile / tpq;
    base = tau * rpq + (tile - tau * tpq) * GN_ROWS;
    end = (tau + 1) * rpq;
    t.lid = g * p.m + tau;
  }
  const int32_t last = base + GN_ROWS - 1 < end - 1 ? base + GN_ROWS - 1 : end - 1;
  const int32_t r = base + 32 * wave + (lane & 31);
  t.valid = r <= last;
  t.active = base + 32 * wave <= last;
  t.r = t.valid ? r : last;
  t.i = (int32_t)div_g(p, (uint32_t)t.r);
  t.h = g * p.G + (t.r - t.i * p.G);
  const int64_t first_q = p.N - p.C;
  const int32_t i_last = (int32_t)div_g(p, (uint32_t)last);
  const int64_t a = first_q + t.i, a_last = first_q + i_last;
  const int32_t pg = (int32_t)(a >> lp), pg_lo = (int32_t)((first_q + div_g(p, (uint32_t)base)) >> lp), pg_hi = (int32_t)(a_last >> lp);
  t.T_ent = visible_len(p, t.lid, pg_hi, lane);
  // tokens visible up to page v = entries up to v, whole pages, less the unseen tail of v itself.  The rows of
  // a tile lie in at most nine pages, so the entries past pg_lo are among the last 64.
  const int32_t e = t.T_ent - 1 - lane >= 0 ? list_at(p, t.lid, t.T_ent - 1 - lane) : -1;
  t.V = 0;
  t.V_last = 0;
  for (int32_t v = pg_lo; v <= pg_hi; ++v) {
    const int32_t whole = (t.T_ent - __builtin_popcountll(__ballot(e > v))) << lp;
    const bool held = __ballot(e == v) != 0;
    if (pg == v) t.V = whole - (held ? p.P - 1 - (int32_t)(a & (p.P - 1)) : 0);
    if (v == pg_hi) t.V_last = whole - (held ? p.P - 1 - (int32_t)(a_last & (p.P - 1)) : 0);
  }
  return t;
}

// K / V tiles of a list, copied tile by tile in ascending order.  Every wave moves RW rows of K and of V.
template <typename T, int D> struct GnStream {
  typedef Gn<T, D> X;
  PageWindow pw;
  int64_t lane_off;   // this lane's row and granule inside the wave's rows, bytes
  int64_t step;       // bytes between the rows of consecutive copy instructions
  int64_t head_off;   // bytes
  __device__ __forceinline__ void init(const Params& p, const GnTile& t, int g, int lane, int32_t first_tok, int lp) {
    lane_off = (int64_t)(lane / X::NG) * p.pool_tok_stride * X::ES;
    step = (int64_t)X::RPI * p.pool_tok_stride * X::ES;
    head_off = (int64_t)g * p.pool_head_stride * X::ES;
    pw.slots = false;
    pw.base = first_tok >> lp;
    pw.fetch(p, t.lid, t.T_ent, pw.base, lane, pw.l_cur, pw.p_cur);
    pw.fetch(p, t.lid, t.T_ent, pw.base + 64, lane, pw.l_nxt, pw.p_nxt);
  }
  __device__ __forceinline__ void copy(const Params& p, const GnTile& t, int wave, int lane, int lp, int32_t tile, uint32_t buf) {
    const int32_t tok = tile * X::KT + wave * X::RW;
    int32_t e = tok >> lp;
    e = e < t.T_ent ? e : t.T_ent - 1;   // (rows past the list's end are masked: any page of the list will do)
    e = __builtin_amdgcn_readfirstlane(e);
    pw.advance(p, t.lid, t.T_ent, e, lane);
    const int64_t o = (int64_t)pw.phys(e) * p.pool_page_stride * X::ES + head_off + (int64_t)(tok & (p.P - 1)) * p.pool_tok_stride * X::ES;
    const uint32_t lrow = lane / X::NG, pos = lane % X::NG;
    const uint32_t dst = buf + wave * X::RW * X::RB;
#pragma unroll
    for (int k = 0; k < X::NI; ++k) {
      const uint32_t row = (wave * X::RW + k * X::RPI + lrow) & 15;   // (the swizzle sees the row index modulo 16)
      const int64_t at = o + lane_off + k * step + (int64_t)((pos ^ X::swz(row)) << 4);
      gn_copy16((const unsigned char*)p.k_pool + at, dst + 1024 * k);
      gn_copy16((const unsigned char*)p.v_pool + at, dst + X::TILE + 1024 * k);
    }
  }
};

// workgroup -> (KV head, row tile, split).  The head varies fastest: workgroups are dealt round-robin to the
// XCDs, so with 1, 2, 4 or 8 KV heads every head keeps to its own XCDs and their L2.
struct GnBlock { int g; int32_t tile, split; };
__device__ __forceinline__ GnBlock gn_block(const Params& p, int32_t tiles, int32_t n_split) {
  const int32_t b = blockIdx.x, rest = b / p.Hkv;
  return {b - rest * p.Hkv, tiles - 1 - rest / n_split, rest % n_split};   // late rows see more pages: they start first
}

// ---- forward ----------------------------------------------------------------------------------
// n_split > 1: O (not normalised) and {running maximum in log2 units, sum} of every row go to
// part[split][KV head][row][D] and part_ml, which the combine kernel merges.
template <typename T, int D>
__global__ __launch_bounds__(GN_THREADS, 2) void fwd_generic_kernel(Params p, int32_t tiles, int32_t n_split, int lp,
                                                                    float* __restrict__ part, float2* __restrict__ part_ml) {
  typedef Gn<T, D> X;
  extern __shared__ __align__(16) unsigned char smem[];
  const int lane = threadIdx.x & 63, hh = lane >> 5, lq = lane & 31, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const GnBlock b = gn_block(p, tiles, n_split);
  const GnTile t = gn_tile(p, b.g, b.tile, wave, lane, lp);
  const int32_t n_kt = (t.V_last + X::KT - 1) / X::KT;
  const int32_t k0 = (int32_t)((int64_t)n_kt * b.split / n_split), k1 = (int32_t)((int64_t)n_kt * (b.split + 1) / n_split);

  uint4 qf[X::NJ];
  const int64_t roff = (int64_t)t.i * p.q_tok_stride + (int64_t)t.h * p.q_head_stride;
#pragma unroll
  for (int j = 0; j < X::NJ; ++j) qf[j] = *reinterpret_cast<const uint4*>((const unsigned char*)((const T*)p.q + roff) + 32 * j + 16 * hh);

  f32x16 of[X::DB];
  gn_zero(of);
  float m_run = -1e30f, l_run = 0.f;
  const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};   // (the row sum is that of the rounded probabilities)
  const float c = p.sm_scale * 1.4426950408889634f;
  const uint32_t lane_row = lq * X::RB + ((hh ^ X::swz(lq)) << 4);
  const int32_t V_min = __builtin_amdgcn_readfirstlane(t.V), V_max = __builtin_amdgcn_readlane(t.V, 31);

  GnStream<T, D> ks;
  if (k0 < k1) {
    ks.init(p, t, b.g, lane, k0 * X::KT, lp);
    ks.copy(p, t, wave, lane, lp, k0, 0);
  }
  wait_copies<0>();
  __syncthreads();
  for (int32_t k = k0; k < k1; ++k) {
    const uint32_t buf = ((k - k0) & 1) * GN_BUF;
    if (k + 1 < k1) ks.copy(p, t, wave, lane, lp, k + 1, buf ^ GN_BUF);
#pragma unroll
    for (int u = 0; u < X::KT / 32; ++u) {
      const int32_t t0 = k * X::KT + 32 * u;
      if (t.active && t0 < V_max) {   // (wave-uniform)
        f32x16 s = gn_chain<T, D>(smem, buf + 32 * u * X::RB, lane_row, qf);
        if (t0 + 32 > V_min) {
          const int32_t rel = t.V - t0 - 4 * hh;
#pragma unroll
          for (int x = 0; x < 16; ++x)
            if (8 * (x >> 2) + (x & 3) >= rel) s[x] = -INFINITY;
        }
        float mx = fmaxf(s[0], s[1]);
#pragma unroll
        for (int x = 2; x < 16; ++x) mx = fmaxf(mx, s[x]);
        const float m_new = fmaxf(m_run, half_max(mx));
        const float alpha = __builtin_amdgcn_exp2f((m_run - m_new) * c), mc = m_new * c;
        m_run = m_new;
        float sum = 0.f;
#pragma unroll
        for (int x = 0; x < 16; x += 2) {
          s[x] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[x], c, -mc));
          s[x + 1] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[x + 1], c, -mc));
          if constexpr (X::BF) sum = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pack2_bf16(s[x], s[x + 1])), ones, sum, false);
          else sum += s[x] + s[x + 1];
        }
        l_run = __builtin_fmaf(l_run, alpha, sum);
        if (__any(alpha != 1.f)) {
#pragma unroll
          for (int db = 0; db < X::DB; ++db)
#pragma unroll
            for (int x = 0; x < 16; ++x) of[db][x] *= alpha;
        }
        gn_tprod<T, D>(smem, buf + X::TILE + 32 * u * X::RB, lane, s, of);
      }
    }
    wait_copies<0>();
    __syncthreads();
  }

  const float l_tot = half_sum(l_run);
  if (!t.valid) return;
  if (n_split > 1) {
    const int64_t at = ((int64_t)b.split * p.Hkv + b.g) * ((int64_t)p.C * p.G) + t.r;
    float* dst = part + at * D;
    gn_emit<T, D>(of, hh, [&](int d, float v0, float v1, float v2, float v3) { gn_store4<float>(dst + d, v0, v1, v2, v3); });
    if (hh == 0) part_ml[at] = make_float2(l_tot > 0.f ? m_run * c : -INFINITY, l_tot);
  } else {
    const float inv = 1.f / l_tot;
    T* dst = (T*)p.o + roff;
    gn_emit<T, D>(of, hh, [&](int d, float v0, float v1, float v2, float v3) { gn_store4<T>(dst + d, v0 * inv, v1 * inv, v2 * inv, v3 * inv); });
    if (hh == 0) p.lse[(int64_t)t.h * p.C + t.i] = (m_run * c + __builtin_amdgcn_logf(l_tot)) * 0.6931471805599453f;
  }
}

// O = sum of the splits' O rescaled to the common maximum / sum of their l; D / 4 lanes per row
template <typename T, int D>
__global__ __launch_bounds__(256) void fwd_combine_kernel(Params p, int32_t n_split, const float* __restrict__ part,
                                                          const float2* __restrict__ part_ml) {
  constexpr int LPR = D / 4;
  const int64_t rows = (int64_t)p.C * p.G, row = (int64_t)blockIdx.x * (256 / LPR) + threadIdx.x / LPR;
  if (row >= rows * p.Hkv) return;
  const int d = (threadIdx.x % LPR) * 4;
  const int g = (int)(row / rows);
  const int32_t r = (int32_t)(row - g * rows), i = (int32_t)div_g(p, (uint32_t)r), h = g * p.G + (r - i * p.G);
  float M = -INFINITY;
  for (int s = 0; s < n_split; ++s) M = fmaxf(M, part_ml[s * rows * p.Hkv + row].x);
  float L = 0.f;
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int s = 0; s < n_split; ++s) {
    const float2 ml = part_ml[s * rows * p.Hkv + row];
    const float w = __builtin_amdgcn_exp2f(ml.x - M);
    const float4 v = *reinterpret_cast<const float4*>(part + (s * rows * p.Hkv + row) * D + d);
    L += ml.y * w;
    acc.x += v.x * w; acc.y += v.y * w; acc.z += v.z * w; acc.w += v.w * w;
  }
  const float inv = 1.f / L;
  gn_store4<T>((T*)p.o + (int64_t)i * p.q_tok_stride + (int64_t)h * p.q_head_stride + d, acc.x * inv, acc.y * inv, acc.z * inv, acc.w * inv);
  if (d == 0) p.lse[(int64_t)h * p.C + i] = (M + __builtin_amdgcn_logf(L)) * 0.6931471805599453f;
}

// ---- dQ -----------------------------------------------------------------------------------------
// Also computes Delta = <dO, O> of its rows, which the dK / dV kernel reads (it runs afterwards).
template <typename T, int D>
__global__ __launch_bounds__(GN_THREADS, (Gn<T, D>::RB == 512 ? 1 : 2)) void dq_generic_kernel(Params p, int32_t tiles, int32_t n_split, int lp,
                                                                                 float* __restrict__ part) {
  typedef Gn<T, D> X;
  extern __shared__ __align__(16) unsigned char smem[];
  const int lane = threadIdx.x & 63, hh = lane >> 5, lq = lane & 31, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const GnBlock b = gn_block(p, tiles, n_split);
  const GnTile t = gn_tile(p, b.g, b.tile, wave, lane, lp);
  const int32_t n_kt = (t.V_last + X::KT - 1) / X::KT;
  const int32_t k0 = (int32_t)((int64_t)n_kt * b.split / n_split), k1 = (int32_t)((int64_t)n_kt * (b.split + 1) / n_split);

  uint4 qf[X::NJ], dof[X::NJ];
  const int64_t roff = (int64_t)t.i * p.q_tok_stride + (int64_t)t.h * p.q_head_stride;
  float delta = 0.f;
#pragma unroll
  for (int j = 0; j < X::NJ; ++j) {
    const int64_t at = roff * X::ES + 32 * j + 16 * hh;
    qf[j] = *reinterpret_cast<const uint4*>((const unsigned char*)p.q + at);
    dof[j] = *reinterpret_cast<const uint4*>((const unsigned char*)p.d_o + at);
    const uint4 ov = *reinterpret_cast<const uint4*>((const unsigned char*)p.o + at);
    const T* x = reinterpret_cast<const T*>(&dof[j]);
    const T* y = reinterpret_cast<const T*>(&ov);
#pragma unroll
    for (int k = 0; k < 16 / X::ES; ++k) delta = __builtin_fmaf(Elem<T>::load(x + k), Elem<T>::load(y + k), delta);
  }
  delta = half_sum(delta);
  if (b.split == 0 && t.valid && hh == 0) p.delta[(int64_t)t.h * p.C + t.i] = delta;
  const float lse2 = p.lse[(int64_t)t.h * p.C + t.i] * 1.4426950408889634f;

  f32x16 dq[X::DB];
  gn_zero(dq);
  const float c = p.sm_scale * 1.4426950408889634f;
  const uint32_t lane_row = lq * X::RB + ((hh ^ X::swz(lq)) << 4);
  const int32_t V_min = __builtin_amdgcn_readfirstlane(t.V), V_max = __builtin_amdgcn_readlane(t.V, 31);

  GnStream<T, D> ks;
  if (k0 < k1) {
    ks.init(p, t, b.g, lane, k0 * X::KT, lp);
    ks.copy(p, t, wave, lane, lp, k0, 0);
  }
  wait_copies<0>();
  __syncthreads();
  for (int32_t k = k0; k < k1; ++k) {
    const uint32_t buf = ((k - k0) & 1) * GN_BUF;
    if (k + 1 < k1) ks.copy(p, t, wave, lane, lp, k + 1, buf ^ GN_BUF);
#pragma unroll
    for (int u = 0; u < X::KT / 32; ++u) {
      const int32_t t0 = k * X::KT + 32 * u;
      if (t.active && t0 < V_max) {
        f32x16 s = gn_chain<T, D>(smem, buf + 32 * u * X::RB, lane_row, qf);
        const f32x16 dp = gn_chain<T, D>(smem, buf + X::TILE + 32 * u * X::RB, lane_row, dof);
        const bool mask = t0 + 32 > V_min;
        const int32_t rel = t.V - t0 - 4 * hh;
#pragma unroll
        for (int x = 0; x < 16; ++x) {
          float pr = __builtin_amdgcn_exp2f(__builtin_fmaf(s[x], c, -lse2));
          if (mask && 8 * (x >> 2) + (x & 3) >= rel) pr = 0.f;
          s[x] = pr * (dp[x] - delta);
        }
        gn_tprod<T, D>(smem, buf + 32 * u * X::RB, lane, s, dq);
      }
    }
    wait_copies<0>();
    __syncthreads();
  }
  if (!t.valid) return;
  if (n_split > 1) {
    float* dst = part + (((int64_t)b.split * p.Hkv + b.g) * ((int64_t)p.C * p.G) + t.r) * D;
    gn_emit<T, D>(dq, hh, [&](int d, float v0, float v1, float v2, float v3) { gn_store4<float>(dst + d, v0, v1, v2, v3); });
  } else {
    T* dst = (T*)p.d_q + roff;
    const float sc = p.sm_scale;
    gn_emit<T, D>(dq, hh, [&](int d, float v0, float v1, float v2, float v3) { gn_store4<T>(dst + d, v0 * sc, v1 * sc, v2 * sc, v3 * sc); });
  }
}

// ---- dK / dV ------------------------------------------------------------------------------------
// A workgroup owns a unit of up to 128 keys of a KV head -- 128 / P consecutive list entries, or (one
// list per query page) one page of the union -- or one slice of the rows that see it.  Wave w holds
// keys 32 w .. + 31.  part[slot][dK | dV][128 keys][D]: slices, added to the pool by the finish kernel.
template <typename T, typename TG, int D>
__global__ __launch_bounds__(GN_THREADS, (Gn<T, D>::RB >= 256 && !(sizeof(T) == 4 && D == 64) ? 1 : 2)) void dkv_generic_kernel(
    Params p, int32_t n_split, int lp, float* __restrict__ part) {
  typedef Gn<T, D> X;
  extern __shared__ __align__(16) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63, hh = lane >> 5, lq = lane & 31, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int32_t bid = blockIdx.x, rest = bid / p.Hkv, g = bid - rest * p.Hkv;
  int32_t e0, sp = 0, q0 = 0, qc = 0, slot = -1;
  if (p.qp) {
    const int32_t n_units = p.unit_count[g];
    if (rest >= n_units) return;
    const int4 un = p.units[(int64_t)g * p.max_units + (n_units - 1 - rest)];
    e0 = un.x; q0 = un.y; qc = un.z; slot = un.w;
  } else {
    const int32_t u = rest / n_split;
    sp = rest - u * n_split;
    e0 = u << (7 - lp);
    if (e0 >= list_len(p, g)) return;
    if (n_split > 1) slot = bid;   // (every slice of every unit has a slot of its own: the workgroup index)
  }
  const int32_t len = owned_len(p, g);
  const int64_t first_q = p.N - p.C;
  // this lane's key
  const int32_t kq = 32 * wave + lq;
  int32_t e = e0 + (p.qp ? 0 : kq >> lp);
  const bool kvalid = p.qp ? kq < p.P : e < len;
  e = e < len ? e : len - 1;
  const bool active = p.qp ? 32 * wave < p.P : e0 + (32 * wave >> lp) < len;
  const int64_t l = owned_at(p, g, e), pos = (l << lp) + (kq & (p.P - 1));
  const int64_t koff = (int64_t)p.page_table[l] * p.pool_page_stride + (int64_t)g * p.pool_head_stride + (int64_t)(kq & (p.P - 1)) * p.pool_tok_stride;
  // rows before r_key do not see the key
  const int32_t r_key = pos > first_q ? (int32_t)(pos - first_q) * p.G : 0;
  const int32_t r_key_max = __builtin_amdgcn_readlane(r_key, 31);
  const int64_t pos0 = owned_at(p, g, e0) << lp;
  const int32_t r_lo = pos0 > first_q ? (int32_t)(pos0 - first_q) * p.G : 0, rows = p.C * p.G;
  // stages of KT rows: [s0, s1) of the chunk's, or stage v % spq of the unit's query page v / spq
  const int32_t rpq = p.P * p.G, spq = (rpq + X::KT - 1) / X::KT;
  const int32_t st_lo = r_lo / X::KT, st_n = (rows + X::KT - 1) / X::KT - st_lo;
  const int32_t s0 = p.qp ? 0 : st_lo + (int32_t)((int64_t)st_n * sp / n_split);
  const int32_t s1 = p.qp ? qc * spq : st_lo + (int32_t)((int64_t)st_n * (sp + 1) / n_split);
  int32_t tau_v = 0;
  if (p.qp && lane < qc) tau_v = p.inv_qp[(int64_t)g * p.m * p.sel_stride + p.inv_off[(int64_t)g * (p.un_stride + 1) + e0] + q0 + lane];

  uint4 kf[X::NJ], vf[X::NJ];
#pragma unroll
  for (int j = 0; j < X::NJ; ++j) {
    const int64_t at = koff * X::ES + 32 * j + 16 * hh;
    kf[j] = *reinterpret_cast<const uint4*>((const unsigned char*)p.k_pool + at);
    vf[j] = *reinterpret_cast<const uint4*>((const unsigned char*)p.v_pool + at);
  }
  f32x16 dk[X::DB], dv[X::DB];
  gn_zero(dk);
  gn_zero(dv);
  const float c = p.sm_scale * 1.4426950408889634f;
  const uint32_t lane_row = lq * X::RB + ((hh ^ X::swz(lq)) << 4);

  // rows [base, end) of stage s
  auto stage_rows = [&](int32_t s, int32_t& base, int32_t& end) {
    if (!p.qp) {
      base = s * X::KT;
      end = rows;
    } else {
      const int32_t v = s / spq, tau = __builtin_amdgcn_readlane(tau_v, v & 63);
      base = tau * rpq + (s - v * spq) * X::KT;
      end = (tau + 1) * rpq;
    }
  };
  float st_l = INFINITY, st_d = 0.f;   // statistics of row `tid` of the stage under way
  auto copy = [&](int32_t s, uint32_t buf) {
    int32_t base, end;
    stage_rows(s, base, end);
    const uint32_t lrow = lane / X::NG, pos16 = lane % X::NG;
    const uint32_t dst = buf + wave * X::RW * X::RB;
#pragma unroll
    for (int k = 0; k < X::NI; ++k) {
      const uint32_t row = wave * X::RW + k * X::RPI + lrow;
      int32_t r = base + (int32_t)row;
      r = r < end ? r : end - 1;
      const int32_t i = (int32_t)div_g(p, (uint32_t)r);
      const int64_t at = ((int64_t)i * p.q_tok_stride + (int64_t)(g * p.G + (r - i * p.G)) * p.q_head_stride) * X::ES +
                         (int64_t)((pos16 ^ X::swz(row & 15)) << 4);
      gn_copy16((const unsigned char*)p.q + at, dst + 1024 * k);
      gn_copy16((const unsigned char*)p.d_o + at, dst + X::TILE + 1024 * k);
    }
    if (tid < X::KT) {
      const int32_t r = base + tid;
      st_l = INFINITY;   // rows past the end: P = 0
      st_d = 0.f;
      if (r < end) {
        const int32_t i = (int32_t)div_g(p, (uint32_t)r);
        const int64_t at = (int64_t)(g * p.G + (r - i * p.G)) * p.C + i;
        st_l = p.lse[at] * 1.4426950408889634f;
        st_d = p.delta[at];
      }
    }
  };
  auto publish = [&](uint32_t buf) {   // buf: GN_BUF * index
    float* st = reinterpret_cast<float*>(smem + GN_STAT + (buf ? 512 : 0));
    if (tid < X::KT) {
      st[tid] = st_l;
      st[64 + tid] = st_d;
    }
  };

  if (s0 < s1) {
    copy(s0, 0);
    publish(0);
  }
  wait_copies<0>();
  __syncthreads();
  for (int32_t s = s0; s < s1; ++s) {
    const uint32_t buf = ((s - s0) & 1) * GN_BUF;
    if (s + 1 < s1) copy(s + 1, buf ^ GN_BUF);
    int32_t base, end;
    stage_rows(s, base, end);
    const float* st = reinterpret_cast<const float*>(smem + GN_STAT + (buf ? 512 : 0));
#pragma unroll
    for (int u = 0; u < X::KT / 32; ++u) {
      if (active) {
        f32x16 pr = gn_chain<T, D>(smem, buf + 32 * u * X::RB, lane_row, kf);
        f32x16 ds = gn_chain<T, D>(smem, buf + X::TILE + 32 * u * X::RB, lane_row, vf);
        const bool mask = base + 32 * u < r_key_max;   // (wave-uniform)
        const int32_t rel = r_key - base - 32 * u - 4 * hh;
#pragma unroll
        for (int a = 0; a < 4; ++a) {
          const float4 l4 = *reinterpret_cast<const float4*>(st + 32 * u + 8 * a + 4 * hh);
          const float4 d4 = *reinterpret_cast<const float4*>(st + 64 + 32 * u + 8 * a + 4 * hh);
          const float lv[4] = {l4.x, l4.y, l4.z, l4.w}, dl[4] = {d4.x, d4.y, d4.z, d4.w};
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            float v = __builtin_amdgcn_exp2f(__builtin_fmaf(pr[4 * a + q], c, -lv[q]));
            if (mask && 8 * a + q < rel) v = 0.f;
            pr[4 * a + q] = v;
            ds[4 * a + q] = v * (ds[4 * a + q] - dl[q]);
          }
        }
        gn_tprod<T, D>(smem, buf + X::TILE + 32 * u * X::RB, lane, pr, dv);
        gn_tprod<T, D>(smem, buf + 32 * u * X::RB, lane, ds, dk);
      }
    }
    if (s + 1 < s1) publish(buf ^ GN_BUF);
    wait_copies<0>();
    __syncthreads();
  }

  const float sc = p.sm_scale;
  if (slot >= 0) {
    float* dst = part + ((int64_t)slot * 2 * GN_ROWS + kq) * D;
    if (kvalid) {
      gn_emit<T, D>(dk, hh, [&](int d, float v0, float v1, float v2, float v3) { gn_store4<float>(dst + d, v0 * sc, v1 * sc, v2 * sc, v3 * sc); });
      dst += GN_ROWS * D;
      gn_emit<T, D>(dv, hh, [&](int d, float v0, float v1, float v2, float v3) { gn_store4<float>(dst + d, v0, v1, v2, v3); });
    }
  } else if (kvalid) {
    TG* pk = (TG*)p.dk_pool + koff;
    TG* pv = (TG*)p.dv_pool + koff;
    gn_emit<T, D>(dk, hh, [&](int d, float v0, float v1, float v2, float v3) { gn_add4<TG>(pk + d, v0 * sc, v1 * sc, v2 * sc, v3 * sc); });
    gn_emit<T, D>(dv, hh, [&](int d, float v0, float v1, float v2, float v3) { gn_add4<TG>(pv + d, v0, v1, v2, v3); });
  }
}

// What is left of a backward with splits, in one launch: workgroups below dq_blocks add the dQ partials (D / 4
// lanes per row), the others add the slices of a dK / dV unit to the pool (one thread per four dims).
template <typename T, typename TG, int D>
__global__ __launch_bounds__(256) void bwd_finish_kernel(Params p, int32_t dq_split, const float* __restrict__ dq_part, int32_t dq_blocks,
                                                         int32_t kv_split, const float* __restrict__ kv_part, int lp) {
  constexpr int LPR = D / 4, BPU = 2 * GN_ROWS * LPR / 256;   // workgroups per unit
  if ((int32_t)blockIdx.x < dq_blocks) {
    const int64_t rows = (int64_t)p.C * p.G, row = (int64_t)blockIdx.x * (256 / LPR) + threadIdx.x / LPR;
    if (row >= rows * p.Hkv) return;
    const int d = (threadIdx.x % LPR) * 4, g = (int)(row / rows);
    const int32_t r = (int32_t)(row - g * rows), i = (int32_t)div_g(p, (uint32_t)r), h = g * p.G + (r - i * p.G);
    float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int s = 0; s < dq_split; ++s) {
      const float4 v = *reinterpret_cast<const float4*>(dq_part + (s * rows * p.Hkv + row) * D + d);
      a.x += v.x; a.y += v.y; a.z += v.z; a.w += v.w;
    }
    const float sc = p.sm_scale;
    gn_store4<T>((T*)p.d_q + (int64_t)i * p.q_tok_stride + (int64_t)h * p.q_head_stride + d, a.x * sc, a.y * sc, a.z * sc, a.w * sc);
    return;
  }
  const int32_t b = (int32_t)blockIdx.x - dq_blocks, blk = b % BPU, ug = b / BPU, u = ug / p.Hkv, g = ug - u * p.Hkv;
  const int e4 = blk * 256 + threadIdx.x, which = e4 / (GN_ROWS * LPR), kq = (e4 / LPR) % GN_ROWS, d = (e4 % LPR) * 4;
  int64_t slot, next;
  int32_t e;
  if (p.qp) {
    if (u >= p.multi_count[g] || kq >= p.P) return;
    e = p.multi_list[(int64_t)g * p.max_multi + u];
    kv_split = p.un_ns[(int64_t)g * p.un_stride + e];
    slot = p.un_pbase[(int64_t)g * p.un_stride + e];
    next = 1;
  } else {
    e = (u << (7 - lp)) + (kq >> lp);
    if (e >= list_len(p, g)) return;
    slot = ((int64_t)u * kv_split) * p.Hkv + g;
    next = p.Hkv;
  }
  const int64_t l = owned_at(p, g, e);
  float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int s = 0; s < kv_split; ++s) {
    const float4 v = *reinterpret_cast<const float4*>(kv_part + (((slot + s * next) * 2 + which) * GN_ROWS + kq) * D + d);
    a.x += v.x; a.y += v.y; a.z += v.z; a.w += v.w;
  }
  TG* pool = (TG*)(which == 0 ? p.dk_pool : p.dv_pool) + (int64_t)p.page_table[l] * p.pool_page_stride + (int64_t)g * p.pool_head_stride +
             (int64_t)(kq & (p.P - 1)) * p.pool_tok_stride + d;
  gn_add4<TG>(pool, a.x, a.y, a.z, a.w);
}

// ---- host side ----------------------------------------------------------------------------------
static inline size_t gn_up(size_t x) { return (x + 255) & ~(size_t)255; }

// Splits: enough workgroups for two per compute unit, no split shorter than two tiles of the longest list
static int32_t gn_row_splits(const Params& p, int32_t max_len, int32_t kt) {
  const int64_t wgs = (int64_t)gn_tiles(p.C, p.G, p.P, p.m, p.qp) * p.Hkv;
  const int64_t longest = p.qp ? p.sel_stride : max_len;
  const int64_t want = 512 / (wgs > 0 ? wgs : 1), most = longest * p.P / (2 * kt);
  int64_t s = want < most ? want : most;
  s = s < 1 ? 1 : s > 32 ? 32 : s;
  return (int32_t)s;
}
static int32_t gn_key_units(const Params& p, int32_t max_len) {
  return (int32_t)(((int64_t)max_len * p.P + GN_ROWS - 1) / GN_ROWS);
}
static int32_t gn_key_splits(const Params& p, int32_t max_len, int32_t kt) {
  if (p.qp) return 1;
  const int64_t wgs = (int64_t)gn_key_units(p, max_len) * p.Hkv;
  const int64_t want = 512 / (wgs > 0 ? wgs : 1), most = ((int64_t)p.C * p.G + kt - 1) / kt / 2;
  int64_t s = want < most ? want : most;
  s = s < 1 ? 1 : s > 16 ? 16 : s;
  return (int32_t)s;
}
static int32_t gn_kt(const Params& p, bool bf) { return p.D * (bf ? 2 : 4) == 512 ? 32 : 64; }

static size_t gn_row_part_bytes(const Params& p, int32_t split) {
  return split > 1 ? gn_up((size_t)split * p.Hq * p.C * p.D * 4) : 0;
}
size_t fwd_generic_workspace_bytes(const Params& p, bool bf, int32_t max_len) {
  const int32_t s = gn_row_splits(p, max_len, gn_kt(p, bf));
  return s > 1 ? gn_row_part_bytes(p, s) + gn_up((size_t)s * p.Hq * p.C * 8) : 256;
}
static size_t gn_key_part_bytes(const Params& p, int32_t max_len, int32_t split) {
  const size_t slots = p.qp ? (size_t)p.Hkv * qp_max_pslots(p, p.sel_stride) : split > 1 ? (size_t)gn_key_units(p, max_len) * p.Hkv * split : 0;
  return gn_up(slots * 2 * GN_ROWS * p.D * 4);
}
size_t bwd_generic_workspace_bytes(const Params& p, bool bf, int32_t max_len) {
  const int32_t kt = gn_kt(p, bf);
  return gn_up((size_t)p.Hq * p.C * sizeof(float)) + gn_row_part_bytes(p, gn_row_splits(p, max_len, kt)) +
         gn_key_part_bytes(p, max_len, gn_key_splits(p, max_len, kt));
}

template <typename T, int D>
static hipError_t fwd_generic(const Params& p, int32_t max_len, void* ws, size_t ws_bytes, hipStream_t st) {
  static DeviceOnce lds_once;
  if (hipError_t e = ensure_max_dynamic_lds(lds_once, (const void*)fwd_generic_kernel<T, D>, GN_LDS); e != hipSuccess) return e;
  const int lp = __builtin_ctz(p.P);
  int32_t ns = gn_row_splits(p, max_len, Gn<T, D>::KT);
  if (ns > 1 && (!ws || ws_bytes < fwd_generic_workspace_bytes(p, Gn<T, D>::BF, max_len))) ns = 1;   // (the forward also runs without a workspace)
  float* part = (float*)ws;
  float2* ml = (float2*)((unsigned char*)ws + gn_row_part_bytes(p, ns));
  const int32_t tiles = gn_tiles(p.C, p.G, p.P, p.m, p.qp);
  ProfScope prof_("attn_fwd_generic", st);
  fwd_generic_kernel<T, D><<<dim3((unsigned)tiles * p.Hkv * ns), dim3(GN_THREADS), GN_LDS, st>>>(p, tiles, ns, lp, part, ml);
  if (ns > 1) {
    constexpr int RPB = 256 / (D / 4);
    fwd_combine_kernel<T, D><<<dim3((unsigned)(((int64_t)p.Hq * p.C + RPB - 1) / RPB)), dim3(256), 0, st>>>(p, ns, part, ml);
  }
  return hipGetLastError();
}
hipError_t launch_fwd_generic(const Params& p, bool bf, int32_t max_len, void* ws, size_t ws_bytes, hipStream_t st) {
  if (bf) return p.D == 128 ? fwd_generic<bf16_t, 128>(p, max_len, ws, ws_bytes, st) : fwd_generic<bf16_t, 64>(p, max_len, ws, ws_bytes, st);
  return p.D == 128 ? fwd_generic<float, 128>(p, max_len, ws, ws_bytes, st) : fwd_generic<float, 64>(p, max_len, ws, ws_bytes, st);
}

template <typename T, typename TG, int D>
static hipError_t bwd_generic(Params p, int32_t max_len, void* ws, hipStream_t st) {
  static DeviceOnce once_q, once_kv;
  if (hipError_t e = ensure_max_dynamic_lds(once_q, (const void*)dq_generic_kernel<T, D>, GN_LDS); e != hipSuccess) return e;
  if (hipError_t e = ensure_max_dynamic_lds(once_kv, (const void*)dkv_generic_kernel<T, TG, D>, GN_LDS); e != hipSuccess) return e;
  const int lp = __builtin_ctz(p.P);
  const int32_t kt = Gn<T, D>::KT, ns = gn_row_splits(p, max_len, kt), nk = gn_key_splits(p, max_len, kt);
  unsigned char* w = (unsigned char*)ws;
  p.delta = (float*)w;
  w += gn_up((size_t)p.Hq * p.C * sizeof(float));
  float* dq_part = (float*)w;
  float* kv_part = (float*)(w + gn_row_part_bytes(p, ns));
  const int32_t tiles = gn_tiles(p.C, p.G, p.P, p.m, p.qp);
  const int32_t units = p.qp ? p.max_units : gn_key_units(p, max_len);
  ProfScope prof_("attn_bwd_generic", st);
  dq_generic_kernel<T, D><<<dim3((unsigned)tiles * p.Hkv * ns), dim3(GN_THREADS), GN_LDS, st>>>(p, tiles, ns, lp, dq_part);
  dkv_generic_kernel<T, TG, D><<<dim3((unsigned)units * p.Hkv * nk), dim3(GN_THREADS), GN_LDS, st>>>(p, nk, lp, kv_part);
  if (ns > 1 || nk > 1 || p.qp) {
    constexpr int RPB = 256 / (D / 4), BPU = 2 * GN_ROWS * (D / 4) / 256;
    const int32_t dq_blocks = ns > 1 ? (int32_t)(((int64_t)p.Hq * p.C + RPB - 1) / RPB) : 0;
    const int64_t kv_blocks = (int64_t)(p.qp ? p.max_multi : nk > 1 ? units : 0) * p.Hkv * BPU;
    bwd_finish_kernel<T, TG, D><<<dim3((unsigned)(dq_blocks + kv_blocks)), dim3(256), 0, st>>>(p, ns, dq_part, dq_blocks, nk, kv_part, lp);
  }
  return hipGetLastError();
}
// max_len: host-side upper bound of the list length (of the union with one list per query page)
hipError_t launch_bwd_generic(const Params& p, bool bf, int32_t max_len, void* ws, hipStream_t st) {
#define OOMB_BWD(T, TG) (p.D == 128 ? bwd_generic<T, TG, 128>(p, max_len, ws, st) : bwd_generic<T, TG, 64>(p, max_len, ws, st))
  if (bf) return p.grad_is_bf16 ? OOMB_BWD(bf16_t, bf16_t) : OOMB_BWD(bf16_t, float);
  return p.grad_is_bf16 ? OOMB_BWD(float, bf16_t) : OOMB_BWD(float, float);
#undef OOMB_BWD
}

}  // namespace oomb
