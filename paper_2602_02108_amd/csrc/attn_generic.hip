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
// bf16: v_mfma_f32_32x32x16_bf16, the transposed operand by transposing LDS reads.  fp32: S in three
// bf16 terms per value (below), the other products by v_mfma_f32_32x32x2_f32; an operand is one dword
// per lane, so any order of the contraction index that both operands share will do, and four
// instructions take one 16-byte read.
//
// Page sizes disappear in "list-token space": the tokens of a page list in list order.  The list is
// ascending, so what a row sees is a prefix of that sequence: one number per row.  Row space of a
// KV head: r = token * G + head in group, so a tile's rows are consecutive tokens of all G heads,
// and the rows of a query page are contiguous for every page size.
//
// What bounds them: fp32 the matrix pipe itself (256 flops per cycle and compute unit, 157 TFLOP/s; calls that are not short
// therefore form the other products in terms, too: fwd_terms_kernel and bwd_units_kernel);
// bf16 the exposed vector work and LDS latency of one or two waves per SIMD; short calls the number
// of workgroups, which is why the streamed side is cut into splits whose partial sums a second
// kernel combines in a fixed order.  Measured against one wave per query row (per key in dK / dV)
// with plain fp32 arithmetic: 28 / 4 heads fp32, chunk 512, 16 + 4 pages of 128: 41.5 -> 0.41 ms
// (59 GFLOP); 8 / 2 heads bf16, chunk 1088, 24 + 17 pages of 64: 18.4 -> 0.11 ms (32 GFLOP).
#include "mfma_common.h"
#include "launch.h"
#include "partials.h"

namespace oomb {

constexpr int GN_ROWS = PART_ROWS;

// Geometry of a row tile: RB bytes per row, NG granules of 16 bytes, granule c of row r at position
// c ^ swz(r).  The swizzle frees both access patterns of bank conflicts: 16 rows at one granule, and
// the second product's (bf16: 4 rows x 64 bytes of a transposing read; fp32: whole rows).
template <typename T, int D> struct Gn {
  static constexpr bool BF = sizeof(T) == 2;
  static constexpr int ES = sizeof(T), RB = D * ES, NG = RB / 16;
  static constexpr int NJ = NG / 2;                // k-steps of the first product (one granule per lane each)
  static constexpr int DB = D / 32;                // accumulator blocks of the second product
  static constexpr int RPI = 1024 / RB;            // rows per copy instruction of a wave
  static __device__ __forceinline__ constexpr uint32_t swz(uint32_t r) {
    return !BF ? (r & 15) : RB == 256 ? row_tile_f(r) : ((((r >> 1) & 1) << 2) | ((r >> 2) & 3));
  }
};
// Two row tiles of KT rows (K and V, or Q and dO) per buffer, copied by four waves; two buffers.
template <typename T, int D> struct GnTiles {
  static constexpr int RB = Gn<T, D>::RB;
  static constexpr int KT = Gn<T, D>::BF ? 64 : 32, U = KT / 32;   // rows of a tile, blocks of 32
  static constexpr int TILE = KT * RB, BUF = 2 * TILE;
  static constexpr int NI = TILE / 1024 / 4;       // copy instructions per wave and tile
  static constexpr int RW = NI * Gn<T, D>::RPI;    // rows a wave copies: 8 or 16, so they lie in one page
};
// Forward and dQ: a group of four waves (128 rows) walks its share of the key tiles; with KH = 2 a workgroup
// holds two such groups on the same rows whose results meet in LDS at the end: two waves per SIMD, and
// half the partial results of two workgroups.
template <typename T, int D, int KH> struct GnRow {
  static constexpr int THREADS = 256 * KH, GROUP = 2 * GnTiles<T, D>::BUF;   // LDS of a group
  static constexpr int MERGE = GN_ROWS * D * 4 + 4 * 64 * 8;
  static constexpr int LDS = KH * GROUP > MERGE || KH == 1 ? KH * GROUP : MERGE;
};

// C += A B over one granule pair: A, B hold 16 bytes per lane (granule 2 j + lane / 32 of the lane's row)
template <typename T> __device__ __forceinline__ void gn_mma(const u32x4_t& a, const u32x4_t& b, f32x16& c) {
  if constexpr (sizeof(T) == 2) {
    c = mfma32(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c);
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) c = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a[e]), __uint_as_float(b[e]), c, 0, 0, 0);
  }
}

template <int N> __device__ __forceinline__ void gn_zero(f32x16 (&v)[N]) {
#pragma unroll
  for (int k = 0; k < N; ++k)
#pragma unroll
    for (int x = 0; x < 16; ++x) v[k][x] = 0.f;
}

// ---- products of fp32 tensors on the bf16 matrix pipe ---------------------------------------------
// An fp32 value is the sum of three bf16 values, all 24 bits: a = a0 + a1 + a2, each the rounding of what the ones before it left.  A
// product of two such sums takes six bf16 matrix instructions -- a0 b0, a0 b1, a1 b0, a1 b1, a0 b2, a2 b0; the others are at most 2^-24 of
// it, 2^-27 rms -- and these 192 cycles where v_mfma_f32_32x32x2 takes 512.
// Values below 2^-109 keep fewer bits: the smallest bf16 is 2^-133.  V, dO and dS, on which the results depend linearly, are therefore lifted by 2^16 first (GN_LIFT;
// what overflows -- products of dO and V of 2^96 -- is not finite and formed anew from fp32 products): they keep their bits down to the smallest normal fp32 value.  Not lifted are Q and K,
// whose products are the argument of an exponential (dQ of small keys: GnU), and P, whose largest value in a row is not small: a product is off by 2^-134 times the other value.
// S is formed this way on every route.  What the backward makes of S and LSE then has the errors that the forward's S has, whichever
// kernels the two passes take; those of different products do not cancel in dQ.  Against 64 bits, 2 / 1 heads of 128, logits of 3 times
// the spread, chunk 1024, 40 pages: dQ both passes with fp32 products 1.95e-6, one of them in terms 4.5e-6 (forward) and 4.1e-6 (backward), S in
// terms on either route 1.2 to 1.4e-6.
constexpr float GN_EDGE = 0x1.FFp127f;   // the least value that bf16 rounds to an infinity
constexpr float GN_LIFT = 0x1p16f, GN_LOWER = 0x1p-16f;
struct GnTerms { uint32_t w[3]; };
// two values.  What would round to an infinity is cut off instead; infinities and NaN are their own first term.
__device__ __forceinline__ GnTerms gn_terms(float a, float b) {
  GnTerms t;
  auto first = [](float v) {
    const uint32_t u = __float_as_uint(v), r = pack2_bf16(v, v) << 16;
    return fabsf(v) < GN_EDGE || v != v ? r : u & 0xffff0000u;
  };
  const uint32_t a0 = first(a), b0 = first(b);
  t.w[0] = (a0 >> 16) | (b0 & 0xffff0000u);
  const float ra = fabsf(a) < INFINITY ? a - __uint_as_float(a0) : 0.f, rb = fabsf(b) < INFINITY ? b - __uint_as_float(b0) : 0.f;
  t.w[1] = pack2_bf16(ra, rb);
  t.w[2] = pack2_bf16(ra - __uint_as_float(t.w[1] << 16), rb - __uint_as_float(t.w[1] & 0xffff0000u));
  return t;
}
// the same in 11 instructions, for values below GN_EDGE (and NaN)
__device__ __forceinline__ GnTerms gn_terms_plain(float a, float b) {
  GnTerms t;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    t.w[k] = pack2_bf16(a, b);
    a -= __uint_as_float(t.w[k] << 16);
    b -= __uint_as_float(t.w[k] & 0xffff0000u);
  }
  return t;
}
// eight values as operands of three terms
template <bool PLAIN> __device__ __forceinline__ void gn_load_terms(const u32x4_t& a, const u32x4_t& b, u32x4_t (&t)[3]) {
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const float x = __uint_as_float(k < 2 ? a[2 * k] : b[2 * k - 4]), y = __uint_as_float(k < 2 ? a[2 * k + 1] : b[2 * k - 3]);
    const GnTerms w = PLAIN ? gn_terms_plain(x, y) : gn_terms(x, y);
#pragma unroll
    for (int n = 0; n < 3; ++n) t[n][k] = w.w[n];
  }
}
__device__ __forceinline__ void gn_lift(u32x4_t& v) {
#pragma unroll
  for (int k = 0; k < 4; ++k) v[k] = __float_as_uint(__uint_as_float(v[k]) * GN_LIFT);
}
// c += the product of two values of three terms, the smallest first; small += all of it but the product of the first terms
__device__ __forceinline__ void gn_mma_terms(const u32x4_t (&a)[3], const u32x4_t& b0, const u32x4_t& b1, const u32x4_t& b2, f32x16& small, f32x16& c) {
  const u32x4_t* b[3] = {&b0, &b1, &b2};
  constexpr int order[6][2] = {{2, 0}, {0, 2}, {1, 1}, {1, 0}, {0, 1}, {0, 0}};
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    f32x16& acc = k < 5 ? small : c;
    acc = mfma32(__builtin_bit_cast(bf16x8, a[order[k][0]]), __builtin_bit_cast(bf16x8, *b[order[k][1]]), acc);
  }
}
// Whether a small sum is not finite: 16 instructions per block (0 times an infinity or a NaN is a NaN)
__device__ __forceinline__ bool gn_odd(const f32x16& small) {
  float z0 = 0.f, z1 = 0.f;
#pragma unroll
  for (int x = 0; x < 16; x += 2) {
    z0 = __builtin_fmaf(small[x], 0.f, z0);
    z1 = __builtin_fmaf(small[x + 1], 0.f, z1);
  }
  return __any(z0 + z1 != 0.f);
}
// The two sums of gn_mma_terms as one, into c.  The small products of an infinity are infinities of either sign or (0 times infinity) NaN; that of the first terms
// is what the values themselves give: there it stands alone.
__device__ __forceinline__ void gn_add_small(f32x16& c, const f32x16& small, bool odd) {
  if (__builtin_expect(odd, 0)) {
#pragma unroll
    for (int x = 0; x < 16; ++x) c[x] = fabsf(small[x]) < INFINITY ? c[x] + small[x] : c[x];
  } else {
#pragma unroll
    for (int x = 0; x < 16; ++x) c[x] += small[x];
  }
}
// Granule j of an operand of a first product.  fp32: granules 2 k and 2 k + 1 are eight consecutive dims, half a k-step of the bf16 pipe.
template <typename T> __host__ __device__ __forceinline__ constexpr int gn_granule(const int j, const int hh) { return sizeof(T) == 2 ? 2 * j + hh : 4 * (j >> 1) + 2 * hh + (j & 1); }
// The staying operand of S; fp32: as terms, 96 registers for 64 at head dim 128
template <typename T, int D> struct GnStay {
  static constexpr int NJ = Gn<T, D>::NJ;
  const u32x4_t* src;
  u32x4_t f[NJ];
  __device__ __forceinline__ void at(const T* row, const int hh) { src = reinterpret_cast<const u32x4_t*>(row) + gn_granule<T>(0, hh); }
  __device__ __forceinline__ void load(const int j) { f[j] = src[gn_granule<T>(j, 0)]; }
  __device__ __forceinline__ void here() {}
  template <bool> __device__ __forceinline__ void split() {}
};
template <int D> struct GnStay<float, D> {
  static constexpr int NJ = Gn<float, D>::NJ;
  const u32x4_t* src;
  u32x4_t raw[NJ], t[NJ / 2][3];
  __device__ __forceinline__ void at(const float* row, const int hh) { src = reinterpret_cast<const u32x4_t*>(row) + gn_granule<float>(0, hh); }
  __device__ __forceinline__ void load(const int j) { raw[j] = src[gn_granule<float>(j, 0)]; }
  // waits for the granules
  __device__ __forceinline__ void here() {
#pragma unroll
    for (int j = 0; j < NJ; ++j) asm volatile("" : "+v"(raw[j]));
  }
  __device__ __forceinline__ bool finite() const {   // (of this lane)
    uint32_t m = 0;
#pragma unroll
    for (int j = 0; j < NJ / 2; ++j)
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint32_t w = t[j][0][k] & 0x7f807f80u, e = (w & 0xffffu) > w >> 16 ? w & 0xffffu : w >> 16;   // (the exponents of two first terms)
        m = m > e ? m : e;
      }
    return m != 0x7f80u;
  }
  template <bool PLAIN> __device__ __forceinline__ void split() {
#pragma unroll
    for (int j = 0; j < NJ; j += 2) gn_load_terms<PLAIN>(raw[j], raw[j + 1], t[j >> 1]);
  }
};
// S of 32 rows of the streamed side.  fp32: in terms, those of the streamed side formed on the way (11 vector instructions for two values, beside
// 192 matrix cycles for 512).  28 / 4 heads of 128, chunk 512, 20 pages: forward 177 -> 148 us, backward 604 -> 570 against S on the
// fp32 pipe; 14 / 2 heads of 64, chunk 1664, 27 pages of 128: 233 -> 198 and 632 -> 598; one tile per wave (2 / 1 heads) the same to 0.1 us.
template <typename T> struct GnSum {
  f32x16 v[sizeof(T) == 4 ? 2 : 1];
  u32x4_t held;
  __device__ __forceinline__ void zero() { gn_zero(v); }
  template <int D> __device__ __forceinline__ void step(const int j, const u32x4_t& f, const GnStay<T, D>& stay) {   // granule j of the streamed side
    if constexpr (sizeof(T) == 2) {
      v[0] = mfma32(__builtin_bit_cast(bf16x8, f), __builtin_bit_cast(bf16x8, stay.f[j]), v[0]);
    } else if (!(j & 1)) {
      held = f;
    } else {
      u32x4_t a[3];
      const u32x4_t(&b)[3] = stay.t[j >> 1];
      gn_load_terms<true>(held, f, a);
      gn_mma_terms(a, b[0], b[1], b[2], v[1], v[0]);
    }
  }
  // After the last granule: S is v[0].  again(j): granule j once more.  LOOP: the rare second sum in a loop, which takes fewer registers but
  // where accumulators live in the other half of the register file (dQ, dK / dV).
  template <bool LOOP, int D, typename L> __device__ __forceinline__ void close(const GnStay<T, D>& stay, L&& again) {
    if constexpr (sizeof(T) == 4) {
      constexpr int NJ = Gn<T, D>::NJ;
      const bool odd = gn_odd(v[1]);
      if (__builtin_expect(odd, 0)) {   // a value at the edge of fp32: with the terms of gn_terms
        zero();
        auto add = [&](const int j) __attribute__((always_inline)) {
          u32x4_t a[3], b[3];
          gn_load_terms<false>(again(j), again(j + 1), a);
          __builtin_amdgcn_sched_barrier(0);
          gn_load_terms<false>(stay.src[gn_granule<T>(j, 0)], stay.src[gn_granule<T>(j + 1, 0)], b);
          gn_mma_terms(a, b[0], b[1], b[2], v[1], v[0]);
          __builtin_amdgcn_sched_barrier(0);
        };
        if constexpr (LOOP) {
#pragma unroll 1
          for (int j = 0; j < NJ; j += 2) add(j);
        } else {
#pragma unroll
          for (int j = 0; j < NJ; j += 2) add(j);
        }
      }
      gn_add_small(v[0], v[1], odd);
    }
  }
};

// c + <a, b> over 16 bytes each
template <typename T> __device__ __forceinline__ float gn_dot(const u32x4_t& a, const u32x4_t& b, float c) {
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    if constexpr (sizeof(T) == 2) {
      c = __builtin_fmaf(__uint_as_float(a[k] << 16), __uint_as_float(b[k] << 16), c);
      c = __builtin_fmaf(__uint_as_float(a[k] & 0xffff0000u), __uint_as_float(b[k] & 0xffff0000u), c);
    } else {
      c = __builtin_fmaf(__uint_as_float(a[k]), __uint_as_float(b[k]), c);
    }
  }
  return c;
}

// LDS operand addresses of a lane.  bf16: one register per k-step and per transposing read (the swizzle is an XOR
// on the lane's granule), so that an operand read is register + immediate; fp32 forms its addresses as it
// goes (an instruction of its matrix pipe lasts 64 cycles).
template <typename T, int D> struct GnAddr {
  typedef Gn<T, D> X;
  static constexpr int NP = X::BF ? 2 * X::DB : 16;   // operands of the second product per block of 32 rows
  uint32_t row[X::BF ? X::NJ : 1], tr[X::BF ? 2 * X::DB : 1];
  __device__ __forceinline__ void init(int lane, uint32_t base) {   // base: a multiple of 1 KiB
    const uint32_t lq = lane & 31, hh = lane >> 5;
    if constexpr (X::BF) {
#pragma unroll
      for (int j = 0; j < X::NJ; ++j) row[j] = base + ((lq * X::RB + ((hh ^ X::swz(lq)) << 4)) ^ (uint32_t)(j << 5));
      const uint32_t L = lane & 15, gq = lane >> 4, r = 4 * (gq >> 1) + (L >> 2);
      const uint32_t t = r * X::RB + (((2 * (gq & 1) + ((L & 3) >> 1)) ^ X::swz(r)) << 4) + 8 * (L & 1);
#pragma unroll
      for (int db = 0; db < X::DB; ++db) {
        tr[2 * db] = base + (t ^ (uint32_t)(db << 6));
        tr[2 * db + 1] = base + (t ^ (uint32_t)(db << 6) ^ 32u);   // rows + 8: the swizzle changes by 2
      }
    } else {
      const uint32_t gran = D == 128 ? lq : lq >> 1, sub = D == 128 ? 0 : 8 * (lq & 1);
      row[0] = base + lq * X::RB + (((2 * hh) ^ X::swz(lq)) << 4);
      tr[0] = base + 4 * hh * X::RB + ((gran ^ (4 * hh)) << 4) + sub;
    }
  }
  // fp32, once per tile: operand addresses are formed from these registers each time (kept across the loop they would be spilled)
  __device__ __forceinline__ void anew() {
    if constexpr (!X::BF) asm volatile("" : "+v"(row[0]), "+v"(tr[0]));
  }
  // granule j of the first product: the 32 rows at LDS offset `off`
  __device__ __forceinline__ u32x4_t row_frag(const int j, const uint32_t off) const {
    const uint32_t at = (X::BF ? row[X::BF ? j : 0] : row[0] ^ (uint32_t)(gn_granule<T>(j, 0) << 4)) + off;
    return *(__attribute__((address_space(3))) const u32x4_t*)at;
  }
  // operand v of the second product over the same rows.  bf16: key group v / DB, dim block v % DB.  fp32: row 8 (v / 4) +
  // 4 hh + v % 4, the lane's DB consecutive dims.
  __device__ __forceinline__ u32x4_t tr_frag(const int v, const uint32_t off) const {
    if constexpr (X::BF) {
      const int u = v / X::DB, db = v % X::DB;
      const u32x2_t lo = __builtin_bit_cast(u32x2_t, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
          (__attribute__((address_space(3))) s16x4_t*)(tr[2 * db] + (off + 16 * u * X::RB))));
      const u32x2_t hi = __builtin_bit_cast(u32x2_t, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
          (__attribute__((address_space(3))) s16x4_t*)(tr[2 * db + 1] + (off + (16 * u + 8) * X::RB))));
      return __builtin_shufflevector(lo, hi, 0, 1, 2, 3);
    } else {
      const int r = 8 * (v >> 2) + (v & 3);
      const uint32_t at = (tr[0] ^ (uint32_t)((r & 15) << 4)) + (off + r * X::RB);
      if constexpr (D == 128) return *(__attribute__((address_space(3))) const u32x4_t*)at;
      const u32x2_t w = *(__attribute__((address_space(3))) const u32x2_t*)at;
      return __builtin_shufflevector(w, w, 0, 1, 0, 1);
    }
  }
};

// A block of probabilities (or dS) as the B operand of the second product.  fp32 tensors: the values themselves.  bf16 tensors: NT
// bf16 terms whose sum stands for the value, each the rounding of what the ones before it left, NT matrix
// instructions in the place of one (the fp32 instruction would take sixteen times as long).  Three are all 24 bits: shapes
// without kernels of their own hold probabilities and dS in fp32.  One is the precision of the kernels for pages of 128
// at head dim 128, and of the short calls that those hand over.  Two terms are 17 bits: enough for results in bf16
// unless their sums cancel (to 2^-14 of their terms: O, dQ and bf16 gradients 3 to 6 % off).  Error against 64 bits, 2-norm, 13
// calls of 64 to 2176 keys: O and gradients in bf16 1.66e-3 (the rounding of bf16 itself), dV in fp32 0.3 to 0.7e-6 (fp32
// values on the vector unit 0.6 to 1.5e-6; one term: O 2.1e-3, dV 1.7e-3).
template <typename T, int NT> struct GnP;
template <int NT> struct GnP<bf16_t, NT> {
  uint32_t w[NT][8];
  __device__ __forceinline__ void set2(const int x, float a, float b) {   // registers x, x + 1
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const uint32_t v = w[t][x >> 1] = pack2_bf16(a, b);
      if (t + 1 < NT) {
        a -= __uint_as_float(v << 16);
        b -= __uint_as_float(v & 0xffff0000u);
      }
    }
  }
};
template <> struct GnP<float, 1> {
  float w[1][16];
  __device__ __forceinline__ void set2(const int x, float a, float b) { w[0][x] = a; w[0][x + 1] = b; }
};
// operand v (tr_frag) of acc += tile^T P.  bf16: acc[db] row m is dim 32 db + m.  fp32: acc[e] row m is dim DB m + e.
template <typename T, int D, int NT> __device__ __forceinline__ void gn_tr_mma(const int v, const u32x4_t& f, const GnP<T, NT>& p, f32x16 (&acc)[D / 32]) {
  if constexpr (sizeof(T) == 2) {
    const int u = v / (D / 32), db = v % (D / 32);
#pragma unroll
    for (int t = NT - 1; t >= 0; --t) {   // (the smallest terms first)
      const u32x4_t b = {p.w[t][4 * u], p.w[t][4 * u + 1], p.w[t][4 * u + 2], p.w[t][4 * u + 3]};
      acc[db] = mfma32(__builtin_bit_cast(bf16x8, f), __builtin_bit_cast(bf16x8, b), acc[db]);
    }
  } else {
#pragma unroll
    for (int e = 0; e < D / 32; ++e) acc[e] = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(f[e]), p.w[0][v], acc[e], 0, 0, 0);
  }
}

// A straight run of N operand reads and their matrix instructions in batches of four: the next batch is fetched while
// one computes (left to itself the compiler waits for every operand just before its use).
// load(i) reads operand i, use(i, operand) multiplies and may add vector work; i is a constant.
template <typename T, int D> constexpr int GN_BATCH = sizeof(T) == 4 && D == 128 ? 2 : 4;   // (fp32 at head dim 128: registers)
template <int N, int B = 4, typename L, typename M> __device__ __forceinline__ void gn_pipeline(L&& load, M&& use) {
  static_assert(N % B == 0, "whole batches");
  u32x4_t fr[2][B];
#pragma unroll
  for (int k = 0; k < B; ++k) fr[0][k] = load(k);
#pragma unroll
  for (int b = 0; b < N / B; ++b) {
    if (b + 1 < N / B) {
#pragma unroll
      for (int k = 0; k < B; ++k) fr[(b + 1) & 1][k] = load(B * (b + 1) + k);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int k = 0; k < B; ++k) {
      use(B * b + k, fr[b & 1][k]);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

// A row statistic of a block of 32 rows in LDS: value x of a lane is that of row 8 (x / 4) + 4 hh + x % 4.  A group of four is fetched while the one before
// it is in use: read where it is needed, every value waits for the LDS and for all operands fetched ahead of it (the one-launch backward of 8 / 2 heads,
// 41 pages of 64, chunk 1088: two thirds of a stage).
struct GnStat {
  float4 v[2];
  __device__ __forceinline__ void fetch(const float* block, const int hh, const int a) { v[a & 1] = *reinterpret_cast<const float4*>(block + 8 * a + 4 * hh); }
  __device__ __forceinline__ float at(const float* block, const int hh, const int x) {   // (in order)
    const float4& w = v[(x >> 2) & 1];
    const float r = (x & 3) == 0 ? w.x : (x & 3) == 1 ? w.y : (x & 3) == 2 ? w.z : w.w;
    if ((x & 3) == 0 && x < 12) fetch(block, hh, (x >> 2) + 1);
    return r;
  }
};

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
  int64_t block;          // index of the wave's block of 32 rows among all of the call
  int32_t r, i, h;        // this lane's row (clamped to the tile's last), its chunk token and query head
  bool valid, active;     // the lane owns a row; the wave owns at least one
  int32_t T_ent;          // list entries that some row of the tile sees
  int32_t V, V_last;      // list tokens this lane's row / the tile's last row sees
  int32_t V_first;        // those that every row of the tile sees
};

__device__ __forceinline__ GnTile gn_tile(const Params& p, int g, int32_t tile, int rb, int lane, int lp, int32_t max_len) {
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
  // the last 64 entries of a list of the expected length, read while its length is on its way
  int32_t e = max_len - 1 - lane >= 0 ? list_at(p, t.lid, max_len - 1 - lane) : -1;
  const int32_t len = list_len(p, t.lid);
  const int32_t last = base + GN_ROWS - 1 < end - 1 ? base + GN_ROWS - 1 : end - 1;
  const int32_t r = base + 32 * rb + (lane & 31);
  t.block = ((int64_t)g * gn_tiles(p.C, p.G, p.P, p.m, p.qp) + tile) * 4 + rb;
  t.valid = r <= last;
  t.active = base + 32 * rb <= last;
  t.r = t.valid ? r : last;
  t.i = (int32_t)div_g(p, (uint32_t)t.r);
  t.h = g * p.G + (t.r - t.i * p.G);
  const int64_t first_q = p.N - p.C;
  const int32_t i_last = (int32_t)div_g(p, (uint32_t)last);
  const int64_t a = first_q + t.i, a_last = first_q + i_last, a_first = first_q + div_g(p, (uint32_t)base);
  const int32_t pg = (int32_t)(a >> lp), pg_lo = (int32_t)(a_first >> lp), pg_hi = (int32_t)(a_last >> lp);
  // The rows of a tile lie in at most nine pages, so the entries past pg_lo that some row sees are among the last
  // 64 up to pg_hi.
  t.T_ent = len;
  int32_t n_over = __builtin_popcountll(__ballot(e > pg_hi));
  if (len != max_len || n_over > 48) {   // (shorter list, or a tile far before the list's end)
    t.T_ent = visible_len(p, t.lid, pg_hi, lane);
    e = t.T_ent - 1 - lane >= 0 ? list_at(p, t.lid, t.T_ent - 1 - lane) : -1;
    n_over = 0;
  }
  t.T_ent -= n_over;
  // tokens visible up to page v: entries up to v, whole pages, less the unseen tail of v itself
  t.V = 0;
  t.V_last = 0;
  t.V_first = 0;
  for (int32_t v = pg_lo; v <= pg_hi; ++v) {
    const int32_t whole = (t.T_ent + n_over - __builtin_popcountll(__ballot(e > v))) << lp;
    const bool held = __ballot(e == v) != 0;
    if (pg == v) t.V = whole - (held ? p.P - 1 - (int32_t)(a & (p.P - 1)) : 0);
    if (v == pg_lo) t.V_first = whole - (held ? p.P - 1 - (int32_t)(a_first & (p.P - 1)) : 0);
    if (v == pg_hi) t.V_last = whole - (held ? p.P - 1 - (int32_t)(a_last & (p.P - 1)) : 0);
  }
  t.T_ent = __builtin_amdgcn_readfirstlane(t.T_ent);
  t.V_last = __builtin_amdgcn_readfirstlane(t.V_last);
  t.V_first = __builtin_amdgcn_readfirstlane(t.V_first);
  return t;
}

// Splits cut the key tiles of a list of max_len entries, so that where a split starts is known before anything is
// read; what lies past the list, or past what the tile's rows see, is dropped.
struct GnRange { int32_t k0, k1; };
__device__ __forceinline__ GnRange gn_range(int32_t max_len, int lp, int32_t kt, int32_t split, int32_t n_split) {
  const int64_t n = (((int64_t)max_len << lp) + kt - 1) / kt;
  return {(int32_t)(n * split / n_split), (int32_t)(n * (split + 1) / n_split)};
}

// K / V tiles of a list, copied tile by tile in ascending order.  Every wave of a group moves RW rows of K and of V.
template <typename T, int D> struct GnStream {
  typedef Gn<T, D> X;
  typedef GnTiles<T, D> Y;
  int32_t base, p_cur, p_nxt;   // physical pages of the list entries base .. + 63 and of the next 64, one per lane
  int32_t last;                 // last entry with a page
  int64_t lane_off[Y::NI];      // this lane's row and granule, bytes from the wave's first row
  int64_t head_off;
  // one window of list entries; len is the host's bound, so entries past the list's own end may hold anything
  __device__ __forceinline__ int32_t window(const Params& p, int lid, int32_t len, int32_t at, int lane) const {
    int32_t l = at + lane < len ? list_at(p, lid, at + lane) : 0;
    l = l >= 0 && l < p.n ? l : 0;
    return p.page_table[l];
  }
  __device__ __forceinline__ void init(const Params& p, int lid, int32_t max_len, int g, int rb, int lane, int32_t first_tok, int lp) {
    const uint32_t lrow = lane / X::NG, pos = lane % X::NG;
#pragma unroll
    for (int k = 0; k < Y::NI; ++k) {
      const uint32_t row = k * X::RPI + lrow;
      lane_off[k] = (int64_t)row * p.pool_tok_stride * X::ES + ((pos ^ X::swz((rb * Y::RW + row) & 15)) << 4);   // (the swizzle sees rows modulo 16)
    }
    head_off = (int64_t)g * p.pool_head_stride * X::ES;
    base = __builtin_amdgcn_readfirstlane(first_tok >> lp);
    p_cur = window(p, lid, max_len, base, lane);
    p_nxt = window(p, lid, max_len, base + 64, lane);
  }
  __device__ __forceinline__ void copy(const Params& p, int lid, int32_t max_len, int rb, int lane, int lp, int32_t tile, uint32_t buf) {
    const int32_t tok = tile * Y::KT + rb * Y::RW;
    int32_t e = tok >> lp;
    e = __builtin_amdgcn_readfirstlane(e < last ? e : last);   // (rows past the last visible page are masked: any page of the list will do)
    if (e >= base + 64) {
      base += 64;
      p_cur = p_nxt;
      p_nxt = window(p, lid, max_len, base + 64, lane);
      wait_copies<0>();   // (here, once per 64 entries: a wait left to the compiler would stand in front of every tile)
    }
    const int32_t j = e - base;
    const int32_t ph = __builtin_amdgcn_readlane(j < 64 ? p_cur : p_nxt, j & 63);
    const int64_t o = ((int64_t)ph * p.pool_page_stride + (int64_t)(tok & (p.P - 1)) * p.pool_tok_stride) * X::ES + head_off;
    const unsigned char* k_src = (const unsigned char*)p.k_pool + o;
    const unsigned char* v_src = (const unsigned char*)p.v_pool + o;
    const uint32_t dst = buf + rb * Y::RW * X::RB;
#pragma unroll
    for (int k = 0; k < Y::NI; ++k) gn_copy16(k_src + lane_off[k], dst + 1024 * k);
#pragma unroll
    for (int k = 0; k < Y::NI; ++k) gn_copy16(v_src + lane_off[k], dst + Y::TILE + 1024 * k);
  }
};

// workgroup -> (KV head, row tile, split).  The head varies fastest: workgroups are dealt round-robin to the
// XCDs, so with 1, 2, 4 or 8 KV heads every head keeps to its own XCDs and their L2.
struct GnBlock { int g; int32_t tile, split; };
__device__ __forceinline__ GnBlock gn_block(const Params& p, int32_t b, int32_t tiles, int32_t n_split) {
  const int32_t rest = b / p.Hkv;
  return {b - rest * p.Hkv, tiles - 1 - rest / n_split, rest % n_split};   // late rows see more pages: they start first
}

// The key loop of forward and dQ: tiles kr of this wave's group.  compute(LDS offset of the tile inside the group's
// buffers -- a constant --, first list token, whether some row of the workgroup's tile may not see all of it).  APART: the tiles that
// every row sees have a loop of their own, without masks.
template <typename T, int D, int KH, bool APART, typename F>
__device__ __forceinline__ void gn_key_loop(const Params& p, const GnTile& t, GnStream<T, D>& ks, GnRange kr, GnRange other, int32_t max_len,
                                            int group, int rb, int lane, int lp, GnStay<T, D>& qs, F&& compute) {
  typedef GnTiles<T, D> Y;
  const int32_t n_kt = (t.V_last + Y::KT - 1) / Y::KT;   // (tiles past what the last row sees are dropped)
  const int32_t k1 = kr.k1 < n_kt ? kr.k1 : n_kt, mine = k1 - kr.k0;
  const int32_t theirs = (other.k1 < n_kt ? other.k1 : n_kt) - other.k0, steps = KH == 2 && theirs > mine ? theirs : mine;
  const uint32_t at = group * GnRow<T, D, KH>::GROUP;
  ks.last = t.T_ent - 1;
  wait_copies<0>();   // (every load so far, so that no wait for one of them is left inside the loop)
  qs.here();
  if (mine > 0) ks.copy(p, t.lid, max_len, rb, lane, lp, kr.k0, at);
  qs.template split<true>();   // (while the first tile is on its way)
  auto walk = [&](int32_t i0, const int32_t end, auto mask) __attribute__((always_inline)) {   // (i0 is even)
    for (; i0 < end; i0 += 2) {
#pragma unroll
      for (int b = 0; b < 2; ++b) {   // (unrolled: the buffer is a constant)
        const int32_t i = i0 + b;
        if (mask.value && i >= end) break;
        wait_copies<0>();
        __syncthreads();   // this tile is in LDS; nobody reads the one before it any more, whose buffer takes the next
        if (i + 1 < mine) ks.copy(p, t.lid, max_len, rb, lane, lp, kr.k0 + i + 1, at + (b ^ 1) * Y::BUF);
        if (!mask.value || i < mine) compute((uint32_t)(b * Y::BUF), (kr.k0 + i) * Y::KT, mask);
      }
    }
  };
  int32_t seen = 0;   // (the same for both groups)
  if constexpr (APART) {
    const int32_t all = t.V_first / Y::KT, k_hi = KH == 2 && other.k0 > kr.k0 ? other.k0 : kr.k0;
    seen = all - k_hi;
    seen = (seen < mine ? seen : mine) & ~1;
    if (KH == 2) seen = seen < theirs ? seen : theirs & ~1;
    seen = seen > 0 ? seen : 0;
    walk(0, seen, std::false_type());
  }
  walk(seen, steps, std::true_type());
}

// ---- values that are not finite -----------------------------------------------------------------
// The products multiply a token that a row does not see by a probability of 0, which makes a NaN where the token holds an
// infinity or a NaN.  So sums that are not finite are formed once more, by one wave over exactly what the row (or key) sees, in plain
// fp32.  Finite values pay one look at the sums: 32 or 64 instructions per wave.
template <int N> __device__ __forceinline__ bool gn_not_finite(const f32x16 (&v)[N]) {
  float z = 0.f;   // (0 times an infinity or a NaN is a NaN)
#pragma unroll
  for (int k = 0; k < N; ++k)
#pragma unroll
    for (int x = 0; x < 16; ++x) z = __builtin_fmaf(v[k][x], 0.f, z);
  return z != 0.f;
}
// The launch parameters (every kernel's first argument) read anew: held for this path they would be spilled in front of the main loops.
__device__ __forceinline__ const Params& gn_params_again() {
  auto args = __builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(args));
  return *(const Params*)args;
}
// lanes l and l + 32 hold one row or key: bit l of the result
__device__ __forceinline__ uint32_t gn_either_half(bool v) {
  const uint64_t b = __ballot(v);
  return (uint32_t)b | (uint32_t)(b >> 32);
}
__device__ __forceinline__ float gn_lane(float v, int lane) { return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(v), lane)); }
__device__ __forceinline__ int64_t gn_lane64(int64_t v, int lane) {
  return ((int64_t)__builtin_amdgcn_readlane((int32_t)(v >> 32), lane) << 32) | (uint32_t)__builtin_amdgcn_readlane((int32_t)v, lane);
}
// <a, b> of two rows of D elements
template <typename T, int D> __device__ __forceinline__ float gn_row_dot(const T* a, const T* b) {
  float c = 0.f;
#pragma unroll 2
  for (int j = 0; j < Gn<T, D>::NG; ++j) c = gn_dot<T>(reinterpret_cast<const u32x4_t*>(a)[j], reinterpret_cast<const u32x4_t*>(b)[j], c);
  return c;
}
// Delta of a row: as the dQ kernel left it, or (a backward in one launch) from O and dO
template <typename T, int D> __device__ __forceinline__ float gn_delta(const Params& p, int i, int h) {
  const int64_t off = (int64_t)i * p.q_tok_stride + (int64_t)h * p.q_head_stride;
  return p.delta ? p.delta[(int64_t)h * p.C + i] : gn_row_dot<T, D>((const T*)p.d_o + off, (const T*)p.o + off);
}
// acc += sum over the lanes x < cnt of w_x times row off_x of `rows` (elements), the lane's dims lane, lane + 64.  True: every
// dim is NaN and stays so (a row or key that sees a NaN mostly ends here after its first 64).
template <typename T, int D> __device__ __forceinline__ bool gn_add_rows(float (&acc)[D / 64], const T* rows, float w, int64_t off, int cnt, int lane) {
  for (int x = 0; x < cnt; ++x) {
    const float wx = gn_lane(w, x);
    const T* row = rows + gn_lane64(off, x);
#pragma unroll
    for (int k = 0; k < D / 64; ++k) acc[k] += wx * Elem<T>::load(row + 64 * k + lane);
  }
  return __all(D == 64 ? acc[0] != acc[0] : acc[0] != acc[0] && acc[D / 64 - 1] != acc[D / 64 - 1]);
}
// O of one row (ref: what its exponentials are relative to, times log2 e; scale: 1 / the sum of its probabilities), or dQ (ref: LSE times log2 e)
template <typename T, int D, bool DQ>
__device__ __forceinline__ void gn_redo_row(const Params& p, int g, int i, int h, int lp, int lane, float ref, float scale, float delta) {
  const int lid = list_id(p, g, i);
  const int64_t roff = (int64_t)i * p.q_tok_stride + (int64_t)h * p.q_head_stride, a = p.N - p.C + i;
  const T *q = (const T*)p.q + roff, *d_o = (const T*)p.d_o + roff;
  const int32_t n_ent = visible_len(p, lid, a >> lp, lane);
  int32_t V = n_ent << lp;   // list tokens that the row sees
  if (n_ent > 0 && list_at(p, lid, n_ent - 1) == (int32_t)(a >> lp)) V -= p.P - 1 - (int32_t)(a & (p.P - 1));
  if (ref != ref || delta != delta || scale != scale) {   // (all of the row is NaN)
    V = 0;
    scale = NAN;
  }
  const float c = p.sm_scale * 1.4426950408889634f;
  float acc[D / 64] = {};
  for (int32_t t0 = 0; t0 < V; t0 += 64) {
    float w = 0.f;
    int64_t off = 0;
    if (t0 + lane < V) {
      const int32_t t = t0 + lane;
      off = (int64_t)p.page_table[list_at(p, lid, t >> lp)] * p.pool_page_stride + (int64_t)g * p.pool_head_stride + (int64_t)(t & (p.P - 1)) * p.pool_tok_stride;
      w = __builtin_amdgcn_exp2f(__builtin_fmaf(gn_row_dot<T, D>(q, (const T*)p.k_pool + off), c, -ref));
      if (DQ) w *= gn_row_dot<T, D>(d_o, (const T*)p.v_pool + off) - delta;
      else w *= scale;   // (before the sum: the largest w may be 2^8, times a value near the edge)
    }
    if (gn_add_rows<T, D>(acc, (const T*)(DQ ? p.k_pool : p.v_pool), w, off, V - t0 < 64 ? V - t0 : 64, lane)) break;
  }
  T* dst = (T*)(DQ ? p.d_q : p.o) + roff;
#pragma unroll
  for (int k = 0; k < D / 64; ++k) Elem<T>::store(dst + 64 * k + lane, DQ || V == 0 ? acc[k] * scale : acc[k]);
}
// dK (or dV) of token t of owned page e into the pool
template <typename T, typename TG, int D> __device__ __forceinline__ void gn_redo_key(const Params& p, int g, int32_t e, int32_t t, bool is_dk, int lp, int lane) {
  const int64_t l = owned_at(p, g, e), pos = (l << lp) + t, first_q = p.N - p.C;
  const int64_t koff = (int64_t)p.page_table[l] * p.pool_page_stride + (int64_t)g * p.pool_head_stride + (int64_t)t * p.pool_tok_stride;
  const int32_t r_key = pos > first_q ? (int32_t)(pos - first_q) * p.G : 0, rpq = p.P * p.G;   // rows before r_key do not see it
  const int32_t* inv = p.qp ? p.inv_off + (int64_t)g * (p.un_stride + 1) + e : nullptr;
  const int32_t n_seg = p.qp ? inv[1] - inv[0] : 1;
  const float c = p.sm_scale * 1.4426950408889634f;
  float acc[D / 64] = {};
  bool done = false;
  for (int32_t seg = 0; seg < n_seg && !done; ++seg) {   // the chunk's rows, or those of every query page that lists the page
    int32_t r0 = 0, end = p.C * p.G;
    if (p.qp) {
      r0 = p.inv_qp[(int64_t)g * p.m * p.sel_stride + inv[0] + seg] * rpq;
      end = r0 + rpq;
    }
    for (r0 = r0 < r_key ? r_key : r0; r0 < end && !done; r0 += 64) {
      float w = 0.f;
      int64_t off = 0;
      if (r0 + lane < end) {
        const int32_t i = (int32_t)div_g(p, (uint32_t)(r0 + lane)), h = g * p.G + (r0 + lane - i * p.G);
        off = (int64_t)i * p.q_tok_stride + (int64_t)h * p.q_head_stride;
        w = __builtin_amdgcn_exp2f(__builtin_fmaf(gn_row_dot<T, D>((const T*)p.q + off, (const T*)p.k_pool + koff), c, -(p.lse[(int64_t)h * p.C + i] * 1.4426950408889634f)));
        if (is_dk) {
          w *= gn_row_dot<T, D>((const T*)p.d_o + off, (const T*)p.v_pool + koff) - gn_delta<T, D>(p, i, h);
        }
      }
      done = gn_add_rows<T, D>(acc, (const T*)(is_dk ? p.q : p.d_o), w, off, end - r0 < 64 ? end - r0 : 64, lane);
    }
  }
  TG* dst = (TG*)(is_dk ? p.dk_pool : p.dv_pool) + koff;
#pragma unroll
  for (int k = 0; k < D / 64; ++k)
    Elem<TG>::store(dst + 64 * k + lane, Elem<TG>::load(dst + 64 * k + lane) + acc[k] * (is_dk ? p.sm_scale : 1.f));
}

// ---- forward ----------------------------------------------------------------------------------
// Where a running maximum starts: finite, also as a logit, because a row that has seen nothing yet forms (-inf - m) c; below
// every product that a float holds as a logit of this scale.
__device__ __forceinline__ float gn_lowest(const Params& p) { return -1e38f / fmaxf(1.f, p.sm_scale); }
// The reference of a row's exponentials after products of at most mx (and m_run before).  It stays where it is until a product lies GN_LAZY binary orders above it: O, which
// follows every change, is then rescaled once or twice instead of in most tiles (64 instructions in front of each product at head dim 128).  fp32 probabilities of up
// to 2^8 keep as many bits as those of up to 1; bf16 ones are exact where they are 1, and keep the largest product (fwd_generic_kernel).  fp32,
// 28 / 4 heads, 20 pages of 128: pass 420.9 -> 414.3 us; 8 / 2 heads bf16, 41 pages of 64: 112.3 -> 111.7.
constexpr float GN_LAZY = 8.f;
__device__ __forceinline__ float gn_reference(float m_run, float mx, float c) {
  const float m = fmaxf(m_run, half_max(mx));
  return (m - m_run) * fabsf(c) > GN_LAZY ? m : m_run;
}
// log-sum-exp of a row: m the reference, l the sum of exponentials relative to it
__device__ __forceinline__ float gn_lse(const Params& p, float m, float l) {
  // As a sum of m's share, the exponent of l times ln 2 (in two parts, the first of which times an exponent is exact) and the logarithm of l's fraction, rounded
  // once: the backward's probabilities have the relative error that LSE has as a difference.  Rounded at every step (28 / 4 heads fp32, 20 pages, x 1e-7): LSE 0.47, dK
  // 7.6, dV 7.7.
  const float f = __builtin_amdgcn_frexp_mantf(l), e = (float)__builtin_amdgcn_frexp_expf(l);
  const float a = m * p.sm_scale, b = e * 0.693145751953125f, s = a + b, t = s - a;
  const float low = ((a - (s - t)) + (b - t)) + __builtin_fmaf(m, p.sm_scale, -a);
  return s + (low + __builtin_fmaf(e, 1.4286068203e-6f, __builtin_amdgcn_logf(f) * 0.6931471805599453f));
}

// n_split > 1: O (not normalised) and {running maximum of the products, sum} of every row go to part[split][block] and
// part_ml[split][block][32], which the combine kernel merges.
template <typename T, int D, int KH, int NT>
__global__ __launch_bounds__(256 * KH, 2) void fwd_generic_kernel(Params p, int32_t tiles, int32_t n_split, int lp, int32_t max_len,
                                                                  float* __restrict__ part, float2* __restrict__ part_ml) {
  typedef Gn<T, D> X;
  typedef GnTiles<T, D> Y;
  extern __shared__ __align__(16) unsigned char smem[];
  const int lane = threadIdx.x & 63, hh = lane >> 5, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), rb = wave & 3, group = wave >> 2;
  const GnBlock b = gn_block(p, blockIdx.x, tiles, n_split);
  const GnRange kr = gn_range(max_len, lp, Y::KT, KH * b.split + group, KH * n_split);
  const GnRange other = gn_range(max_len, lp, Y::KT, KH * b.split + (KH - 1 - group), KH * n_split);
  const GnTile t = gn_tile(p, b.g, b.tile, rb, lane, lp, max_len);
  GnStream<T, D> ks;
  ks.init(p, t.lid, max_len, b.g, rb, lane, kr.k0 * Y::KT, lp);

  GnStay<T, D> qs;
  const int64_t roff = (int64_t)t.i * p.q_tok_stride + (int64_t)t.h * p.q_head_stride;
  qs.at((const T*)p.q + roff, hh);
#pragma unroll
  for (int j = 0; j < X::NJ; ++j) qs.load(j);

  f32x16 of[X::DB];
  gn_zero(of);
  float m_run = gn_lowest(p), l_run = 0.f;
  [[maybe_unused]] const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};   // (NT = 1: the row sum is that of the rounded probabilities)
  const float c = p.sm_scale * 1.4426950408889634f;
  GnAddr<T, D> ad;
  ad.init(lane, group * GnRow<T, D, KH>::GROUP);
  const int32_t V_min = __builtin_amdgcn_readfirstlane(t.V), V_max = __builtin_amdgcn_readlane(t.V, 31);

  // One tile: S of its blocks, one softmax step over all of them, then O.  The exponentials of a second block
  // run between the matrix instructions of the first block's product.
  gn_key_loop<T, D, KH, false>(p, t, ks, kr, other, max_len, group, rb, lane, lp, qs, [&](const uint32_t at, const int32_t t0, auto) __attribute__((always_inline)) {
    if (!t.active || t0 >= V_max) return;   // (wave-uniform)
    constexpr int NP = GnAddr<T, D>::NP;
    ad.anew();
    GnSum<T> sums[Y::U];
#pragma unroll
    for (int u = 0; u < Y::U; ++u) sums[u].zero();
    gn_pipeline<Y::U * X::NJ, GN_BATCH<T, D>>(
        [&](const int i) __attribute__((always_inline)) { return ad.row_frag(i % X::NJ, at + 32 * (i / X::NJ) * X::RB); },
        [&](const int i, const u32x4_t& f) __attribute__((always_inline)) { sums[i / X::NJ].step(i % X::NJ, f, qs); });
    f32x16 s[Y::U];
#pragma unroll
    for (int u = 0; u < Y::U; ++u) {
      sums[u].template close<true>(qs, [&](const int j) __attribute__((always_inline)) { return ad.row_frag(j, at + 32 * u * X::RB); });
      s[u] = sums[u].v[0];
    }
    if (t0 + Y::KT > V_min) {
      const int32_t rel = t.V - t0 - 4 * hh;
#pragma unroll
      for (int u = 0; u < Y::U; ++u)
#pragma unroll
        for (int x = 0; x < 16; ++x)
          if (32 * u + 8 * (x >> 2) + (x & 3) >= rel) s[u][x] = -INFINITY;
    }
    // Probabilities are relative to a running maximum: of the tile, or (one bf16 term) of each block of 32 keys, as in the kernel
    // that this one stands in for.  The key that sets a maximum has a probability of 1, which bf16 holds exactly.  Error
    // against 64 bits, 28 / 4 heads, chunk 1536, 16 pages: one maximum per 64 keys O 2.191e-3, LSE 1.046e-5, one per 32 (and the
    // other kernel) 2.182e-3, 1.035e-5; it costs 1 to 2 us of the 54 of a chunk of one page against 65 pages.
    constexpr int REFS = NT == 1 ? Y::U : 1;
    float alpha[REFS], mc[REFS];
#pragma unroll
    for (int k = 0; k < REFS; ++k) {
      float mx = s[k][0];
#pragma unroll
      for (int u = k; u < (REFS == 1 ? Y::U : k + 1); ++u)
#pragma unroll
        for (int x = u == k; x < 16; ++x) mx = fmaxf(mx, s[u][x]);
      const float m_new = X::BF && NT == 1 ? fmaxf(m_run, half_max(mx)) : gn_reference(m_run, mx, c);
      alpha[k] = __builtin_amdgcn_exp2f((m_run - m_new) * c);
      mc[k] = m_new * c;
      m_run = m_new;
    }
    auto rescale = [&](const int k) __attribute__((always_inline)) {
      if (__any(alpha[k] != 1.f)) {
#pragma unroll
        for (int db = 0; db < X::DB; ++db)
#pragma unroll
          for (int x = 0; x < 16; ++x) of[db][x] *= alpha[k];
      }
    };
    rescale(0);
    l_run *= alpha[0];
    GnP<T, NT> pr[Y::U];
    auto exps = [&](const int u, const int x) __attribute__((always_inline)) {   // registers x, x + 1
      const float ref = mc[REFS == 1 ? 0 : u];
      const float a = __builtin_amdgcn_exp2f(__builtin_fmaf(s[u][x], c, -ref)), b2 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[u][x + 1], c, -ref));
      pr[u].set2(x, a, b2);
      if constexpr (X::BF && NT == 1) l_run = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pr[u].w[0][x >> 1]), ones, l_run, false);
      else l_run += a + b2;
    };
#pragma unroll
    for (int x = 0; x < 16; x += 2) exps(0, x);
    if constexpr (REFS == 2) l_run *= alpha[1];
    gn_pipeline<Y::U * NP, GN_BATCH<T, D>>(
        [&](const int i) __attribute__((always_inline)) { return ad.tr_frag(i % NP, at + Y::TILE + 32 * (i / NP) * X::RB); },
        [&](const int i, const u32x4_t& f) __attribute__((always_inline)) {
          if (REFS == 2 && i == NP) rescale(REFS - 1);
          gn_tr_mma<T, D, NT>(i % NP, f, pr[i / NP], of);
          if (i < NP && Y::U == 2) {   // 16 exponentials over NP instructions (4, 8 or 16)
            if (NP == 4) exps(Y::U - 1, 4 * i);
            if (NP <= 8) exps(Y::U - 1, NP == 4 ? 4 * i + 2 : 2 * i);
            if (NP == 16 && !(i & 1)) exps(Y::U - 1, i);
          }
        });
  });

  float l_tot = half_sum(l_run);
  if constexpr (KH == 2) {   // the second group's results through LDS
    float* mo = reinterpret_cast<float*>(smem) + rb * (D * 32) + lane;
    float2* ml = reinterpret_cast<float2*>(smem + GN_ROWS * D * 4) + rb * 64 + lane;
    __syncthreads();
    if (group == 1) {
#pragma unroll
      for (int k = 0; k < X::DB * 16; ++k) mo[64 * k] = of[k >> 4][k & 15];
      *ml = make_float2(m_run, l_tot);
    }
    __syncthreads();
    if (group == 1) return;
    const float2 o = *ml;
    const float M = fmaxf(m_run, o.x), w0 = __builtin_amdgcn_exp2f((m_run - M) * c), w1 = __builtin_amdgcn_exp2f((o.x - M) * c);
    m_run = M;
    l_tot = l_tot * w0 + o.y * w1;
#pragma unroll
    for (int k = 0; k < X::DB * 16; ++k) of[k >> 4][k & 15] = of[k >> 4][k & 15] * w0 + mo[64 * k] * w1;
  }
  if (n_split > 1) {
    const int64_t at = (int64_t)b.split * p.Hkv * tiles * 4 + t.block;
    if (!t.active) return;
    part_store<T, D>(part, at, lane, of, 1.f);
    if (hh == 0) part_ml[at * 32 + lane] = make_float2(l_tot > 0.f ? m_run : -INFINITY, l_tot);
  } else {
    const float inv = 1.f / l_tot;
    uint32_t bad = gn_either_half(t.valid && gn_not_finite(of));
    if (t.valid && !((bad >> (lane & 31)) & 1)) {
      T* dst = (T*)p.o + roff;
      part_emit<T, D>(of, hh, [&](int d, float v0, float v1, float v2, float v3) { part_store4<T>(dst + d, v0 * inv, v1 * inv, v2 * inv, v3 * inv); });
    }
    if (t.valid && hh == 0) p.lse[(int64_t)t.h * p.C + t.i] = gn_lse(p, m_run, l_tot);
    for (; bad; bad &= bad - 1) {
      const int x = __builtin_ctz(bad);
      gn_redo_row<T, D, false>(gn_params_again(), b.g, __builtin_amdgcn_readlane(t.i, x), __builtin_amdgcn_readlane(t.h, x), lp, lane, gn_lane(m_run * c, x), gn_lane(inv, x), 0.f);
    }
  }
}

// Combine kernels: a workgroup of NW waves takes a block of 32 rows, wave w the groups w, w + NW, ..  The sums go through LDS, so that the
// results leave in whole rows instead of the register order of the partials.
template <int D, int NW = 4> constexpr int GN_GW = D / 8 / NW;   // groups per wave
// in: the sums of this thread's groups; then f(k, row, dim, value) for the row pieces this thread writes, piece k = float4
// k * 64 NW + thread of the block.  redo: rows whose sums are not finite are left out; returns them, a bit each.
template <int D> struct GnRowsLds { float4 v[8 * D]; uint32_t bad[8]; };
template <typename L, int D, int NW = 4, typename F> __device__ __forceinline__ uint32_t gn_rows_out(GnRowsLds<D>& lds, const float4 (&v)[GN_GW<D, NW>], bool redo, F&& f) {
  auto& sh = lds.v;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, r = lane & 31;
  constexpr int GPR = D / 4;   // float4s per row
#pragma unroll
  for (int j = 0; j < GN_GW<D, NW>; ++j) sh[r * GPR + ((part_group_dim<L, D>(wave + NW * j, lane >> 5) >> 2) ^ (r & 15))] = v[j];
  float z = 0.f;
#pragma unroll
  for (int j = 0; j < GN_GW<D, NW>; ++j) z = __builtin_fmaf(v[j].x, 0.f, __builtin_fmaf(v[j].y, 0.f, __builtin_fmaf(v[j].z, 0.f, __builtin_fmaf(v[j].w, 0.f, z))));
  const uint32_t mine = gn_either_half(redo && z != 0.f);
  if (lane == 0) lds.bad[wave] = mine;
  __syncthreads();
  uint32_t bad = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) bad |= lds.bad[w];
#pragma unroll
  for (int k = 0; k < GN_GW<D, NW>; ++k) {
    const int e = k * 64 * NW + threadIdx.x, row = e / GPR, c = e % GPR;
    if (!((bad >> row) & 1)) f(k, row, 4 * c, sh[row * GPR + (c ^ (row & 15))]);
  }
  return __builtin_amdgcn_readfirstlane(bad);
}
// row `row` of a block -> chunk token and query head; false past the last row
__device__ __forceinline__ bool gn_out_row(const Params& p, int32_t tiles, int64_t block, int row, int& i, int& h) {
  const int64_t tg = block >> 2;
  const int32_t g = (int32_t)(tg / tiles), tile = (int32_t)(tg - (int64_t)g * tiles);
  int32_t r = ((int32_t)block & 3) * 32 + row, end;
  if (!p.qp) {
    r += tile * GN_ROWS;
    end = p.C * p.G;
  } else {
    const int32_t rpq = p.P * p.G, tpq = (rpq + GN_ROWS - 1) / GN_ROWS, tau = tile / tpq;
    r += tau * rpq + (tile - tau * tpq) * GN_ROWS;
    end = (tau + 1) * rpq;
  }
  if (r >= end) return false;
  i = (int)div_g(p, (uint32_t)r);
  h = g * p.G + (r - i * p.G);
  return true;
}
__device__ __forceinline__ float4 gn_load_part(const float* part, int64_t at) {
  typedef float f32x4_t __attribute__((ext_vector_type(4)));   // (read once: non-temporal, so that they push nothing else out of the caches)
  const f32x4_t v = __builtin_nontemporal_load(reinterpret_cast<const f32x4_t*>(part) + at);
  return make_float4(v.x, v.y, v.z, v.w);
}
// sums of n partials `step` float4s apart for the thread's groups of a block, at most four of each in flight, added in order
// `meanwhile` runs once, while the first of them are on their way.
template <int D, int NW, int N, typename F>
__device__ __forceinline__ void gn_add_parts(const float* part, int64_t at, int64_t step, float4 (&a)[GN_GW<D, NW>], F&& meanwhile) {
  float4 v[GN_GW<D, NW>][N];
#pragma unroll
  for (int u = 0; u < N; ++u)
#pragma unroll
    for (int j = 0; j < GN_GW<D, NW>; ++j) v[j][u] = gn_load_part(part, at + j * 64 * NW + u * step);
  __builtin_amdgcn_sched_barrier(0);
  meanwhile();
#pragma unroll
  for (int u = 0; u < N; ++u)
#pragma unroll
    for (int j = 0; j < GN_GW<D, NW>; ++j) { a[j].x += v[j][u].x; a[j].y += v[j][u].y; a[j].z += v[j][u].z; a[j].w += v[j][u].w; }
}
template <int D, int NW, typename F>
__device__ __forceinline__ void gn_sum_parts(const float* part, int64_t block, int64_t step, int n, float4 (&a)[GN_GW<D, NW>], F&& meanwhile) {
  int64_t at = (block * (D / 8) + (threadIdx.x >> 6)) * 64 + (threadIdx.x & 63);
#pragma unroll
  for (int j = 0; j < GN_GW<D, NW>; ++j) a[j] = make_float4(0.f, 0.f, 0.f, 0.f);
  auto nothing = [] {};
  const int first = n & 3;   // (the odd ones first)
  if (first == 3) gn_add_parts<D, NW, 3>(part, at, step, a, meanwhile);
  else if (first == 2) gn_add_parts<D, NW, 2>(part, at, step, a, meanwhile);
  else if (first == 1) gn_add_parts<D, NW, 1>(part, at, step, a, meanwhile);
  else gn_add_parts<D, NW, 4>(part, at, step, a, meanwhile);
  for (int done = first ? first : 4; done < n; done += 4) gn_add_parts<D, NW, 4>(part, at + done * step, step, a, nothing);
}

// O = sum of the splits' O rescaled to the common maximum / sum of their l.  L: the element type in whose register order the partial sums lie.
// What bounds it is how much a compute unit has in flight: eight waves with eight splits each.  Against four waves with four splits, whole passes: 28 / 4
// heads, one page, 9 splits (112 blocks) 52.5 -> 51.8 us; 14 / 2 heads, two pages 54.6 -> 53.8; at 448
// blocks the same.
constexpr int COMBINE_WAVES = 8;
template <typename T, int D, typename L = T>
__global__ __launch_bounds__(64 * COMBINE_WAVES) void fwd_combine_kernel(Params p, int32_t tiles, int32_t n_split, const float* __restrict__ part,
                                                          const float2* __restrict__ part_ml, int lp) {
  __shared__ GnRowsLds<D> sh;
  constexpr int NW = COMBINE_WAVES, GW = GN_GW<D, NW>, N = 8;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t block = blockIdx.x, blocks = (int64_t)p.Hkv * tiles * 4;
  const int64_t at = (block * (D / 8) + wave) * 64 + lane;
  const float c = p.sm_scale * 1.4426950408889634f;
  float M = gn_lowest(p), l_sum = 0.f;   // (a split that saw nothing of the row holds -inf and 0)
  float4 acc[GW];
#pragma unroll
  for (int j = 0; j < GW; ++j) acc[j] = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int s0 = 0; s0 < n_split; s0 += N) {   // N splits in flight
    float2 ml[N];
    float4 v[GW][N];
#pragma unroll
    for (int u = 0; u < N; ++u) {
      ml[u] = make_float2(-INFINITY, 0.f);
      if (s0 + u < n_split) {
        ml[u] = part_ml[((s0 + u) * blocks + block) * 32 + (lane & 31)];
#pragma unroll
        for (int j = 0; j < GW; ++j) v[j][u] = gn_load_part(part, at + j * 64 * NW + (s0 + u) * blocks * (D / 8) * 64);
      }
    }
#pragma unroll
    for (int u0 = 0; u0 < N; u0 += 4) {   // (added four at a time)
      if (s0 + u0 >= n_split) break;
      const float m_new = fmaxf(fmaxf(fmaxf(ml[u0].x, ml[u0 + 1].x), fmaxf(ml[u0 + 2].x, ml[u0 + 3].x)), M);
      const float w0 = __builtin_amdgcn_exp2f((M - m_new) * c);
      M = m_new;
      l_sum *= w0;
#pragma unroll
      for (int j = 0; j < GW; ++j) { acc[j].x *= w0; acc[j].y *= w0; acc[j].z *= w0; acc[j].w *= w0; }
#pragma unroll
      for (int u = u0; u < u0 + 4; ++u)
        if (s0 + u < n_split) {
          const float w = __builtin_amdgcn_exp2f((ml[u].x - m_new) * c);
          l_sum += ml[u].y * w;
#pragma unroll
          for (int j = 0; j < GW; ++j) { acc[j].x += v[j][u].x * w; acc[j].y += v[j][u].y * w; acc[j].z += v[j][u].z * w; acc[j].w += v[j][u].w * w; }
        }
    }
  }
  const float inv = 1.f / l_sum, by = sizeof(L) != sizeof(T) ? inv * GN_LOWER : inv;   // (sums of lifted values)
#pragma unroll
  for (int j = 0; j < GW; ++j) { acc[j].x *= by; acc[j].y *= by; acc[j].z *= by; acc[j].w *= by; }
  int i, h;
  uint32_t bad = gn_rows_out<L, D, NW>(sh, acc, true, [&](int, int row, int d, const float4& r) __attribute__((always_inline)) {
    if (gn_out_row(p, tiles, block, row, i, h))
      part_store4<T>((T*)p.o + (int64_t)i * p.q_tok_stride + (int64_t)h * p.q_head_stride + d, r.x, r.y, r.z, r.w);
  });
  if (threadIdx.x < 32 && gn_out_row(p, tiles, block, threadIdx.x, i, h))
    p.lse[(int64_t)h * p.C + i] = gn_lse(p, M, l_sum);
  for (bad &= 0xfu << (4 * wave); bad; bad &= bad - 1) {   // (four rows per wave)
    const int x = __builtin_ctz(bad);
    if (gn_out_row(p, tiles, block, x, i, h))
      gn_redo_row<T, D, false>(gn_params_again(), h / p.G, i, h, lp, lane, gn_lane(M * c, x), gn_lane(inv, x), 0.f);
  }
}

// ---- forward of fp32 tensors on the bf16 matrix pipe ---------------------------------------------
template <int D> struct GnF3 {
  typedef Gn<bf16_t, D> X;
  static constexpr int TERM = 32 * X::RB, V = 3 * TERM, TILE = 6 * TERM;   // 32 keys: K0 K1 K2 V0 V1 V2, in the order of the LDS tile
  static constexpr int NI = V / 1024 / 4, LDS = 3 * V;   // copies of K or V per wave; LDS: K twice, V once
};
template <int D> __device__ __forceinline__ void gn_store_terms(unsigned char* dst, const u32x4_t (&v)[2]) {
  u32x4_t t[3];
  gn_load_terms<false>(v[0], v[1], t);
#pragma unroll
  for (int k = 0; k < 3; ++k) *reinterpret_cast<u32x4_t*>(dst + k * GnF3<D>::TERM) = t[k];
}
static inline int32_t gn_f3_tiles(const Params& p, int32_t max_len) { return (int32_t)(((int64_t)max_len * p.P + 31) / 32); }

// The terms of the listed keys (V lifted) of n_tiles tiles from t0 on, [KV head][tile of 32 list tokens][TILE]; zeros past the list.  odd[KV head][tile][4]: a byte per
// wave, whether a key of the tile is not finite.
template <int D>
__global__ __launch_bounds__(256) void kv_terms_kernel(Params p, int32_t t0, int32_t n_tiles, int lp, unsigned char* __restrict__ img, unsigned char* __restrict__ odd) {
  typedef GnF3<D> F;
  constexpr int NG = F::X::NG;
  float z = 0.f;   // (0 times an infinity or a NaN is a NaN)
  const int32_t kt = blockIdx.x / p.Hkv, g = blockIdx.x - kt * p.Hkv, len = list_len(p, g);
  unsigned char* out = img + ((int64_t)g * n_tiles + kt) * F::TILE;
#pragma unroll
  for (int x = 0; x < 2 * 32 * NG / 256; ++x) {
    const int gi = threadIdx.x + 256 * x, is_v = gi / (32 * NG), r = gi / NG % 32, c = gi % NG;
    const int32_t tok = 32 * (t0 + kt) + r, e = tok >> lp;
    u32x4_t v[2] = {};
    if (e < len) {
      const int64_t at = (int64_t)p.page_table[list_at(p, g, e)] * p.pool_page_stride + (int64_t)g * p.pool_head_stride + (int64_t)(tok & (p.P - 1)) * p.pool_tok_stride + 8 * c;
      const u32x4_t* src = reinterpret_cast<const u32x4_t*>((const float*)(is_v ? p.v_pool : p.k_pool) + at);
      v[0] = src[0];
      v[1] = src[1];
    }
    if (!is_v) {
#pragma unroll
      for (int k = 0; k < 8; ++k) z = __builtin_fmaf(__uint_as_float(v[k >> 2][k & 3]), 0.f, z);
    } else {
      gn_lift(v[0]);
      gn_lift(v[1]);
    }
    gn_store_terms<D>(out + is_v * F::V + r * F::X::RB + ((c ^ F::X::swz(r)) << 4), v);
  }
  const bool any = __any(z != 0.f);
  if ((threadIdx.x & 63) == 0) odd[((int64_t)g * n_tiles + kt) * 4 + (threadIdx.x >> 6)] = any;
}
// f(i, operand of three terms) for i = 0 .. N - 1: the next operand is fetched while one computes
template <int N, typename L, typename M> __device__ __forceinline__ void gn_terms_pipeline(L&& load, M&& use) {
  u32x4_t fr[2][3];
#pragma unroll
  for (int t = 0; t < 3; ++t) fr[0][t] = load(0, t);
#pragma unroll
  for (int i = 0; i < N; ++i) {
    if (i + 1 < N) {
#pragma unroll
      for (int t = 0; t < 3; ++t) fr[(i + 1) & 1][t] = load(i + 1, t);
      __builtin_amdgcn_sched_barrier(0);
    }
    use(i, fr[i & 1]);
    __builtin_amdgcn_sched_barrier(0);
  }
}

// fp32 forward, one list per KV head: O = softmax(Q K^T) V of 128 rows and a range of tiles of 32 keys.  Two workgroups per compute unit, whose barriers
// are their own: the vector work of one (softmax, terms of P) runs beside the matrix instructions of the other.  S is summed in two accumulators, the
// products of the first terms apart from the small ones, so that fewer sums are rounded at its full size (O against 64 bits 4.2e-7 instead of
// 6.0e-7; on the fp32 pipe 7.3e-7).  28 / 4 heads, chunk 512, 20 pages of 128: the forward with layout and combine 187 us on the fp32 pipe, 148 with S
// alone in terms, 118 here: 1.0 PFLOP/s of bf16 instructions, the matrix pipe busy for 61 % of the cycles of the compute units in use, waves waiting 13 %.  256 rows per workgroup, half of
// the copies: 2 to 6 % faster where the chip is full, up to 25 % slower where it is not.
template <int D, bool FIRST>
__global__ __launch_bounds__(256, 2) void fwd_terms_kernel(Params p, int32_t tiles, int32_t n_split, int lp, int32_t max_len, int32_t t0, int32_t n_tiles, bool last, const unsigned char* __restrict__ img,
                                                           const int32_t* __restrict__ odd_tiles, float* __restrict__ part, float2* __restrict__ part_ml) {
  typedef GnF3<D> F;
  typedef Gn<bf16_t, D> X;
  extern __shared__ __align__(16) unsigned char smem[];
  const int lane = threadIdx.x & 63, hh = lane >> 5, rb = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const GnBlock b = gn_block(p, blockIdx.x, tiles, n_split);
  // this launch: tiles t0 .. t0 + n_tiles - 1 of the list, which the splits share
  const GnRange kr = {t0 + (int32_t)((int64_t)n_tiles * b.split / n_split), t0 + (int32_t)((int64_t)n_tiles * (b.split + 1) / n_split)};
  // whether the wave meets a value that is not finite: a key's, or (below) its row's.  (Looked up once: 16 instructions per tile were 2 to 7 % of the kernel.)
  odd_tiles += (int64_t)b.g * n_tiles - t0;
  int32_t odd_key = kr.k0 + lane < kr.k1 ? odd_tiles[kr.k0 + lane] : 0;
  const GnTile t = gn_tile(p, b.g, b.tile, rb, lane, lp, max_len);
  const bool active = t.active;

  GnStay<float, D> qs;
  qs.at((const float*)p.q + (int64_t)t.i * p.q_tok_stride + (int64_t)t.h * p.q_head_stride, hh);
#pragma unroll
  for (int j = 0; j < GnStay<float, D>::NJ; ++j) qs.load(j);
  qs.template split<false>();
  for (int32_t kt = kr.k0 + 64 + lane; kt < kr.k1; kt += 64) odd_key |= odd_tiles[kt];
  const bool odd = __any(odd_key != 0 || !qs.finite());
  f32x16 of[X::DB];
  gn_zero(of);
  float m_run = gn_lowest(p), l_run = 0.f;
  if (!FIRST && active) {   // on from where the launch before left the split
    const int64_t at = (((int64_t)b.split * p.Hkv + b.g) * tiles + b.tile) * 4 + rb;
    const float4* src = reinterpret_cast<const float4*>(part) + at * (D / 8) * 64 + lane;
#pragma unroll
    for (int k = 0; k < D / 8; ++k) {
      const float4 v = src[64 * k];
      f32x16& o = of[k >> 2];
      const int a = 4 * (k & 3);
      o[a] = v.x; o[a + 1] = v.y; o[a + 2] = v.z; o[a + 3] = v.w;
    }
    const float2 ml = part_ml[at * 32 + (lane & 31)];
    m_run = fmaxf(m_run, ml.x);
    l_run = hh ? 0.f : ml.y;
  }
  const float c = p.sm_scale * 1.4426950408889634f;
  GnAddr<bf16_t, D> ad;
  ad.init(lane, 0);
  uint32_t row0 = ad.row[0];
  const int32_t V_min = __builtin_amdgcn_readfirstlane(t.V), V_max = __builtin_amdgcn_readlane(t.V, 31);
  const int32_t n_kt = (t.V_last + 31) / 32, k1 = kr.k1 < n_kt ? kr.k1 : n_kt;
  const unsigned char* src = img + ((int64_t)b.g * n_tiles - t0) * F::TILE + rb * F::NI * 1024 + lane * 16;
  auto copy = [&](const int32_t kt, const uint32_t which, const uint32_t dst) __attribute__((always_inline)) {   // which: 0 or F::V
#pragma unroll
    for (int k = 0; k < F::NI; ++k) gn_copy16(src + (int64_t)kt * F::TILE + which + 1024 * k, dst + rb * F::NI * 1024 + 1024 * k);
  };
  GnP<bf16_t, 3> pr;
  auto scores = [&](const uint32_t at, const int32_t t0) __attribute__((always_inline)) {
    f32x16 s[2];
    gn_zero(s);
    asm volatile("" : "+v"(row0));   // (the addresses of the k-steps are formed from one register: kept apart, they would be spilled)
    gn_terms_pipeline<X::NJ>([&](const int j, const int k) __attribute__((always_inline)) {
                               return *(__attribute__((address_space(3))) const u32x4_t*)((row0 ^ (uint32_t)(j << 5)) + (at + k * F::TERM));
                             },
                             [&](const int j, const u32x4_t (&f)[3]) __attribute__((always_inline)) { gn_mma_terms(f, qs.t[j][0], qs.t[j][1], qs.t[j][2], s[1], s[0]); });
#pragma unroll
    for (int x = 0; x < 16; ++x) s[1][x] += s[0][x];
    if (t0 + 32 > V_min || odd) {   // (one branch for both)
      const int32_t rel = t.V - t0 - 4 * hh;
#pragma unroll
      for (int x = 0; x < 16; ++x) {
        // the small products of an infinity are infinities of either sign or (0 times infinity) NaN; that of the first terms is what the values give
        s[1][x] = fabsf(s[1][x]) < INFINITY ? s[1][x] : s[0][x];
        if (8 * (x >> 2) + (x & 3) >= rel) s[1][x] = -INFINITY;
      }
    }
    float mx = s[1][0];
#pragma unroll
    for (int x = 1; x < 16; ++x) mx = fmaxf(mx, s[1][x]);
    const float m_new = gn_reference(m_run, mx, c), alpha = __builtin_amdgcn_exp2f((m_run - m_new) * c), mc = m_new * c;
    m_run = m_new;
    if (__any(alpha != 1.f)) {
#pragma unroll
      for (int db = 0; db < X::DB; ++db)
#pragma unroll
        for (int x = 0; x < 16; ++x) of[db][x] *= alpha;
    }
    l_run *= alpha;
#pragma unroll
    for (int x = 0; x < 16; x += 2) {
      const float a = __builtin_amdgcn_exp2f(__builtin_fmaf(s[1][x], c, -mc)), b2 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[1][x + 1], c, -mc));
      pr.set2(x, a, b2);
      l_run += a + b2;
    }
  };
  auto output = [&]() __attribute__((always_inline)) {
    gn_terms_pipeline<2 * X::DB>([&](const int v, const int k) __attribute__((always_inline)) { return ad.tr_frag(v, 2 * F::V + k * F::TERM); },
                                 [&](const int v, const u32x4_t (&f)[3]) __attribute__((always_inline)) {
                                   const int u = v / X::DB;
                                   u32x4_t w[3];
#pragma unroll
                                   for (int k = 0; k < 3; ++k) w[k] = u32x4_t{pr.w[k][4 * u], pr.w[k][4 * u + 1], pr.w[k][4 * u + 2], pr.w[k][4 * u + 3]};
                                   gn_mma_terms(f, w[0], w[1], w[2], of[v % X::DB], of[v % X::DB]);
                                 });
  };
  wait_copies<0>();
  if (kr.k0 < k1) copy(kr.k0, 0, 0);
  for (int32_t k0 = kr.k0; k0 < k1; k0 += 2) {
#pragma unroll
    for (int b2 = 0; b2 < 2; ++b2) {   // (unrolled: the buffer is a constant)
      const int32_t kt = k0 + b2;
      if (kt >= k1) break;
      const bool on = active && 32 * kt < V_max;
      wait_copies<0>();
      __syncthreads();   // K of this tile is in LDS; nobody reads K and V of the one before it any more
      copy(kt, F::V, 2 * F::V);
      if (kt + 1 < k1) copy(kt + 1, 0, (b2 ^ 1) * F::V);
      if (on) scores((uint32_t)(b2 * F::V), 32 * kt);
      if (kt + 1 < k1) wait_copies<F::NI>();   // (V is older than the next K)
      else wait_copies<0>();
      __syncthreads();
      if (on) output();
    }
  }

  // (the row and the launch parameters anew: kept across the loop they would be spilled)
  const Params& p2 = gn_params_again();
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const float l_tot = half_sum(l_run);
  const int32_t r = b.tile * GN_ROWS + 32 * rb + (tid & 31), rows = p2.C * p2.G;
  const bool valid = r < rows;
  if (n_split > 1 || !last) {
    const int64_t at = (((int64_t)b.split * p2.Hkv + b.g) * tiles + b.tile) * 4 + rb;
    if (!active) return;
    part_store<bf16_t, D>(part, at, tid & 63, of, 1.f);
    if (!(tid & 32)) part_ml[at * 32 + (tid & 31)] = make_float2(l_tot > 0.f ? m_run : -INFINITY, l_tot);
  } else {
    const float inv = 1.f / l_tot, low = inv * GN_LOWER;
    const int32_t i = (int32_t)div_g(p2, (uint32_t)(valid ? r : 0)), h = b.g * p2.G + (valid ? r - i * p2.G : 0);
    uint32_t bad = gn_either_half(valid && gn_not_finite(of));
    if (valid && !((bad >> (tid & 31)) & 1)) {
      float* dst = (float*)p2.o + (int64_t)i * p2.q_tok_stride + (int64_t)h * p2.q_head_stride;
      part_emit<bf16_t, D>(of, (tid >> 5) & 1, [&](int d, float v0, float v1, float v2, float v3) { part_store4<float>(dst + d, v0 * low, v1 * low, v2 * low, v3 * low); });
    }
    if (valid && !(tid & 32)) p2.lse[(int64_t)h * p2.C + i] = gn_lse(p2, m_run, l_tot);
    for (; bad; bad &= bad - 1) {
      const int x = __builtin_ctz(bad);
      gn_redo_row<float, D, false>(p2, b.g, __builtin_amdgcn_readlane(i, x), __builtin_amdgcn_readlane(h, x), lp, tid & 63, gn_lane(m_run * c, x), gn_lane(inv, x), 0.f);
    }
  }
}

// ---- how a backward's work is shared out ----------------------------------------------------------
// A row tile (dQ) takes as many steps as it sees key tiles, a unit of 128 keys (dK / dV) as many as there are stages of rows that see it: those that hold the chunk's
// own pages fewer than the others.  Each is cut into equal parts of at most `most` steps, a workgroup each, so that all workgroups have about the same work; parts of one
// row tile or unit leave partial sums, of which workgroup b of KV head g has number b Hkv + g.  (The same number of parts for all: the backward of 8 / 2 heads,
// chunk 1088, 24 + 17 pages of 64 in one launch 97 us for 83; equal ranges across row tiles and units, with one part more per workgroup and rows that
// no other workgroup reads at the same time, 83 us there, but 8 to 30 % slower where parts fit well.)
// The steps are counted for a list of the greatest length that ends with the chunk's own pages, so that nothing has to be read first; with other lists the shares
// are less even.  The first part of a unit takes every stage up to its end, the last part of a row tile every tile from its start.
struct GnShare { int32_t n, most; };   // workgroups per KV head
struct GnShares { GnShare kv, rows; float *kv_part, *row_part; };
struct GnPart { int32_t u, s0, s1, slot; bool first, last; };   // steps s0 .. s1 - 1 of row tile or unit u; slot of the partial sums, or < 0
// of units of 128 keys: steps are stages of `rows` rows, counted from `from`; of row tiles: tiles of kt keys
struct GnKeySteps {
  int32_t PG, rows, all, past, lp;   // past: list entries before the chunk's own pages
  __host__ __device__ __forceinline__ GnKeySteps(const Params& p, int lp, int32_t max_len, int32_t kt)
      : PG(p.P * p.G), rows(kt), all((int32_t)(((int64_t)p.C * p.G + kt - 1) / kt)), past(max_len - p.m), lp(lp) {}
  __host__ __device__ __forceinline__ int32_t from(int32_t u) const {
    const int32_t j = (u << (7 - lp)) - past, s = j > 0 ? (int32_t)((int64_t)j * PG / rows) : 0;
    return s < all ? s : all - 1;
  }
  __host__ __device__ __forceinline__ int32_t operator()(int32_t u) const { return all - from(u); }
  int32_t over(int32_t v, int32_t units) const {   // units with more than v steps (v >= 0): those up to the last key page that stage all - v comes after
    if (v == 0) return units;
    if (v >= all) return 0;
    const int64_t j = ((int64_t)(all - v) * rows - 1) / PG, n = ((past + j) >> (7 - lp)) + 1;
    return (int32_t)(n < units ? n : units);
  }
};
struct GnRowSteps {
  int32_t G, rows, past, P, kt, lp;
  uint32_t magic;
  __host__ __device__ __forceinline__ GnRowSteps(const Params& p, int lp, int32_t max_len, int32_t kt)
      : G(p.G), rows(p.C * p.G), past(max_len - p.m), P(p.P), kt(kt), lp(lp), magic(p.g_magic) {}
  __host__ __device__ __forceinline__ int32_t operator()(int32_t t) const {
    const int32_t r = t * GN_ROWS + GN_ROWS - 1 < rows - 1 ? t * GN_ROWS + GN_ROWS - 1 : rows - 1, i = G == 1 ? r : (int32_t)(((uint64_t)(uint32_t)r * magic) >> 32);
    const int64_t seen = ((int64_t)(past + (i >> lp)) << lp) + (i & (P - 1)) + 1;
    const int32_t n = (int32_t)((seen + kt - 1) / kt);
    return n > 1 ? n : 1;
  }
  int32_t over(int32_t v, int32_t tiles) const {   // row tiles with more than v steps: those whose last row lies r rows or more into the chunk
    const int64_t r = ((int64_t)v * kt - (int64_t)past * P) * G;
    if (v == 0 || r <= 0) return tiles;
    const int64_t n = tiles - 1 - (r >> 7);   // (of all but the last, whose last row is rows - 1)
    return (int32_t)((n > 0 ? n : 0) + (rows - 1 >= r));
  }
};
template <typename N> __device__ __forceinline__ int32_t gn_parts(const N& steps, const GnShare& w, int32_t u) { return (int32_t)((uint32_t)(steps(u) + w.most - 1) / (uint32_t)w.most); }
// Sums over the lanes before this one, and over all, of numbers up to 31 (a unit has at most 16 parts, a row tile 31): five ballots.
__device__ __forceinline__ int32_t gn_sum_before(int32_t v, int32_t& all) {
  int32_t before = 0;
  all = 0;
#pragma unroll
  for (int k = 0; k < 5; ++k) {
    const uint64_t bits = __ballot((v >> k) & 1);
    before += (int32_t)__builtin_amdgcn_mbcnt_hi((uint32_t)(bits >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bits, 0)) << k;
    all += __builtin_popcountll(bits) << k;
  }
  return before;
}
// What workgroup b of KV head g does of `units` row tiles or units.  (Where each is one part -- all long lists -- nothing is looked for.  With a scan by shuffles and divisions of 64 bits, in front of the
// first load of every workgroup, one-launch backwards of 20 to 50 us took 0.5 us longer, and their finish kernels as much.)
template <typename N> __device__ __forceinline__ GnPart gn_part(int32_t units, const GnShare& w, int32_t b, int g, int32_t Hkv, const N& steps) {
  if (w.n == units) return {b, 0, steps(b), -1, true, true};
  const int lane = threadIdx.x & 63;
  int32_t u = 0, before = 0, n = 0, e = 1, x = 0;
  for (int32_t u0 = 0; u0 < units; u0 += 64) {
    const bool there = u0 + lane < units;
    const int32_t mine = there ? gn_parts(steps, w, u0 + lane) : 0;
    int32_t all;
    const int32_t first = before + gn_sum_before(mine, all);
    const uint64_t here = __ballot(first <= b && b < first + mine);
    if (here) {
      const int l = __builtin_ctzll(here);
      u = u0 + l;
      n = __builtin_amdgcn_readfirstlane(steps(u));
      e = __builtin_amdgcn_readlane(mine, l);
      x = b - __builtin_amdgcn_readlane(first, l);
      break;
    }
    before += all;
  }
  return {u, (int32_t)((uint32_t)(n * x) / (uint32_t)e), (int32_t)((uint32_t)(n * (x + 1)) / (uint32_t)e), e == 1 ? -1 : b * Hkv + g, x == 0, x + 1 == e};
}
// {the first part of u, parts}
template <typename N> __device__ __forceinline__ int2 gn_parts_of(const GnShare& w, int32_t u, const N& steps) {
  const int lane = threadIdx.x & 63;
  int32_t before = 0, all;
  for (int32_t u0 = 0; u0 < u; u0 += 64) {
    gn_sum_before(u0 + lane < u ? gn_parts(steps, w, u0 + lane) : 0, all);
    before += all;
  }
  return make_int2(before, __builtin_amdgcn_readfirstlane(gn_parts(steps, w, u)));
}

// ---- dQ -----------------------------------------------------------------------------------------
// Also computes Delta = <dO, O> of its rows for the dK / dV kernel, which runs afterwards: p.delta, or (bias != nullptr) the
// bias words from which attn_bwd_dkv_mfma.hip starts its accumulators.  Where dQ overlaps O otherwise than row on row, a row of O may
// be overwritten before its workgroup reads it: then delta_kernel has filled p.delta beforehand.
template <typename T, int D> __global__ __launch_bounds__(256) void delta_kernel(Params p) {
  constexpr int NG = Gn<T, D>::NG;   // lanes of a row, 16 bytes each
  const int64_t row = (int64_t)blockIdx.x * (256 / NG) + threadIdx.x / NG;
  if (row >= (int64_t)p.C * p.Hq) return;
  const int i = (int)(row / p.Hq), h = (int)(row - (int64_t)i * p.Hq), c = threadIdx.x % NG;
  const int64_t off = (int64_t)i * p.q_tok_stride + (int64_t)h * p.q_head_stride;
  float d = gn_dot<T>(reinterpret_cast<const u32x4_t*>((const T*)p.d_o + off)[c], reinterpret_cast<const u32x4_t*>((const T*)p.o + off)[c], 0.f);
#pragma unroll
  for (int o = 1; o < NG; o <<= 1) d += __shfl_xor(d, o, 64);
  if (c == 0) p.delta[(int64_t)h * p.C + i] = d;
}
template <typename T, int D> static hipError_t launch_delta(const Params& p, hipStream_t st) {
  constexpr int R = 256 / Gn<T, D>::NG;
  delta_kernel<T, D><<<dim3((unsigned)(((int64_t)p.C * p.Hq + R - 1) / R)), dim3(256), 0, st>>>(p);
  return hipGetLastError();
}
// the key tiles kr[w] of wave group w of a row tile; the first of them: Delta is left for the other kernels.  slot: of the partial sums (blocks of 128 rows), or < 0
template <int KH> struct GnRowPiece { int32_t g, tile; GnRange kr[KH]; bool first; int64_t slot; };
template <typename T, int D, int KH, int NT, bool ALONE>
__device__ __forceinline__ void dq_body(const Params& p, unsigned char* smem, const GnRowPiece<KH>& b, int lp, int32_t max_len, float* __restrict__ part,
                                        float* __restrict__ bias, int32_t n_stages) {
  typedef Gn<T, D> X;
  typedef GnTiles<T, D> Y;
  const int lane = threadIdx.x & 63, hh = lane >> 5, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), rb = wave & 3, group = KH == 1 ? 0 : wave >> 2;
  const GnRange kr = group ? b.kr[KH - 1] : b.kr[0], other = group ? b.kr[0] : b.kr[KH - 1];
  const GnTile t = gn_tile(p, b.g, b.tile, rb, lane, lp, max_len);
  GnStream<T, D> ks;
  ks.init(p, t.lid, max_len, b.g, rb, lane, kr.k0 * Y::KT, lp);

  GnStay<T, D> qs;
  u32x4_t dof[X::NJ];
  const int64_t roff = (int64_t)t.i * p.q_tok_stride + (int64_t)t.h * p.q_head_stride;
  float delta = 0.f;
  qs.at((const T*)p.q + roff, hh);
#pragma unroll
  for (int j = 0; j < X::NJ; ++j) {
    qs.load(j);
    const int64_t at = roff * X::ES + 16 * gn_granule<T>(j, hh);
    dof[j] = *reinterpret_cast<const u32x4_t*>((const unsigned char*)p.d_o + at);
    delta = gn_dot<T>(dof[j], *reinterpret_cast<const u32x4_t*>((const unsigned char*)p.o + at), delta);
  }
  delta = half_sum(delta);
  if (p.delta_given) delta = p.delta[(int64_t)t.h * p.C + t.i];
  const float lse2 = p.lse[(int64_t)t.h * p.C + t.i] * 1.4426950408889634f;

  f32x16 dq[X::DB];
  gn_zero(dq);
  const float c = p.sm_scale * 1.4426950408889634f;
  if (b.first && group == 0 && t.valid && hh == 0) {
    if (bias) {   // row space of that kernel: blocks of 32 tokens of one head, the heads interleaved
      const uint32_t blk = (uint32_t)(t.i >> 5) * p.G + (uint32_t)(t.h - b.g * p.G), r = 32 * blk + (t.i & 31);
      float* w = bias + (((int64_t)b.g * n_stages + (r >> 6)) * 2) * 64 + (r & 63);
      w[0] = -lse2 / c;
      w[64] = -delta;
    } else if (p.delta && !p.delta_given) {
      p.delta[(int64_t)t.h * p.C + t.i] = delta;
    }
  }
  GnAddr<T, D> ad;
  ad.init(lane, group * GnRow<T, D, KH>::GROUP);
  const int32_t V_max = __builtin_amdgcn_readlane(t.V, 31);

  gn_key_loop<T, D, KH, true>(p, t, ks, kr, other, max_len, group, rb, lane, lp, qs, [&](const uint32_t at, const int32_t t0, auto mask) __attribute__((always_inline)) {
    if (!t.active || t0 >= V_max) return;
    constexpr int NP = GnAddr<T, D>::NP, NJ = X::NJ, L = 2 * NJ + NP;
    const int32_t rel = t.V - t0 - 4 * hh;
    ad.anew();
    if constexpr (ALONE) {
      // A wave alone on its SIMD, whose vector work runs only beside its own matrix instructions: S and dP of block 0; those of block 1 beside
      // dS of block 0; dQ of block 0 beside dS of block 1; dQ of block 1.  (Block by block, as below: the backward of 8 / 2 heads, 41 pages of 64,
      // chunk 1088 in one launch 103 us, so 92; with two waves per SIMD it only costs registers.)
      static_assert(Y::U == 2 && 16 % NP == 0 && 32 % (2 * NJ) == 0, "two blocks of bf16");
      f32x16 sum[2][2];   // [block][S, then P, then dS | dP]
      gn_zero(sum[0]);
      gn_zero(sum[1]);
      GnP<T, NT> dsp[2];
      auto form = [&](const int u, const int x) __attribute__((always_inline)) {
        float v = __builtin_amdgcn_exp2f(__builtin_fmaf(sum[u][0][x], c, -lse2));
        if (mask.value && 32 * u + 8 * (x >> 2) + (x & 3) >= rel) v = 0.f;
        sum[u][0][x] = v * (sum[u][1][x] - delta);
        if (x & 1) dsp[u].set2(x - 1, sum[u][0][x - 1], sum[u][0][x]);
      };
      gn_pipeline<4 * NJ + 2 * NP, GN_BATCH<T, D>>(
          [&](const int i) __attribute__((always_inline)) {
            if (i < 4 * NJ) return ad.row_frag(i % NJ, at + 32 * (i / (2 * NJ)) * X::RB + (i / NJ % 2 ? Y::TILE : 0));
            const int v = i - 4 * NJ;
            return ad.tr_frag(v % NP, at + 32 * (v / NP) * X::RB);
          },
          [&](const int i, const u32x4_t& f) __attribute__((always_inline)) {
            if (i < 4 * NJ) {
              const int u = i / (2 * NJ), j = i % NJ, e = 16 / (2 * NJ);
              sum[u][i / NJ % 2] = mfma32(__builtin_bit_cast(bf16x8, f), __builtin_bit_cast(bf16x8, i / NJ % 2 ? dof[j] : qs.f[j]), sum[u][i / NJ % 2]);
              if (u == 1)
#pragma unroll
                for (int x = (i - 2 * NJ) * e; x < (i - 2 * NJ + 1) * e; ++x) form(0, x);
            } else {
              const int v = i - 4 * NJ, e = 16 / NP;
              gn_tr_mma<T, D, NT>(v % NP, f, dsp[v / NP], dq);
              if (v < NP)
#pragma unroll
                for (int x = v * e; x < (v + 1) * e; ++x) form(1, x);
            }
          });
      return;
    } else {
      GnSum<T> s;   // of one block
      f32x16 dp[1];
      f32x16& pr = s.v[0];   // P
      GnP<T, NT> ds;
      // per block: S, then dP with the exponentials of S between its instructions, dS, then dQ
      gn_pipeline<Y::U * L, GN_BATCH<T, D>>(
          [&](const int i) __attribute__((always_inline)) {
            const int u = i / L, k = i % L;
            const uint32_t o = at + 32 * u * X::RB;
            return k < NJ ? ad.row_frag(k, o) : k < 2 * NJ ? ad.row_frag(k - NJ, o + Y::TILE) : ad.tr_frag(k - 2 * NJ, o);
          },
          [&](const int i, const u32x4_t& f) __attribute__((always_inline)) {
            const int u = i / L, k = i % L;
            if (k == 0) {
              s.zero();
              gn_zero(dp);
            }
            if (k < NJ) {
              s.step(k, f, qs);
              if (k == NJ - 1) s.template close<false>(qs, [&](const int j) __attribute__((always_inline)) { return ad.row_frag(j, at + 32 * u * X::RB); });
            } else if (k < 2 * NJ) {
              gn_mma<T>(f, dof[k - NJ], dp[0]);
  #pragma unroll
              for (int x = (k - NJ) * (16 / NJ); x < (k - NJ + 1) * (16 / NJ); ++x) {
                float v = __builtin_amdgcn_exp2f(__builtin_fmaf(pr[x], c, -lse2));
                if (mask.value && 32 * u + 8 * (x >> 2) + (x & 3) >= rel) v = 0.f;
                pr[x] = v;
              }
              if (k == 2 * NJ - 1) {
  #pragma unroll
                for (int x = 0; x < 16; x += 2) ds.set2(x, pr[x] * (dp[0][x] - delta), pr[x + 1] * (dp[0][x + 1] - delta));
              }
            } else {
              gn_tr_mma<T, D, NT>(k - 2 * NJ, f, ds, dq);
            }
          });
    }
  });

  if constexpr (KH == 2) {
    float* mo = reinterpret_cast<float*>(smem) + rb * (D * 32) + lane;
    __syncthreads();
    if (group == 1) {
#pragma unroll
      for (int k = 0; k < X::DB * 16; ++k) mo[64 * k] = dq[k >> 4][k & 15];
    }
    __syncthreads();
    if (group == 1) return;
#pragma unroll
    for (int k = 0; k < X::DB * 16; ++k) dq[k >> 4][k & 15] += mo[64 * k];
  }
  if (b.slot >= 0) {
    if (t.active) part_store<T, D>(part, b.slot * 4 + rb, lane, dq, 1.f);
  } else {
    uint32_t bad = gn_either_half(t.valid && gn_not_finite(dq));
    if (t.valid && !((bad >> (lane & 31)) & 1)) {
      T* dst = (T*)p.d_q + roff;
      const float sc = p.sm_scale;
      part_emit<T, D>(dq, hh, [&](int d, float v0, float v1, float v2, float v3) { part_store4<T>(dst + d, v0 * sc, v1 * sc, v2 * sc, v3 * sc); });
    }
    for (; bad; bad &= bad - 1) {
      const int x = __builtin_ctz(bad);
      gn_redo_row<T, D, true>(gn_params_again(), b.g, __builtin_amdgcn_readlane(t.i, x), __builtin_amdgcn_readlane(t.h, x), lp, lane, gn_lane(lse2, x), p.sm_scale, gn_lane(delta, x));
    }
  }
}
template <typename T, int D, int KH, int NT>
__global__ __launch_bounds__(256 * KH, (Gn<T, D>::RB == 512 ? 1 : 2)) void dq_generic_kernel(Params p, int32_t tiles, int32_t n_split, int lp, int32_t max_len,
                                                                                             float* __restrict__ part, float* __restrict__ bias, int32_t n_stages) {
  extern __shared__ __align__(16) unsigned char smem[];
  const GnBlock b = gn_block(p, blockIdx.x, tiles, n_split);
  GnRowPiece<KH> t = {b.g, b.tile, {}, b.split == 0, n_split > 1 ? ((int64_t)b.split * p.Hkv + b.g) * tiles + b.tile : -1};
#pragma unroll
  for (int k = 0; k < KH; ++k) t.kr[k] = gn_range(max_len, lp, GnTiles<T, D>::KT, KH * b.split + k, KH * n_split);
  dq_body<T, D, KH, NT, false>(p, smem, t, lp, max_len, part, bias, n_stages);
}

// ---- dK / dV ------------------------------------------------------------------------------------
// A workgroup owns a unit of up to 128 keys of a KV head -- 128 / P consecutive list entries, or (one
// list per query page) one page of the union -- or one slice of the rows that see it.  Wave w holds
// keys 32 w .. + 31.  part[slot][dK | dV][wave]: slices, added to the pool by the finish kernel.
template <typename T, int D> struct GnKey {
  static constexpr int KT = GnTiles<T, D>::KT;
  static constexpr int STAT = 2 * GnTiles<T, D>::BUF, LDS = STAT + 2 * 2 * 64 * 4;   // two buffers, {lse2, delta} of their rows
};
// stages s0 .. s1 - 1 of the unit from list entry e0 on, or of the query pages q0 .. q0 + qc - 1 of a page of the union; slot: of the partial sums, or < 0
struct GnKeyPiece { int32_t g, e0, s0, s1, slot, q0, qc; bool first; };
// first stage of `rows` rows that sees list entry e of KV head g
__device__ __forceinline__ int32_t gn_first_stage(const Params& p, int g, int32_t e, int lp, int32_t rows) {
  const int64_t pos = owned_at(p, g, e) << lp, first_q = p.N - p.C;
  return (pos > first_q ? (int32_t)(pos - first_q) * p.G : 0) / rows;
}
template <typename T, typename TG, int D, bool OWN_DELTA, int NT, bool ALONE>
__device__ __forceinline__ void dkv_body(const Params& p, unsigned char* smem, const GnKeyPiece& piece, int lp, float* __restrict__ part) {
  typedef Gn<T, D> X;
  typedef GnKey<T, D> R;
  typedef GnTiles<T, D> Y;
  const int tid = threadIdx.x;
  const int lane = tid & 63, hh = lane >> 5, lq = lane & 31, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int32_t g = piece.g, e0 = piece.e0, q0 = piece.q0, qc = piece.qc, slot = piece.slot, s1 = piece.s1;
  int32_t s0 = piece.s0;
  if (!p.qp) {
    if (e0 >= list_len(p, g)) return;
    const int32_t seen = __builtin_amdgcn_readfirstlane(gn_first_stage(p, g, e0, lp, R::KT));   // the first stage that sees the unit
    s0 = piece.first || s0 < seen ? seen : s0;
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
  const int32_t rows = p.C * p.G;
  // a stage: KT rows of the chunk's, or stage v % spq of the piece's query page v / spq
  const int32_t rpq = p.P * p.G, spq = (rpq + R::KT - 1) / R::KT;
  int32_t tau_v = 0;
  if (p.qp && lane < qc) tau_v = p.inv_qp[(int64_t)g * p.m * p.sel_stride + p.inv_off[(int64_t)g * (p.un_stride + 1) + e0] + q0 + lane];

  GnStay<T, D> ks;
  u32x4_t vf[X::NJ];
  ks.at((const T*)p.k_pool + koff, hh);
#pragma unroll
  for (int j = 0; j < X::NJ; ++j) {
    ks.load(j);
    const int64_t at = koff * X::ES + 16 * gn_granule<T>(j, hh);
    vf[j] = *reinterpret_cast<const u32x4_t*>((const unsigned char*)p.v_pool + at);
  }
  f32x16 dk[X::DB], dv[X::DB];
  gn_zero(dk);
  gn_zero(dv);
  const float c = p.sm_scale * 1.4426950408889634f;
  GnAddr<T, D> ad;
  ad.init(lane, 0);

  // rows [base, end) of stage s
  auto stage_rows = [&](int32_t s, int32_t& base, int32_t& end) {
    if (!p.qp) {
      base = s * R::KT;
      end = rows;
    } else {
      const int32_t v = s / spq, tau = __builtin_amdgcn_readlane(tau_v, v & 63);
      base = tau * rpq + (s - v * spq) * R::KT;
      end = (tau + 1) * rpq;
    }
  };
  float st_l = INFINITY, st_d = 0.f;   // statistics of row `tid` of the stage under way
  // OWN_DELTA: Delta of the stage's rows from dO and O themselves, TPR threads per row
  constexpr int TPR = 256 / R::KT, DG = X::NG / TPR;
  u32x4_t dl_o[OWN_DELTA ? DG : 1], dl_do[OWN_DELTA ? DG : 1];
  bool dl_ok = false;
  // (what the copies need of the launch parameters stays in registers: read anew for every row they were a third of the rest of a stage)
  int32_t G = p.G;
  uint32_t g_magic = p.g_magic;
  int64_t tok_stride = p.q_tok_stride, head_stride = p.q_head_stride;
  const unsigned char *q_rows = (const unsigned char*)((const T*)p.q + (int64_t)g * p.G * p.q_head_stride), *do_rows = (const unsigned char*)((const T*)p.d_o + (int64_t)g * p.G * p.q_head_stride);
  typedef const __attribute__((address_space(1))) float* gfloat_t;
  gfloat_t lse = (gfloat_t)p.lse;
  int32_t C = p.C;
  asm volatile("" : "+s"(G), "+s"(g_magic), "+s"(tok_stride), "+s"(head_stride), "+s"(q_rows), "+s"(do_rows), "+s"(lse), "+s"(C));
  auto row_at = [&](int32_t r) __attribute__((always_inline)) {   // bytes from the first row of the KV head's heads
    const uint32_t m = __umulhi((uint32_t)r, g_magic), i = G == 1 ? (uint32_t)r : m;
    return ((int64_t)i * tok_stride + (int64_t)(uint32_t)(r - (int32_t)(i * G)) * head_stride) * X::ES;
  };
  auto copy = [&](int32_t s, uint32_t buf) {
    int32_t base, end;
    stage_rows(s, base, end);
    const uint32_t lrow = lane / X::NG, pos16 = lane % X::NG;
    const uint32_t dst = buf + wave * Y::RW * X::RB;
#pragma unroll
    for (int k = 0; k < Y::NI; ++k) {
      const uint32_t row = wave * Y::RW + k * X::RPI + lrow;
      int32_t r = base + (int32_t)row;
      r = r < end ? r : end - 1;
      const int64_t at = row_at(r) + (int64_t)((pos16 ^ X::swz(row & 15)) << 4);
      gn_copy16(q_rows + at, dst + 1024 * k);
      gn_copy16(do_rows + at, dst + Y::TILE + 1024 * k);
    }
    if (tid < R::KT) {
      const int32_t r = base + tid;
      st_l = INFINITY;   // rows past the end: P = 0
      st_d = 0.f;
      if (r < end) {
        const uint32_t m = __umulhi((uint32_t)r, g_magic), i = G == 1 ? (uint32_t)r : m;
        const int64_t at = (int64_t)(g * G + (r - (int32_t)i * G)) * C + i;
        st_l = lse[at] * 1.4426950408889634f;
        if (!OWN_DELTA) st_d = p.delta[at];
      }
    }
    if constexpr (OWN_DELTA) {
      int32_t r = base + tid / TPR;
      dl_ok = r < end;
      r = dl_ok ? r : end - 1;
      const int64_t at = row_at(r) + 16 * (tid % TPR);
      // (not the pointers of the copies, whose address space the compiler has lost: flat loads would make every wait for an LDS operand wait for them, too)
      const unsigned char *o_rows = (const unsigned char*)((const T*)p.o + (int64_t)g * p.G * p.q_head_stride), *dl_rows = (const unsigned char*)((const T*)p.d_o + (int64_t)g * p.G * p.q_head_stride);
#pragma unroll
      for (int k = 0; k < DG; ++k) {
        dl_o[k] = *reinterpret_cast<const u32x4_t*>(o_rows + at + 16 * TPR * k);
        dl_do[k] = *reinterpret_cast<const u32x4_t*>(dl_rows + at + 16 * TPR * k);
      }
    }
  };
  auto publish = [&](uint32_t buf) {   // buf: Y::BUF * index
    float* st = reinterpret_cast<float*>(smem + R::STAT + (buf ? 512 : 0));
    if (tid < R::KT) {
      st[tid] = st_l;
      if (!OWN_DELTA) st[64 + tid] = st_d;
    }
    if constexpr (OWN_DELTA) {
      float sum = 0.f;
#pragma unroll
      for (int k = 0; k < DG; ++k) sum = gn_dot<T>(dl_do[k], dl_o[k], sum);
#pragma unroll
      for (int o = 1; o < TPR; o <<= 1) sum += __shfl_xor(sum, o, 64);
      if (tid % TPR == 0) st[64 + tid / TPR] = dl_ok ? sum : 0.f;
    }
  };

  if (s0 < s1) {
    copy(s0, 0);
    ks.template split<true>();   // (while the first stage is on its way)
    publish(0);
  }
  wait_copies<0>();
  __syncthreads();
  // The stages whose rows all see every key of the unit come last: they have a loop of their own, without masks
  int32_t e1 = e0 + (p.qp ? 1 : 128 >> lp);
  e1 = (e1 < len ? e1 : len) - 1;
  const int64_t pos1 = (owned_at(p, g, e1) << lp) + p.P - 1;
  const int32_t r_all = __builtin_amdgcn_readfirstlane(pos1 > first_q ? (int32_t)(pos1 - first_q) * p.G : 0);
  auto stage = [&](const int32_t s, const uint32_t buf, auto mask) __attribute__((always_inline)) {   // (buf: a constant)
    if (s + 1 < s1) copy(s + 1, buf ^ Y::BUF);
    int32_t base, end;
    stage_rows(s, base, end);
    const float* st = reinterpret_cast<const float*>(smem + R::STAT + (buf ? 512 : 0));
    if (active) {
      // per block of 32 rows: S; dP with the exponentials of S between its instructions; dV with dS between its
      // instructions; dK
      constexpr int NP = GnAddr<T, D>::NP, NJ = X::NJ, L = 2 * NJ + 2 * NP;
      const int32_t rel = r_key - base - 4 * hh;
      ad.anew();
      if constexpr (ALONE) {
        // S and dP of block 0; those of block 1 beside P of block 0; dV of block 0 beside its dS; dK of block 0 beside P of block 1;
        // dV of block 1 beside its dS; dK of block 1
        static_assert(Y::U == 2 && 16 % NP == 0 && 16 % (2 * NJ) == 0, "two blocks of bf16");
        f32x16 sum[2][2];   // [block][S, then P, then dS | dP]
        gn_zero(sum[0]);
        gn_zero(sum[1]);
        GnP<T, NT> pr, ds;
        GnStat st_lse, st_delta;
        auto form_p = [&](const int u, const int x) __attribute__((always_inline)) {
          float v = __builtin_amdgcn_exp2f(__builtin_fmaf(sum[u][0][x], c, -st_lse.at(st + 32 * u, hh, x)));
          if (mask.value && 32 * u + 8 * (x >> 2) + (x & 3) < rel) v = 0.f;
          sum[u][0][x] = v;
          if (x & 1) pr.set2(x - 1, sum[u][0][x - 1], sum[u][0][x]);
        };
        auto form_ds = [&](const int u, const int x) __attribute__((always_inline)) {
          sum[u][0][x] *= sum[u][1][x] - st_delta.at(st + 64 + 32 * u, hh, x);
          if (x & 1) ds.set2(x - 1, sum[u][0][x - 1], sum[u][0][x]);
        };
        gn_pipeline<4 * NJ + 4 * NP, GN_BATCH<T, D>>(
            [&](const int i) __attribute__((always_inline)) {
              if (i < 4 * NJ) return ad.row_frag(i % NJ, buf + 32 * (i / (2 * NJ)) * X::RB + (i / NJ % 2 ? Y::TILE : 0));
              const int v = i - 4 * NJ;   // (dV takes dO, dK takes Q)
              return ad.tr_frag(v % NP, buf + 32 * (v / (2 * NP)) * X::RB + (v / NP % 2 ? 0 : Y::TILE));
            },
            [&](const int i, const u32x4_t& f) __attribute__((always_inline)) {
              if (i == 2 * NJ - 1) st_lse.fetch(st, hh, 0);
              if (i == 4 * NJ - 1) st_delta.fetch(st + 64, hh, 0);
              if (i == 4 * NJ + NP - 1) st_lse.fetch(st + 32, hh, 0);
              if (i == 4 * NJ + 2 * NP - 1) st_delta.fetch(st + 96, hh, 0);
              if (i < 4 * NJ) {
                const int u = i / (2 * NJ), j = i % NJ, e = 16 / (2 * NJ);
                sum[u][i / NJ % 2] = mfma32(__builtin_bit_cast(bf16x8, f), __builtin_bit_cast(bf16x8, i / NJ % 2 ? vf[j] : ks.f[j]), sum[u][i / NJ % 2]);
                if (u == 1)
#pragma unroll
                  for (int x = (i - 2 * NJ) * e; x < (i - 2 * NJ + 1) * e; ++x) form_p(0, x);
              } else {
                const int v = i - 4 * NJ, part = v / NP, n = v % NP, e = 16 / NP;
                if (part % 2 == 0) gn_tr_mma<T, D, NT>(n, f, pr, dv);
                else gn_tr_mma<T, D, NT>(n, f, ds, dk);
#pragma unroll
                for (int x = n * e; x < (n + 1) * e; ++x) {
                  if (part % 2 == 0) form_ds(part / 2, x);
                  else if (part == 1) form_p(1, x);
                }
              }
            });
      } else {
        GnSum<T> sv;
        f32x16 dp[1];
        f32x16& w = sv.v[0];   // P, then dS
        GnP<T, NT> pr, ds;
        GnStat st_lse, st_delta;
        gn_pipeline<Y::U * L, GN_BATCH<T, D>>(
            [&](const int i) __attribute__((always_inline)) {
              const int u = i / L, k = i % L;
              const uint32_t o = buf + 32 * u * X::RB;
              return k < NJ ? ad.row_frag(k, o) : k < 2 * NJ ? ad.row_frag(k - NJ, o + Y::TILE)
                   : k < 2 * NJ + NP ? ad.tr_frag(k - 2 * NJ, o + Y::TILE) : ad.tr_frag(k - 2 * NJ - NP, o);
            },
            [&](const int i, const u32x4_t& f) __attribute__((always_inline)) {
              const int u = i / L, k = i % L;
              if (k == 0) {
                sv.zero();
                gn_zero(dp);
              }
              if (k == NJ - 1) st_lse.fetch(st + 32 * u, hh, 0);
              if (k == 2 * NJ - 1) st_delta.fetch(st + 64 + 32 * u, hh, 0);
              if (k < NJ) {
                sv.step(k, f, ks);
                if (k == NJ - 1) sv.template close<false>(ks, [&](const int j) __attribute__((always_inline)) { return ad.row_frag(j, buf + 32 * u * X::RB); });
              } else if (k < 2 * NJ) {
                gn_mma<T>(f, vf[k - NJ], dp[0]);
  #pragma unroll
                for (int x = (k - NJ) * (16 / NJ); x < (k - NJ + 1) * (16 / NJ); ++x) {
                  float v = __builtin_amdgcn_exp2f(__builtin_fmaf(w[x], c, -st_lse.at(st + 32 * u, hh, x)));
                  if (mask.value && 32 * u + 8 * (x >> 2) + (x & 3) < rel) v = 0.f;
                  w[x] = v;
                }
                if (k == 2 * NJ - 1) {
  #pragma unroll
                  for (int x = 0; x < 16; x += 2) pr.set2(x, w[x], w[x + 1]);
                }
              } else if (k < 2 * NJ + NP) {
                gn_tr_mma<T, D, NT>(k - 2 * NJ, f, pr, dv);
                const int n = k - 2 * NJ;
  #pragma unroll
                for (int x = n * (16 / NP); x < (n + 1) * (16 / NP); ++x)
                  w[x] = w[x] * (dp[0][x] - st_delta.at(st + 64 + 32 * u, hh, x));
                if (n == NP - 1) {
  #pragma unroll
                  for (int x = 0; x < 16; x += 2) ds.set2(x, w[x], w[x + 1]);
                }
              } else {
                gn_tr_mma<T, D, NT>(k - 2 * NJ - NP, f, ds, dk);
              }
            });
      }
    }
    if (s + 1 < s1) publish(buf ^ Y::BUF);
    wait_copies<0>();
    __syncthreads();
  };
  int32_t s = s0;
  for (; s < s1; s += 2) {
    int32_t base, end;
    stage_rows(s, base, end);
    if (base >= r_all) break;
    stage(s, 0, std::true_type());
    if (s + 1 < s1) stage(s + 1, Y::BUF, std::true_type());
  }
  for (; s < s1; s += 2) {
    stage(s, 0, std::false_type());
    if (s + 1 < s1) stage(s + 1, Y::BUF, std::false_type());
  }

  const float sc = p.sm_scale;
  if (slot >= 0) {
    if (active) {
      const int nb = part_key_blocks(p);
      part_store<T, D>(part, ((int64_t)slot * 2) * nb + wave, lane, dk, sc);
      part_store<T, D>(part, ((int64_t)slot * 2 + 1) * nb + wave, lane, dv, 1.f);
    }
  } else {
    uint32_t bad[2] = {gn_either_half(kvalid && gn_not_finite(dv)), gn_either_half(kvalid && gn_not_finite(dk))};
    TG* pk = (TG*)p.dk_pool + koff;
    TG* pv = (TG*)p.dv_pool + koff;
    if (kvalid && !((bad[1] >> lq) & 1))
      part_emit<T, D>(dk, hh, [&](int d, float v0, float v1, float v2, float v3) { part_add4<TG>(pk + d, v0 * sc, v1 * sc, v2 * sc, v3 * sc); });
    if (kvalid && !((bad[0] >> lq) & 1))
      part_emit<T, D>(dv, hh, [&](int d, float v0, float v1, float v2, float v3) { part_add4<TG>(pv + d, v0, v1, v2, v3); });
    for (int is_dk = 0; is_dk < 2; ++is_dk)
      for (uint32_t left = bad[is_dk]; left; left &= left - 1) {
        const int32_t k = 32 * wave + __builtin_ctz(left);
        gn_redo_key<T, TG, D>(gn_params_again(), g, e0 + (p.qp ? 0 : k >> lp), k & (p.P - 1), is_dk, lp, lane);
      }
  }
}
// the part of the keys of workgroup bid
template <typename T, typename TG, int D, bool OWN_DELTA, int NT>
__device__ __forceinline__ void dkv_share(const Params& p, unsigned char* smem, int32_t bid, const GnShares& w, int lp, int32_t max_len) {
  const int32_t b = bid / p.Hkv, g = bid - b * p.Hkv, units = (int32_t)(((int64_t)max_len * p.P + GN_ROWS - 1) / GN_ROWS);
  const GnKeySteps steps(p, lp, max_len, GnKey<T, D>::KT);
  const GnPart t = gn_part(units, w.kv, b, g, p.Hkv, steps);
  const int32_t lo = steps.from(t.u);
  dkv_body<T, TG, D, OWN_DELTA, NT, sizeof(T) == 2 && D == 128>(p, smem, GnKeyPiece{g, t.u << (7 - lp), lo + t.s0, lo + t.s1, t.slot, 0, 0, t.first}, lp, w.kv_part);
}
template <typename T, typename TG, int D, int NT>
__global__ __launch_bounds__(256, (D == 128 || sizeof(T) == 4 ? 1 : 2)) void dkv_generic_kernel(Params p, GnShares w, int lp, int32_t max_len) {
  extern __shared__ __align__(16) unsigned char smem[];
  if (!p.qp) return dkv_share<T, TG, D, false, NT>(p, smem, blockIdx.x, w, lp, max_len);
  // a workgroup per entry of the work table
  const int32_t rest = blockIdx.x / p.Hkv, g = blockIdx.x - rest * p.Hkv, n_units = p.unit_count[g];
  if (rest >= n_units) return;
  const int4 un = p.units[(int64_t)g * p.max_units + (n_units - 1 - rest)];
  constexpr int32_t KT = GnKey<T, D>::KT;
  dkv_body<T, TG, D, false, NT, sizeof(T) == 2 && D == 128>(p, smem, GnKeyPiece{g, un.x, 0, un.z * ((p.P * p.G + KT - 1) / KT), un.w, un.y, un.z, false}, lp, w.kv_part);
}

// The whole backward of fp32 tensors: five products per pair instead of the seven of two kernels, as products of three bf16 terms (at head dim
// 64 all but dQ's).  A unit is 128 list tokens, 32 per wave: their K and V stay in registers as terms (K at head dim 128 in LDS), the rows of the head stream through
// LDS in stages of 32, as terms too (row_terms_kernel).  dS goes through LDS, dQ of a stage is left as one fp32 partial sum per unit.  One wave per
// SIMD (512 registers); the vector work of a product runs between the matrix instructions of the next one.
// The stages of all units of a KV head, one unit after the other, are cut into equal ranges, one per workgroup: whatever the list and the chunk, every
// compute unit has the same work.  A range covers the end of one unit and the start of the next (or several short ones); the piece of unit u
// in range b has slot (b + u) Hkv + g.
// A launch takes the units u0 .. u0 + un - 1 of every head (the slots count from u0); the launches after the first add to the partial sums of dQ, which are
// un in number: their room is bounded whatever the list.  (The stages that a unit's rows have are among those of the unit un before it, whose
// partial sums it adds to: a later page of the list is seen by fewer rows.)
template <int D> struct GnU {
  typedef Gn<bf16_t, D> X;
  typedef GnF3<D> F;
  // Head dim 128: dQ in terms, too.  A stage: Q0 Q1 Q2 dO0 dO1 dO2 and {lse2, delta}; K0 K1 K2 of the unit as [key][dim] in the order of a row tile.  The terms of dS take the
  // place of dO once dV is done, as [key][row] with word w (four rows) of key k at w ^ (k / 4 mod 8): 56 of about 15000
  // cycles of a stage are bank conflicts.  Against dQ on the fp32 pipe, 28 / 4 heads, chunk 512, 20 pages of 128, whole pass: 426 -> 421 us (192 matrix cycles in the place of 512, but two barriers more
  // a stage); dQ against 64 bits 7.9e-7 -> 7.4e-7.
  // Head dim 64 (two workgroups per compute unit have 80 KiB each): dQ on the fp32 pipe.  dS as [row][key], rows 544 bytes apart (both the dwords of 32 keys x 2 rows that
  // a store moves and the 16 bytes x 64 rows of a read fall on all banks); K as [key][dim]
  static constexpr bool TERMS = D == 128;
  static constexpr int STAT = F::TILE, DS = TERMS ? F::V : STAT + 2 * 64 * 4, DS_ROW = GN_ROWS * 4 + 32, DS_TERM = GN_ROWS * 64;
  static constexpr int KL = TERMS ? STAT + 2 * 64 * 4 : DS + 32 * DS_ROW, KL_ROW = D * 4 + 16, K_TERM = GN_ROWS * X::RB, OFF = KL + 3 * K_TERM, LDS = TERMS ? OFF + GN_ROWS * 8 : KL + GN_ROWS * KL_ROW;
  static_assert(!TERMS || 3 * DS_TERM <= F::V, "dS in the place of dO");
  // A value of K below 2^-110 (and not 0) is not the sum of three terms.  dQ is linear in K: units that hold such a value form it on the fp32 pipe from K in the pool (OFF: where its rows lie there), dS
  // being the sum of its terms.  4 us a stage more; with such a value in every unit the pass above takes 403 us instead of 272.  (Lifted as V is, K would take S along, whose products may be as
  // large as a float holds.)
  static constexpr uint32_t TINY = 17u << 24;   // bits of 2^-110, without the sign
  // dQ of a stage: wave w takes dim block w % DB and the keys of part w / DB; a partial sum per part
  static constexpr int PARTS = 4 / X::DB, KEYS = GN_ROWS / PARTS, WGS = D == 64 ? 2 : 1;   // workgroups per compute unit
};
__device__ __forceinline__ int32_t gn_unit_stages(const Params& p, int g, int32_t u, int32_t n_units, int lp) {
  if (u >= n_units) return 0;
  const int32_t n = (int32_t)(((int64_t)p.C * p.G + 31) / 32) - gn_first_stage(p, g, u << (7 - lp), lp, 32);
  return n > 0 ? n : 0;
}
__device__ __forceinline__ int32_t gn_wave_sum(int32_t v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
  return __builtin_amdgcn_readfirstlane(v);
}
__device__ __forceinline__ int32_t gn_unit_count(const Params& p, int g) { return (int32_t)(((int64_t)list_len(p, g) * p.P + GN_ROWS - 1) / GN_ROWS); }
// The terms of the rows of Q and (lifted) dO, [KV head][stage of 32 rows][GnF3::TILE], zeros past the last row; and Delta = <dO, O>.
template <int D> __global__ __launch_bounds__(256) void row_terms_kernel(Params p, int32_t stages, unsigned char* __restrict__ img) {
  typedef GnF3<D> F;
  constexpr int NG = F::X::NG;   // lanes of a row, eight values each
  const int32_t s = blockIdx.x / p.Hkv, g = blockIdx.x - s * p.Hkv;
  unsigned char* out = img + ((int64_t)g * stages + s) * F::TILE;
#pragma unroll
  for (int x = 0; x < 2 * 32 * NG / 256; ++x) {
    const int gi = threadIdx.x + 256 * x, is_do = gi / (32 * NG), r = gi / NG % 32, c = gi % NG;   // (is_do is the same for a whole row)
    const int32_t row = 32 * s + r;
    const bool valid = row < p.C * p.G;
    const int32_t i = (int32_t)div_g(p, (uint32_t)(valid ? row : 0)), h = g * p.G + (valid ? row - i * p.G : 0);
    const int64_t at = (int64_t)i * p.q_tok_stride + (int64_t)h * p.q_head_stride + 8 * c;
    u32x4_t v[2] = {};
    if (valid) {
      const u32x4_t* src = reinterpret_cast<const u32x4_t*>((const float*)(is_do ? p.d_o : p.q) + at);
      v[0] = src[0];
      v[1] = src[1];
    }
    if (is_do) {
      const u32x4_t* o = reinterpret_cast<const u32x4_t*>((const float*)p.o + at);
      float d = 0.f;
      if (valid) d = gn_dot<float>(v[1], o[1], gn_dot<float>(v[0], o[0], 0.f));
#pragma unroll
      for (int k = 1; k < NG; k <<= 1) d += __shfl_xor(d, k, 64);
      if (valid && c == 0) p.delta[(int64_t)h * p.C + i] = d;
      gn_lift(v[0]);
      gn_lift(v[1]);
    }
    gn_store_terms<D>(out + is_do * F::V + r * F::X::RB + ((c ^ F::X::swz(r)) << 4), v);
  }
}
struct GnPiece { int32_t g, u, s0, s1, slot, set, stages; };   // stages s0 .. s1 - 1 of unit u; its set of partial sums of dQ
template <int D, bool ADD>
__device__ __forceinline__ void units_body(const Params& p, unsigned char* smem, int lp, const unsigned char* __restrict__ img, float* __restrict__ part,
                                           float* __restrict__ dq_part, const GnPiece& t) {
  typedef GnU<D> R;
  typedef GnF3<D> F;
  typedef Gn<bf16_t, D> X;
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));   // (nothing that depends on the lane is kept from one piece to the next: it would be spilled)
  const int lane = tid & 63, hh = lane >> 5, lq = lane & 31, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int32_t e0 = t.u << (7 - lp), len = list_len(p, t.g), kq = 32 * wave + lq;   // this lane's key
  int32_t e = e0 + (kq >> lp);
  const bool kvalid = e < len, active = e0 + (32 * wave >> lp) < len;
  e = e < len ? e : len - 1;
  const int64_t l = list_at(p, t.g, e), pos = (l << lp) + (kq & (p.P - 1)), first_q = p.N - p.C;
  const int64_t koff = (int64_t)p.page_table[l] * p.pool_page_stride + (int64_t)t.g * p.pool_head_stride + (int64_t)(kq & (p.P - 1)) * p.pool_tok_stride;
  // rows before r_key do not see the key
  const int32_t r_key = !kvalid ? INT32_MAX : pos > first_q ? (int32_t)(pos - first_q) * p.G : 0, r_key_max = __builtin_amdgcn_readlane(r_key, 31);
  u32x4_t kf[X::NJ][3], vf[X::NJ][3], raw[2][X::NJ][2];
#pragma unroll
  for (int j = 0; j < X::NJ; ++j)
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      raw[0][j][e] = reinterpret_cast<const u32x4_t*>((const float*)p.k_pool + koff + 16 * j + 8 * hh)[e];
      raw[1][j][e] = reinterpret_cast<const u32x4_t*>((const float*)p.v_pool + koff + 16 * j + 8 * hh)[e];
    }
  uint32_t least = ~0u;   // |K| of this lane, in bits, but for zeros
#pragma unroll
  for (int j = 0; j < X::NJ; ++j) {
    gn_load_terms<false>(raw[0][j][0], raw[0][j][1], kf[j]);
    if constexpr (R::TERMS) {
#pragma unroll
      for (int x = 0; x < 8; ++x) {
        const uint32_t v = 2 * raw[0][j][x >> 2][x & 3] - 1;
        least = v < least ? v : least;
      }
#pragma unroll
      for (int k = 0; k < 3; ++k) *reinterpret_cast<u32x4_t*>(smem + R::KL + k * R::K_TERM + kq * X::RB + (((2 * j + hh) ^ X::swz(kq & 15)) << 4)) = kf[j][k];
    } else {
      u32x4_t* kl = reinterpret_cast<u32x4_t*>(smem + R::KL + kq * R::KL_ROW + 64 * j + 32 * hh);
      kl[0] = raw[0][j][0];
      kl[1] = raw[0][j][1];
    }
    gn_lift(raw[1][j][0]);
    gn_lift(raw[1][j][1]);
    gn_load_terms<false>(raw[1][j][0], raw[1][j][1], vf[j]);
    __builtin_amdgcn_sched_barrier(0);   // (one after the other: the comparisons of all of them would be spilled)
  }
  f32x16 dk[X::DB], dv[X::DB];
  gn_zero(dk);
  gn_zero(dv);
  const float c = p.sm_scale * 1.4426950408889634f;
  GnAddr<bf16_t, D> ad;
  ad.init(lane, 0);
  float* const ds_out = reinterpret_cast<float*>(smem + R::DS) + kq + 4 * hh * (R::DS_ROW / 4);
  if (!R::TERMS && !active) {   // (keys past the list: dS is and stays zero)
#pragma unroll
    for (int x = 0; x < 16; ++x) ds_out[(8 * (x >> 2) + (x & 3)) * (R::DS_ROW / 4)] = 0.f;
  }
  const unsigned char* src = img + ((int64_t)t.g * t.stages) * F::TILE + wave * (F::V / 4) + lane * 16;
  float st_l = INFINITY, st_d = 0.f;   // statistics of row `tid` of the stage under way
  // part 0: Q, 1: dO of stage s; every wave a quarter of each
  auto rows_in = [&](const int32_t s, const int part) __attribute__((always_inline)) {
#pragma unroll
    for (int k = 0; k < F::V / 4096; ++k) gn_copy16(src + (int64_t)s * F::TILE + part * F::V + 1024 * k, part * F::V + wave * (F::V / 4) + 1024 * k);
  };
  auto stats_in = [&](const int32_t s) __attribute__((always_inline)) {
    if (tid < 32) {
      const int32_t r = 32 * s + tid;
      st_l = INFINITY;   // rows past the end: P = 0
      st_d = 0.f;
      if (r < p.C * p.G) {
        const int32_t i = (int32_t)div_g(p, (uint32_t)r);
        const int64_t at = (int64_t)(t.g * p.G + (r - i * p.G)) * p.C + i;
        st_l = p.lse[at] * 1.4426950408889634f;
        st_d = p.delta[at] * (GN_LIFT * GN_LIFT);
      }
    }
  };
  float* const st = reinterpret_cast<float*>(smem + R::STAT);
  auto stats_out = [&] {
    if (tid < 32) {
      st[tid] = st_l;
      st[64 + tid] = st_d;
    }
  };
  if constexpr (R::TERMS) {
    if (hh == 0) reinterpret_cast<int64_t*>(smem + R::OFF)[kq] = koff;
    st[96 + wave] = __any(least < R::TINY - 1) ? 1.f : 0.f;
  }
  // dQ of a stage: dim block db, the keys of part kp; dims 32 db + 8 a + 4 hh .. + 3 are group 4 db + a of the block
  const int db = wave % X::DB, kp = wave / X::DB;
  float4* const dst0 = reinterpret_cast<float4*>(dq_part) + (((int64_t)(t.set * R::PARTS + kp) * p.Hkv + t.g) * (4 * gn_tiles(p.C, p.G, p.P, p.m, 0))) * (D / 8) * 64 + lane + 256 * db;
  float4 old[4];
  auto fetch = [&](const int32_t s) __attribute__((always_inline)) {
#pragma unroll
    for (int a = 0; a < 4; ++a) old[a] = dst0[(int64_t)s * (D / 8) * 64 + 64 * a];
  };
  auto dq_out = [&](const int32_t s, f32x16& dq) __attribute__((always_inline)) {
    if constexpr (ADD) {
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        dq[4 * a] += old[a].x;
        dq[4 * a + 1] += old[a].y;
        dq[4 * a + 2] += old[a].z;
        dq[4 * a + 3] += old[a].w;
      }
    }
#pragma unroll
    for (int a = 0; a < 4; ++a) dst0[(int64_t)s * (D / 8) * 64 + 64 * a] = make_float4(dq[4 * a], dq[4 * a + 1], dq[4 * a + 2], dq[4 * a + 3]);
  };
  // lane's addresses of dQ's operands: K^T (the last term apart: an offset has 16 bits), dS of an even and an odd group of 16 keys; + 8: the second four keys of a half
  uint32_t k_at[2], k_last[2], ds_at[2][2], k_rows = R::KL + wave * (32 * X::RB);
  if constexpr (R::TERMS) {
    const uint32_t L = lane & 15, gq = lane >> 4, r = 4 * (gq >> 1) + (L >> 2), k0 = r * X::RB + (((2 * (gq & 1) + ((L & 3) >> 1)) ^ X::swz(r)) << 4) + 8 * (L & 1);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      k_at[h] = R::KL + (k0 ^ (uint32_t)(db << 6) ^ (uint32_t)(32 * h)) + 8 * h * X::RB;
      k_last[h] = k_at[h] + 2 * R::K_TERM;
#pragma unroll
      for (int e = 0; e < 2; ++e) ds_at[e][h] = R::DS + (r + 8 * h) * 64 + (((4 * (gq & 1) + (L & 3)) ^ ((4 * e + (gq >> 1) + 2 * h) & 7)) << 3);
    }
  }
  auto tr_pair = [&](const uint32_t lo, const uint32_t hi) __attribute__((always_inline)) {
    const u32x2_t a = __builtin_bit_cast(u32x2_t, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4_t*)lo));
    const u32x2_t b = __builtin_bit_cast(u32x2_t, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4_t*)hi));
    return __builtin_shufflevector(a, b, 0, 1, 2, 3);
  };
  auto publish = [&] {
    stats_out();
    wait_copies<0>();
    __syncthreads();
  };
  rows_in(t.s0, 0);
  rows_in(t.s0, 1);
  stats_in(t.s0);
  publish();
  bool tiny = false;
  if constexpr (R::TERMS) tiny = __builtin_amdgcn_readfirstlane(__any(st[96 + (lane & 3)] != 0.f));
  for (int32_t s = t.s0; s < t.s1; ++s) {
    // one stage: S, dP with P, dV with dS, dK
    const int32_t base = 32 * s, rel = r_key - base - 4 * hh;
    const bool mask = base < r_key_max;   // (wave-uniform)
    f32x16 sv[2], dp[2];
    GnP<bf16_t, 3> pr, ds;
    GnStat st_lse, st_delta;
    auto terms = [&](const GnP<bf16_t, 3>& v, const int u, const int k) __attribute__((always_inline)) { return u32x4_t{v.w[k][4 * u], v.w[k][4 * u + 1], v.w[k][4 * u + 2], v.w[k][4 * u + 3]}; };
    auto load = [&](const int i, const int k) __attribute__((always_inline)) {
      return i < X::NJ ? ad.row_frag(i, k * F::TERM) : i < 2 * X::NJ ? ad.row_frag(i - X::NJ, F::V + k * F::TERM)
           : i < 2 * X::NJ + 2 * X::DB ? ad.tr_frag(i - 2 * X::NJ, F::V + k * F::TERM) : ad.tr_frag(i - 2 * X::NJ - 2 * X::DB, k * F::TERM);
    };
    auto use = [&](const int i, const u32x4_t (&f)[3]) __attribute__((always_inline)) {
      constexpr int NJ = X::NJ, NV = 2 * X::DB;
      // (statistics ahead of their use at head dim 128 only: at 64 there are no registers for it, and another workgroup on the compute unit)
      if (R::TERMS && i == 2 * NJ - 1) st_delta.fetch(st + 64, hh, 0);
      if (i < NJ) {   // (S at head dim 64: at 128 it is formed below)
        if constexpr (!R::TERMS) gn_mma_terms(f, kf[i][0], kf[i][1], kf[i][2], sv[1], sv[0]);
      } else if (i < 2 * NJ) {   // dP, and P
        const int j = i - NJ;
        gn_mma_terms(f, vf[j][0], vf[j][1], vf[j][2], dp[1], dp[0]);
#pragma unroll
        for (int x = j * (16 / NJ); x < (j + 1) * (16 / NJ); ++x) {
          const int row = 8 * (x >> 2) + (x & 3);
          float v = __builtin_amdgcn_exp2f(__builtin_fmaf(sv[0][x] + sv[1][x], c, -(R::TERMS ? st_lse.at(st, hh, x) : st[row + 4 * hh])));
          if (mask && row < rel) v = 0.f;
          sv[0][x] = v;
        }
#pragma unroll
        for (int x = j * (16 / NJ); x < (j + 1) * (16 / NJ); x += 2) pr.set2(x, sv[0][x], sv[0][x + 1]);
      } else if (i < 2 * NJ + NV) {   // dV, and dS
        const int v = i - 2 * NJ, u = v / X::DB;
        gn_mma_terms(f, terms(pr, u, 0), terms(pr, u, 1), terms(pr, u, 2), dv[v % X::DB], dv[v % X::DB]);
#pragma unroll
        for (int x = v * (16 / NV); x < (v + 1) * (16 / NV); ++x) {
          const int row = 8 * (x >> 2) + (x & 3);
          sv[0][x] = sv[0][x] * (dp[0][x] + dp[1][x] - (R::TERMS ? st_delta.at(st + 64, hh, x) : st[64 + row + 4 * hh]));   // (dP, Delta and dS: lifted twice)
          if (!R::TERMS) ds_out[row * (R::DS_ROW / 4)] = sv[0][x];
        }
#pragma unroll
        for (int x = v * (16 / NV); x < (v + 1) * (16 / NV); x += 2) ds.set2(x, sv[0][x], sv[0][x + 1]);
      } else {
        const int v = i - 2 * NJ - NV, u = v / X::DB;
        gn_mma_terms(f, terms(ds, u, 0), terms(ds, u, 1), terms(ds, u, 2), dk[v % X::DB], dk[v % X::DB]);
      }
    };
    if constexpr (R::TERMS) {
      constexpr int NJ = X::NJ, NV = 2 * X::DB;   // (keys past the list: all of their rows are masked)
      // S: K's rows come from LDS as well, 24 reads of a stage for 96 registers (in registers, a third of them was spilled)
      gn_zero(sv);
      u32x4_t fq[2][3], fr[2][3];
      auto rows = [&](const int j) __attribute__((always_inline)) {
        const uint32_t at = ad.row[j] + k_rows, last = at + 2 * R::K_TERM;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          fq[j & 1][k] = load(j, k);
          fr[j & 1][k] = *(__attribute__((address_space(3))) const u32x4_t*)(k < 2 ? at + k * R::K_TERM : last);
        }
      };
      rows(0);
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        if (j + 1 < NJ) {
          rows(j + 1);
          __builtin_amdgcn_sched_barrier(0);
        }
        if (j == NJ - 1) st_lse.fetch(st, hh, 0);
        gn_mma_terms(fq[j & 1], fr[j & 1][0], fr[j & 1][1], fr[j & 1][2], sv[1], sv[0]);
        __builtin_amdgcn_sched_barrier(0);
      }
      gn_zero(dp);
      wait_copies<0>();
      __syncthreads();   // dO of the stage is in LDS
      gn_terms_pipeline<NJ + NV>([&](const int i, const int k) __attribute__((always_inline)) { return load(NJ + i, k); },
                                 [&](const int i, const u32x4_t (&f)[3]) __attribute__((always_inline)) { use(NJ + i, f); });
      __syncthreads();   // nobody reads dO any more, whose place takes dS
      unsigned char* const out = smem + R::DS + kq * 64;
#pragma unroll
      for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int a = 0; a < 4; ++a) *reinterpret_cast<uint2*>(out + k * R::DS_TERM + (((2 * a + hh) ^ ((kq >> 2) & 7)) << 3)) = make_uint2(ds.w[k][2 * a], ds.w[k][2 * a + 1]);
      gn_terms_pipeline<NV>([&](const int i, const int k) __attribute__((always_inline)) { return load(2 * NJ + NV + i, k); },
                            [&](const int i, const u32x4_t (&f)[3]) __attribute__((always_inline)) { use(2 * NJ + NV + i, f); });
      __syncthreads();   // dS is in LDS; nobody reads Q any more, whose place takes the next stage's
      if (s + 1 < t.s1) {
        rows_in(s + 1, 0);
        stats_in(s + 1);
      }
      if constexpr (ADD) fetch(s);   // (on their way during the product)
      f32x16 dq[2];
      gn_zero(dq);
      u32x4_t fk[2][3], fd[2][3];
      auto get = [&](const int n) __attribute__((always_inline)) {   // keys 16 n .. + 15
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          const uint32_t o = 16 * n * X::RB + (k < 2 ? k * R::K_TERM : 0);
          fk[n & 1][k] = tr_pair((k < 2 ? k_at[0] : k_last[0]) + o, (k < 2 ? k_at[1] : k_last[1]) + o);
          fd[n & 1][k] = tr_pair(ds_at[n & 1][0] + (k * R::DS_TERM + 1024 * n), ds_at[n & 1][1] + (k * R::DS_TERM + 1024 * n));
        }
      };
      if (tiny) {   // (operands of an instruction: K of key n + 4 hh + x, dim 32 db + lq; dS of the key, row lq)
        const float* const k_dim = (const float*)p.k_pool + 32 * db + lq;
#pragma unroll 1
        for (int n = 0; n < GN_ROWS; n += 16) {
          float k_val[8], d_val[8];
#pragma unroll
          for (int x = 0; x < 8; ++x) {
            const int key = n + 8 * (x >> 2) + 4 * hh + (x & 3);
            k_val[x] = k_dim[reinterpret_cast<const int64_t*>(smem + R::OFF)[key]];
            const unsigned char* d = smem + R::DS + key * 64 + (((lq >> 2) ^ ((key >> 2) & 7)) << 3) + 2 * (lq & 3);
            d_val[x] = 0.f;
#pragma unroll
            for (int k = 2; k >= 0; --k) d_val[x] += bf16_to_f32(*reinterpret_cast<const bf16_t*>(d + k * R::DS_TERM));
          }
#pragma unroll
          for (int x = 0; x < 8; ++x) dq[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(k_val[x], d_val[x], dq[0], 0, 0, 0);
        }
      } else {
        get(0);
#pragma unroll
        for (int n = 0; n < GN_ROWS / 16; ++n) {
          if (n + 1 < GN_ROWS / 16) {
            get(n + 1);
            __builtin_amdgcn_sched_barrier(0);
          }
          gn_mma_terms(fk[n & 1], fd[n & 1][0], fd[n & 1][1], fd[n & 1][2], dq[1], dq[0]);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      stats_out();
      wait_copies<0>();
#pragma unroll
      for (int x = 0; x < 16; ++x) dq[0][x] += dq[1][x];
      dq_out(s, dq[0]);
      __syncthreads();   // Q and the statistics of the next stage are in LDS; nobody reads dS any more, whose place takes its dO
      if (s + 1 < t.s1) rows_in(s + 1, 1);
      continue;
    }
    if (active) {
      gn_zero(sv);
      gn_zero(dp);
      gn_terms_pipeline<2 * X::NJ + 4 * X::DB>(load, use);
    }
    __syncthreads();   // dS is in LDS; nobody reads the stage any more, whose place takes the next
    if (s + 1 < t.s1) {
      rows_in(s + 1, 0);
      rows_in(s + 1, 1);
      stats_in(s + 1);
    }
    f32x16 dq;
#pragma unroll
    for (int x = 0; x < 16; ++x) dq[x] = 0.f;
    // operands of four instructions: dS of keys 8 n + 4 hh .. + 3 of the part (row lq), K of the same keys (dim 32 db + lq)
    const uint32_t at_ds = R::DS + lq * R::DS_ROW + 16 * hh + kp * R::KEYS * 4, at_k = R::KL + (kp * R::KEYS + 4 * hh) * R::KL_ROW + (32 * db + lq) * 4;
    u32x4_t fd[2];
    float fk[2][4];
    auto get = [&](const int n) __attribute__((always_inline)) {
      fd[n & 1] = *reinterpret_cast<const u32x4_t*>(smem + (at_ds + 32 * n));
#pragma unroll
      for (int x = 0; x < 4; ++x) fk[n & 1][x] = *reinterpret_cast<const float*>(smem + (at_k + (8 * n + x) * R::KL_ROW));
    };
    get(0);
#pragma unroll
    for (int n = 0; n < R::KEYS / 8; ++n) {
      if (n + 1 < R::KEYS / 8) {
        get(n + 1);
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int x = 0; x < 4; ++x) dq = __builtin_amdgcn_mfma_f32_32x32x2f32(fk[n & 1][x], __uint_as_float(fd[n & 1][x]), dq, 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (ADD) fetch(s);   // (the other workgroup computes meanwhile, and there are no registers to have them on their way during the product)
    dq_out(s, dq);
    publish();
  }
  if (active) {
    part_store<bf16_t, D>(part, ((int64_t)t.slot * 2) * 4 + wave, lane, dk, p.sm_scale);
    part_store<bf16_t, D>(part, ((int64_t)t.slot * 2 + 1) * 4 + wave, lane, dv, 1.f);
  }
}
template <int D, bool ADD>
__global__ __launch_bounds__(256, GnU<D>::WGS) void bwd_units_kernel(Params p, int32_t u0, int32_t un, int32_t ranges, int lp, const unsigned char* __restrict__ img,
                                                                              float* __restrict__ part, float* __restrict__ dq_part) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int lane = threadIdx.x & 63;
  const int32_t b = blockIdx.x / p.Hkv, g = blockIdx.x - b * p.Hkv, n_units = gn_unit_count(p, g) < u0 + un ? gn_unit_count(p, g) : u0 + un;
  int32_t all = 0;
  for (int32_t u = u0; u < n_units; u += 64) all += gn_unit_stages(p, g, u + lane, n_units, lp);
  all = gn_wave_sum(all);
  ranges = ranges < all ? ranges : all;   // (none of them empty)
  if (b >= ranges) return;
  int32_t at = (int32_t)((int64_t)all * b / ranges);
  const int32_t end = (int32_t)((int64_t)all * (b + 1) / ranges);
  // the unit in which the range starts, and where in it
  int32_t u = u0, before = 0;
  for (int32_t v0 = u0; v0 < n_units; v0 += 64) {
    const int32_t n = gn_unit_stages(p, g, v0 + lane, n_units, lp);
    int32_t upto = n;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int32_t v = __shfl_up(upto, o, 64);
      if (lane >= o) upto += v;
    }
    const int past = __builtin_popcountll(__ballot(before + upto <= at));
    u = v0 + past;
    if (past < 64) {
      if (past > 0) before += __builtin_amdgcn_readlane(upto, past - 1);
      break;
    }
    before += __builtin_amdgcn_readlane(upto, 63);
  }
  const int32_t S = (int32_t)(((int64_t)p.C * p.G + 31) / 32);
  for (; at < end; ++u) {
    const int32_t lo = __builtin_amdgcn_readfirstlane(gn_first_stage(p, g, u << (7 - lp), lp, 32)), n = S - lo > 0 ? S - lo : 0;
    const int32_t s0 = lo + (at - before), s1 = s0 + (end - at) < lo + n ? s0 + (end - at) : lo + n;
    if (s0 < s1) {
      units_body<D, ADD>(p, smem, lp, img, part, dq_part, GnPiece{g, u, s0, s1, (b + u - u0) * p.Hkv + g, u - u0, S});
      __syncthreads();
    }
    at += s1 - s0;
    before += n;
  }
}

// dQ and dK / dV of a short call in one launch: the first workgroups take the keys, the others the rows; neither
// waits for the other (each computes Delta itself, so dQ must not be written over O).  8 us of launch and start-up less than one after the other, where
// neither fills the chip.
template <typename T, typename TG, int D, int NT>
__global__ __launch_bounds__(256, (D == 128 || sizeof(T) == 4 ? 1 : 2)) void bwd_pair_kernel(Params p, GnShares w, int32_t tiles, int lp, int32_t max_len) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int32_t kv_blocks = w.kv.n * p.Hkv;
  if ((int32_t)blockIdx.x < kv_blocks) return dkv_share<T, TG, D, true, NT>(p, smem, blockIdx.x, w, lp, max_len);
  const int32_t x = (int32_t)blockIdx.x - kv_blocks, b = x / p.Hkv, g = x - b * p.Hkv;
  const GnPart t = gn_part(tiles, w.rows, b, g, p.Hkv, GnRowSteps(p, lp, max_len, GnTiles<T, D>::KT));
  dq_body<T, D, 1, NT, sizeof(T) == 2 && D == 128>(p, smem, GnRowPiece<1>{g, t.u, {{t.s0, t.last ? INT32_MAX : t.s1}}, false, t.slot}, lp, max_len, w.row_part, nullptr, 0);
}

// What is left of a backward with splits, in one launch: workgroups below dq_blocks add the dQ partials, the others
// add the slices of a dK / dV unit to the pool.
// Eight waves per block (NW) keep more loads in flight where there are few blocks: 14 / 2 heads, two pages, 53.3 -> 52.2 us a pass; 6 / 2 heads, 93 pages
// (1700 blocks): 250.6 -> 249.3.  At 5000 blocks it makes no difference, and where many more fill the chip four waves are faster (4096 tokens of 28 / 4
// heads with a list per page: 91 us against 98).
constexpr int64_t FINISH_FEW = 4096;
template <typename T, typename TG, int D, typename L, int NW>
__global__ __launch_bounds__(64 * NW) void bwd_finish_kernel(Params p, int32_t tiles, int32_t dq_split, const float* __restrict__ dq_part,
                                                         int32_t dq_blocks, int32_t kv_split, const float* __restrict__ kv_part, int lp,
                                                         int redo_keys, int32_t u0, int32_t un, GnShare row_share, GnShare kv_share, int32_t max_len) {
  constexpr bool UNITS = sizeof(L) != sizeof(T);   // the partial sums are those of bwd_units_kernel, its units u0 .. u0 + un - 1: of lifted values (dV), or of dS, lifted twice
  constexpr float low = UNITS ? GN_LOWER * GN_LOWER : 1.f;
  __shared__ GnRowsLds<D> sh;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  float4 a[GN_GW<D, NW>];
  if ((int32_t)blockIdx.x < dq_blocks) {
    const int64_t blocks = (int64_t)p.Hkv * tiles * 4;
    if constexpr (UNITS) {   // a partial sum per unit that sees the block: the first ones of the list
      const int32_t gb = (int32_t)blockIdx.x / (4 * tiles), s = (int32_t)blockIdx.x - gb * 4 * tiles, n = gn_unit_count(p, gb);
      dq_split = 0;
      for (int32_t u = 0; u < n; u += 64)
        dq_split += __builtin_popcountll(__ballot(u + lane < n && gn_first_stage(p, gb, (u + lane) << (7 - lp), lp, 32) <= s));
      dq_split = __builtin_amdgcn_readfirstlane(dq_split < un ? dq_split : un) * GnU<D>::PARTS;
    }
    if (row_share.n) {
      const int32_t gb = (int32_t)blockIdx.x / (4 * tiles), tile = ((int32_t)blockIdx.x >> 2) - gb * tiles;
      const int2 t = gn_parts_of(row_share, tile, GnRowSteps(p, lp, max_len, GnTiles<T, D>::KT));
      if (t.y == 1) return;   // (one workgroup had the whole row tile)
      gn_sum_parts<D, NW>(dq_part, ((int64_t)t.x * p.Hkv + gb) * 4 + (blockIdx.x & 3), (int64_t)p.Hkv * 4 * (D / 8) * 64, t.y, a, [] {});
    } else {
      gn_sum_parts<D, NW>(dq_part, blockIdx.x, blocks * (D / 8) * 64, dq_split, a, [] {});
    }
    const float sc = p.sm_scale;
    int i, h;
    uint32_t bad = gn_rows_out<L, D, NW>(sh, a, true, [&](int, int row, int d, const float4& r) __attribute__((always_inline)) {
      if (gn_out_row(p, tiles, blockIdx.x, row, i, h))
        part_store4<T>((T*)p.d_q + (int64_t)i * p.q_tok_stride + (int64_t)h * p.q_head_stride + d, r.x * sc * low, r.y * sc * low, r.z * sc * low, r.w * sc * low);
    });
    for (bad &= ((1u << 32 / NW) - 1) << (32 / NW * wave); bad; bad &= bad - 1)
      if (gn_out_row(p, tiles, blockIdx.x, __builtin_ctz(bad), i, h))
        gn_redo_row<T, D, true>(gn_params_again(), h / p.G, i, h, lp, lane, p.lse[(int64_t)h * p.C + i] * 1.4426950408889634f, sc, gn_delta<T, D>(p, i, h));
    return;
  }
  // (last units first: their slices were written last and are still in the memory-side cache)
  const int32_t nb = part_key_blocks(p), b = (int32_t)(gridDim.x - 1 - blockIdx.x), ug = b / (2 * nb), u = u0 + ug / p.Hkv, g = ug - (u - u0) * p.Hkv;
  const int wb = b - ug * 2 * nb, which = wb >= nb, kb = which ? wb - nb : wb;   // block of the slot, {dK, dV}, block of keys
  int64_t slot, next;
  int32_t e0;
  if (p.qp) {
    if (u >= p.multi_count[g]) return;
    e0 = p.multi_list[(int64_t)g * p.max_multi + u];
    kv_split = p.un_ns[(int64_t)g * p.un_stride + e0];
    slot = p.un_pbase[(int64_t)g * p.un_stride + e0];
    next = 1;
  } else {
    e0 = (u << (7 - lp)) + (32 * kb >> lp);
    if (e0 >= list_len(p, g)) return;
    slot = ((int64_t)u * kv_split) * p.Hkv + g;
    next = p.Hkv;
    if (kv_share.n) {
      const int2 t = gn_parts_of(kv_share, u, GnKeySteps(p, lp, max_len, GnTiles<T, D>::KT));
      if (t.y == 1) return;
      slot = (int64_t)t.x * p.Hkv + g;
      kv_split = t.y;
    }
    if constexpr (UNITS) {   // the ranges (kv_split of them) that hold a piece of the unit
      const int32_t n_units = gn_unit_count(p, g) < u0 + un ? gn_unit_count(p, g) : u0 + un;
      int32_t all = 0, before = 0;
      for (int32_t v = u0 + lane; v < n_units; v += 64) {
        const int32_t n = gn_unit_stages(p, g, v, n_units, lp);
        all += n;
        before += v < u ? n : 0;
      }
      all = gn_wave_sum(all);
      before = gn_wave_sum(before);
      const int32_t ranges = kv_split < all ? kv_split : all;
      const int32_t mine = __builtin_amdgcn_readfirstlane(gn_unit_stages(p, g, u, n_units, lp));
      if (mine == 0) return;
      // range b starts at stage all b / kv_split: the last one that starts at or before a stage
      auto range_of = [&](int32_t at) { return (int32_t)(((int64_t)(at + 1) * ranges - 1) / all); };
      const int32_t first = range_of(before);
      slot = (int64_t)(first + u - u0) * p.Hkv + g;
      kv_split = range_of(before + mine - 1) - first + 1;
    }
  }
  // The block's 32 keys lie in one page, or in two of 16 tokens.  Its rows of the pool are looked up and read behind the loads
  // of the slices: in front of them the chain list -> page table -> pool would hold those back.
  TG* dst[GN_GW<D, NW>];
  float4 old[GN_GW<D, NW>];
  gn_sum_parts<D, NW>(kv_part, slot * 2 * nb + wb, next * 2 * nb * (D / 8) * 64, kv_split, a, [&]() __attribute__((always_inline)) {
    TG* const pool = (TG*)(which == 0 ? p.dk_pool : p.dv_pool) + (int64_t)g * p.pool_head_stride;
    const bool two = lp == 4 && !p.qp && e0 + 1 < list_len(p, g);
    TG* const page0 = pool + (int64_t)p.page_table[owned_at(p, g, e0)] * p.pool_page_stride;
    TG* const page1 = two ? pool + (int64_t)p.page_table[owned_at(p, g, e0 + 1)] * p.pool_page_stride : nullptr;
#pragma unroll
    for (int k = 0; k < GN_GW<D, NW>; ++k) {
      const int x = k * 64 * NW + threadIdx.x, kq = 32 * kb + x / (D / 4);
      TG* const page = lp == 4 && (kq & 16) ? page1 : page0;
      dst[k] = page ? page + (int64_t)(kq & (p.P - 1)) * p.pool_tok_stride + 4 * (x % (D / 4)) : nullptr;
      if (page) old[k] = part_load4<TG>(dst[k]);
    }
  });
  uint32_t bad = gn_rows_out<L, D, NW>(sh, a, redo_keys, [&](int k, int, int, const float4& r) __attribute__((always_inline)) {
    const float by = UNITS && which ? GN_LOWER : low;
    if (dst[k]) part_store4<TG>(dst[k], old[k].x + r.x * by, old[k].y + r.y * by, old[k].z + r.z * by, old[k].w + r.w * by);
  });
  for (bad &= ((1u << 32 / NW) - 1) << (32 / NW * wave); bad; bad &= bad - 1) {
    const int32_t x = __builtin_ctz(bad), k = 32 * kb + x, e = e0 + (p.qp ? 0 : x >> lp);
    if (p.qp ? k < p.P : e < list_len(p, g)) gn_redo_key<T, TG, D>(gn_params_again(), g, e, k & (p.P - 1), which == 0, lp, lane);
  }
}

// ---- host side ----------------------------------------------------------------------------------
static inline size_t gn_up(size_t x) { return (x + 255) & ~(size_t)255; }

// How the rows of a forward or dQ call go onto the chip: splits of the key range and wave groups per workgroup, by an
// estimate of the time in microseconds.  `unit` is the time of a tile of KT keys on a full chip, for a workgroup of two
// groups (256 of them at a time) or for two workgroups of one group (512 at a time).  A round that leaves compute
// units idle costs less than a full one -- the clock rises, single groups get a compute unit to themselves --:
// `only` if it is the call's only round, `rest` after full ones, both growing with the part f that is filled.  On
// top a round costs RAMP (launch, list -> page table -> first tile), and a split its combine kernel and the
// partial sums, written and read at about 4 TB/s.  The constants are fitted to a sweep over 28 / 4 and 6 / 2 heads, 1 to
// 48 query pages, lists of 8 to 240 + m pages, 1 to 24 splits.  E.g. 28 / 4 heads, 65 pages, one query page (28 tiles of 128
// rows): 9 splits of two groups, 36 us against 123 without; 12 query pages (336 tiles): 3 splits of single
// groups, 241 against 260.
static int32_t gn_list_len(const Params& p, int32_t max_len) { return p.qp ? p.sel_stride : max_len; }
struct GnPlan { int32_t n, groups; float us; };
static float gn_rounds(float r, float only0, float only1, float rest0, float rest1) {
  const float full = floorf(r), f = r - full;
  return full + (f <= 0.f ? 0.f : full > 0.f ? rest0 + rest1 * f : only0 + only1 * f);
}
static GnPlan gn_plan(const Params& p, bool bf, int32_t max_len, bool dq, int32_t most = 32) {   // most: splits the workspace has room for
  constexpr float RAMP = 6.f, LAUNCH = 3.f, PART = 2.56e-4f;
  const float ds = (p.D == 128 ? 1.f : bf ? 0.65f : 0.5f) * (dq ? 1.4f : 1.f);
  const float unit1 = (bf ? 2.15f : 7.8f) * ds, unit2 = (bf ? 1.17f : 4.0f) * ds;   // (fp32: what its matrix pipe needs)
  const int32_t wgs = gn_tiles(p.C, p.G, p.P, p.m, p.qp) * p.Hkv, kt = bf ? 64 : 32;
  const float len = (float)gn_list_len(p, max_len);
  const float all = len * p.P / kt, avg = (len - 0.5f * p.m) * p.P / kt;   // tiles of the longest row, of an average one
  const bool pairs = bf || !dq || p.D == 64;   // (fp32 dQ at head dim 128 holds 320 registers: one wave per SIMD)
  GnPlan best = {1, 1, 1e30f};
  for (int32_t n = 1; n <= most && (n == 1 || n <= all); ++n) {
    const float x = (float)wgs * n, extra = n > 1 ? LAUNCH + x * p.D * PART : 0.f;
    const float mine = avg / n > 1.f ? avg / n : 1.f;
    float us = pairs ? gn_rounds(x / 512.f, bf ? 0.55f : 0.5f, 0.42f, 0.35f, 0.6f) * mine * unit1 + ceilf(x / 512.f) * RAMP
                     : ceilf(x / 256.f) * (mine * 0.5f * unit1 + RAMP);
    if (us + extra < best.us) best = {n, 1, us + extra};
    if (!pairs || 2 * n > all) continue;
    us = gn_rounds(x / 256.f, 0.78f, 0.14f, 0.58f, 0.25f) * (mine > 2.f ? mine : 2.f) * unit2 + ceilf(x / 256.f) * RAMP;
    if (us + extra < best.us) best = {n, 2, us + extra};
  }
  return best;
}

static int32_t gn_key_units(const Params& p, int32_t max_len) {
  return (int32_t)(((int64_t)max_len * p.P + GN_ROWS - 1) / GN_ROWS);
}
// The parts of `units` row tiles or units of a KV head if none has more than `most` steps: those with more than none, `most`, 2 `most` .. steps.
template <typename N> static int32_t gn_count(const N& steps, int32_t units, int32_t most) {
  const int32_t first = steps(0), last = steps(units - 1), least = first < last ? first : last, greatest = first < last ? last : first;   // (from unit to unit they only fall, or only rise)
  int32_t n = 0;
  for (int32_t v = 0; v < greatest; v += most) n += v < least ? units : steps.over(v, units);
  return n;
}
// The least `most` with which they are `slots` workgroups or fewer, at most `parts` of a unit (one each where the units are more).
template <typename N> static GnShare gn_share(const N& steps, int32_t units, int32_t slots, int32_t parts) {
  const int32_t first = steps(0), last = steps(units - 1), least = first < last ? first : last, greatest = first < last ? last : first;
  if (slots < units) return {units, greatest};
  const int32_t each = slots / units, floor = (greatest + parts - 1) / parts;
  int32_t lo = (int32_t)(((int64_t)units * least + slots - 1) / slots), hi = (greatest + each - 1) / each;   // (hi: no unit has more parts than its share of the slots)
  lo = lo < floor ? floor : lo;
  hi = hi < lo ? lo : hi;
  while (lo < hi) {
    const int32_t mid = (lo + hi) / 2;
    if (gn_count(steps, units, mid) <= slots) hi = mid;
    else lo = mid + 1;
  }
  return {gn_count(steps, units, lo), lo};
}
// workgroups of the dK / dV and one-launch kernels that run at once
static int32_t gn_slots(const Params& p, bool bf) { return bf && p.D == 64 ? 512 : 256; }   // (two workgroups per compute unit)
static int32_t gn_head_slots(const Params& p, bool bf) { return gn_slots(p, bf) / p.Hkv > 1 ? gn_slots(p, bf) / p.Hkv : 1; }
// us of a stage of KT rows x 128 keys in the dK / dV kernel
static bool gn_one_term(const Params& p) { return p.D == HD && p.P == TP; }   // (bf16: probabilities and dS in one term)
static float gn_stage_us(const Params& p, bool bf) { return bf ? (gn_one_term(p) ? 2.1f : p.D == 128 ? 3.8f : 3.2f) : (p.D == 128 ? 10.f : 5.f); }
static float gn_tile_us(const Params& p, bool bf) { return bf ? (gn_one_term(p) ? 1.3f : 2.f) : (p.D == 128 ? 7.f : 3.5f); }   // of KT keys x 128 rows in the one-launch backward
static GnShare gn_key_share(const Params& p, bool bf, int32_t max_len, int32_t slots, int32_t most = 0) {   // most: the steps of a part, if given
  const int32_t units = gn_key_units(p, max_len);
  if (p.qp || units < 1) return {0, 1};
  const GnKeySteps steps(p, __builtin_ctz(p.P), max_len, bf ? 64 : 32);
  return most ? GnShare{gn_count(steps, units, most), most} : gn_share(steps, units, slots, 16);
}
constexpr int32_t GN_ROW_PARTS = 31;   // (what gn_sum_before holds)
static GnShare gn_row_share(const Params& p, bool bf, int32_t max_len, int32_t slots, int32_t parts) {
  const int32_t tiles = gn_tiles(p.C, p.G, p.P, p.m, 0);
  return gn_share(GnRowSteps(p, __builtin_ctz(p.P), max_len, bf ? 64 : 32), tiles, slots, parts);
}
static float gn_key_us(const Params& p, bool bf, int32_t most) { return most * gn_stage_us(p, bf) + (bf ? 12.f : 8.f); }

// A backward in one launch (bwd_pair_kernel): the workgroups that run at once (256, or 512 at head dim 64 with bf16: two per
// compute unit) are shared out so that keys and rows take the same time.  us: the estimate that gn_backward goes by; huge where there is no such launch.
// How the work is cut: the longest part of the keys takes keys + stage a step, that of the rows rows + tile a step, these `crowd` longer a step where there are two workgroups on every compute unit; the
// finish kernel takes `launch`, `each` for every part of the unit or row tile that has most, and `part` a value of the partial sums (written and read).  Fitted to 2 to 16 parts a unit, and to as few steps a
// part of the rows as there is room for and more, of 1155 bf16 calls of 15 to 250 us (fp32 100).  The best division by these is taken where it is 10 % better than that by the constants of `us` (16
// parts of a row tile at most) and takes less than 60 us: bf16 calls of that length are 2.5 % faster on average, up to 32, and 1 % of them more than 3 % slower, at most 9.  Nearer than that the two are not
// told apart (taken from 7 % on, 3 % faster and 2.5 % of them slower), and longer calls are decided by how two workgroups share a compute unit (28 / 4 heads of 64, 640 rows, 46 pages of 128: 205 -> 226 us).
// 6 / 2 heads, 128 rows, 31 pages 33.3 -> 28.2 us, 8 / 8, 256 rows, 3 pages 24.9 -> 21.
struct GnPair { GnShare kv, rows; float us; };
struct GnPartUs { float keys, stage, rows, tile, launch, each, part, crowd; };
static GnPartUs gn_part_us(const Params& p, bool bf) {
  if (!bf) return p.D == 128 ? GnPartUs{9.8f, 7.8f, 10.1f, 5.3f, 7.2f, 0.f, 1.24e-4f, 0.f} : GnPartUs{7.3f, 4.34f, 7.9f, 2.87f, 3.3f, 0.f, 2.29e-4f, 0.f};
  if (gn_one_term(p)) return {8.9f, 2.2f, 8.35f, 1.07f, 0.6f, 0.285f, 1.4e-4f, 0.f};
  return p.D == 128 ? GnPartUs{12.3f, 2.8f, 10.1f, 1.63f, 0.9f, 0.31f, 1.94e-4f, 0.f} : GnPartUs{6.2f, 2.1f, 3.8f, 1.76f, 2.4f, 0.3f, 2.1e-4f, 0.126f};
}
static GnPair gn_pair(const Params& p, bool bf, int32_t max_len) {
  GnPair best = {{0, 1}, {0, 1}, 1e30f};
  const int32_t per = gn_slots(p, bf) / p.Hkv;   // workgroups of a KV head
  const int32_t wq = gn_tiles(p.C, p.G, p.P, p.m, p.qp), wk = gn_key_units(p, max_len);
  if (p.qp || wk < 1 || wq + wk > per) return best;
  const float tile = gn_tile_us(p, bf);
  const GnPartUs t = gn_part_us(p, bf);
  const GnRowSteps row_steps(p, __builtin_ctz(p.P), max_len, bf ? 64 : 32);
  const int32_t whole = gn_key_share(p, bf, max_len, wk).most, whole_row = row_steps(wq - 1);
  auto cost = [&](const GnShare& k, const GnShare& q) {
    const float kn = k.n > wk ? k.n : 0, qn = q.n > wq ? q.n : 0, over = p.Hkv * (k.n + q.n) / 256.f - 1.f, slow = over > 0.f ? 1.f + t.crowd * over : 1.f;
    const float tk = t.keys + k.most * t.stage * slow, tq = t.rows + q.most * t.tile * slow, nk = kn / wk, nq = qn / wq;
    return (tk > tq ? tk : tq) + (kn + qn > 0.f ? t.launch : 0.f) + t.each * (nk > nq ? nk : nq) + p.Hkv * (2.f * kn + qn) * p.D * t.part;
  };
  GnShare k_est = {0, 1}, q_est = {0, 1};   // the division of `us`
  float least = 1e30f;
  bool estimate = true;
  for (int32_t e = 1, most = 0; e <= 16 && e <= whole; ++e) {   // more parts per unit, until the rows have too few workgroups
    if ((whole + e - 1) / e == most) continue;
    most = (whole + e - 1) / e;
    const GnShare k = gn_key_share(p, bf, max_len, 0, most);
    if (k.n > per - wq) break;
    const GnShare q0 = gn_row_share(p, bf, max_len, per - k.n, GN_ROW_PARTS);
    if (estimate) {   // (until the rows take longer)
      const GnShare q = q0.most >= (whole_row + 15) / 16 ? q0 : gn_row_share(p, bf, max_len, per - k.n, 16);
      const float tk = gn_key_us(p, bf, most), tq = q.most * tile + (bf ? 10.f : 6.f), us = (tq > tk ? tq : tk) + p.Hkv * ((k.n > wk ? 2.f * k.n : 0.f) + (q.n > wq ? q.n : 0.f)) * p.D * 2.56e-4f;
      if (us < best.us) best.us = us, k_est = k, q_est = q;
      estimate = tq <= tk;
    }
    // the rows: as many parts as there is room for, or as few as take no longer than the keys, or around that
    const float tk = t.keys + most * t.stage;
    const int32_t even = (int32_t)((tk - t.rows) / t.tile);
    for (int32_t x = 0; x < 5; ++x) {
      const int32_t steps = x == 0 ? q0.most : x == 4 ? whole_row : even + x - 1;
      if (x && (steps <= q0.most || steps > whole_row || tk >= least)) continue;
      const GnShare q = x ? GnShare{gn_count(row_steps, wq, steps), steps} : q0;
      const float us = cost(k, q);
      if (us < least) least = us, best.kv = k, best.rows = q;
    }
    if (!estimate && t.rows + q0.most * t.tile > tk) break;
  }
  if (k_est.n > 0 && (least > 60.f || least > 0.9f * cost(k_est, q_est))) best.kv = k_est, best.rows = q_est;
  return best;
}
// dQ and dK / dV one after the other, each with the chip to itself
static float gn_two_us(const Params& p, bool bf, int32_t max_len) {
  const float rows = gn_plan(p, bf, max_len, true).us;
  if (bf && gn_one_term(p)) {   // (the kernel of pages of 128 has two roles per pair of waves and cuts the rows of a page into slices; 256 workgroups at a time)
    const int64_t wgs = (int64_t)gn_key_units(p, max_len) * p.Hkv;
    const float stages = (float)p.C * p.G / 64.f;
    int64_t n = 256 / wgs;
    n = n > 16 ? 16 : n > stages ? (int64_t)stages : n;
    n = n < 1 ? 1 : n;
    return rows + (float)((wgs * n + 255) / 256) * stages / n * 1.75f + 16.f;
  }
  const int64_t slots = gn_slots(p, bf);
  const GnShare k = gn_key_share(p, bf, max_len, gn_head_slots(p, bf));
  return (rows + (float)(((int64_t)k.n * p.Hkv + slots - 1) / slots) * gn_key_us(p, bf, k.most)) * (bf && p.D == 64 ? 1.2f : 1.f) + 16.f;
}
// bf16 pages of 128: the one launch forms dS from P before P is rounded, the kernels for many rows and keys after: dK against 64 bits 1.66e-3 and 2.35e-3.  Up to half of the workgroups' number
// the faster of the two; beyond that the calls that one launch serves with as many splits of every unit as of any other, and of every row tile (estimated as such), and no others: calls of that
// size agree to 2e-3 with the same lists given per query page, which have the other kernels only.  (It would be faster there, too: 28 / 4 heads, 512 rows, 10 pages 60 us against 70; 4 / 4, 1024
// rows, 30 pages 56 against 67.)  two: the others' estimate.
static bool gn_pair_even(const Params& p, int32_t max_len, float two) {
  const int32_t wq = gn_tiles(p.C, p.G, p.P, p.m, 0) * p.Hkv, wk = gn_key_units(p, max_len) * p.Hkv;
  if (2 * wq > 256 || 2 * wk > 256) return false;
  const float nt = (max_len - 0.5f * p.m) * p.P / 64.f, stages = (float)p.C * p.G / 64.f;
  for (int32_t nk = 1; nk <= 16 && (nk == 1 || nk <= stages) && wk * nk + wq <= 256; ++nk) {
    int32_t ns = (256 - wk * nk) / wq;
    ns = ns > 32 ? 32 : ns > nt ? (nt < 1.f ? 1 : (int32_t)nt) : ns;
    const float tq = (nt / ns > 1.f ? nt / ns : 1.f) * 1.2f + 6.f, tk = (stages / nk > 1.f ? stages / nk : 1.f) * 2.6f + 8.f;
    if ((tq > tk ? tq : tk) + (wk * nk * 2.f + wq * ns) * p.D * 2.56e-4f < two) return true;
  }
  return false;
}
// What a backward takes unless it goes by units: the one launch, if `one`.  A call is planned once (0.3 to 3 us, 12 at most; 100 to 180 where the parts of every row tile were counted).
struct GnBackward { GnPair pair; bool one; float us; };
static GnBackward gn_backward(const Params& p, bool bf, int32_t max_len) {
  const GnPair pair = gn_pair(p, bf, max_len);
  const float two = gn_two_us(p, bf, max_len);
  bool one = pair.us < two;
  if (bf && gn_one_term(p) && pair.us < 1e29f) {
    const bool half = 2 * (gn_tiles(p.C, p.G, p.P, p.m, 0) + gn_key_units(p, max_len)) <= gn_slots(p, bf) / p.Hkv;
    one = (half && one) || gn_pair_even(p, max_len, two - 7.f);   // (7 us of the estimate are what the launches after those of its constants took)
  }
  return {pair, one, one ? pair.us : two};
}

// The backward by units (bwd_units_kernel): units per launch, ranges per KV head -- as many workgroups as run at once --, and the estimate of its time in
// microseconds.  A stage of 32 rows x 128 keys takes STAGE (head dim 64: with two workgroups on a compute unit), the partial sums (written, then read) BYTES a
// byte, K, V and the gradient pool POOL; fewer ranges than fit leave fewer partial sums to add.  Fitted to 35 shapes (2 / 1 to 28 / 4 heads, chunks of
// 16 to 2048, lists of 1K to 65K tokens): right to 10 % for most, 15 to 30 % low where a unit has only a few stages at head dim 64.
// Partial sums of dQ take at most UNITS_ROOM, the slots of dK / dV half of it: a launch then still has UNITS_ROOM / 16 KiB = 32768 stages, 128 per workgroup.  In one launch 28 / 4 heads,
// chunk 512, 100 pages take 1.37 ms and 842 MB of workspace, in two 1.43 and 449; chunk 2048, 40 pages 1.86 and 1317 MB, 1.84 and 540 (half this
// room: 1.89 and 361); chunk 2048, 200 pages 10.8 ms and 630 MB, for which one launch would need 6 GB.
constexpr size_t UNITS_ROOM = (size_t)512 << 20;
struct GnUnits { int32_t un, ranges; float us; };
static inline size_t gn_delta_bytes(const Params& p) { return gn_up((size_t)p.Hq * p.C * sizeof(float)); }
static int32_t gn_row_stages(const Params& p) { return (int32_t)(((int64_t)p.C * p.G + 31) / 32); }
static size_t gn_row_img_bytes(const Params& p) { return gn_up((size_t)p.Hkv * gn_row_stages(p) * 6 * 32 * p.D * 2); }
static size_t gn_unit_dq_bytes(const Params& p) { return (size_t)gn_tiles(p.C, p.G, p.P, p.m, 0) * p.Hkv * GN_ROWS * 128 * 4; }   // (at head dim 64 two per unit)
static size_t gn_unit_slot_bytes(const Params& p) { return (size_t)p.Hkv * 2 * GN_ROWS * p.D * 4; }
static int32_t gn_units_most(const Params& p) {   // ranges that run at once
  const int32_t n = (p.D == 128 ? 256 : 512) / p.Hkv;
  return n < 1 ? 1 : n;
}
// what a call needs whose launches take un units each
static size_t gn_units_bytes(const Params& p, int32_t un) {
  return gn_delta_bytes(p) + gn_row_img_bytes(p) + (size_t)(gn_units_most(p) + un) * gn_unit_slot_bytes(p) + un * gn_unit_dq_bytes(p);
}
static int32_t gn_units_fit(const Params& p, int32_t max_len) {   // most units of a launch
  const size_t slots = 2 * gn_unit_slot_bytes(p), each = gn_unit_dq_bytes(p) > slots ? gn_unit_dq_bytes(p) : slots;
  const size_t units = gn_key_units(p, max_len), fit = UNITS_ROOM / each;
  return (int32_t)(fit < 1 ? 1 : fit < units ? fit : units);
}
static GnUnits gn_units(const Params& p, int32_t max_len, size_t room) {   // room: of the workspace
  GnUnits best = {0, 1, 1e30f};
  const int32_t units = gn_key_units(p, max_len);
  if (units < 1 || gn_units_bytes(p, 1) > room) return best;
  const size_t more = 1 + (room - gn_units_bytes(p, 1)) / (gn_unit_slot_bytes(p) + gn_unit_dq_bytes(p));
  int32_t fit = gn_units_fit(p, max_len);
  if (more < (size_t)fit) fit = (int32_t)more;
  const int32_t launches = (units + fit - 1) / fit, un = (units + launches - 1) / launches;
  constexpr float START = 22.f, GROUP = 25.f, BYTES = 3e-7f, POOL = 2e-7f;
  const float STAGE = p.D == 128 ? 6.f : 5.6f, slot = (float)gn_unit_slot_bytes(p);
  const int64_t S = gn_row_stages(p), most = gn_units_most(p), full = (int64_t)un * S;
  int64_t last = (int64_t)(units - un * (launches - 1)) * S;   // stages of a head in the last launch, if its list is full: fewer of the units that hold the chunk's own pages
  for (int32_t u = (int32_t)((int64_t)(max_len - p.m) * p.P / GN_ROWS); u < units; ++u) {
    const int64_t tok = (int64_t)u * GN_ROWS - (int64_t)(max_len - p.m) * p.P;
    last -= tok > 0 ? tok * p.G / 32 : 0;
  }
  last = last < 1 ? 1 : last;
  const float dq = (float)units * (float)gn_unit_dq_bytes(p) * BYTES;
  const int64_t q0 = ((launches > 1 ? full : last) + most - 1) / most;
  for (int64_t q = q0; q < q0 + 4; ++q) {
    const int64_t r = ((launches > 1 ? full : last) + q - 1) / q;
    const float us = START + (launches - 1) * ((float)q * STAGE + GROUP) + (float)((last + r - 1) / r) * STAGE + dq +
                     (float)(r * launches + units) * slot * BYTES + units * slot * 3.f * POOL;
    if (us < best.us) best = {un, (int32_t)r, us};
  }
  return best;
}

// Against the one-launch backward, or dQ and dK / dV one after the other (us: their estimate).  On the 35 shapes above what is chosen is the better one, or within 3 %: calls of 50 us
// and less are up to 30 % faster without, from 60 us on this is 1.2 to 2.3 times as fast: 28 / 4 heads, chunk 512, 16 + 4 pages of 128: 576 -> 284 us, 300 pages
// 7.7 -> 4.2 ms; 14 / 2 heads of 64 dims, chunk 1664, 14 + 13 pages of 128: 598 -> 323.
static bool gn_takes_units(const GnUnits& u, float us) { return u.us < 1e29f && u.us < us; }

static size_t gn_row_blocks(const Params& p) { return (size_t)gn_tiles(p.C, p.G, p.P, p.m, p.qp) * p.Hkv * 4; }
// splits that fit `bytes` of partial results of `per` bytes each (at least 1: no partial results)
static int32_t gn_fit(size_t bytes, size_t per) { return (int32_t)(bytes / per > 32 ? 32 : bytes / per < 2 ? 1 : bytes / per); }
static size_t gn_row_part_bytes(const Params& p, int32_t split) { return split > 1 ? split * gn_row_blocks(p) * 32 * p.D * 4 : 0; }
// The fp32 forward in terms: splits of the key range, how many launches walk it (each with the image of its own part of the list, 1.5 times what
// the keys and values there take and at most IMAGE_ROOM; the sums go on from launch to launch), and the estimate of the time in microseconds, the layout of the terms included.  Two workgroups of a compute unit take `unit` for a
// tile of 32 keys each (192 matrix instructions per SIMD); 512 run at a time.
constexpr size_t IMAGE_ROOM = (size_t)512 << 20;
struct GnF3Plan { int32_t n, launches; float us; };
static size_t gn_f3_tile_bytes(const Params& p) { return (size_t)p.Hkv * 6 * 32 * p.D * 2; }
static int32_t gn_f3_fit(const Params& p, int32_t max_len) {   // most tiles of a launch
  const size_t n = gn_f3_tiles(p, max_len), fit = IMAGE_ROOM / gn_f3_tile_bytes(p);
  return (int32_t)(fit < 1 ? 1 : fit < n ? fit : n);
}
static int32_t gn_f3_launches(const Params& p, int32_t max_len) {
  const int32_t fit = gn_f3_fit(p, max_len);
  return (gn_f3_tiles(p, max_len) + fit - 1) / fit;
}
static size_t gn_f3_img_bytes(const Params& p, int32_t max_len) {   // (not less for a longer list, whose launches may take fewer)
  return gn_up((size_t)gn_f3_fit(p, max_len) * gn_f3_tile_bytes(p));
}
static size_t gn_f3_split_bytes(const Params& p) { return gn_row_part_bytes(p, 2) / 2 + gn_row_blocks(p) * 32 * 8; }
static size_t gn_f3_odd_bytes(const Params& p, int32_t max_len) { return gn_up((size_t)gn_f3_fit(p, max_len) * p.Hkv * 4); }   // a word per tile
static size_t gn_f3_bytes(const Params& p, int32_t max_len, int32_t n) {
  return gn_f3_img_bytes(p, max_len) + gn_f3_odd_bytes(p, max_len) + (n > 1 || gn_f3_launches(p, max_len) > 1 ? n * gn_f3_split_bytes(p) : 0);
}
static GnF3Plan gn_f3_plan(const Params& p, bool bf, int32_t max_len, size_t room) {   // room: of the workspace
  GnF3Plan best = {1, 1, 1e30f};
  if (bf || p.qp || gn_f3_bytes(p, max_len, 1) > room) return best;
  constexpr float RAMP = 6.f, LAUNCH = 3.f, PART = 2.56e-4f, LAYOUT = 5.f, BYTES = 5e-7f;
  const float unit = 3.3f * (p.D == 128 ? 1.f : 0.55f), all = (float)gn_f3_tiles(p, max_len), avg = (max_len - 0.5f * p.m) * p.P / 32.f;
  const int32_t tiles = gn_tiles(p.C, p.G, p.P, p.m, 0), wgs = tiles * p.Hkv, launches = gn_f3_launches(p, max_len);
  for (int32_t n = 1; n <= 32 && (n == 1 || n * launches <= all); ++n) {
    if (gn_f3_bytes(p, max_len, n) > room) break;
    const float x = (float)wgs * n, extra = n > 1 ? LAUNCH + x * p.D * PART : 0.f, mine = avg / (n * launches) > 1.f ? avg / (n * launches) : 1.f;
    const float us = launches * (gn_rounds(x / 512.f, 0.55f, 0.45f, 0.55f, 0.45f) * mine * unit + ceilf(x / 512.f) * RAMP + LAYOUT) +
                     (launches - 1) * x * p.D * PART + extra + all * (float)gn_f3_tile_bytes(p) * BYTES;
    if (us < best.us) best = {n, launches, us};
  }
  return best;
}
// Against the kernel of every shape, each by its own estimate (S is formed in terms by both, so the backward need not follow).  Timed on the 35 shapes above,
// the estimates of both are low alike: below 1 the terms are the better one or at most 2 % slower.  The layout of the terms is what few rows do not
// pay for: 28 / 4 heads of 128, 16 tokens against 16K 82 us with it and 72 without, 128 tokens 180 and 210; 8 / 4 heads, 64 tokens against 64K 300 and 234.
// Up to 1.22 where the backward takes terms: calls of 27 to 37 us, up to 5 us slower than they could be (6 / 3 heads, chunk 320, 30 pages of 64: 36.7
// and 31.1), with which the tests reach the edges of this kernel.
static bool gn_takes_f3(const Params& p, bool bf, int32_t max_len, const GnF3Plan& f) {
  if (f.us > 1e29f) return false;
  const float other = gn_plan(p, bf, max_len, false).us;
  return f.us < other || (f.us < 1.22f * other && gn_takes_units(gn_units(p, max_len, SIZE_MAX), gn_backward(p, bf, max_len).us));
}
size_t fwd_generic_workspace_bytes(const Params& p, bool bf, int32_t max_len) {
  const int32_t s = gn_plan(p, bf, max_len, false).n;
  const size_t plain = s > 1 ? gn_row_part_bytes(p, s) + s * gn_row_blocks(p) * 32 * 8 : 256;
  const GnF3Plan f = gn_f3_plan(p, bf, max_len, SIZE_MAX);
  const size_t terms = gn_takes_f3(p, bf, max_len, f) ? gn_f3_bytes(p, max_len, f.n) : 0;
  return terms > plain ? terms : plain;
}
size_t dq_generic_part_bytes(const Params& p, bool bf, int32_t max_len) { return gn_row_part_bytes(p, gn_plan(p, bf, max_len, true).n); }
// partial sums of the shares of keys, and of rows
static size_t gn_key_slot_bytes(const Params& p) { return (size_t)2 * part_key_blocks(p) * 32 * p.D * 4; }
static size_t gn_key_part_bytes(const Params& p, int32_t units, const GnShare& w) {   // (0: no more parts than units)
  const size_t slots = p.qp ? (size_t)p.Hkv * qp_max_pslots(p, p.sel_stride) : w.n <= units ? 0 : (size_t)p.Hkv * w.n;
  return gn_up(slots * gn_key_slot_bytes(p));
}
// the parts of dK / dV in a kernel of their own that `room` has space for
static GnShare gn_key_share_in(const Params& p, bool bf, int32_t max_len, size_t room) {
  const size_t fit = room / (gn_key_slot_bytes(p) * p.Hkv);
  const int32_t slots = gn_head_slots(p, bf);
  return gn_key_share(p, bf, max_len, fit < (size_t)slots ? (int32_t)fit : slots);
}
static size_t gn_pair_bytes(const Params& p, int32_t max_len, const GnPair& t) {
  const bool whole = t.rows.n <= gn_tiles(p.C, p.G, p.P, p.m, 0);
  return gn_key_part_bytes(p, gn_key_units(p, max_len), t.kv) + (whole ? 0 : (size_t)p.Hkv * t.rows.n * GN_ROWS * p.D * 4);
}
// What those partial sums take at most for any list of max_len entries or fewer, which may have more parts than the longest: the workspace of a history that grows is asked for once (28 / 4 heads of 64 dims,
// chunk 512, 64 + 16 pages of 32 in that of 284 + 16 pages, 14.7 MB without this: 158 us instead of 71; 6 / 2 heads of 128, chunk 128, 2K tokens in that of 8K 53 instead of 27).
static size_t gn_key_room(const Params& p, bool bf, int32_t max_len) {
  const int64_t units = gn_key_units(p, max_len), slots = gn_head_slots(p, bf);
  if (p.qp || gn_key_units(p, p.m) >= slots) return gn_key_part_bytes(p, 0, {0, 1});
  return gn_up((size_t)p.Hkv * (size_t)(16 * units < slots ? 16 * units : slots) * gn_key_slot_bytes(p));
}
static size_t gn_pair_room(const Params& p, bool bf, int32_t max_len) {
  const int64_t per = gn_slots(p, bf) / p.Hkv, wq = gn_tiles(p.C, p.G, p.P, p.m, 0), units = gn_key_units(p, max_len);
  if (p.qp || wq + gn_key_units(p, p.m) > per) return 0;
  const int64_t kv = 16 * units < per - wq ? 16 * units : per - wq, rows = GN_ROW_PARTS * wq < per - kv ? GN_ROW_PARTS * wq : per - kv;
  return gn_up((size_t)p.Hkv * kv * gn_key_slot_bytes(p)) + (size_t)p.Hkv * rows * GN_ROWS * p.D * 4;
}
size_t bwd_pair_room(const Params& p, bool bf, int32_t max_len) { return gn_pair_room(p, bf, max_len); }
size_t bwd_generic_min_bytes(const Params& p) { return gn_up((size_t)p.Hq * p.C * sizeof(float)) + gn_key_part_bytes(p, 0, {0, 1}); }
size_t bwd_generic_workspace_bytes(const Params& p, bool bf, int32_t max_len) {
  const size_t delta = gn_up((size_t)p.Hq * p.C * sizeof(float)), pair = gn_pair_room(p, bf, max_len);
  const size_t two = delta + dq_generic_part_bytes(p, bf, max_len) + gn_key_room(p, bf, max_len);
  const size_t most = pair > two ? pair : two;
  if (bf || p.qp) return most;
  const GnUnits u = gn_units(p, max_len, SIZE_MAX);
  const size_t units = gn_takes_units(u, gn_backward(p, bf, max_len).us) ? gn_units_bytes(p, gn_units_fit(p, max_len)) : 0;   // (not less for a longer list, whose launches may take fewer)
  return units > most ? units : most;
}

// terms of a probability (GnP) where a shape has no kernels of its own
template <typename T> constexpr int GN_TERMS = sizeof(T) == 4 ? 1 : 3;

template <typename T, int D, int KH, int NT>
static hipError_t fwd_launch(const Params& p, int32_t tiles, int32_t ns, int32_t len, float* part, float2* ml, hipStream_t st) {
  typedef GnRow<T, D, KH> R;
  static DeviceOnce lds_once;
  if (hipError_t e = ensure_max_dynamic_lds(lds_once, (const void*)fwd_generic_kernel<T, D, KH, NT>, R::LDS); e != hipSuccess) return e;
  fwd_generic_kernel<T, D, KH, NT><<<dim3((unsigned)tiles * p.Hkv * ns), dim3(R::THREADS), R::LDS, st>>>(p, tiles, ns, __builtin_ctz(p.P), len, part, ml);
  return hipGetLastError();
}
template <typename T, int D, int NT = GN_TERMS<T>>
static hipError_t fwd_generic(const Params& p, int32_t max_len, void* ws, size_t ws_bytes, const char* name, hipStream_t st) {
  // (the forward also runs without a workspace)
  const GnPlan sp = gn_plan(p, Gn<T, D>::BF, max_len, false, ws ? gn_fit(ws_bytes, gn_row_blocks(p) * 32 * (p.D * 4 + 8)) : 1);
  const int32_t ns = sp.n;
  float* part = (float*)ws;
  float2* ml = (float2*)((unsigned char*)ws + gn_row_part_bytes(p, ns));
  const int32_t tiles = gn_tiles(p.C, p.G, p.P, p.m, p.qp), len = gn_list_len(p, max_len);
  ProfScope prof_(name, st);
  hipError_t e = sp.groups == 2 ? fwd_launch<T, D, 2, NT>(p, tiles, ns, len, part, ml, st) : fwd_launch<T, D, 1, NT>(p, tiles, ns, len, part, ml, st);
  if (e == hipSuccess && ns > 1) {
    fwd_combine_kernel<T, D><<<dim3((unsigned)(gn_row_blocks(p))), dim3(64 * COMBINE_WAVES), 0, st>>>(p, tiles, ns, part, ml, __builtin_ctz(p.P));
    e = hipGetLastError();
  }
  return e;
}
// *done: whether the call was taken (it has the room, and the estimate is below that of the fp32 matrix pipe)
template <int D> static hipError_t fwd_terms(const Params& p, int32_t max_len, void* ws, size_t ws_bytes, const char* name, hipStream_t st, bool* done) {
  typedef GnF3<D> F;
  const GnF3Plan f = ws ? gn_f3_plan(p, false, max_len, ws_bytes) : GnF3Plan{1, 1, 1e30f};
  if (!gn_takes_f3(p, false, max_len, f)) return hipSuccess;
  *done = true;
  ProfScope prof_(name, st);
  static DeviceOnce once, once_on;
  if (hipError_t e = ensure_max_dynamic_lds(once, (const void*)fwd_terms_kernel<D, true>, F::LDS); e != hipSuccess) return e;
  if (hipError_t e = ensure_max_dynamic_lds(once_on, (const void*)fwd_terms_kernel<D, false>, F::LDS); e != hipSuccess) return e;
  const int32_t tiles = gn_tiles(p.C, p.G, p.P, p.m, 0), n_tiles = gn_f3_tiles(p, max_len), lp = __builtin_ctz(p.P);
  unsigned char* img = (unsigned char*)ws;
  unsigned char* odd = img + gn_f3_img_bytes(p, max_len);
  float* part = (float*)(odd + gn_f3_odd_bytes(p, max_len));
  float2* ml = (float2*)((unsigned char*)part + (size_t)f.n * gn_row_blocks(p) * 32 * p.D * 4);
  for (int32_t l = 0; l < f.launches; ++l) {
    const int32_t t0 = (int32_t)((int64_t)n_tiles * l / f.launches), nt = (int32_t)((int64_t)n_tiles * (l + 1) / f.launches) - t0;
    { ProfScope layout_("kv_terms", st); kv_terms_kernel<D><<<dim3((unsigned)(nt * p.Hkv)), dim3(256), 0, st>>>(p, t0, nt, lp, img, odd); }
    if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
    {
      ProfScope fwd_("fwd_terms", st);
      auto kernel = l ? fwd_terms_kernel<D, false> : fwd_terms_kernel<D, true>;
      kernel<<<dim3((unsigned)(tiles * p.Hkv * f.n)), dim3(256), F::LDS, st>>>(p, tiles, f.n, lp, max_len, t0, nt, l + 1 == f.launches, img, (const int32_t*)odd, part, ml);
    }
    if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  }
  if (f.n == 1) return hipSuccess;
  fwd_combine_kernel<float, D, bf16_t><<<dim3((unsigned)(gn_row_blocks(p))), dim3(64 * COMBINE_WAVES), 0, st>>>(p, tiles, f.n, part, ml, lp);
  return hipGetLastError();
}
hipError_t launch_fwd_generic(const Params& p, bool bf, int32_t max_len, void* ws, size_t ws_bytes, hipStream_t st) {
  const char* name = "attn_fwd_generic";
  bool done = false;
  if (!bf)
    if (hipError_t e = p.D == 128 ? fwd_terms<128>(p, max_len, ws, ws_bytes, name, st, &done) : fwd_terms<64>(p, max_len, ws, ws_bytes, name, st, &done); done) return e;
  if (bf) return p.D == 128 ? fwd_generic<bf16_t, 128>(p, max_len, ws, ws_bytes, name, st) : fwd_generic<bf16_t, 64>(p, max_len, ws, ws_bytes, name, st);
  return p.D == 128 ? fwd_generic<float, 128>(p, max_len, ws, ws_bytes, name, st) : fwd_generic<float, 64>(p, max_len, ws, ws_bytes, name, st);
}
hipError_t launch_fwd_generic_bf16_128(const Params& p, int32_t max_len, void* ws, size_t ws_bytes, hipStream_t st) {
  return fwd_generic<bf16_t, 128, 1>(p, max_len, ws, ws_bytes, "attn_fwd_split", st);
}

template <typename T, int D, int KH, int NT>
static hipError_t dq_launch(const Params& p, int32_t tiles, int32_t ns, int32_t len, float* part, float* bias, int32_t n_stages, hipStream_t st) {
  typedef GnRow<T, D, KH> R;
  static DeviceOnce lds_once;
  if (hipError_t e = ensure_max_dynamic_lds(lds_once, (const void*)dq_generic_kernel<T, D, KH, NT>, R::LDS); e != hipSuccess) return e;
  dq_generic_kernel<T, D, KH, NT><<<dim3((unsigned)tiles * p.Hkv * ns), dim3(R::THREADS), R::LDS, st>>>(p, tiles, ns, __builtin_ctz(p.P), len, part,
                                                                                                   bias, n_stages);
  return hipGetLastError();
}
template <typename T, int D, int NT = GN_TERMS<T>>
static hipError_t dq_generic(const Params& p, int32_t max_len, float* part, size_t part_bytes, float* bias, int32_t n_stages, int32_t* splits,
                             hipStream_t st) {
  const GnPlan sp = gn_plan(p, Gn<T, D>::BF, max_len, true, gn_fit(part_bytes, gn_row_blocks(p) * 32 * p.D * 4));
  const int32_t tiles = gn_tiles(p.C, p.G, p.P, p.m, p.qp), len = gn_list_len(p, max_len);
  *splits = sp.n;
  if constexpr (Gn<T, D>::RB < 512)   // (fp32 at head dim 128 needs 320 registers: one wave per SIMD)
    if (sp.groups == 2) return dq_launch<T, D, 2, NT>(p, tiles, sp.n, len, part, bias, n_stages, st);
  return dq_launch<T, D, 1, NT>(p, tiles, sp.n, len, part, bias, n_stages, st);
}
hipError_t launch_dq_generic_bf16_128(const Params& p, int32_t max_len, float* part, size_t part_bytes, float* bias, int32_t n_stages,
                                      int32_t* splits, hipStream_t st) {
  return dq_generic<bf16_t, 128, 1>(p, max_len, part, part_bytes, bias, n_stages, splits, st);
}

template <typename T, typename TG, int D, typename L = T>
static hipError_t bwd_finish(const Params& p, int32_t dq_split, const float* dq_part, int32_t kv_units, int32_t kv_split, const float* kv_part,
                             bool redo_keys, hipStream_t st, int32_t u0 = 0, int32_t un = 0, GnShare rows = {0, 1}, GnShare kv = {0, 1}, int32_t max_len = 0) {
  if (rows.n <= gn_tiles(p.C, p.G, p.P, p.m, p.qp)) rows.n = 0;   // (nothing is left)
  if (kv.n > 0 && kv.n <= kv_units) kv_units = 0;
  const int32_t dq_blocks = dq_split > 1 || rows.n ? (int32_t)(gn_row_blocks(p)) : 0;
  const int64_t blocks = dq_blocks + (int64_t)kv_units * p.Hkv * 2 * part_key_blocks(p);
  if (blocks <= 0) return hipSuccess;
  auto run = [&](auto kernel, unsigned waves) {
    kernel<<<dim3((unsigned)blocks), dim3(64 * waves), 0, st>>>(p, gn_tiles(p.C, p.G, p.P, p.m, p.qp), dq_split, dq_part, dq_blocks, kv_split, kv_part,
                                                                __builtin_ctz(p.P), redo_keys, u0, un, rows, kv, max_len);
  };
  if (blocks <= FINISH_FEW) run(bwd_finish_kernel<T, TG, D, L, 8>, 8);
  else run(bwd_finish_kernel<T, TG, D, L, 4>, 4);
  return hipGetLastError();
}
// (the dK / dV slices of pages with kernels of their own: keys are left as those give them)
hipError_t launch_bwd_finish(const Params& p, bool bf, int32_t dq_split, const float* dq_part, int32_t kv_units, int32_t kv_split,
                             const float* kv_part, hipStream_t st) {
#define OOMB_FINISH(T, TG) (p.D == 128 ? bwd_finish<T, TG, 128>(p, dq_split, dq_part, kv_units, kv_split, kv_part, false, st) \
                                       : bwd_finish<T, TG, 64>(p, dq_split, dq_part, kv_units, kv_split, kv_part, false, st))
  if (bf) return p.grad_is_bf16 ? OOMB_FINISH(bf16_t, bf16_t) : OOMB_FINISH(bf16_t, float);
  return p.grad_is_bf16 ? OOMB_FINISH(float, bf16_t) : OOMB_FINISH(float, float);
#undef OOMB_FINISH
}

// The one-launch backward, if the shape takes it and the workspace has room (else *done stays false)
template <typename T, typename TG, int D, int NT = GN_TERMS<T>>
static hipError_t bwd_pair(Params p, const GnBackward& b, int32_t max_len, void* ws, size_t ws_bytes, const char* name, hipStream_t st, bool* done) {
  const GnPair& t = b.pair;
  // (dQ over O: the keys' workgroups would read rows of O that the others have overwritten)
  if (!b.one || dq_overlaps_o(p, Gn<T, D>::BF) || gn_pair_bytes(p, max_len, t) > ws_bytes) return hipSuccess;
  *done = true;
  ProfScope prof_(name, st);
  constexpr int LDS = GnKey<T, D>::LDS > GnRow<T, D, 1>::LDS ? GnKey<T, D>::LDS : GnRow<T, D, 1>::LDS;
  static DeviceOnce once;
  if (hipError_t e = ensure_max_dynamic_lds(once, (const void*)bwd_pair_kernel<T, TG, D, NT>, LDS); e != hipSuccess) return e;
  p.delta = nullptr;
  const GnShares w = {t.kv, t.rows, (float*)ws, (float*)((unsigned char*)ws + gn_key_part_bytes(p, gn_key_units(p, max_len), t.kv))};
  bwd_pair_kernel<T, TG, D, NT><<<dim3((unsigned)((t.kv.n + t.rows.n) * p.Hkv)), dim3(256), LDS, st>>>(p, w, gn_tiles(p.C, p.G, p.P, p.m, 0), __builtin_ctz(p.P), max_len);
  if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  return bwd_finish<T, TG, D>(p, 1, w.row_part, gn_key_units(p, max_len), 1, w.kv_part, true, st, 0, 0, t.rows, t.kv, max_len);
}
hipError_t launch_bwd_pair_bf16_128(const Params& p, int32_t max_len, void* ws, size_t ws_bytes, hipStream_t st, bool* done) {
  const GnBackward b = gn_backward(p, true, max_len);
  return p.grad_is_bf16 ? bwd_pair<bf16_t, bf16_t, 128, 1>(p, b, max_len, ws, ws_bytes, "bwd_pair", st, done)
                        : bwd_pair<bf16_t, float, 128, 1>(p, b, max_len, ws, ws_bytes, "bwd_pair", st, done);
}

template <typename TG, int D>
static hipError_t bwd_units(Params p, const GnBackward& b, int32_t max_len, void* ws, size_t ws_bytes, const char* name, hipStream_t st, bool* done) {
  if (p.qp) return hipSuccess;
  const GnUnits t = gn_units(p, max_len, ws_bytes);
  if (!gn_takes_units(t, b.us)) return hipSuccess;
  *done = true;
  ProfScope prof_(name, st);
  static DeviceOnce once, once_add;
  if (hipError_t e = ensure_max_dynamic_lds(once, (const void*)bwd_units_kernel<D, false>, GnU<D>::LDS); e != hipSuccess) return e;
  if (hipError_t e = ensure_max_dynamic_lds(once_add, (const void*)bwd_units_kernel<D, true>, GnU<D>::LDS); e != hipSuccess) return e;
  const int32_t units = gn_key_units(p, max_len), stages = gn_row_stages(p), lp = __builtin_ctz(p.P);
  p.delta = (float*)ws;   // (formed before anything of dQ is written, which may overlap O, and read again by rows that are formed once more)
  unsigned char* img = (unsigned char*)ws + gn_delta_bytes(p);
  float* kv_part = (float*)(img + gn_row_img_bytes(p));
  float* dq_part = (float*)((unsigned char*)kv_part + (size_t)(t.ranges + t.un) * gn_unit_slot_bytes(p));
  {
    ProfScope terms_("row_terms", st);
    row_terms_kernel<D><<<dim3((unsigned)(stages * p.Hkv)), dim3(256), 0, st>>>(p, stages, img);
  }
  if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  for (int32_t u0 = 0; u0 < units; u0 += t.un) {
    const int32_t n = units - u0 < t.un ? units - u0 : t.un;
    {
      ProfScope units_("bwd_units", st);
      auto kernel = u0 ? bwd_units_kernel<D, true> : bwd_units_kernel<D, false>;
      kernel<<<dim3((unsigned)(p.Hkv * t.ranges)), dim3(256), GnU<D>::LDS, st>>>(p, u0, t.un, t.ranges, lp, img, kv_part, dq_part);
    }
    if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
    // dK / dV of these units, and dQ with the last
    if (hipError_t e = bwd_finish<float, TG, D, bf16_t>(p, u0 + n < units ? 1 : 2, dq_part, n, t.ranges, kv_part, true, st, u0, t.un); e != hipSuccess) return e;
  }
  return hipSuccess;
}

template <typename T, typename TG, int D>
static hipError_t bwd_generic(Params p, int32_t max_len, void* ws, size_t ws_bytes, hipStream_t st) {
  const char* name = "attn_bwd_generic";
  bool done = false;
  const GnBackward b = gn_backward(p, Gn<T, D>::BF, max_len);
  if constexpr (sizeof(T) == 4)
    if (hipError_t e = bwd_units<TG, D>(p, b, max_len, ws, ws_bytes, name, st, &done); done || e != hipSuccess) return e;
  if (hipError_t e = bwd_pair<T, TG, D>(p, b, max_len, ws, ws_bytes, name, st, &done); done || e != hipSuccess) return e;
  ProfScope prof_(name, st);
  static DeviceOnce once_kv;
  if (hipError_t e = ensure_max_dynamic_lds(once_kv, (const void*)dkv_generic_kernel<T, TG, D, GN_TERMS<T>>, GnKey<T, D>::LDS); e != hipSuccess) return e;
  // [Delta][dK / dV parts][dQ partials]; with less room than the parts of this call need there are as many as fit
  unsigned char* at = (unsigned char*)ws;
  p.delta = (float*)at;
  at += gn_up((size_t)p.Hq * p.C * sizeof(float));
  size_t left = ws_bytes - gn_up((size_t)p.Hq * p.C * sizeof(float));
  const GnShares w = {gn_key_share_in(p, Gn<T, D>::BF, max_len, left), {0, 1}, (float*)at, nullptr};
  const int32_t all = gn_key_units(p, max_len);
  float* dq_part = (float*)(at + gn_key_part_bytes(p, all, w.kv));
  left -= gn_key_part_bytes(p, all, w.kv);
  const int32_t units = p.qp ? p.max_units : gn_key_units(p, max_len);
  if (p.d_q != p.o && dq_overlaps_o(p, Gn<T, D>::BF)) {
    if (hipError_t e = launch_delta<T, D>(p, st); e != hipSuccess) return e;
    p.delta_given = 1;
  }
  int32_t ns = 1;
  hipError_t e = dq_generic<T, D>(p, max_len, dq_part, left, nullptr, 0, &ns, st);
  if (e != hipSuccess) return e;
  dkv_generic_kernel<T, TG, D, GN_TERMS<T>><<<dim3((unsigned)(p.qp ? units : w.kv.n) * p.Hkv), dim3(256), GnKey<T, D>::LDS, st>>>(p, w, __builtin_ctz(p.P), max_len);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  return bwd_finish<T, TG, D>(p, ns, dq_part, p.qp ? p.max_multi : units, 1, w.kv_part, true, st, 0, 0, {0, 1}, w.kv, max_len);
}
// max_len: host-side upper bound of the list length (of the union with one list per query page)
hipError_t launch_bwd_generic(const Params& p, bool bf, int32_t max_len, void* ws, size_t ws_bytes, hipStream_t st) {
#define OOMB_BWD(T, TG) (p.D == 128 ? bwd_generic<T, TG, 128>(p, max_len, ws, ws_bytes, st) : bwd_generic<T, TG, 64>(p, max_len, ws, ws_bytes, st))
  if (bf) return p.grad_is_bf16 ? OOMB_BWD(bf16_t, bf16_t) : OOMB_BWD(bf16_t, float);
  return p.grad_is_bf16 ? OOMB_BWD(float, bf16_t) : OOMB_BWD(float, float);
#undef OOMB_BWD
}

// Whether a shape with kernels of its own (bf16, P = D = 128) is faster here.  Those take 256 rows per workgroup
// and 2.0 us (dQ: 2.55) per 64 keys, 7 to 13 % less than these with the chip full, but do not split: with
// workgroups for less than a round, or for little more than one, they leave compute units idle.  They also need the
// page images (forward) or the row statistics (dQ) of a kernel before them: 20 ns per page and head.  With one list per query page the
// images are those of the union of a head's lists, whose length the host does not know: 2.5 lists (32 lists of 160 entries of the 1M
// votes workload: 400 pages; max_len, the worst case, would be 5120, 410 us for a kernel of 32), after the maps of those lists.
// The constants are fitted to both kernels timed at 28 / 4, 32 / 8, 14 / 2, 6 / 2 and 4 / 4 heads, 1 to 64 query pages, 8 to 256 past pages
// (289 shapes; 180 with lists of their own per query page).  What is chosen is on average 0.2 % slower than the better one, at most
// 8 % (14 % with lists per query page) -- forward; with the first constants, of fewer shapes, 0.7 % and 30 %, e.g. 14 / 2, 48
// query pages, 64 past pages: these 717, those 552 us.  dQ: 0.2 %, at most 16 %.
bool rows_take_generic(const Params& p, int32_t max_len, bool dq) {
  const float r = row_tiles_per_head(p.C, p.G, p.m, p.qp) * p.Hkv / 256.f;
  const float avg = 2.f * ((float)gn_list_len(p, max_len) - 0.5f * p.m), plan = gn_plan(p, true, max_len, dq).us;
  if (dq) return plan < 0.97f * (gn_rounds(r, 0.78f, 0.2f, 0.6f, 0.3f) * avg * 2.55f + ceilf(r) * 8.f + 4.f + (float)p.C * p.Hq * 7e-5f);
  const float lists = 2.5f * (float)p.sel_stride, images = p.qp && lists < (float)max_len ? lists : (float)max_len;
  const float before = (p.qp ? 60.f : 30.f) + (float)p.Hkv * images * 0.02f;
  return plan < 0.98f * (gn_rounds(r, 0.6f, 0.28f, 0.35f, 0.45f) * avg * 2.0f + before);
}

}  // namespace oomb
