// Offloaded KV cache (paper Sec. 4.3): the K / V pools and their gradient pools live in
// pinned host memory; the pages a chunk attends are fetched into small device staging
// pools, the attention kernels run on those, and the gradients of the fetched pages are
// added back to the host pools.
//
// The copies are kernels that read (write) the pinned host memory directly over the
// host link with 16-byte accesses, tile by tile ((page, KV head) = P rows): the
// page list never leaves the device, so no host round trip sits between the selection
// and the transfer, and a fetch on its own stream overlaps whatever computes meanwhile.
// They run on a FEW workgroups that walk the tiles: host accesses take microseconds, and
// a grid that covers the chip fills the memory pipeline of every compute unit with them,
// which stalls a concurrently running kernel almost completely (measured: with 128 or more
// workgroups nothing overlaps); 10 to 12 workgroups of 256 threads saturate the link (55 GB/s in, 47 GB/s each
// way) and disturb only the compute units they sit on.
//   offload_plan       which KV heads hold each page (bit mask over the lists: one list per
//                      KV head, or one per KV head and query page) and the staging slot of
//                      every held page (ascending logical page order), one workgroup.  The
//                      slot table is the page table of the staging pools; it never points
//                      past their capacity (a page that does not fit gets slot 0 and the
//                      count of held pages tells the caller)
//   offload_fetch      stage[slot][g] = host[page_table[l]][g]  (K and V) for the held
//                      (page, head) tiles, optionally zeroing the gradient staging tiles
//   offload_writeback  host[page_table[l]][g] += stage[slot][g]  (dK and dV)
#include <cstdlib>

#include "common.h"
#include "launch.h"

namespace oomb {

constexpr int PLAN_THREADS = 1024;

// lists: p.sel [Hkv][lists_per_head][p.sel_stride], p.sel_count [Hkv][lists_per_head]
__global__ __launch_bounds__(PLAN_THREADS) void offload_plan_kernel(Params p, int32_t lists_per_head, int32_t stage_cap,
                                                                    int32_t* __restrict__ stage_table,
                                                                    int32_t* __restrict__ slot_pages,
                                                                    uint32_t* __restrict__ head_mask,
                                                                    int32_t* __restrict__ n_slots) {
  __shared__ int32_t wave_tot[PLAN_THREADS / 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int32_t n = (int32_t)p.n;
  for (int32_t l = tid; l < n; l += PLAN_THREADS) head_mask[l] = 0u;
  __syncthreads();
  const int32_t per_head = lists_per_head * p.sel_stride;
  for (int g = 0; g < p.Hkv; ++g)
    for (int32_t e = tid; e < per_head; e += PLAN_THREADS) {
      const int32_t q = e / p.sel_stride, j = e - q * p.sel_stride;
      if (j >= p.sel_count[g * lists_per_head + q]) continue;
      const int32_t l = p.sel[(int64_t)g * per_head + e];
      if (l >= 0 && l < n) atomicOr(&head_mask[l], 1u << g);  // (a bit set: independent of the order)
    }
  __syncthreads();
  // exclusive scan of "held" over the logical pages: every thread takes a run of consecutive pages
  const int32_t per = (n + PLAN_THREADS - 1) / PLAN_THREADS;
  const int32_t l0 = tid * per < n ? tid * per : n, l1 = l0 + per < n ? l0 + per : n;
  int32_t mine = 0;
  for (int32_t l = l0; l < l1; ++l) mine += head_mask[l] != 0u;
  int32_t inc = mine;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int32_t t = __shfl_up(inc, o, 64);
    if (lane >= o) inc += t;
  }
  if (lane == 63) wave_tot[wave] = inc;
  __syncthreads();
  int32_t before = 0, total = 0;
  for (int w = 0; w < PLAN_THREADS / 64; ++w) {
    const int32_t t = wave_tot[w];
    if (w < wave) before += t;
    total += t;
  }
  int32_t at = before + inc - mine;
  for (int32_t l = l0; l < l1; ++l) {
    if (head_mask[l]) {
      stage_table[l] = at < stage_cap ? at : 0;
      if (at < stage_cap) slot_pages[at] = l;
      ++at;
    } else {
      stage_table[l] = -1;
    }
  }
  if (tid == 0) {
    n_slots[0] = total < stage_cap ? total : stage_cap;  // slots in use
    n_slots[1] = total;                                   // pages held: more than stage_cap = overflow
  }
}

// Tile (slot s, KV head g): P rows of D elements, in granules of 16 bytes.  The workgroups walk the held tiles with a stride of
// `step`; a batch is BATCH granules per thread and tensor.  The link needs about 120 KB of reads under way, and a wave waits for
// the stores that it issued before a load as well (one counter): so the loads of a batch are issued before the stores of the
// batch in front of it, over the ends of tiles too.
constexpr int BATCH = 4, TRANSFER_THREADS = 256;
typedef uint32_t Granule __attribute__((ext_vector_type(4)));
struct TileWalk {
  const Params& p;
  const int32_t* slot_pages;
  const uint32_t* head_mask;
  int32_t tiles, step, tile, shift, total, x;   // granules of a row: 1 << shift; of a tile: total
  int64_t host, stage;                          // element offsets of the tile in the two pools

  __device__ __forceinline__ TileWalk(const Params& p_, const int32_t* slot_pages_, const uint32_t* head_mask_, const int32_t* n_slots,
                                      int32_t stage_cap, int32_t first, int32_t step_, int elem)
      : p(p_), slot_pages(slot_pages_), head_mask(head_mask_), step(step_), tile(first - step_), shift(__builtin_ctz(p_.D * elem / 16)),
        total(p_.P << shift), x(0), host(0), stage(0) {
    tiles = (n_slots[0] < stage_cap ? n_slots[0] : stage_cap) * p.Hkv;
    next_tile();
  }
  __device__ __forceinline__ bool more() const { return tile < tiles; }
  __device__ __forceinline__ void next_tile() {
    x = 0;
    for (tile += step; tile < tiles; tile += step) {
      const int32_t slot = tile / p.Hkv, g = tile - slot * p.Hkv, l = slot_pages[slot];
      if (l < 0 || l >= p.n || !((head_mask[l] >> g) & 1u)) continue;
      host = (int64_t)p.page_table[l] * p.pool_page_stride + (int64_t)g * p.pool_head_stride;
      stage = (int64_t)slot * p.pool_page_stride + (int64_t)g * p.pool_head_stride;
      return;
    }
  }
  __device__ __forceinline__ void next() {
    x += BATCH * TRANSFER_THREADS;
    if (x >= total) next_tile();
  }
  // granule u of this thread in the batch at x0: byte offset inside a tile (a thread past the end repeats its first granule,
  // or the tile's last one)
  __device__ __forceinline__ bool granule(int u, int elem, int64_t& off) const {
    const int32_t e = x + u * TRANSFER_THREADS + (int32_t)threadIdx.x, i = e < total ? e : total - 1;
    off = (int64_t)(i >> shift) * p.pool_tok_stride * elem + 16 * (i & ((1 << shift) - 1));
    return e < total;
  }
};

// K and V of the held tiles into the staging pools.  The last `zero_wgs` workgroups clear the gradient staging tiles instead:
// that is work for the device's memory and would only hold the link's workgroups up.
__global__ __launch_bounds__(TRANSFER_THREADS) void offload_fetch_kernel(Params p, const int32_t* __restrict__ slot_pages,
                                                            const uint32_t* __restrict__ head_mask, const int32_t* __restrict__ n_slots,
                                                            int32_t stage_cap, const unsigned char* __restrict__ a_host,
                                                            const unsigned char* __restrict__ b_host, unsigned char* __restrict__ a_stage,
                                                            unsigned char* __restrict__ b_stage, unsigned char* __restrict__ ga_stage,
                                                            unsigned char* __restrict__ gb_stage, int es, int gs, int zero_wgs) {
  const int movers = gridDim.x - zero_wgs;
  if ((int)blockIdx.x >= movers) {
    TileWalk w(p, slot_pages, head_mask, n_slots, stage_cap, blockIdx.x - movers, zero_wgs, gs);
    for (; w.more(); w.next())
#pragma unroll
      for (int u = 0; u < BATCH; ++u) {
        int64_t off;
        if (!w.granule(u, gs, off)) continue;
        *reinterpret_cast<Granule*>(ga_stage + w.stage * gs + off) = Granule{0, 0, 0, 0};
        *reinterpret_cast<Granule*>(gb_stage + w.stage * gs + off) = Granule{0, 0, 0, 0};
      }
    return;
  }
  TileWalk w(p, slot_pages, head_mask, n_slots, stage_cap, blockIdx.x, movers, es);
  struct Held { Granule a[BATCH], b[BATCH]; int64_t to[BATCH]; } even, odd;
  auto load = [&](Held& h) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < BATCH; ++u) {
      int64_t off;
      const bool in = w.granule(u, es, off);
      h.a[u] = *reinterpret_cast<const Granule*>(a_host + w.host * es + off);
      h.b[u] = *reinterpret_cast<const Granule*>(b_host + w.host * es + off);
      h.to[u] = in ? w.stage * es + off : -1;
    }
    w.next();
  };
  auto store = [&](const Held& h) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < BATCH; ++u)
      if (h.to[u] >= 0) {
        *reinterpret_cast<Granule*>(a_stage + h.to[u]) = h.a[u];
        *reinterpret_cast<Granule*>(b_stage + h.to[u]) = h.b[u];
      }
  };
  if (!w.more()) return;
  load(even);
  for (;;) {
    if (!w.more()) { store(even); break; }
    load(odd);
    store(even);
    if (!w.more()) { store(odd); break; }
    load(even);
    store(odd);
  }
}

// host += staged gradients of the held tiles (dK and dV)
template <typename TG>
__global__ __launch_bounds__(TRANSFER_THREADS) void offload_writeback_kernel(Params p, const int32_t* __restrict__ slot_pages,
                                                                const uint32_t* __restrict__ head_mask, const int32_t* __restrict__ n_slots,
                                                                int32_t stage_cap, unsigned char* a_host, unsigned char* b_host,
                                                                const unsigned char* __restrict__ a_stage,
                                                                const unsigned char* __restrict__ b_stage) {
  constexpr int GS = (int)sizeof(TG), EPG = 16 / GS;  // elements per granule
  TileWalk w(p, slot_pages, head_mask, n_slots, stage_cap, blockIdx.x, gridDim.x, GS);
  struct Held { Granule ha[BATCH], hb[BATCH], sa[BATCH], sb[BATCH]; int64_t to[BATCH]; } even, odd;
  auto load = [&](Held& h) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < BATCH; ++u) {
      int64_t off;
      const bool in = w.granule(u, GS, off);
      h.ha[u] = __builtin_nontemporal_load(reinterpret_cast<const Granule*>(a_host + w.host * GS + off));
      h.hb[u] = __builtin_nontemporal_load(reinterpret_cast<const Granule*>(b_host + w.host * GS + off));
      h.sa[u] = *reinterpret_cast<const Granule*>(a_stage + w.stage * GS + off);
      h.sb[u] = *reinterpret_cast<const Granule*>(b_stage + w.stage * GS + off);
      h.to[u] = in ? w.host * GS + off : -1;
    }
    w.next();
  };
  auto add = [&](unsigned char* at, Granule h, Granule s) {
    TG* he = reinterpret_cast<TG*>(&h);
    const TG* se = reinterpret_cast<const TG*>(&s);
#pragma unroll
    for (int e = 0; e < EPG; ++e) Elem<TG>::store(he + e, Elem<TG>::load(he + e) + Elem<TG>::load(se + e));
    __builtin_nontemporal_store(h, reinterpret_cast<Granule*>(at));
  };
  auto store = [&](const Held& h) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < BATCH; ++u)
      if (h.to[u] >= 0) {
        add(a_host + h.to[u], h.ha[u], h.sa[u]);
        add(b_host + h.to[u], h.hb[u], h.sb[u]);
      }
  };
  if (!w.more()) return;
  load(even);
  for (;;) {
    if (!w.more()) { store(even); break; }
    load(odd);
    store(even);
    if (!w.more()) { store(odd); break; }
    load(even);
    store(odd);
  }
}

// A pointer the device can dereference: device memory, or host memory that the runtime has
// pinned and mapped.  Returns nullptr for anything else (so that nothing is launched on it).
void* device_view(const void* ptr) {
  if (!ptr) return nullptr;
  hipPointerAttribute_t attr;
  if (hipPointerGetAttributes(&attr, ptr) != hipSuccess) {
    (void)hipGetLastError();
    return nullptr;
  }
  if (attr.type != hipMemoryTypeHost && attr.type != hipMemoryTypeDevice && attr.type != hipMemoryTypeManaged) return nullptr;
  return attr.devicePointer;
}

// Workgroups of a transfer kernel (OOMB_OFFLOAD_WGS overrides the default, for experiments), and those that clear gradient
// staging tiles beside a fetch.  Each takes a compute unit from the attention that the transfer hides behind.  Long transfers, those
// that are hidden, take the fewest that carry what the link does; short ones two more, for their ends and host memory that is cold.
// 1M tokens, 28 / 4 heads, 128 pages (2560 tiles of capacity), movers + clearing: step with overlapped transfers / with transfers
// in series / fetch / write-back in ms,
//   12 + 48: 4.85 / 7.24 / 0.76 / 1.81    12 + 4: 4.87 / 7.23 / 0.76 / 1.81    10 + 4: 4.81 / 7.22 / 0.76 / 1.80    8 + 4: 4.77 / 7.33 / 0.77 / 1.88
// (12 that wait for their own stores: 4.79 / 7.43 / 0.87 / 1.89; the step without transfers: 4.35).  Steps in series, inputs that change, 12 + 48,
// 12 + 4, 10 + 48 in us: 384 tiles 541, 541, 560; 564 tiles 616, 618, 642; 1280 tiles 2628, 2631, 2658.
constexpr int ZERO_WGS = 4;
constexpr int64_t LONG_TRANSFER = 2048;   // tiles of the staging pools' capacity
static unsigned transfer_wgs(int64_t tiles) {
  static int forced = -1;
  if (forced < 0) {
    const char* e = std::getenv("OOMB_OFFLOAD_WGS");
    const int v = e ? std::atoi(e) : 0;
    forced = v < 1 ? 0 : v;
  }
  const int v = forced ? forced : tiles >= LONG_TRANSFER ? 10 : 12;
  return (unsigned)(tiles < v ? (tiles > 0 ? tiles : 1) : v);
}

hipError_t launch_offload_plan(const Params& p, int32_t lists_per_head, int32_t stage_cap, int32_t* stage_table,
                               int32_t* slot_pages, uint32_t* head_mask, int32_t* n_slots, hipStream_t st) {
  ProfScope prof_("offload_plan", st);
  offload_plan_kernel<<<dim3(1), dim3(PLAN_THREADS), 0, st>>>(p, lists_per_head, stage_cap, stage_table, slot_pages, head_mask,
                                                              n_slots);
  return hipGetLastError();
}

hipError_t launch_offload_fetch(const Params& p, bool is_bf16, const int32_t* slot_pages, const uint32_t* head_mask,
                                const int32_t* n_slots, int32_t stage_cap, void* host_k, void* host_v, void* stage_k,
                                void* stage_v, void* stage_dk, void* stage_dv, hipStream_t st) {
  ProfScope prof_("offload_fetch", st);
  const int64_t tiles = (int64_t)stage_cap * p.Hkv;
  const int zero_wgs = stage_dk ? (int)(tiles < ZERO_WGS ? tiles : ZERO_WGS) : 0;
  offload_fetch_kernel<<<dim3(transfer_wgs(tiles) + zero_wgs), dim3(TRANSFER_THREADS), 0, st>>>(
      p, slot_pages, head_mask, n_slots, stage_cap, (const unsigned char*)host_k, (const unsigned char*)host_v, (unsigned char*)stage_k,
      (unsigned char*)stage_v, (unsigned char*)stage_dk, (unsigned char*)stage_dv, is_bf16 ? 2 : 4, p.grad_is_bf16 ? 2 : 4, zero_wgs);
  return hipGetLastError();
}

hipError_t launch_offload_writeback(const Params& p, const int32_t* slot_pages, const uint32_t* head_mask,
                                    const int32_t* n_slots, int32_t stage_cap, void* stage_dk, void* stage_dv, void* host_dk,
                                    void* host_dv, hipStream_t st) {
  ProfScope prof_("offload_writeback", st);
  const dim3 grid(transfer_wgs((int64_t)stage_cap * p.Hkv)), block(TRANSFER_THREADS);
  auto* kernel = p.grad_is_bf16 ? &offload_writeback_kernel<bf16_t> : &offload_writeback_kernel<float>;
  kernel<<<grid, block, 0, st>>>(p, slot_pages, head_mask, n_slots, stage_cap, (unsigned char*)host_dk, (unsigned char*)host_dv,
                                 (const unsigned char*)stage_dk, (const unsigned char*)stage_dv);
  return hipGetLastError();
}

}  // namespace oomb
