// GroupGEMM kernels of layer0 (gathered rows of x times W1, activation fused) and layer1 (h times W2), the top-k
// reduction in its three places (a kernel of its own, data-movement workgroups inside the layer1 kernel, the layer1
// epilogue), the one-launch variant of the two GroupGEMMs, and the plan-time weight packing, for gfx950.
//
// Design (paper Section 3.2.1 maps to CDNA4 like this):
//  * one persistent workgroup per compute unit walks a device-built tile schedule; a workgroup is either a
//    GEMM workgroup or a data-movement workgroup, chosen by its index (the division point of Section 3.2.2); the
//    data movement there is to do on one GPU: reducing finished column panels of layer1, prefetching weight panels;
//  * a GEMM workgroup is 4 wavefronts, one per SIMD; a tile is BM x 256 outputs with BM = 256, 192, 128 or 64, and
//    accumulates in fp32 with v_mfma_f32_16x16x32_bf16.  What bounds the kernel is the power limit, and per flop this one draws
//    less than v_mfma_f32_32x32x16_bf16 (half the accumulator traffic; register-only loops: 2061 against 1835 TFLOP/s).  8192
//    tokens of the Mixtral-shaped layer, 32x32x16 -> 16x16x32 and direct epilogue: main loop 91 -> 82 us per layer0
//    tile (1140 cycles per K step in both, 1.60 -> 1.78 GHz), epilogue 5.4 -> 4.2 us, the layer 4338 -> 4077 us;
//    Sweeping the blocks back and forth, one operand of two changing per MFMA, draws less again: 8192 tokens 4042 -> 4005 us, 16384 of
//    them with plain weights 8035 -> 7960, 16384 of 16 experts of F = 6400 3830 -> 3800 (which operand stays longer makes no difference);
//  * operands go global -> LDS directly (global_load_lds_dwordx4, 16 bytes per lane, no registers in between):
//    B through a ring of 4 stages of depth 32, A through a ring of 5 blocks of half the tile's rows by depth 64, so
//    that a load of A fetches whole 128-byte lines (8 rows per instruction); rows of A are gathered through
//    per-lane row offsets that stay in registers for the whole tile (the row-index caching of Section 4);
//  * A is read from LDS with ds_read_b128 (K-contiguous rows, XOR-swizzled by row); B either as the weights are
//    stored (K x N) with ds_read_b64_tr_b16, which hands every lane the 4 K-consecutive values of its column, or, with
//    packed weights (k_pack_weights: every stage already an LDS image in operand order), with one ds_read_b128;
//  * a layer0 tile waits for the ready flag of the source segment of its last row (Section 2.2.1: a tile
//    cannot start before all of its tokens have arrived);
//  * the tile schedules are built on the device (index_build.hip): one queue of 32-byte item records per XCD,
//    taken with one atomic per tile, a tile ahead, and stolen from the other XCDs' queues at the end.
#include <atomic>
#include <mutex>

#include "moe_device.h"

namespace moe {

constexpr int BK = kTileK, NS = kStages, BN = kTileN;
constexpr int kMaxPanels = 128;   // column panels whose publication can be batched per workgroup
constexpr int B_STAGE = BK * BN * 2;  // 16 KiB

__device__ __forceinline__ bf16x8 lds_read_a(uint32_t addr) {
  return *(const bf16x8 __attribute__((address_space(3)))*)(uintptr_t)addr;
}
// Packed weights: a fragment (32 columns x 16 values of K) lies in LDS in lane order, 16 bytes per lane.
__device__ __forceinline__ bf16x8 lds_read_b_packed(uint32_t a) {
  return *(const bf16x8 __attribute__((address_space(3)))*)(uintptr_t)a;
}
// acc += B A with the accumulator staying where it is.  The instruction's result may go elsewhere than its addend came from;
// with all 256 accumulation registers taken the register allocator uses that, outside the loop, to move half of a
// 256-row tile's accumulators to vector registers and back (300 moves per tile).  The compiler does not know this for an
// MFMA: whoever reads the accumulator next waits for it (the next MFMA on it is 32 away at least).
__device__ __forceinline__ void mfma_in_place(f32x4& acc, bf16x8 b, bf16x8 a) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(b), "v"(a));
}
// 16 bytes per lane from sbase + voff straight into LDS at lds_base + lane * 16.  Written as asm so that the
// compiler's wait-count pass does not serialise later LDS reads behind it; completion is awaited by hand
// with s_waitcnt vmcnt.
// STREAM: with the non-temporal hint (GemmParams::stream_rows).
template <bool STREAM = false>
__device__ __forceinline__ void dma16(const void* sbase, uint32_t voff, uint32_t lds_base) {
  if constexpr (STREAM)
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 nt" ::"v"(voff), "s"(sbase), "s"(lds_base)
                 : "memory");
  else
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(voff), "s"(sbase), "s"(lds_base)
                 : "memory");
}
// The same in two instructions with an MFMA between them (M0 wants a cycle before it is used): the LDS address, a base in a
// scalar register plus a constant, and the load.  Nothing between the two may touch M0:
// the scheduling barriers around both leave the MFMA alone there, and the compiler has no other use for M0 in these kernels.
template <int OFF>
__device__ __forceinline__ void dma16_address(uint32_t lds_base) {
  if constexpr (OFF == 0) asm volatile("s_mov_b32 m0, %0" ::"s"(lds_base) : "memory", "m0");
  else asm volatile("s_add_u32 m0, %0, %1" ::"s"(lds_base), "n"(OFF) : "memory", "scc", "m0");
}
template <bool STREAM = false>
__device__ __forceinline__ void dma16_load(const void* sbase, uint32_t voff) {
  if constexpr (STREAM) asm volatile("global_load_lds_dwordx4 %0, %1 nt" ::"v"(voff), "s"(sbase) : "memory");
  else asm volatile("global_load_lds_dwordx4 %0, %1" ::"v"(voff), "s"(sbase) : "memory");
}
// Waits until at most N LDS reads are outstanding, in a form the compiler knows: it adds no waits of its own for the
// fragments that have landed by then (one in front of every fragment's first MFMA otherwise).
template <int N>
__device__ __forceinline__ void wait_lds_reads() {
  __builtin_amdgcn_s_waitcnt(0xc07f | (N << 8));
}
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// Top-k weighted reduction of one unit: kCombineChunk tokens x one 256-column panel of Y.  A thread owns 8 columns
// (16 bytes) of every 8th token of the unit; the rows of several tokens are requested before any is used, because
// with one workgroup per compute unit only loads in flight can cover the memory latency.
template <int K>
__device__ __forceinline__ void combine_unit_k(const GemmParams& p, int panel, int chunk, int k_runtime) {
  constexpr int KK = K > 0 ? K : 1;
  constexpr int TB = K == 0 ? 1 : (K <= 2 ? 8 : (K <= 4 ? 4 : 2));   // tokens per batch of a thread
  constexpr int NB = kCombineChunk / 8 / TB;                           // batches per unit
  const int tid = threadIdx.x;
  const int cg = tid & 31, ts = tid >> 5;
  const size_t col = (size_t)panel * BN + cg * 8;
  if (K == 0) {
    // any other k: one token at a time
    for (int i0 = 0; i0 < kCombineChunk / 8; i0++) {
      const int t = chunk * kCombineChunk + i0 * 8 + ts;
      if (t >= p.T) continue;
      float acc[8];
#pragma unroll
      for (int c = 0; c < 8; c++) acc[c] = 0.f;
      for (int j = 0; j < k_runtime; j++) {
        const int row = p.inv_perm[t * k_runtime + j];
        const float w = p.topk_weights[t * k_runtime + j];
        const u32x4 v = *(const u32x4*)(p.C + (size_t)row * p.ldc + col);
#pragma unroll
        for (int c = 0; c < 4; c++) {
          acc[2 * c] += w * __uint_as_float(v[c] << 16);
          acc[2 * c + 1] += w * __uint_as_float(v[c] & 0xffff0000u);
        }
      }
      u32x4 o;
#pragma unroll
      for (int c = 0; c < 4; c++) {
        bf16x2 pr = {(__bf16)acc[2 * c], (__bf16)acc[2 * c + 1]};
        o[c] = __builtin_bit_cast(uint32_t, pr);
      }
      *(u32x4*)(p.out + (size_t)t * p.H + col) = o;
    }
    return;
  }
  // Two batches in flight: the rows of batch i+1 are requested before batch i is summed and stored.
  float w[2][TB][KK];
  u32x4 v[2][TB][KK];
  auto request = [&](int buf, int batch) {
    int row[TB][KK];
#pragma unroll
    for (int b = 0; b < TB; b++) {
      const int t = chunk * kCombineChunk + (batch * TB + b) * 8 + ts;
      const int tt = t < p.T ? t : p.T - 1;
#pragma unroll
      for (int j = 0; j < KK; j++) {
        row[b][j] = p.inv_perm[tt * KK + j];
        w[buf][b][j] = p.topk_weights[tt * KK + j];
      }
    }
#pragma unroll
    for (int b = 0; b < TB; b++)
#pragma unroll
      for (int j = 0; j < KK; j++) v[buf][b][j] = *(const u32x4*)(p.C + (size_t)row[b][j] * p.ldc + col);
  };
  auto finish = [&](int buf, int batch) {
#pragma unroll
    for (int b = 0; b < TB; b++) {
      const int t = chunk * kCombineChunk + (batch * TB + b) * 8 + ts;
      float acc[8];
#pragma unroll
      for (int c = 0; c < 8; c++) acc[c] = 0.f;
#pragma unroll
      for (int j = 0; j < KK; j++)
#pragma unroll
        for (int c = 0; c < 4; c++) {
          acc[2 * c] += w[buf][b][j] * __uint_as_float(v[buf][b][j][c] << 16);
          acc[2 * c + 1] += w[buf][b][j] * __uint_as_float(v[buf][b][j][c] & 0xffff0000u);
        }
      if (t < p.T) {
        u32x4 o;
#pragma unroll
        for (int c = 0; c < 4; c++) {
          bf16x2 pr = {(__bf16)acc[2 * c], (__bf16)acc[2 * c + 1]};
          o[c] = __builtin_bit_cast(uint32_t, pr);
        }
        *(u32x4*)(p.out + (size_t)t * p.H + col) = o;
      }
    }
  };
  static_assert(NB % 2 == 0, "batches are processed in pairs");
  request(0, 0);
#pragma unroll 1
  for (int i = 0; i < NB; i += 2) {
    request(1, i + 1);
    finish(0, i);
    if (i + 2 < NB) request(0, i + 2);
    finish(1, i + 1);
  }
}

__device__ __forceinline__ void combine_unit(const GemmParams& p, int panel, int chunk) {
  switch (p.k) {
    case 1: combine_unit_k<1>(p, panel, chunk, 1); break;
    case 2: combine_unit_k<2>(p, panel, chunk, 2); break;
    case 4: combine_unit_k<4>(p, panel, chunk, 4); break;
    case 8: combine_unit_k<8>(p, panel, chunk, 8); break;
    default: combine_unit_k<0>(p, panel, chunk, p.k); break;
  }
}

// Claims combine units until none are left.  A unit of panel n may start once every M-tile of that panel is done.
// all_at_once: the panels are all published together at the end of the GEMM work (no data-movement workgroups), so
// the workgroup waits for the last panel once and needs a single acquire instead of one per panel.
__device__ __forceinline__ void combine_loop(const GemmParams& p, int32_t* lds_slot, bool all_at_once) {
  const int n_panels = p.H / BN;
  const int n_chunks = (p.T + kCombineChunk - 1) / kCombineChunk;
  const int total = n_panels * n_chunks;
  const uint32_t need = (uint32_t)*p.n_tiles;
  int acquired_panel = -1;
  if (all_at_once) {
    __syncthreads();
    if (threadIdx.x == 0) {
      bool ok = true;
      for (int n = 0; n < n_panels && ok; n++) ok = spin_until_ge(&p.panel_done[n], need, p.spin_limit);
      if (!ok) atomicExch(p.status, (int)MOE_ERR_TIMEOUT);
      *lds_slot = ok;
    }
    __syncthreads();
    if (!*lds_slot) return;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    acquired_panel = n_panels;   // everything is acquired
  }
  while (true) {
    __syncthreads();
    if (threadIdx.x == 0) {
      int u = atomicAdd(p.combine_counter, 1);
      if (u < total && !all_at_once) {
        const int panel = u / n_chunks;
        if (panel != acquired_panel && !spin_until_ge(&p.panel_done[panel], need, p.spin_limit)) {
          atomicExch(p.status, (int)MOE_ERR_TIMEOUT);
          u = total;
        }
      }
      *lds_slot = u;
    }
    __syncthreads();
    const int u = *lds_slot;
    if (u >= total) break;
    const int panel = u / n_chunks;
    if (!all_at_once && panel != acquired_panel) {
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
      acquired_panel = panel;
    }
    combine_unit(p, panel, u % n_chunks);
  }
}

// ---------------------------------------------------------------------------------------------
// Schedule queues: XCD x owns the list positions base[x] + i * stride, i < len[x].
// ---------------------------------------------------------------------------------------------
struct Queue {
  int own_len, own_base;   // this workgroup's XCD, read once
};
__device__ __forceinline__ int queue_pos(const GemmParams& p, int x, int i) {
  return (p.queue_base ? p.queue_base[x] : x) + i * p.queue_stride;
}
// The heads lie 256 bytes apart in launches of more than a round (Workspace::queue_heads): with all of them in one line the atomics of 256 workgroups that
// end a tile together took several us (1000 tokens of 64 experts with F = 1408: 245 -> 241 us, and with late tickets 263 -> 237).
constexpr int kLateRounds = 2;   // rounds at the end of a queue in which an item is taken late, see run_tile
// Takes the next item of XCD x's queue; returns its list position or -1 when that queue is used up.
__device__ __forceinline__ int take_from(const GemmParams& p, int x, int len, int base) {
  if (len == 0) return -1;
  const int i = __hip_atomic_fetch_add(&p.queue_heads[x * p.head_stride], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return i < len ? base + i * p.queue_stride : -1;
}
// The other XCDs' leftovers, nearest first; -1 when every queue is used up.  All heads and lengths are read first
// (one round trip): at the end of a kernel, and in small problems, most queues are empty and an atomic on each
// of them from every workgroup would serialise on the counters.
__device__ __forceinline__ int steal(const GemmParams& p, int xcd) {
  int head[kXcds], len[kXcds];
#pragma unroll
  for (int d = 1; d < kXcds; d++) {
    const int x = (xcd + d) & (kXcds - 1);
    head[d] = __hip_atomic_load(&p.queue_heads[x * p.head_stride], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    len[d] = p.queue_len[x];
  }
#pragma unroll
  for (int d = 1; d < kXcds; d++) {
    if (head[d] >= len[d]) continue;
    const int x = (xcd + d) & (kXcds - 1);
    const int idx = take_from(p, x, len[d], queue_pos(p, x, 0));
    if (idx >= 0) return idx;
  }
  return -1;
}
// Data-movement workgroup that runs ahead of the GEMM workgroups of its XCD (the specialisation of Section 3.2.1 put
// to local use): it follows the head of the XCD's queue and reads one word of every 128-byte line of the packed
// weight panel of the items about to be handed out, so that the panel is on its way from HBM into the Infinity Cache
// (and this XCD's L2) before a GEMM workgroup's three K steps of lead have to cover the miss.  Pays where a weight
// panel serves few M-tiles (many small experts): there the GEMM workgroups wait for HBM, not for the matrix cores.
// `part` of `n_parts`: the workgroups sharing an XCD split every panel between them.  The loop ends when the queue is
// handed out, or when its head has not moved for about a second (the GEMM side waiting for a ready flag): a
// workgroup that stops prefetching costs time, never correctness.
constexpr int kPrefetchUnroll = 16;
__device__ __forceinline__ void prefetch_loop(const GemmParams& p, int xcd, int part, int n_parts) {
  const int len = p.queue_len[xcd];
  const int base = queue_pos(p, xcd, 0);
  const uint64_t panel_bytes = (uint64_t)(p.K / BK) * B_STAGE;
  const int lines = (int)(panel_bytes / 128);
  const int tid = threadIdx.x;
  int i = 0, last_expert = -1, last_n = -1;
  uint32_t idle = 0, sink = 0;
  while (i < len) {
    const int head = uniform(__hip_atomic_load(&p.queue_heads[xcd * p.head_stride], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    if (head >= len) break;   // everything handed out: nothing left to be ahead of
    // items handed out a while ago are being streamed by their workgroups already
    if (i < head - p.prefetch_behind) i = head - p.prefetch_behind;
    if (i >= head + p.prefetch_ahead) {
      if (++idle > (1u << 20)) break;
      __builtin_amdgcn_s_sleep(32);
      continue;
    }
    idle = 0;
    const int expert = uniform(p.items[base + i * p.queue_stride].expert);
    const int n_tile = uniform(p.items[base + i * p.queue_stride].n_tile);
    i++;
    if (expert == last_expert && n_tile == last_n) continue;   // the M-tiles of a block share the panel
    last_expert = expert;
    last_n = n_tile;
    const char* src = p.B + ((uint64_t)expert * p.n_tiles_n + n_tile) * panel_bytes;
    for (int l0 = part * 256 * kPrefetchUnroll; l0 < lines; l0 += n_parts * 256 * kPrefetchUnroll) {
      uint32_t v[kPrefetchUnroll];
#pragma unroll
      for (int u = 0; u < kPrefetchUnroll; u++) {
        const int l = l0 + u * 256 + tid;
        v[u] = l < lines ? *(const uint32_t*)(src + (size_t)l * 128) : 0u;
      }
#pragma unroll
      for (int u = 0; u < kPrefetchUnroll; u++) sink ^= v[u];
    }
  }
  if (p.K < 0) p.status[63] = (int32_t)sink;   // never true: keeps the loads
}
// The last n_prefetch workgroups of a launch take the prefetch role (multiples of 8: workgroup b runs on XCD b % 8,
// so any 8 consecutive workgroups cover the 8 XCDs).
__device__ __forceinline__ bool prefetch_role(const GemmParams& p) {
  const int first = (int)gridDim.x - p.n_prefetch;
  if (p.n_prefetch <= 0 || (int)blockIdx.x < first) return false;
  prefetch_loop(p, blockIdx.x & (kXcds - 1), ((int)blockIdx.x - first) >> 3, p.n_prefetch >> 3);
  return true;
}

__device__ __forceinline__ void block_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

#ifdef MOE_TILE_TRACE
// Measurement build only (tile_trace.py compiles the library with -DMOE_TILE_TRACE): every workgroup notes, per tile,
// the time (100 MHz device clock) at which it started on it, had the operands of the first K step in LDS, finished
// the main loop and finished the epilogue; and, in core clock cycles, how long the main loop took and how much of that
// its first wavefront spent at the synchronisation point of each K step (waiting for its operand loads to land and
// for the other wavefronts).
constexpr int kTraceWgs = 256, kTraceTiles = 128, kTraceWords = 6;
__device__ uint64_t g_trace_stamp[2][kTraceWgs][kTraceTiles][kTraceWords];
__device__ int32_t g_trace_kind[2][kTraceWgs][kTraceTiles];
__device__ int32_t g_trace_count[2][kTraceWgs];
// (The count is kept in LDS, slot: a load from global memory here would make the compiler wait for everything in
// flight, the successor's first operand loads included.)
__device__ __forceinline__ void trace_tile(int layer, int kind, uint64_t t0, uint64_t t1, uint64_t t2, uint64_t t3,
                                           uint64_t loop_cycles, uint64_t sync_cycles, volatile uint32_t* slot) {
  if (threadIdx.x != 0 || blockIdx.x >= kTraceWgs) return;
  const int n = (int)slot[layer];
  if (n >= kTraceTiles) return;
  slot[layer] = (uint32_t)(n + 1);
  g_trace_stamp[layer][blockIdx.x][n][0] = t0;
  g_trace_stamp[layer][blockIdx.x][n][1] = t1;
  g_trace_stamp[layer][blockIdx.x][n][2] = t2;
  g_trace_stamp[layer][blockIdx.x][n][3] = t3;
  g_trace_stamp[layer][blockIdx.x][n][4] = loop_cycles;
  g_trace_stamp[layer][blockIdx.x][n][5] = sync_cycles;
  g_trace_kind[layer][blockIdx.x][n] = kind;
  g_trace_count[layer][blockIdx.x] = n + 1;
}
#define MOE_TRACE_STAMP(var) var = wall_clock64()
#define MOE_TRACE_CYCLES(var) var = clock64()
#define MOE_TRACE_ADD_CYCLES(sum, since) sum += clock64() - since
#else
#define MOE_TRACE_STAMP(var)
#define MOE_TRACE_CYCLES(var)
#define MOE_TRACE_ADD_CYCLES(sum, since)
#endif

// Publishes one finished M-tile of column panel `panel` to the data-movement side: every wavefront makes its stores
// visible device-wide, then one thread bumps the panel's counter.
__device__ __forceinline__ void publish_panel(const GemmParams& p, int panel) {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
  __syncthreads();
  if (threadIdx.x == 0) __hip_atomic_fetch_add(&p.panel_done[panel], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// What a workgroup knows about a tile before it starts on it.
struct Tile {
  int idx;        // list position, -1: none
  ItemRec rec;
  int arow[8];    // rows of A this lane loads, per half of the tile's rows (layer0: gathered token rows, layer1: rows of h)
  int pre;        // 1: the loads of its first NS-1 stages were issued during the previous tile's epilogue
};
__device__ __forceinline__ ItemRec make_uniform(ItemRec r) {
  r.m_tile = uniform(r.m_tile); r.n_tile = uniform(r.n_tile); r.expert = uniform(r.expert); r.row0 = uniform(r.row0);
  r.nrows = uniform(r.nrows); r.ready_seg = uniform(r.ready_seg);
  // (192 rows: a ragged tile of 129 to 192 rows was padded to 256.  us per gate + layer, 256 / 192: 150 rows for each of 16 experts of F = 6400 569 /
  // 536, 162 for each of 64 of F = 2560 822 / 779, 425 for each of 64 of F = 1408 512 / 488, 412 for each of 64 of F = 2560 1412 / 1371)
  r.kind = r.nrows <= 64 ? 0 : (r.nrows <= 128 ? 1 : (r.nrows <= 192 ? 3 : 2));   // the variant that computes it: the lowest that holds its rows
  return r;
}
__device__ __forceinline__ ItemRec load_item(const GemmParams& p, int idx) { return make_uniform(p.items[idx]); }
// Global offsets and running base pointers of a tile's operand loads.
struct LoadState {
  uint32_t aoff[8], boff[4];
  const char* Ab;
  const char* Bb;
};

// LDS of a tile of BM rows.  B is kept in a ring of NSX stages of one K step, loaded NSX - 1 steps ahead; A in a ring
// of NSX + 1 blocks in front of it, a block being one half of the tile's rows by 64
// values of K (128 bytes per row: whole cache lines of the operand, 8 rows per load instruction; fetching the 64
// bytes of one K step per row, 16 rows per instruction, is 1-2 % slower).  Block b = 2d + h holds rows [h*BM/2, (h+1)*BM/2) for
// K steps 2d and 2d+1; a block per K step is loaded, NSX - 1 steps ahead like B.
// NSX is 4 (three steps of lead) except for the 64-row tiles of the ragged expert ends, which get 6: a K step of
// theirs is 16 MFMAs of 16 cycles per wavefront, so three steps of lead are a third of a memory round trip and the tile would
// spend half its time waiting for its operands; their small A blocks leave the LDS for two more B stages.
constexpr int kDeepStages = 6;
constexpr int a_block_bytes(int bm) { return bm * 64; }
constexpr int b_ring_offset(int bm, int nsx) { return (nsx + 1) * a_block_bytes(bm); }
// The reduction in the layer1 epilogue lists its tokens in 2 KiB that are free at the end of a tile even when the successor's
// first loads are under way (A blocks 0..2, B stages 0..2): A block 3 of a 256-row tile, the space behind the rings otherwise.
constexpr int kListBytes = 2048;
constexpr int list_offset(int bm, int nsx) { return bm == 256 ? 3 * a_block_bytes(bm) : b_ring_offset(bm, nsx) + nsx * B_STAGE; }
constexpr int kLdsBytes = b_ring_offset(256, NS) + NS * B_STAGE;   // 144 KiB; covers the smaller tiles' layouts too
static_assert(list_offset(192, NS) + kListBytes <= kLdsBytes && list_offset(128, NS) + kListBytes <= kLdsBytes && list_offset(64, kDeepStages) + kListBytes <= kLdsBytes, "the list fits");
static_assert(kLdsBytes <= 160 * 1024 - 16384, "LDS of a compute unit, less the kernels' static variables");

// Rows of A the lane loads for a tile of the given variant: LA = 1, 2, 3 or 4 loads per block and two blocks (row
// halves) per tile; a load covers 8 rows, 8 lanes per row.  arow[h * LA + j]: row half h, load j.
template <int MODE>
__device__ __forceinline__ void load_arows(const GemmParams& p, Tile& t, int lane, int w) {
  const int la = t.rec.kind == 3 ? 3 : 1 << t.rec.kind;
#pragma unroll
  for (int i = 0; i < 8; i++) {
    if (i < 2 * la) {
      const int h = i >= la, j = i - h * la;
      const int r = h * (32 * la) + (w * la + j) * 8 + (lane >> 3);
      const int sr = t.rec.row0 + (r < t.rec.nrows ? r : t.rec.nrows - 1);   // past the ragged end: the last row again
      t.arow[i] = MODE != MODE_L1 ? p.a_rows[sr] : sr;
    }
  }
}

// Address set-up of a tile and its first loads: A blocks and B stages 0 .. NSX-2, in the order A0 A1 B0 A2 B1 ...
// A(NSX-2) B(NSX-3) B(NSX-2) (what K step 0 needs first, then a block and a stage per further step).
// A: lane l of a load fetches the 16 bytes at position (l & 7) ^ ((row / 2) & 7) of its row's 128-byte line, so that
// the line lands in LDS (linearly, 16 bytes per lane) with its chunks XOR-swizzled by row: the 16 rows one pass of
// ds_read_b128 touches then fall on distinct banks.
template <int WM, int MT, int NT, int MODE, bool PK, bool STREAM, int NSX>
__device__ __forceinline__ void setup_and_issue(const GemmParams& p, uint32_t lds0, const Tile& t, LoadState& ls, int lane,
                                                int w, bool issue) {
  constexpr int BM = WM * MT * 32;
  constexpr int A_BLOCK = a_block_bytes(BM);
  constexpr int B_RING = b_ring_offset(BM, NSX);
  constexpr int LA = BM / 64, LB = 4;
  constexpr int LEAD = NSX - 1;   // K steps the loads run ahead
#pragma unroll
  for (int i = 0; i < 2 * LA; i++) {
    const int r = (w * LA + i % LA) * 8 + (lane >> 3);   // row inside the block
    const int c = (lane & 7) ^ ((r >> 1) & 7);
    ls.aoff[i] = (uint32_t)t.arow[i] * p.lda_bytes + c * 16;
  }
  const int col0 = (MODE == MODE_L0_SWIGLU) ? t.rec.n_tile * (BN / 2) : t.rec.n_tile * BN;
#pragma unroll
  for (int j = 0; j < LB; j++) {
    if (PK) {
      // packed weights: a stage is 16 KiB in a row, already in its LDS order
      ls.boff[j] = (uint32_t)((w * LB + j) * 1024 + lane * 16);
      continue;
    }
    const int kr = (w * LB + j) * 2 + (lane >> 5);
    const int cpb = lane & 31;
    const int blk = (cpb >> 1) ^ ((kr & 3) | (((kr >> 3) & 1) << 2));   // 16-column blocks, XOR-swizzled by row
    const int c8 = (blk * 2 + (cpb & 1)) * 8;  // column of the tile this lane fetches
    int gcol;
    if (MODE == MODE_L0_SWIGLU) {
      // a wavefront's 32*NT columns are [gate | up] of the same 16*NT hidden units
      const int region = c8 / (NT * 32), within = c8 % (NT * 32);
      const int half = within / (NT * 16), fo = within % (NT * 16);
      gcol = half * p.F + col0 + region * (NT * 16) + fo;
    } else {
      gcol = col0 + c8;
    }
    ls.boff[j] = ((uint32_t)kr * p.ldb + gcol) * 2;
  }
  ls.Ab = uniform(p.A);
  ls.Bb = PK ? uniform(p.B + ((uint64_t)t.rec.expert * p.n_tiles_n + t.rec.n_tile) * ((uint64_t)(p.K / BK) * B_STAGE))
             : uniform(p.B + (uint64_t)t.rec.expert * p.b_expert_bytes);
  const size_t bstep = PK ? (size_t)B_STAGE : (size_t)BK * p.ldb * 2;
  if (issue) {
    auto a_block = [&](int b) {
#pragma unroll
      for (int j = 0; j < LA; j++)
        dma16(ls.Ab + (b >> 1) * 128, ls.aoff[(b & 1) * LA + j], lds0 + b * A_BLOCK + (w * LA + j) * 1024);
    };
    auto b_stage = [&](int st) {
#pragma unroll
      for (int j = 0; j < LB; j++) dma16<STREAM>(ls.Bb + st * bstep, ls.boff[j], lds0 + B_RING + st * B_STAGE + (w * LB + j) * 1024);
    };
    a_block(0);
    a_block(1);
    b_stage(0);
#pragma unroll
    for (int st = 2; st < LEAD; st++) {
      a_block(st);
      b_stage(st - 1);
    }
    b_stage(LEAD - 1);
  }
  ls.Bb += LEAD * bstep;   // ls.Ab stays the row start: the K position of A comes from the block number
}

// Workgroup-wide: is the source segment of tile t there?  block = true waits for it (up to the spin limit).
template <int MODE>
__device__ __forceinline__ bool segment_ready(const GemmParams& p, const Tile& t, volatile int32_t* lds_slot, bool block) {
  if (MODE == MODE_L1 || p.seg_ready == nullptr) return true;
  if (threadIdx.x == 0) {
    const uint32_t* flag = &p.seg_ready[t.rec.ready_seg];
    bool ok;
    if (block) {
      ok = spin_until_ge(flag, p.ready_epoch, p.spin_limit);
      if (!ok) atomicExch(p.status, (int)MOE_ERR_TIMEOUT);
    } else {
      ok = __hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM) >= p.ready_epoch;
    }
    lds_slot[1] = ok;
  }
  __syncthreads();
  const bool ok = lds_slot[1] != 0;
  __syncthreads();
  if (ok) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "");
  return ok;
}

// One tile of BM = WM*MT*32 rows by 256 columns: address set-up and first loads, main loop, epilogue.  While the
// tile runs the workgroup finds out what its next tile is without waiting for any of the round trips: the queue
// atomic is issued up front; once the last operand load has landed (a step and a half before the end) its result is shared
// through LDS and the item record is requested.  A tile followed by one of the same height also starts the
// successor's first operand stages during its own epilogue (next.pre = 1); otherwise only the rows of A the next
// tile gathers are requested, after the epilogue.  next.idx = -1: no further tile.
template <int WM, int MT, int NT, int MODE, bool PK, bool STREAM, int NSX = NS>
__device__ __forceinline__ void run_tile(const GemmParams& p, char* smem, volatile int32_t* lds_slot, const Tile& cur,
                                         Tile& next, int xcd, const Queue& q, int& pending_panel,
                                         volatile int32_t* lds_panel_count_ptr, volatile uint32_t* lds_mask) {
  constexpr int WN = 4 / WM;
  constexpr int BM = WM * MT * 32;
  static_assert(WN * NT * 32 == BN, "tile must be 256 columns wide");
  constexpr int A_BLOCK = a_block_bytes(BM);
  constexpr int B_RING = b_ring_offset(BM, NSX);
  constexpr int AB = NSX + 1;     // blocks of the A ring
  constexpr int LEAD = NSX - 1;   // K steps the loads run ahead; odd, so that the steps without loads at the end start on an odd step
  static_assert(LEAD % 2 == 1 && (BM != 256 || NSX == NS), "see list_offset: A block 3 of a 256-row tile is free at its end");
  constexpr int LA = BM / 64;  // A loads per lane per K step (one block)
  constexpr int LB = 4;        // B loads per lane per K step (one stage)
  constexpr int LS = LA + LB;

#ifdef MOE_TILE_TRACE
  uint64_t tt0 = 0, tt1 = 0, tt2 = 0, tt3 = 0, tc_loop = 0, tc_sync = 0, tc_mark = 0;
#endif
  MOE_TRACE_STAMP(tt0);
  const uint32_t lds0 = (uint32_t)(uintptr_t)smem;
  // The thread index is made opaque per tile: otherwise the lane-dependent address constants of all three tile
  // heights are hoisted out of the tile loop, kept live across it and spilled.
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = w / WN, wn = w % WN;
  const int g = lane >> 4, j16 = lane & 15;   // (also of the MFMA's operands: K group and row / column of a fragment)
  const int row0 = uniform(cur.rec.row0), nrows = uniform(cur.rec.nrows), n_tile = uniform(cur.rec.n_tile);
  const int col0 = (MODE == MODE_L0_SWIGLU) ? n_tile * (BN / 2) : n_tile * BN;

  // LDS read addresses of a lane: a_rd[parity of the K step] inside an A block (fragment 0: 16 rows by 32 values of K, the
  // lane's row is lane % 16 and its 8 values of K are those at lane / 16), b_rd inside a B stage (fragment 0 of the wavefront)
  uint32_t a_rd[2], b_rd;
  {
    const int s = (j16 >> 1) & 7;
#pragma unroll
    for (int sub = 0; sub < 2; sub++) a_rd[sub] = lds0 + j16 * 128 + (((sub * 4 + g) ^ s) << 4);
    if (PK) {
      // column block of the packed tile this wavefront's columns begin with: SwiGLU tiles hold [4 gate | 4 up] blocks of the
      // same 128 hidden units, of which a wavefront takes the gate and up blocks of its own units (see b_frag_offset)
      const int c = MODE == MODE_L0_SWIGLU ? wn * (NT / 2) : wn * NT;
      b_rd = lds0 + B_RING + c * 1024 + (g >> 1) * (B_STAGE / 2) + (g & 1) * 512 + j16 * 16;
    } else {
      const int krow = 8 * g + (j16 >> 2);
      const int swz = (j16 >> 2) | ((g & 1) << 2);
      b_rd = lds0 + B_RING + krow * 512 + (((wn * NT * 2) ^ swz) << 5) + (j16 & 3) * 8;
    }
  }
  // Measurement aid: the fences a tile-granular hand-off between the two GroupGEMMs would need (a layer1 tile
  // acquiring what layer0 tiles on other XCDs released), without the hand-off itself.
  if (MODE == MODE_L1 && p.handoff_fences) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  // address set-up and the first loads (A blocks 0..2, B stages 0..2)
  LoadState ls;
  setup_and_issue<WM, MT, NT, MODE, PK, STREAM, NSX>(p, lds0, cur, ls, lane, w, !cur.pre);
  const char* Ab = uniform(ls.Ab);
  const char* Bb = uniform(ls.Bb);
  const size_t bstep = PK ? (size_t)B_STAGE : (size_t)BK * p.ldb * 2;

  // Not cleared: the MFMAs of the tile's first K step take a zero constant as their addend instead (clearing 256
  // accumulator registers is 256 instructions, 0.8 us of a tile with the matrix cores idle).
  constexpr int MA = 2 * MT, NB = 2 * NT;     // 16-row and 16-column blocks of the wavefront
  constexpr int HA = MA / 2, HB = NB / 2;     // ... of a half of them
  f32x4 acc[MA][NB];

  // Per K step and lane: LA loads of A (block kt+LEAD: the other half of the rows than the block before, 64 values of K)
  // and LB loads of B (stage kt+LEAD).  The loads are issued one at a time between groups of MFMAs: a burst would fill
  // the vector-memory queue and stall the MFMAs queued behind it.
  using P0 = std::integral_constant<int, 0>;
  using P1 = std::integral_constant<int, 1>;
  // Where K step kt finds its operands in the rings and where its loads go, kept incrementally: written as
  // (kt ...) % AB the compiler turns the read addresses into per-lane vectors that it rebases every step, and the
  // scalar divisions pile up at the top of the loop, where no MFMA covers them (2 % of the kernel's time).
  struct Ring {
    uint32_t oa, ob;      // LDS offsets of the A block of row half 0 of kt's pair of steps and of B stage kt
    uint32_t a0, a1;      // A blocks of step kt, row halves 0 and 1 (LDS offsets)
    uint32_t an0, an1;    // ... of step kt + 1
    uint32_t b, bn;       // B stage kt, kt + 1
    uint32_t adst, bdst;  // slots of A block kt + LEAD and B stage kt + LEAD
  };
  auto wrap_a = [](uint32_t x) { return x >= (uint32_t)AB * A_BLOCK ? x - (uint32_t)AB * A_BLOCK : x; };
  auto wrap_b = [](uint32_t x) {
    if constexpr ((NSX & (NSX - 1)) == 0) return x & ((uint32_t)NSX * B_STAGE - 1);   // (offsets are multiples of B_STAGE)
    else return x >= (uint32_t)NSX * B_STAGE ? x - (uint32_t)NSX * B_STAGE : x;
  };
  // The state of the step after r's, whose parity is PARNEW: the A ring's part and the B ring's part (worked out in
  // different groups of MFMAs, see half1 and half2).
  auto advance_a = [&](const Ring& r, Ring& n, auto parnew) {
    constexpr int PARNEW = decltype(parnew)::value;
    n.oa = PARNEW == 0 ? wrap_a(r.oa + 2 * A_BLOCK) : r.oa;   // an even step begins a new pair of A blocks
    n.a0 = r.an0;
    n.a1 = r.an1;
    if (PARNEW == 0) {
      n.an0 = n.a0;
      n.an1 = n.a1;
    } else {
      n.an0 = wrap_a(n.oa + 2 * A_BLOCK);
      n.an1 = wrap_a(n.oa + 3 * A_BLOCK);
    }
    n.adst = wrap_a(n.oa + (uint32_t)(LEAD + PARNEW) * A_BLOCK);
  };
  auto advance_b = [&](const Ring& r, Ring& n) {
    n.ob = wrap_b(r.ob + B_STAGE);
    n.b = r.bn;
    n.bn = wrap_b(n.ob + B_STAGE);
    n.bdst = wrap_b(n.ob + (uint32_t)LEAD * B_STAGE);
  };
  Ring ring, next_ring;   // K step 0; the step after it (filled in as the step goes)
  ring.oa = 0;
  ring.ob = 0;
  ring.a0 = ring.an0 = 0;
  ring.a1 = ring.an1 = A_BLOCK;
  ring.b = 0;
  ring.bn = B_STAGE;
  ring.adst = (uint32_t)LEAD * A_BLOCK;
  ring.bdst = (uint32_t)LEAD * B_STAGE;
  next_ring = ring;
  const char* a_src = Ab + ((LEAD - 1) / 2) * 128;   // what the A block of an even step is loaded from; + 128: of the odd step after it
  // The read addresses of a K step as one per-lane base per operand (64-row tiles: the two halves of the rows lie in two A
  // blocks) plus constants that go into the instructions' offset fields.
  //   A: fragment f of a half is f * 2 KiB further on; 128- and 256-row tiles: a wavefront's rows fill one block
  //   B (packed): fragment f is b_frag_offset(f) further on; plain: the bits of f that the row's swizzle is XORed into
  struct StepBases { uint32_t a_lo, a_hi, b; };
  auto step_bases = [&](uint32_t blk0, uint32_t blk1, uint32_t b_off, int parity) {
    StepBases sb;
    sb.a_lo = (WM == 2 ? (wm ? blk1 : blk0) : blk0) + a_rd[parity];
    sb.a_hi = WM == 2 ? sb.a_lo + (uint32_t)HA * 2048 : blk1 + a_rd[parity];
    sb.b = b_off + b_rd;
    return sb;
  };
  auto b_frag_offset = [](int f) {
    const int nt = f >> 1;
    return (uint32_t)(MODE == MODE_L0_SWIGLU ? (nt / (NT / 2)) * 4 + nt % (NT / 2) : nt) * 1024 + (uint32_t)(f & 1) * 256;
  };
  static_assert(WM == 1 || 2 * MT * 16 * WM == BM, "a wavefront's rows fill one A block");
  auto read_b = [&](uint32_t base, int f) {
    if constexpr (PK) return lds_read_b_packed(base + b_frag_offset(f));
    const uint32_t at = base ^ (uint32_t)(f << 5);
    return lds_read_b(at, at + 4 * 512);
  };
  // A K step of a wavefront is MA x NB MFMAs of 16 x 16 x 32, taken as four quadrants of the blocks in an order that
  // changes one operand's half at a time and alternates between even and odd steps:
  //   even: (A lo, B lo) (A lo, B hi) | (A hi, B hi) (A hi, B lo)      odd: B lo and hi swapped
  // A half of an operand is then dead two quadrants before its successor is needed, so that one register set of
  // fragments is enough: quadrant 0 reads this step's other half of B and A hi, quadrant 2 the next step's A lo, quadrant 3
  // the half of B that the next step begins with.  Between quadrants 1 and 2 lies the workgroup barrier, with every read of
  // this step long returned.
  bf16x8 af[MA], bfr[NB];
  StepBases now, nxt;
  now = step_bases(ring.a0, ring.a1, ring.b, 0);
  nxt = now;
  // Group gi (of 8, two per quadrant) of a K step of parity PAR: its MFMAs with its LDS reads between them, one per MFMA.
  // reads_next: false in the last step of the tile.
  using First = std::integral_constant<int, 0>;    // the tile's first step: nothing accumulated yet
  using Middle = std::integral_constant<int, 1>;
  using Last = std::integral_constant<int, 2>;     // one of the last LEAD steps (see mfma_in_place)
  // side: scalar work for the step to come, spread between the MFMAs.  load: the group's operand load.
  // In-order issue and 16 cycles per MFMA: what stands between two MFMAs should be three instructions at most, so the
  // reads come behind the first MFMAs, the load behind the reads, in two parts.
  constexpr int PER = HA * HB / 2;                              // MFMAs of a group
  constexpr int kLoadAt = PER == 8 ? 5 : (PER == 6 ? 3 : (PER == 4 ? 2 : 1));   // ... ahead of the load
  auto group = [&](auto par, auto gi, auto where, bool reads_next, auto side, auto load_address, auto load) {
    constexpr int PAR = decltype(par)::value, G = decltype(gi)::value, Q = G / 2;
    constexpr int WHERE = decltype(where)::value;
    constexpr int a0 = (Q >= 2) * HA, b0 = ((Q == 0 || Q == 3) ? PAR : 1 - PAR) * HB;
    constexpr int bx = (1 - PAR) * HB;               // the half of B this step ends and the next one begins without ...
    constexpr int READS = G == 0 || G == 6 ? (PK ? HB : 2 * HB) : (G == 1 || G == 4 ? HA : 0);
    constexpr int TAKE = READS > kLoadAt ? (READS + kLoadAt - 1) / kLoadAt : 1;   // reads behind one MFMA
    const int n_reads = G < 4 || reads_next ? READS : 0;
    if constexpr (G == 0) {
      wait_lds_reads<PK ? HB / 2 : HB>();            // A lo and half of the columns of quadrant 0
#pragma unroll
      for (int f = 0; f < HB; f++) bfr[bx + f] = read_b(now.b, bx + f);
    } else if constexpr (G == 1) {
#pragma unroll
      for (int f = 0; f < HA; f++) af[HA + f] = lds_read_a(now.a_hi + f * 2048);
    } else if constexpr (G == 2) {
      wait_lds_reads<HA>();                          // the columns of quadrant 1
    } else if constexpr (G == 4) {
      if (reads_next) {
#pragma unroll
        for (int f = 0; f < HA; f++) af[f] = lds_read_a(nxt.a_lo + f * 2048);
        }
    } else if constexpr (G == 6) {
      if (reads_next) {
#pragma unroll
        for (int f = 0; f < HB; f++) bfr[bx + f] = read_b(nxt.b, bx + f);
        }
    }
    side();
    auto multiply = [&](auto lo, auto hi) {
#pragma unroll
      for (int i = decltype(lo)::value; i < decltype(hi)::value; i++) {
        // the operand half that was read last is the outer one: its fragments are needed one by one
        // ... and every other sweep of the inner one runs backwards, so that from one MFMA to the next one operand changes, never both
        const int m = (G & 1) * PER + i, out = Q < 2 ? m / HA : m / HB, back = (out & 1) * ((Q < 2 ? HA : HB) - 1);
        const int in = Q < 2 ? m % HA : m % HB, at = back ? back - in : in;
        const int ma = a0 + (Q < 2 ? at : out), nb = b0 + (Q < 2 ? out : at);
        if constexpr (WHERE == Last::value && MA * NB == 64) mfma_in_place(acc[ma][nb], bfr[nb], af[ma]);
        else if constexpr (WHERE == First::value) acc[ma][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bfr[nb], af[ma], (f32x4){0}, 0, 0, 0);
        else acc[ma][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bfr[nb], af[ma], acc[ma][nb], 0, 0, 0);
      }
    };
    using L0 = std::integral_constant<int, 0>;
    using L1 = std::integral_constant<int, kLoadAt>;
    using L2 = std::integral_constant<int, kLoadAt + 1>;
    using L3 = std::integral_constant<int, PER>;
    multiply(L0{}, L1{});
#pragma unroll
    for (int i = 0; i < kLoadAt; i++) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      if (i * TAKE < n_reads) __builtin_amdgcn_sched_group_barrier(0x100, TAKE, 0);
      else __builtin_amdgcn_sched_group_barrier(0x006, 2, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
    load_address();
    __builtin_amdgcn_sched_barrier(0);
    multiply(L1{}, L2{});
    __builtin_amdgcn_sched_barrier(0);
    load();
    __builtin_amdgcn_sched_barrier(0);
    multiply(L2{}, L3{});
    __builtin_amdgcn_sched_barrier(0);
  };
  // first half of K step kt (parity PAR): quadrants 0 and 1, and the loads of A block kt+LEAD
  auto half1 = [&](auto par, bool do_issue, auto where) {
    constexpr int PAR = decltype(par)::value;
    const char* src = a_src + PAR * 128;
    const uint32_t dst = lds0 + ring.adst + w * LA * 1024;
    auto part = [&](auto gi) {
      constexpr int q = decltype(gi)::value;
      const bool load = do_issue && q < LA;
      group(par, gi, where, true,
            [&]() {
              if (q == 2) nxt = step_bases(ring.an0, ring.an1, ring.bn, 1 - PAR);   // where the next step reads
              if (q == 3) advance_a(ring, next_ring, std::integral_constant<int, 1 - PAR>{});   // the A ring's next positions
            },
            [&]() { if (load) dma16_address<q * 1024>(dst); },
            [&]() { if (load) dma16_load(src, ls.aoff[((PAR + LEAD) & 1) * LA + (q < LA ? q : 0)]); });
    };
    part(std::integral_constant<int, 0>{});
    part(std::integral_constant<int, 1>{});
    part(std::integral_constant<int, 2>{});
    part(std::integral_constant<int, 3>{});
  };
  // second half: quadrants 2 and 3, and the loads of B stage kt+LEAD
  auto half2 = [&](auto par, bool do_issue, auto where, bool reads_next) {
    constexpr int PAR = decltype(par)::value;
    const uint32_t dst = lds0 + B_RING + ring.bdst + w * LB * 1024;
    auto part = [&](auto gi) {
      constexpr int q = decltype(gi)::value - 4;
      group(par, gi, where, reads_next, [&]() { if (q == 3) advance_b(ring, next_ring); },   // the B ring's next positions
            [&]() { if (do_issue) dma16_address<q * 1024>(dst); }, [&]() { if (do_issue) dma16_load<STREAM>(Bb, ls.boff[q]); });
    };
    part(std::integral_constant<int, 4>{});
    part(std::integral_constant<int, 5>{});
    part(std::integral_constant<int, 6>{});
    part(std::integral_constant<int, 7>{});
    ring = next_ring;
    now = nxt;
    if (PAR == 1) a_src += 128;
  };

  // The next item of this XCD's queue is requested before anything else of this tile is outstanding; the
  // operand loads of the first stages were issued before (by the previous tile, or by the kernel for the first).
  // Not so in the last rounds of a queue (late): there an item goes to whoever ends first, and not, a tile ahead, to a workgroup that
  // may be at the start of a tall tile while another runs out of short ones.  2047 tokens of 8 experts with F = 3584: 48 short
  // tiles waited for the second round of tall ones, layer0 262 -> 225 us, the layer 414 -> 381; 1100 of 16 with F = 6400 568 -> 539;
  // where all tiles take the same time it costs 0.3 %.  One round instead of two loses half of it.
  int next_raw = 0;
  const int taken = (cur.idx - q.own_base) >> (p.queue_stride == 1 ? 0 : 3);   // position in the own queue (a stolen item: anything)
  const int round = (int)(gridDim.x / kXcds);
  const bool late = p.head_stride > 1 && q.own_len > round && (uint32_t)(taken + kLateRounds * round) >= (uint32_t)q.own_len;   // (up to one round: all gone at the start)
  if (tid == 0 && !late) next_raw = take_from(p, xcd, q.own_len, q.own_base);
  // A tile starts the loads of a successor of its own height during its epilogue, which needs the successor's
  // segment to be there already: the ready flags are sampled here (lane s of the first wavefront reads
  // flag s) and looked at when the successor is known.  A flag raised later than this only costs the early start.
  constexpr bool kCanPre = true;   // (kept as a switch: the early start costs about 30 VGPRs)
  constexpr int kKind = WM == 1 ? 0 : (MT == 4 ? 2 : (MT == 3 ? 3 : 1));   // what ItemRec::kind says of this variant's tiles
  const bool flags_on = MODE != MODE_L1 && p.seg_ready != nullptr;
  uint32_t flag_v = 0;
  if (kCanPre && flags_on && tid < p.n_segments)
    flag_v = __hip_atomic_load(&p.seg_ready[tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);

  // Blocks of 16 rows that the epilogue of the tile before stored ahead of this tile's first loads (layer0: while the
  // gather rows of this tile came back), and the stores it issued behind them: younger than those loads, they need not be
  // waited for with them.
  constexpr int kPreBlock = MODE == MODE_L1 ? 0 : 2;
  constexpr int kPreStores = (MA - kPreBlock) * ((MODE == MODE_L0_SWIGLU) ? NB / 4 : NB / 2);
  const int nk = p.K / BK;  // even and >= 4 (checked on the host)
  // A blocks 0 and 1 and B stage 0 landed?  Everything issued after them (A blocks 2 .. LEAD-1, B stages 1 .. LEAD-1, and
  // what the previous tile's epilogue stored behind them) may still be outstanding; memory operations return in order.
  const bool started_early = cur.pre != 0;
  if (started_early) wait_vmcnt<(LEAD - 2) * LA + (LEAD - 1) * LB + kPreStores>();
  else wait_vmcnt<(LEAD - 2) * LA + (LEAD - 1) * LB>();
  block_barrier();
  MOE_TRACE_STAMP(tt1);
  MOE_TRACE_CYCLES(tc_loop);
#pragma unroll
  for (int f = 0; f < HA; f++) af[f] = lds_read_a(now.a_lo + f * 2048);
#pragma unroll
  for (int f = 0; f < HB; f++) bfr[f] = read_b(now.b, f);

  int kt = 0;
  auto step = [&](auto par, auto where) {
    half1(par, true, where);
    // B stage kt+1 and the A blocks of step kt+1 (up to block kt+2) have landed for this lane; younger, in issue
    // order: B stage kt+2, blocks and stages kt+3 .. kt+LEAD-1, A block kt+LEAD: LEAD-2 steps' worth of loads.
    // After the barrier they have for all, and all are done reading step kt.  The scheduler must not move MFMAs of the
    // first half behind the barrier: they are what covers the latency of the half's LDS reads before the wait.
    __builtin_amdgcn_sched_barrier(0);
    MOE_TRACE_CYCLES(tc_mark);
    if (decltype(where)::value == First::value && started_early) wait_vmcnt<(LEAD - 2) * LS + kPreStores>();
    else wait_vmcnt<(LEAD - 2) * LS>();
    wait_lds_reads<0>();
    block_barrier();
    MOE_TRACE_ADD_CYCLES(tc_sync, tc_mark);
    __builtin_amdgcn_sched_barrier(0);
    half2(par, true, where, true);
    Bb += bstep;
    kt++;
  };
  const int kt_end = nk - LEAD;   // odd; at least 1 (the caller picks NSX so that nk > LEAD)
  step(P0{}, First{});   // kt_end is odd: an even number of steps with loads follows
  while (kt + 2 <= kt_end) {
    step(P1{}, Middle{});
    step(P0{}, Middle{});
  }

  // The last LEAD steps (parities 1, 0, ..., 1) issue nothing.  With r steps still to come after the current one, what
  // is younger than the loads the step waits for is B stage kt+2 and the blocks and stages of the r-2 steps after it.
  static_assert(LEAD == 3 || LEAD == 5, "the steps without loads are written out for these two");
  if constexpr (LEAD == 5) {
    half1(P1{}, false, Last{});
    __builtin_amdgcn_sched_barrier(0);
    wait_vmcnt<LB + 2 * LS>();
    block_barrier();
    __builtin_amdgcn_sched_barrier(0);
    half2(P1{}, false, Last{}, true);
    kt++;
    half1(P0{}, false, Last{});
    __builtin_amdgcn_sched_barrier(0);
    wait_vmcnt<LB + LS>();
    block_barrier();
    __builtin_amdgcn_sched_barrier(0);
    half2(P0{}, false, Last{}, true);
    kt++;
  }
  if (tid == 0 && late) next_raw = take_from(p, xcd, q.own_len, q.own_base);
  half1(P1{}, false, Last{});
  wait_vmcnt<LB>();   // younger than the last A block: the last B stage (and a late ticket)
  block_barrier();
  half2(P1{}, false, Last{}, true);
  kt++;
  half1(P0{}, false, Last{});
  wait_vmcnt<0>();
  // No operand load is in flight any more, so memory operations the compiler waits for by itself no longer stall
  // behind them: thread 0 turns its queue ticket into a list position (stealing from other XCDs if its own queue is
  // used up) and hands it to the workgroup across the barrier; everybody then asks for the item record, whose
  // latency the remaining step and a half covers.
  uint64_t ready_mask = ~0ull;
  if (kCanPre && flags_on) ready_mask = __ballot(tid < p.n_segments && flag_v >= p.ready_epoch);
  if (tid == 0) {
    if (next_raw < 0) next_raw = steal(p, xcd);
    lds_slot[0] = next_raw;
    if (kCanPre && flags_on) {
      lds_mask[0] = (uint32_t)ready_mask;
      lds_mask[1] = (uint32_t)(ready_mask >> 32);
    }
  }
  block_barrier();
  next.idx = uniform((int)lds_slot[0]);
  if (kCanPre && flags_on)
    ready_mask = (uint32_t)uniform((int)lds_mask[0]) | ((uint64_t)(uint32_t)uniform((int)lds_mask[1]) << 32);
  ItemRec raw_rec;
  if (next.idx >= 0) raw_rec = p.items[next.idx];
  half2(P0{}, false, Last{}, true);
  kt++;
  half1(P1{}, false, Last{});
  half2(P1{}, false, Last{}, false);
  if constexpr (MA * NB == 64) {
    asm volatile("s_nop 15\n\ts_nop 3" ::: "memory");   // the last results are there (the compiler does not see MFMAs in mfma_in_place)
    __builtin_amdgcn_sched_barrier(0);
  }

  // The previous tile is published only now: its stores have drained during this tile's main loop, so the release
  // does not wait for them (publishing right after the stores would stall the next tile behind the store burst).
  if (MODE == MODE_L1 && pending_panel >= 0) {
    publish_panel(p, pending_panel);
    pending_panel = -1;
  }
  if (MODE != MODE_L1 && p.handoff_fences) __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");   // the previous tile's stores
  block_barrier();   // every wavefront is done reading the operand stages
  MOE_TRACE_STAMP(tt2);
#ifdef MOE_TILE_TRACE
  tc_loop = clock64() - tc_loop;
#endif

  if (next.idx >= 0) next.rec = make_uniform(raw_rec);
  // early start of the successor (see above): its gather rows are requested now, its first loads after the first
  // 32-row block of the epilogue, into LDS the epilogue does not use
  bool do_pre = false;
  if (kCanPre && !p.no_pre && next.idx >= 0 && next.rec.kind == kKind && ((ready_mask >> (next.rec.ready_seg & 63)) & 1)) do_pre = true;
  next.pre = do_pre;
  if (kCanPre && do_pre) load_arows<MODE>(p, next, lane, w);

  // Epilogue.  The MFMAs ran with the operands swapped (B fragment first), so a lane holds, for output row
  // lane % 16 of each 16x16 block, the four consecutive columns from 4 * (lane / 16) on.  Two neighbouring blocks become one
  // 16-byte store per lane -- 16 rows of 64 bytes -- by exchanging quarter rows between them (v_permlane16_swap): lanes
  // 16 .. 31 and 48 .. 63 end up with the second block, and a lane with the 8 columns from 8 * (lane / 32) on of its block.
  // (Staged through LDS for rows of 128 bytes the epilogue of a layer1 tile took 4.5 us: round trips and address
  // arithmetic that one wavefront per SIMD cannot hide.)
  constexpr int OUT_NB = (MODE == MODE_L0_SWIGLU) ? NB / 2 : NB;   // 16-column blocks of output per wavefront
  static_assert(OUT_NB % 2 == 0, "blocks are stored in pairs");
  int lane_e = lane;   // opaque again: the epilogue's addresses are computed here, not before the main loop
  asm volatile("" : "+v"(lane_e));
  const int col_base = (MODE == MODE_L0_SWIGLU) ? col0 + wn * (NT * 16) : col0 + wn * (NT * 32);
  // The wavefront's rows as a buffer that ends with the tile's last row: what lies behind it is not stored, without a branch,
  // so that the number of stores is the same for every tile (kPreStores).
  const int first_row = wm * (MT * 32);
  const uint32_t row_bytes = p.ldc * 2;
  const __amdgpu_buffer_rsrc_t c_rows = __builtin_amdgcn_make_buffer_rsrc(
      (void*)uniform((const char*)(p.C + (size_t)(row0 + first_row) * p.ldc + col_base)), 0,
      uniform(nrows > first_row ? (int)((nrows - first_row) * row_bytes) : 0), 0x00020000);
  uint32_t c_off = (lane_e & 15) * row_bytes + ((lane_e >> 4) & 1) * 32 + (lane_e >> 5) * 16;
#pragma unroll
  for (int ma = 0; ma < MA; ma++) {
    __builtin_amdgcn_sched_barrier(0);   // one block of rows at a time: keeps the temporaries few
    if constexpr (kCanPre) {
      if (ma == kPreBlock && do_pre) {
        if (flags_on) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "");
        LoadState ls_next;
        setup_and_issue<WM, MT, NT, MODE, PK, STREAM, NSX>(p, lds0, next, ls_next, lane_e, w, true);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    // (read out here: the compiler would otherwise move all accumulators to vector registers first, more than there are)
#pragma unroll
    for (int nb = 0; nb < NB; nb++) asm volatile("" : "+a"(acc[ma][nb]));
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int pr = 0; pr < OUT_NB / 2; pr++) {
      if (MODE == MODE_L0_GELU) __builtin_amdgcn_sched_barrier(0);  // bounds the live activation temporaries
      uint32_t d[2][2];
#pragma unroll
      for (int b = 0; b < 2; b++) {
        const int nb = 2 * pr + b;
        float v[4];
#pragma unroll
        for (int i = 0; i < 4; i++) {
          if (MODE == MODE_L0_SWIGLU) v[i] = silu(acc[ma][nb][i]) * acc[ma][nb + NB / 2][i];
          else if (MODE == MODE_L0_GELU) v[i] = gelu_erf(acc[ma][nb][i]);
          else v[i] = acc[ma][nb][i];
        }
        const bf16x2 lo = {(__bf16)v[0], (__bf16)v[1]}, hi = {(__bf16)v[2], (__bf16)v[3]};
        d[b][0] = __builtin_bit_cast(uint32_t, lo);
        d[b][1] = __builtin_bit_cast(uint32_t, hi);
      }
      u32x4 o;
#pragma unroll
      for (int j = 0; j < 2; j++) {
        const auto x = __builtin_amdgcn_permlane16_swap(d[0][j], d[1][j], false, false);
        o[j] = x[0];
        o[2 + j] = x[1];
      }
      __builtin_amdgcn_raw_buffer_store_b128(o, c_rows, c_off + pr * 64, 0, 0);
    }
    c_off += 16 * row_bytes;
  }
  if (MODE == MODE_L1 && p.fused_combine) {
    if (p.batch_publish) {
      if (tid == 0) lds_panel_count_ptr[n_tile] += 1;
    } else {
      pending_panel = n_tile;
    }
  }
  // Top-k reduction in the layer1 epilogue (the vertical fusion Section 3.2.1 weighs against its specialised
  // blocks).  The k rows of a token lie in tiles of different experts, finished by different workgroups at different
  // times, so the tile still writes its rows of Y; then every row announces itself on a counter per (token, column
  // panel), and the row that finds the other k-1 already there reduces the token: it reads the k rows back in slot
  // order and writes the output row -- the same sum in the same order as the stand-alone kernel, whoever comes last.
  // Nobody waits for anybody; the price is one device-wide release per tile (the rows must be visible before they are
  // announced) and one acquire.
  if (MODE == MODE_L1 && p.epilogue_combine) {
    volatile int32_t* last_list = (volatile int32_t*)(smem + list_offset(BM, NSX));   // free, see list_offset
    int32_t* last_count = (int32_t*)(smem + list_offset(BM, NSX) + 256 * 4);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    __syncthreads();
    if (tid == 0) *last_count = 0;
    __syncthreads();
    const int n_panels = p.H / BN;
    if (tid < nrows) {
      const int t = p.perm[row0 + tid] / p.k;
      const uint32_t before = __hip_atomic_fetch_add(&p.arrive[(size_t)t * n_panels + n_tile], 1u, __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_AGENT);
      if (before + 1 == (uint32_t)p.k) last_list[atomicAdd(last_count, 1)] = t;
    }
    __syncthreads();
    const int n_last = uniform(*(volatile int32_t*)last_count);
    if (n_last > 0) {
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
      const size_t col = (size_t)n_tile * BN + (tid & 31) * 8;
      for (int e = tid >> 5; e < n_last; e += 8) {
        const int t = last_list[e];
        float acc[8];
#pragma unroll
        for (int c = 0; c < 8; c++) acc[c] = 0.f;
        for (int j = 0; j < p.k; j++) {
          const int row = p.inv_perm[t * p.k + j];
          const float wj = p.topk_weights[t * p.k + j];
          const u32x4 v = *(const u32x4*)(p.C + (size_t)row * p.ldc + col);
#pragma unroll
          for (int c = 0; c < 4; c++) {
            acc[2 * c] += wj * __uint_as_float(v[c] << 16);
            acc[2 * c + 1] += wj * __uint_as_float(v[c] & 0xffff0000u);
          }
        }
        u32x4 o;
#pragma unroll
        for (int c = 0; c < 4; c++) {
          bf16x2 pr = {(__bf16)acc[2 * c], (__bf16)acc[2 * c + 1]};
          o[c] = __builtin_bit_cast(uint32_t, pr);
        }
        *(u32x4*)(p.out + (size_t)t * p.H + col) = o;
      }
    }
    __syncthreads();   // the list is read out before the next tile's epilogue writes it
  }
  // rows of A the next tile gathers (requested only now: held across the epilogue they push it into spilling)
  if (next.idx >= 0 && !do_pre) load_arows<MODE>(p, next, lane, w);
#ifdef MOE_TILE_TRACE
  MOE_TRACE_STAMP(tt3);
  trace_tile(MODE == MODE_L1 ? 1 : 0, kKind + (cur.pre ? 4 : 0), tt0, tt1, tt2, tt3, tc_loop, tc_sync, lds_mask + 2);
#endif
}

template <int MODE, bool PK, bool STREAM>
__global__ __launch_bounds__(256, 1) void k_group_gemm(GemmParams p) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  __shared__ int32_t lds_slot[2];
  __shared__ uint32_t lds_mask[4];   // 0, 1: ready flags seen by the workgroup; 2, 3: tiles noted by a measurement build
  __shared__ int32_t lds_panel_count[kMaxPanels];   // layer1, batched publication: tiles finished per column panel
  const int tid = threadIdx.x;
#ifdef MOE_TILE_TRACE
  if (tid == 0) {   // a workgroup that gets no tile in this launch has noted none
    lds_mask[2] = lds_mask[3] = 0;
    if (blockIdx.x < kTraceWgs) g_trace_count[MODE == MODE_L1 ? 1 : 0][blockIdx.x] = 0;
  }
#endif
  if (MODE == MODE_L1) {
    for (int i = tid; i < kMaxPanels; i += 256) lds_panel_count[i] = 0;
  }
  if (PK && prefetch_role(p)) return;
  if (MODE == MODE_L1 && (int)blockIdx.x >= p.n_mfma) {
    if (p.fused_combine) combine_loop(p, &lds_slot[1], false);
    return;
  }
  const int lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int xcd = blockIdx.x & (kXcds - 1);
  // Whether weights are loaded with the hint is a fact of the expert: those of one tile (see stream_rows on the host side).  By the mean of the rows
  // alone, every tile of a launch alike, the tiles of a crowded expert fetched its weights from HBM one after the other.  us per gate + layer,
  // popularity falling as rank^-0.3, 3 sets of weights in turn, none / by the mean / so: 225 rows for each of 8 experts of F = 14336
  // 824 / 882 / 814, 64 of F = 2560 949 / 1005 / 942; rank^-1.2, 125 rows for each of 16 of F = 6400 691 / 674 / 612; even, 200 for each of 64 of F =
  // 2560 828 / 801 / 799; tiles of 128 rows for 150, 16 of F = 6400 641 / 814 / 641.
  __shared__ uint64_t lds_stream[STREAM ? kMaxExperts / 64 : 1];   // a bit per expert
  static_assert(kMaxExperts == 256, "an expert per thread");
  int my_rows = 0;
  if (STREAM) my_rows = p.counts[min(tid, p.E - 1)];
  Queue q;
  q.own_len = p.queue_len[xcd];
  q.own_base = queue_pos(p, xcd, 0);
  int pending_panel = -1;   // layer1: column panel of the last finished tile, not yet published
  // 64-row tiles run with the deeper operand rings whenever the reduction is long enough to fill them
  const bool deep64 = p.deep_short_tiles && p.K / BK > kDeepStages - 1;

  // first tile: found synchronously
  Tile cur, next;
  auto take_sync = [&](Tile& t) {
    if (tid == 0) {
      int idx = take_from(p, xcd, q.own_len, q.own_base);
      if (idx < 0) idx = steal(p, xcd);
      lds_slot[0] = idx;
    }
    __syncthreads();
    t.idx = uniform((int)lds_slot[0]);
    t.pre = 0;
    __syncthreads();
    if (t.idx >= 0) {
      t.rec = load_item(p, t.idx);
      load_arows<MODE>(p, t, lane, w);
    }
  };
  take_sync(cur);
  if (STREAM) {
    const uint64_t few = __ballot(my_rows <= p.stream_rows);
    if (lane == 0) lds_stream[w] = few;
  }
  while (cur.idx >= 0) {
    // every wavefront is done with the LDS of the previous tile before its slots are refilled
    __syncthreads();
    if (!cur.pre && !segment_ready<MODE>(p, cur, lds_slot, true)) {
      take_sync(cur);   // timed out (status says so): give the tile up and take another one
      continue;
    }
    next.idx = -1;
    auto run = [&](auto hint) {
      constexpr bool S = decltype(hint)::value;
      if (cur.rec.kind == 2) run_tile<2, 4, 4, MODE, PK, S>(p, smem, lds_slot, cur, next, xcd, q, pending_panel, lds_panel_count, lds_mask);
      else if (cur.rec.kind == 1) run_tile<2, 2, 4, MODE, PK, S>(p, smem, lds_slot, cur, next, xcd, q, pending_panel, lds_panel_count, lds_mask);
      else if (cur.rec.kind == 3) run_tile<2, 3, 4, MODE, PK, S>(p, smem, lds_slot, cur, next, xcd, q, pending_panel, lds_panel_count, lds_mask);
      else if (deep64) run_tile<1, 2, 2, MODE, PK, S, kDeepStages>(p, smem, lds_slot, cur, next, xcd, q, pending_panel, lds_panel_count, lds_mask);
      else run_tile<1, 2, 2, MODE, PK, S>(p, smem, lds_slot, cur, next, xcd, q, pending_panel, lds_panel_count, lds_mask);
    };
    if constexpr (STREAM) {
      const int e = cur.rec.expert;
      const uint32_t few = ((const uint32_t*)lds_stream)[e >> 5];
      if ((uniform((int)few) >> (e & 31)) & 1) run(std::true_type{});
      else run(std::false_type{});
    } else {
      run(std::false_type{});
    }
    cur = next;
  }
  if (MODE == MODE_L1 && p.fused_combine) {
    if (p.batch_publish) {
      // no data-movement workgroup is waiting for single tiles: one release for everything this workgroup wrote
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
      __syncthreads();
      for (int i = tid; i < p.H / BN; i += 256)
        if (lds_panel_count[i] > 0)
          __hip_atomic_fetch_add(&p.panel_done[i], (uint32_t)lds_panel_count[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    } else if (pending_panel >= 0) {
      publish_panel(p, pending_panel);
    }
    combine_loop(p, &lds_slot[1], p.batch_publish != 0);
  }
}

// ---------------------------------------------------------------------------------------------
// Both GroupGEMMs in one persistent launch (the pipelining between the layers of Fig. 3/4 without a kernel boundary
// in between).  A workgroup first walks the layer0 queues exactly as k_group_gemm does, counting its finished tiles
// per M-tile in LDS; every publish_every tiles, and when the layer0 queues are used up, it makes its stores visible
// device-wide (one agent-scope release for all tiles since the last one: a release per tile would cost a tenth of
// layer0) and adds its counts to tile_done[].  It then walks the layer1 queues; a layer1 tile of M-tile m starts once
// tile_done[m] has reached the number of layer0 column tiles.  No deadlock: a workgroup only reaches layer1 after
// every layer0 item has been handed out, and the workgroups holding them wait for nothing but the ready flags (a
// bounded wait).  Once a workgroup has seen every workgroup finish layer0 it stops checking, and only then lets a
// tile start its successor's loads early.
// ---------------------------------------------------------------------------------------------
template <int MODE0, bool PK>
__global__ __launch_bounds__(256, 1) void k_fused_layers(GemmParams p0, GemmParams p1, FuseParams f) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  __shared__ int32_t lds_slot[2];
  __shared__ uint32_t lds_mask[4];   // 0, 1: ready flags seen by the workgroup; 2, 3: tiles noted by a measurement build
  __shared__ int32_t lds_panel_count[kMaxPanels];      // unused here; run_tile takes it
  __shared__ int32_t lds_tile_cnt[kScheduleTileCap];   // layer0 tiles this workgroup finished per M-tile, not yet published
  const int tid = threadIdx.x;
#ifdef MOE_TILE_TRACE
  if (tid == 0) {
    lds_mask[2] = lds_mask[3] = 0;
    if (blockIdx.x < kTraceWgs) g_trace_count[0][blockIdx.x] = g_trace_count[1][blockIdx.x] = 0;
  }
#endif
  for (int i = tid; i < kScheduleTileCap; i += 256) lds_tile_cnt[i] = 0;
  for (int i = tid; i < kMaxPanels; i += 256) lds_panel_count[i] = 0;
  const int lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int xcd = blockIdx.x & (kXcds - 1);
  const int n_tiles = min(*p0.n_tiles, (int)kScheduleTileCap);
  int pending_panel = -1;
  __syncthreads();

  auto take_sync = [&](const GemmParams& p, const Queue& q, Tile& t, auto mode) {
    constexpr int MODE = decltype(mode)::value;
    if (tid == 0) {
      int idx = take_from(p, xcd, q.own_len, q.own_base);
      if (idx < 0) idx = steal(p, xcd);
      lds_slot[0] = idx;
    }
    __syncthreads();
    t.idx = uniform((int)lds_slot[0]);
    t.pre = 0;
    __syncthreads();
    if (t.idx >= 0) {
      t.rec = load_item(p, t.idx);
      load_arows<MODE>(p, t, lane, w);
    }
  };
  // all stores of this workgroup so far become visible device-wide, then its counts are added
  auto publish = [&]() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    __syncthreads();
    for (int i = tid; i < n_tiles; i += 256) {
      const int c = lds_tile_cnt[i];
      if (c > 0) {
        __hip_atomic_fetch_add(&f.tile_done[i], (uint32_t)c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        lds_tile_cnt[i] = 0;
      }
    }
    __syncthreads();
  };

  // ---- layer0
  {
    using M0 = std::integral_constant<int, MODE0>;
    Queue q;
    q.own_len = p0.queue_len[xcd];
    q.own_base = queue_pos(p0, xcd, 0);
    Tile cur, next;
    int since_publish = 0;
    take_sync(p0, q, cur, M0{});
    while (cur.idx >= 0) {
      __syncthreads();
      if (!cur.pre && !segment_ready<MODE0>(p0, cur, lds_slot, true)) {
        take_sync(p0, q, cur, M0{});   // timed out (status says so): the tile is given up
        continue;
      }
      next.idx = -1;
      const int m_tile = cur.rec.m_tile;
      if (cur.rec.kind == 2) run_tile<2, 4, 4, MODE0, PK, false>(p0, smem, lds_slot, cur, next, xcd, q, pending_panel, lds_panel_count, lds_mask);
      else if (cur.rec.kind == 1) run_tile<2, 2, 4, MODE0, PK, false>(p0, smem, lds_slot, cur, next, xcd, q, pending_panel, lds_panel_count, lds_mask);
      else if (cur.rec.kind == 3) run_tile<2, 3, 4, MODE0, PK, false>(p0, smem, lds_slot, cur, next, xcd, q, pending_panel, lds_panel_count, lds_mask);
      else run_tile<1, 2, 2, MODE0, PK, false>(p0, smem, lds_slot, cur, next, xcd, q, pending_panel, lds_panel_count, lds_mask);
      if (tid == 0 && (unsigned)m_tile < (unsigned)kScheduleTileCap) lds_tile_cnt[m_tile] += 1;
      cur = next;
      if (++since_publish >= f.publish_every && cur.idx >= 0) {
        // (if the successor's first loads are already in flight the fence waits for them too; the tile code's own
        // waits then find them done)
        publish();
        since_publish = 0;
      }
    }
    __syncthreads();
    publish();
    if (tid == 0) __hip_atomic_fetch_add(f.wgs_done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }

  // ---- layer1
  {
    using M1 = std::integral_constant<int, MODE_L1>;
    if ((int)blockIdx.x >= p1.n_mfma) return;
    GemmParams q1 = p1;
    q1.no_pre = 1;
    bool all_seen = false;
    Queue q;
    q.own_len = q1.queue_len[xcd];
    q.own_base = queue_pos(q1, xcd, 0);
    Tile cur, next;
    take_sync(q1, q, cur, M1{});
    while (cur.idx >= 0) {
      __syncthreads();
      if (!all_seen) {
        // the rows of this M-tile: wait until every layer0 column tile of it has been published
        if (tid == 0) {
          const uint32_t m = (uint32_t)cur.rec.m_tile < (uint32_t)kScheduleTileCap ? (uint32_t)cur.rec.m_tile : 0u;
          bool ok = spin_until_ge(&f.tile_done[m], (uint32_t)f.n_tiles_n0, q1.spin_limit ? q1.spin_limit : (1u << 26));
          if (!ok) atomicExch(q1.status, (int)MOE_ERR_TIMEOUT);
          const uint32_t done = __hip_atomic_load(f.wgs_done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          lds_slot[1] = (ok ? 1 : 0) | (done >= gridDim.x ? 2 : 0);
        }
        __syncthreads();
        const int st = lds_slot[1];
        __syncthreads();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        if (!(st & 1)) {
          take_sync(q1, q, cur, M1{});   // timed out: give the tile up
          continue;
        }
        if (st & 2) {
          all_seen = true;     // every workgroup has published everything: nothing left to wait for
          q1.no_pre = 0;
        }
      }
      next.idx = -1;
      if (cur.rec.kind == 2) run_tile<2, 4, 4, MODE_L1, PK, false>(q1, smem, lds_slot, cur, next, xcd, q, pending_panel, lds_panel_count, lds_mask);
      else if (cur.rec.kind == 1) run_tile<2, 2, 4, MODE_L1, PK, false>(q1, smem, lds_slot, cur, next, xcd, q, pending_panel, lds_panel_count, lds_mask);
      else if (cur.rec.kind == 3) run_tile<2, 3, 4, MODE_L1, PK, false>(q1, smem, lds_slot, cur, next, xcd, q, pending_panel, lds_panel_count, lds_mask);
      else run_tile<1, 2, 2, MODE_L1, PK, false>(q1, smem, lds_slot, cur, next, xcd, q, pending_panel, lds_panel_count, lds_mask);
      cur = next;
    }
  }
}

// The kernels need more dynamic LDS than the default limit.  The attribute belongs to the function on one device; it is
// set once per function and device (a bit per device, set after the call succeeded: two threads racing set it twice,
// which is harmless) and never inside a launch that may be under stream capture.
static hipError_t allow_large_lds(const void* kern, int lds_bytes) {
  struct Entry { const void* kern; std::atomic<uint64_t> devices; };
  static Entry entries[16];
  static std::atomic<int> n_entries{0};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const uint64_t bit = 1ull << (dev & 63);
  const int n = n_entries.load(std::memory_order_acquire);
  for (int i = 0; i < n; i++)
    if (entries[i].kern == kern && (entries[i].devices.load(std::memory_order_acquire) & bit)) return hipSuccess;
  e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
  if (e != hipSuccess) return e;
  for (int i = 0; i < n; i++)
    if (entries[i].kern == kern) {
      entries[i].devices.fetch_or(bit, std::memory_order_release);
      return hipSuccess;
    }
  static std::mutex mu;
  std::lock_guard<std::mutex> lock(mu);
  const int m = n_entries.load(std::memory_order_acquire);
  for (int i = 0; i < m; i++)
    if (entries[i].kern == kern) {
      entries[i].devices.fetch_or(bit, std::memory_order_release);
      return hipSuccess;
    }
  if (m < 16) {
    entries[m].kern = kern;
    entries[m].devices.store(bit, std::memory_order_release);
    n_entries.store(m + 1, std::memory_order_release);
  }
  return hipSuccess;   // table full: the attribute is simply set again next time
}

template <int MODE0, bool PK>
static hipError_t launch_fused(const GemmParams& p0, const GemmParams& p1, const FuseParams& f, int grid, hipStream_t st) {
  constexpr int lds = kLdsBytes;
  auto kern = k_fused_layers<MODE0, PK>;
  hipError_t e = allow_large_lds((const void*)kern, lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(grid), dim3(256), lds, st, p0, p1, f);
  return hipGetLastError();
}

hipError_t launch_fused_layers(const GemmParams& p0, const GemmParams& p1, const FuseParams& f, int act, int grid, hipStream_t st) {
  if (act == MOE_ACT_SWIGLU)
    return p0.b_packed ? launch_fused<MODE_L0_SWIGLU, true>(p0, p1, f, grid, st) : launch_fused<MODE_L0_SWIGLU, false>(p0, p1, f, grid, st);
  return p0.b_packed ? launch_fused<MODE_L0_GELU, true>(p0, p1, f, grid, st) : launch_fused<MODE_L0_GELU, false>(p0, p1, f, grid, st);
}

template <int MODE, bool PK>
static hipError_t launch_gemm(const GemmParams& p, int grid, hipStream_t st) {
  constexpr int lds = kLdsBytes;
  auto kern = p.stream_rows > 0 ? k_group_gemm<MODE, PK, true> : k_group_gemm<MODE, PK, false>;
  hipError_t e = allow_large_lds((const void*)kern, lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(grid), dim3(256), lds, st, p);
  return hipGetLastError();
}

hipError_t launch_layer0(const GemmParams& p, int act, int grid, hipStream_t st) {
  if (act == MOE_ACT_SWIGLU) return p.b_packed ? launch_gemm<MODE_L0_SWIGLU, true>(p, grid, st) : launch_gemm<MODE_L0_SWIGLU, false>(p, grid, st);
  return p.b_packed ? launch_gemm<MODE_L0_GELU, true>(p, grid, st) : launch_gemm<MODE_L0_GELU, false>(p, grid, st);
}

hipError_t launch_layer1(const GemmParams& p, int grid, hipStream_t st) {
  return p.b_packed ? launch_gemm<MODE_L1, true>(p, grid, st) : launch_gemm<MODE_L1, false>(p, grid, st);
}

// ---------------------------------------------------------------------------------------------
// Weight packing (once per set of weights, outside the forward): B [E][K][ldb] row-major becomes, per expert, column
// tile and K step of 32, the 16 KiB LDS image of that stage: 16 fragments of 1 KiB, fragment (kk, c) = 16 values of K
// (kk-th half of the step) x 32 columns (c-th block of the tile), lane l of a wavefront owning the 8 K-consecutive
// values k = kk*16 + (l/32)*8 .. +7 of column l%32 -- the operand layout of v_mfma_f32_32x32x16_bf16; the 16 columns by 32
// values that v_mfma_f32_16x16x32_bf16 takes are four pieces of 256 bytes of two of them.  A tile's stages
// follow each other in memory, so a workgroup streams one contiguous run per tile.
// Column blocks: plain layers, block c = columns [32c, 32c+32) of the tile.  SwiGLU W1 ([gate | up] column halves): tile
// n covers hidden units [128n, 128n+128); blocks 0..3 are their gate columns, blocks 4..7 their up columns.
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_pack_weights(const uint16_t* __restrict__ B, uint16_t* __restrict__ out, int K, int ldb,
                                                      int n_tiles_n, int swiglu_F, size_t total_chunks) {
  // one 16-byte chunk (8 values of K for one column) per thread step
  const int nk = K / BK;
  for (size_t ch = (size_t)blockIdx.x * 256 + threadIdx.x; ch < total_chunks; ch += (size_t)gridDim.x * 256) {
    const int l = (int)(ch & 63);
    const int frag = (int)((ch >> 6) & 15);
    const size_t stage = ch >> 10;
    const int kt = (int)(stage % nk);
    const size_t en = stage / nk;
    const int n = (int)(en % n_tiles_n);
    const size_t e = en / n_tiles_n;
    const int kk = frag >> 3, c = frag & 7;
    const int k0 = kt * BK + kk * 16 + (l >> 5) * 8;
    int col;
    if (swiglu_F > 0) col = (c >> 2) * swiglu_F + n * (BN / 2) + (c & 3) * 32 + (l & 31);
    else col = n * BN + c * 32 + (l & 31);
    const uint16_t* src = B + (e * K + k0) * (size_t)ldb + col;
    u32x4 v;
#pragma unroll
    for (int i = 0; i < 4; i++) v[i] = (uint32_t)src[(size_t)(2 * i) * ldb] | ((uint32_t)src[(size_t)(2 * i + 1) * ldb] << 16);
    *(u32x4*)(out + ch * 8) = v;
  }
}

hipError_t launch_pack_weights(const void* B, void* out, int E, int K, int ldb, int n_tiles_n, int swiglu_F, hipStream_t st) {
  const size_t total_chunks = (size_t)E * n_tiles_n * (K / BK) * (B_STAGE / 16);
  if (total_chunks == 0) return hipSuccess;
  size_t grid = (total_chunks + 255) / 256;
  if (grid > 256 * 32) grid = 256 * 32;
  hipLaunchKernelGGL(k_pack_weights, dim3((unsigned)grid), dim3(256), 0, st, (const uint16_t*)B, (uint16_t*)out, K, ldb, n_tiles_n,
                     swiglu_F, total_chunks);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// Stand-alone top-k weighted reduction (used when the layer1 kernel runs without data-movement workgroups).  HBM-bound: 32
// lanes own 256 columns of TOKENS tokens and request the rows of all of them before any is used (8 in flight per lane; walked
// one row at a time, index and row a dependent pair of loads each, 8192 tokens with k = 4 and H = 2048 took 35.5 us, 4.7
// TB/s; now 28.8, 5.8 TB/s).  K = 0: any other k, one row at a time.
// ---------------------------------------------------------------------------------------------
constexpr int combine_tokens(int k) { return k == 1 || k == 2 ? 4 : (k == 4 ? 2 : 1); }
constexpr int kCombineResident = 2048;   // workgroups the device holds at once; up to there one token per 32 lanes (more to start)
template <int K, int TOKENS>
__global__ __launch_bounds__(256) void k_combine(CombineParams p, int n_panels, int n_units) {
  constexpr int KK = K > 0 ? K : 1;
  const int u = blockIdx.x * 8 + (threadIdx.x >> 5);
  if (u >= n_units) return;
  const int group = u / n_panels;
  const size_t col = (size_t)(u - group * n_panels) * BN + (threadIdx.x & 31) * 8;
  const int t0 = group * TOKENS, k = K > 0 ? K : p.k;
  float acc[TOKENS][8];
  auto add = [&](float (&a)[8], float w, const u32x4& v) {
#pragma unroll
    for (int c = 0; c < 4; c++) {
      a[2 * c] += w * __uint_as_float(v[c] << 16);
      a[2 * c + 1] += w * __uint_as_float(v[c] & 0xffff0000u);
    }
  };
#pragma unroll
  for (int i = 0; i < TOKENS; i++)
#pragma unroll
    for (int c = 0; c < 8; c++) acc[i][c] = 0.f;
  if constexpr (K > 0) {
    int row[TOKENS][KK];
    float w[TOKENS][KK];
    u32x4 v[TOKENS][KK];
#pragma unroll
    for (int i = 0; i < TOKENS; i++) {
      const int t = min(t0 + i, p.T - 1);
#pragma unroll
      for (int j = 0; j < KK; j++) {
        row[i][j] = p.inv_perm[t * KK + j];
        w[i][j] = p.topk_weights[t * KK + j];
      }
    }
#pragma unroll
    for (int i = 0; i < TOKENS; i++)
#pragma unroll
      for (int j = 0; j < KK; j++) v[i][j] = *(const u32x4*)(p.Y + (size_t)row[i][j] * p.H + col);
    __builtin_amdgcn_sched_barrier(0);   // all requested by here
#pragma unroll
    for (int i = 0; i < TOKENS; i++)
#pragma unroll
      for (int j = 0; j < KK; j++) add(acc[i], w[i][j], v[i][j]);
  } else {
    for (int j = 0; j < k; j++)
      add(acc[0], p.topk_weights[t0 * k + j], *(const u32x4*)(p.Y + (size_t)p.inv_perm[t0 * k + j] * p.H + col));
  }
#pragma unroll
  for (int i = 0; i < TOKENS; i++) {
    if (t0 + i >= p.T) break;
    u32x4 o;
#pragma unroll
    for (int c = 0; c < 4; c++) {
      const bf16x2 pr = {(__bf16)acc[i][2 * c], (__bf16)acc[i][2 * c + 1]};
      o[c] = __builtin_bit_cast(uint32_t, pr);
    }
    *(u32x4*)(p.out + (size_t)(t0 + i) * p.H + col) = o;
  }
}

__global__ __launch_bounds__(256) void k_zero_u32(uint32_t* __restrict__ ptr, size_t n) {
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) ptr[i] = 0u;
}

hipError_t launch_zero_u32(uint32_t* ptr, size_t n, hipStream_t st) {
  if (n == 0) return hipSuccess;
  size_t grid = (n + 255) / 256;
  if (grid > 1024) grid = 1024;
  hipLaunchKernelGGL(k_zero_u32, dim3((unsigned)grid), dim3(256), 0, st, ptr, n);
  return hipGetLastError();
}

template <int K, int TOKENS = combine_tokens(K)>
static hipError_t launch_combine_k(const CombineParams& p, hipStream_t st) {
  const int n_panels = p.H / BN, n_units = (p.T + TOKENS - 1) / TOKENS * n_panels;   // (T * H < 2^31)
  if constexpr (TOKENS > 1) {
    if (p.T * n_panels <= 8 * kCombineResident) return launch_combine_k<K, 1>(p, st);
  }
  hipLaunchKernelGGL((k_combine<K, TOKENS>), dim3((n_units + 7) / 8), dim3(256), 0, st, p, n_panels, n_units);
  return hipGetLastError();
}

hipError_t launch_combine(const CombineParams& p, hipStream_t st) {
  if (p.T == 0) return hipSuccess;
  switch (p.k) {
    case 1: return launch_combine_k<1>(p, st);
    case 2: return launch_combine_k<2>(p, st);
    case 4: return launch_combine_k<4>(p, st);
    case 8: return launch_combine_k<8>(p, st);
    default: return launch_combine_k<0>(p, st);
  }
}

}  // namespace moe

#ifdef MOE_TILE_TRACE
// Measurement build only.  reset != 0: forget the tiles noted so far.  Otherwise copies out, per layer (0, 1) and
// workgroup (256), the number of tiles noted, and per tile (128 slots) the four time stamps, the two cycle counts and the height class
// (0 / 1 / 3 / 2 for 64 / 128 / 192 / 256 rows, +4 when the tile's first loads were started by its predecessor).  Host pointers.
extern "C" int moe_debug_tile_trace(int reset, uint64_t* stamps, int32_t* kinds, int32_t* counts) {
  if (hipDeviceSynchronize() != hipSuccess) return MOE_ERR_HIP;
  if (reset) {
    static const int32_t zeros[2][moe::kTraceWgs] = {};
    return hipMemcpyToSymbol(HIP_SYMBOL(moe::g_trace_count), zeros, sizeof(zeros)) == hipSuccess ? MOE_OK : MOE_ERR_HIP;
  }
  if (!stamps || !kinds || !counts) return MOE_ERR_INVALID_ARG;
  if (hipMemcpyFromSymbol(stamps, HIP_SYMBOL(moe::g_trace_stamp), sizeof(uint64_t) * 2 * moe::kTraceWgs * moe::kTraceTiles * moe::kTraceWords) != hipSuccess ||
      hipMemcpyFromSymbol(kinds, HIP_SYMBOL(moe::g_trace_kind), sizeof(int32_t) * 2 * moe::kTraceWgs * moe::kTraceTiles) != hipSuccess ||
      hipMemcpyFromSymbol(counts, HIP_SYMBOL(moe::g_trace_count), sizeof(int32_t) * 2 * moe::kTraceWgs) != hipSuccess)
    return MOE_ERR_HIP;
  return MOE_OK;
}
#endif

