// GroupGEMM of small batches (a few rows per expert: decoding), for gfx950.
//
// What bounds it is the stream of weights from HBM: every expert that some token picked is read once for a handful of
// rows.  The persistent tile kernel (grouped_gemm.hip) keeps that stream going only while it has a 64 x 256 tile or two
// per compute unit; with few rows there are few tiles (layer1 of one token of 8 experts, H = 4096: 32), and the rest of
// the chip idles.  Here the unit of work is one wavefront's: 16 to 64 columns of one expert by up to 32 rows.
//  * A wavefront sums all of K, 32 values at a time with the tile kernel's instruction in the tile kernel's order: an output has
//    the same bits whichever kernel computes it, whatever the batch around it.  (K split over 8 wavefronts that added their
//    parts up had not, and was not faster: below.)
//  * It keeps a ring of operands in registers, loaded 2 to 8 steps of 64 values of K ahead, and meets nobody; its rows of A go
//    through a private piece of LDS (8 whole lines per load instruction, then one ds_read_b128 per fragment: read as
//    fragments from memory they took a third longer at 8 rows).
//  * The first loads of the next unit are issued before this one is written, and several wavefronts share a SIMD, so that the
//    stream does not stop at the ends of units.
//  * Packed weights arrive in MFMA operand order (a fragment is 4 pieces of 256 bytes).  With SwiGLU a wavefront has the gate and
//    the up columns of its hidden units.  Plain weights are loaded as they lie (rows of K, whole 128-byte lines) and
//    transposed through LDS with ds_read_b64_tr_b16; with SwiGLU the two wavefronts of a workgroup take gate and up and
//    exchange halves at the end (in 64-byte pieces, both in one wavefront: 61 us against 47 on layer0 of 33 tokens, F = 1792).
//  * A unit of layer0 waits for the source segment of its tile alone; where that is missing for good the others are computed.
//  * There is no schedule: wavefronts walk the units with a fixed stride.  An expert with more rows than a unit holds is several
//    units per columns, next to each other on one XCD, so that its weights come from HBM once.  (With the parts of all experts
//    one after the other they came once per part: 128 tokens of 64 experts, popularity falling as rank^-1.2, 450 / 247 us per
//    layer0 / layer1 launch, now 390 / 200; the tile kernel 335 / 182.  256 tokens of 64 experts of F = 1408 116 / 131 ->
//    96 / 52, tile kernel 95 / 51.)  The row blocks and rows of A that a unit does not have cost nothing: no MFMA, loads
//    beyond the end of the buffer.
// us for both layers, tile kernel -> K in 8 parts -> this one: Mixtral-shaped packed, 1 token 263 -> 135 -> 134 (704 MB: 5.3
// TB/s), 16 tokens 532 -> 485 -> 490 (2.8 GB: 5.8 TB/s; a copy of 1 GiB moves 4.4 TB/s, half of it writes); 64 experts of
// F = 2560, 48 tokens 636 -> 610 -> 614; plain, 8 experts of F = 1792, 33 tokens 102 -> 82 -> 77.
// Then with non-temporal loads of B (gate and layer together): 1 token 134 -> 121 (704 MB: 6.3 TB/s over the two launches), 16 tokens 480
// -> 430 (6.8 TB/s), 48 of 64 experts 614 -> 560, 33 plain 82 -> 76.
#include "moe_device.h"

namespace moe {

constexpr int kDecodeWaves = 2;                    // of a workgroup
constexpr int kUnitChunk = 2;                      // consecutive units on one XCD
constexpr uint32_t kRowsEnd = 1u << 31;            // no row of A has an offset of this or more; past it a load returns zeros
constexpr int kDecodeTileCap = 384;                // tiles of a batch the kernel is used for: at most 4096 / 64 full ones and 256 others
static_assert(kDecodeTileCap % 64 == 0 && kDecodeTileCap >= kDecodeRowsPerExpert * kMaxExperts / 64 + kMaxExperts &&
              kDecodeTileCap >= kDecodeCachedRows / 64 + kMaxExperts && kDecodeCachedRows < 65536, "tiles of the largest batch");
constexpr int kStageBytes = kTileK * kTileN * 2;   // packed weights: one K step of one column tile
constexpr int kPlainPitch = 144;                   // bytes between rows of K in the transposing buffer (64 columns + padding)
constexpr int kNonTemporal = 2;                    // cache policy of a buffer load: the nt bit
constexpr int kStepK = 64;                         // K of one ring slot: a whole 128-byte line of every row of A

// The memory from ptr on (the same in every lane) as a buffer: loads then take one 32-bit offset per lane and one scalar
// offset, and no 64-bit address per load sits in vector registers.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer(const char* ptr, uint32_t bytes = 0xffffffff) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)uniform(ptr), 0, bytes, 0x00020000);
}

// What a workgroup's wavefronts find their units in: the rows of the batch in slots, the tiles of the table or the experts.
struct UnitTable {
  int32_t unit0[kDecodeTileCap];   // units of the slots before
  uint16_t row0[kDecodeTileCap], rows[kDecodeTileCap];
  uint8_t expert[kDecodeTileCap], seg[kDecodeTileCap];
  uint16_t token[kOwnIndexRows];   // own_index: row -> token
  int32_t n_units;
};

// unit0 and n_units from the rows of n slots; for one wavefront.
__device__ __forceinline__ void number_units(UnitTable& L, int n, int rows_per_unit, int n_groups) {
  const int lane = threadIdx.x & 63;
  int n_units = 0;
#pragma unroll 1
  for (int i0 = 0; i0 < n; i0 += 64) {
    const int rows = i0 + lane < n ? L.rows[i0 + lane] : 0;
    const int mine = (rows + rows_per_unit - 1) / rows_per_unit * n_groups;
    int incl = mine;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const int o = __shfl_up(incl, d);
      if (lane >= d) incl += o;
    }
    L.unit0[i0 + lane] = n_units + incl - mine;   // (the capacity is a multiple of 64)
    n_units += uniform(__shfl(incl, 63));
  }
  if (lane == 0) L.n_units = n_units;
}

// The tile table of the index build.  All of it is asked for at once, before the number of tiles is known.
__device__ __forceinline__ int load_table(UnitTable& L, const DecodeParams& p, int rows_per_unit, int n_groups, bool flagged) {
  const int n_tiles = min(*p.n_tiles, kDecodeTileCap);
  for (int i = threadIdx.x; i < p.n_slots; i += kDecodeWaves * 64) {
    L.row0[i] = (uint16_t)p.tile_row0[i];
    L.rows[i] = (uint16_t)p.tile_rows[i];
    L.expert[i] = (uint8_t)p.tile_expert[i];
    if (flagged) L.seg[i] = (uint8_t)p.tile_ready[i];
  }
  __syncthreads();
  if (threadIdx.x < 64) number_units(L, n_tiles, rows_per_unit, n_groups);
  __syncthreads();
  return n_tiles;
}

// The index of a batch of up to kOwnIndexRows pairs, by every workgroup for itself from the expert ids: stable ranks by ballots over runs
// of 64 pairs, as k_index_small makes them.  The slots are the experts.  That launch of one workgroup takes 5 us whatever the batch, and the
// table it leaves is three dependent round trips to memory at the start of a GroupGEMM launch; the ids are one.  out: the
// workgroup that leaves the index of this forward in the workspace too, as k_index_small does without schedules, for the reduction and whoever
// asks for it.  us per gate + layer, with k_index_small / so: 1 token of 8 experts of F = 1792 37.7 / 34.0, 16 tokens 70.2 / 67.5, 33 plain
// 78.4 / 76.3, 1 token of F = 14336 121 / 119; 64 experts of F = 1408, 128 pairs 164.5 / 162.4, 256 184.6 / 183.5, 384 188.0 / 187.9, 512 193.1 /
// 194.4; 4 of H = 256, F = 512, 256 24.5 / 22.2, 384 24.4 / 23.4, 512 24.4 / 24.7; 64 of H = F = 512, 384 35.0 / 34.4, 512 35.0 / 36.1.  With more
// experts there is more to number: 128 of F = 1024, popularity falling as rank^-1.2, 256 pairs 75.3 / 74.6, 384 93.0 / 94.0,
// 512 97.1 / 99.1; 256 experts of F = 1024 128 pairs 103.4 / 105.0, 256 144.4 / 146.8.
__device__ __forceinline__ void own_index(UnitTable& L, const DecodeParams& p, int rows_per_unit, int n_groups, const IndexParams& ip, bool out) {
  constexpr int kRuns = kOwnIndexRows / 64;
  const int tid = threadIdx.x, lane = tid & 63, E = p.E, R = p.R;
  __shared__ int32_t tile0[kMaxExperts + 1];   // out: tiles of the experts before
  if (tid < 64) {
    int key[kRuns], rank[kRuns];
#pragma unroll
    for (int i = 0; i < kRuns; i++) key[i] = i * 64 + lane < R ? p.topk_ids[i * 64 + lane] : -1;
    for (int e = lane; e < E; e += 64) L.rows[e] = 0;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
    for (int i = 0; i < kRuns; i++) {
      if (i * 64 >= R) break;
      const bool valid = i * 64 + lane < R;
      int e = key[i];
      if (valid && (unsigned)e >= (unsigned)E) {   // not an expert: reported through the status word, counted as the last expert
        if (out) ip.ws.status[5] = ip.forward_serial;
        e = E - 1;
      }
      uint64_t same = __ballot(valid);
#pragma unroll
      for (int bit = 0; bit < 8; bit++) {
        const uint64_t b = __ballot((e >> bit) & 1);
        same &= ((e >> bit) & 1) ? b : ~b;
      }
      const uint64_t below = same & ((1ull << lane) - 1ull);
      const int before = valid ? L.rows[e] : 0;   // in the runs before
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      if (valid && below == 0) L.rows[e] = (uint16_t)(before + __popcll(same));
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      key[i] = e;
      rank[i] = before + __popcll(below);
    }
    int rows_before = 0;
#pragma unroll 1
    for (int e0 = 0; e0 < E; e0 += 64) {
      const int rows = e0 + lane < E ? L.rows[e0 + lane] : 0;
      int incl = rows;
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) {
        const int o = __shfl_up(incl, d);
        if (lane >= d) incl += o;
      }
      if (e0 + lane < E) {
        L.row0[e0 + lane] = (uint16_t)(rows_before + incl - rows);
        L.expert[e0 + lane] = (uint8_t)(e0 + lane);
      }
      rows_before += uniform(__shfl(incl, 63));
    }
    number_units(L, E, rows_per_unit, n_groups);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
    for (int i = 0; i < kRuns; i++) {
      const int q = i * 64 + lane;
      if (q < R) {
        const int pos = L.row0[key[i]] + rank[i], t = q / p.k;
        L.token[pos] = (uint16_t)t;
        if (out) {
          ip.ws.perm[pos] = q;
          ip.ws.inv_perm[q] = pos;
          ip.ws.row_token[pos] = t;
        }
      }
    }
    if (out) {
      const int tile_m = ip.tile_m;
      int tiles_before = 0;
#pragma unroll 1
      for (int e0 = 0; e0 < E; e0 += 64) {
        const int rows = e0 + lane < E ? L.rows[e0 + lane] : 0, tiles = (rows + tile_m - 1) / tile_m;
        int incl = tiles;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
          const int o = __shfl_up(incl, d);
          if (lane >= d) incl += o;
        }
        if (e0 + lane < E) tile0[e0 + lane] = tiles_before + incl - tiles;
        tiles_before += uniform(__shfl(incl, 63));
      }
      if (lane == 0) tile0[E] = tiles_before;
      const int waves = waves_now(ip, lane);
      if (lane == 0) ip.ws.status[7] = waves;
    }
  }
  __syncthreads();
  if (!out) return;
  for (int i = tid; i < ip.n_tiles_n1; i += kDecodeWaves * 64) ip.ws.panel_done[i] = 0;
  for (int i = tid; i < ip.max_tiles + 1; i += kDecodeWaves * 64) ip.ws.tile_done[i] = 0;
  if (tid < 2 * kXcds) ip.ws.queue_heads[tid * ip.ws.head_stride] = 0;
  if (tid == 0) {
    const int n_tiles = tile0[E];
    ip.ws.status[0] = 0;
    ip.ws.status[1] = n_tiles;
    ip.ws.status[2] = n_tiles * ip.n_tiles_n0;
    ip.ws.status[3] = n_tiles * ip.n_tiles_n1;
    ip.ws.status[4] = 0;
    ip.ws.status[6] = kScheduleOwed;
    ip.ws.offsets[E] = R;
  }
  for (int e = tid; e < E; e += kDecodeWaves * 64) {
    const int rows = L.rows[e], row0 = L.row0[e], tile_m = ip.tile_m;
    ip.ws.counts[e] = rows;
    ip.ws.offsets[e] = row0;
    for (int i = 0; i * tile_m < rows; i++) {
      const int m = tile0[e] + i, n = min(rows - i * tile_m, tile_m);
      const int last = L.token[row0 + i * tile_m + n - 1];
      int s = 0;
      while (s + 1 < ip.s.S && ip.seg_offsets[s + 1] <= last) s++;
      ip.ws.tile_expert[m] = e;
      ip.ws.tile_row0[m] = row0 + i * tile_m;
      ip.ws.tile_rows[m] = n;
      ip.ws.tile_kind[m] = height_class(n);
      ip.ws.tile_ready[m] = s;
    }
  }
}

// NB: 16-column blocks of weights of a wavefront (SwiGLU: half of them gate, half up columns of the same hidden units);
// RB: 8-row groups of A that are loaded (a unit is up to 8 RB rows); U: steps in flight; EU: wavefronts a SIMD holds; STREAM:
// the loads of B are non-temporal (DecodeParams::b_stream).
template <int MODE, bool PK, int NB, int RB, int U, int EU, bool STREAM>
__global__ __launch_bounds__(kDecodeWaves * 64) __attribute__((amdgpu_waves_per_eu(EU))) void k_decode_gemm(DecodeParams p, IndexParams ip) {
  constexpr bool kPair = MODE == MODE_L0_SWIGLU;
  constexpr int ROWS = 8 * RB;
  constexpr int RR = (RB + 1) / 2;                     // 16-row blocks
  constexpr bool kInWave = kPair && PK;                // gate and up columns of a hidden unit in one wavefront ...
  constexpr bool kTwoWaves = kPair && !PK;             // ... or in the workgroup's two
  constexpr int OB = kInWave ? NB / 2 : NB;            // 16-column blocks of C of a unit
  constexpr int NBL = NB * 2;                          // 16-byte loads of B per lane and step
  constexpr int kABytes = RR * 16 * kStepK * 2;        // rows of A of one step, in LDS
  constexpr int kWaveBytes = kABytes + (PK ? 0 : kTileK * kPlainPitch);   // operands on their way through LDS
  constexpr bool kAhead = U >= 4 && (RB == 1 || !PK);  // a step's rows of A go through LDS a step ahead
  static_assert(PK || NB == 4 || (NB == 2 && !kPair), "plain weights: rows of K in pieces of 64 or 128 bytes");
  static_assert(!kAhead || U % 2 == 0, "the fragments of A alternate between two sets of registers");
  __shared__ __attribute__((aligned(16))) f32x4 swap_lds[kTwoWaves ? 2 : 1][2][kTwoWaves ? RR * 2 : 1][kTwoWaves ? 64 : 1];
  __shared__ __attribute__((aligned(128))) char operands[kDecodeWaves * kWaveBytes];
  __shared__ UnitTable L;
  __shared__ int given_up[2][2];   // [turn][wavefront]: no rows for this unit

  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  // Source segments that have arrived.  A unit waits for its tile's segment only, and starts early where that is there.
  uint64_t there = ~0ull;
  bool patient = true;   // false once a wait has run out: what is missing then is not waited for again
  auto look = [&]() {
    const bool up = lane < p.n_segments && __hip_atomic_load(&p.seg_ready[lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM) >= p.ready_epoch;
    there = __ballot(up);
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "");
  };
  if (MODE == MODE_L1 && p.own_index && blockIdx.x == 0 && tid == 0) {   // what layer0 had to say of its waits, see start_when_there
    if (p.status[kTimedOutAt] == p.forward_serial) p.status[0] = (int)MOE_ERR_TIMEOUT;
    p.status[kTimedOutAt] = 0;
  }
  const bool flagged = MODE != MODE_L1 && p.seg_ready != nullptr;
  if (flagged) look();

  // Units: (slot of the table, columns, row part), the parts fastest.
  const int nk = p.K / kStepK;
  const int n_groups = p.N / (OB * 16);
  constexpr bool kMayWriteIndex = MODE != MODE_L1;
  const int index_blocks = kMayWriteIndex && p.own_index ? kXcds : 0;   // at the front of the grid, see own_index
  if (kMayWriteIndex && index_blocks && blockIdx.x > 0 && (int)blockIdx.x < index_blocks) return;
  const int block = (int)blockIdx.x - index_blocks;
  int n_slots;
  if (p.own_index) {
    n_slots = p.E;
    own_index(L, p, ROWS, n_groups, ip, kMayWriteIndex && block < 0);
    if (kMayWriteIndex && block < 0) return;
  } else {
    n_slots = load_table(L, p, ROWS, n_groups, flagged);
  }
  const int n_units = uniform(L.n_units);
  // the source segment of a token: those that end at it or before
  const int seg_end = flagged && p.own_index && lane < p.n_segments - 1 ? ip.seg_offsets[lane + 1] : 0x7fffffff;
  auto segment_of = [&](int token) { return (int)__popcll(__ballot(seg_end <= token)); };
  // Chunks of kUnitChunk consecutive units go to the XCDs in turn, so that the parts of an expert's rows read its weights at the
  // same time through one L2; inside an XCD its wavefronts (SwiGLU of plain weights: workgroups) take the units in turn.
  const int xcd = block % kXcds;
  const int stride = ((int)gridDim.x - index_blocks) / kXcds * (kTwoWaves ? 1 : kDecodeWaves);
  struct Unit {
    int turn, cg, row0, nrows, expert, seg;   // nrows = 0: there is no further unit
    int row[RB];                 // per lane: rows 8 g + lane / 8 of A (as loaded: used in start, so that nothing waits for them here)
  };
  auto find = [&](int turn) {
    Unit t;
    t.turn = turn;
    t.nrows = t.seg = 0;
    const int index = (turn / kUnitChunk * kXcds + xcd) * kUnitChunk + turn % kUnitChunk;
    if (index < n_units) {
      int slot = -1;   // the last one whose units begin at this one or before (slots without units share the next one's)
      for (int i0 = 0; i0 < n_slots; i0 += 64) slot += __popcll(__ballot(i0 + lane < n_slots && L.unit0[i0 + lane] <= index));
      slot = uniform(slot);
      const int in_slot = index - uniform(L.unit0[slot]), rows = uniform((int)L.rows[slot]), parts = (rows + ROWS - 1) / ROWS;
      const int part = in_slot % parts;
      t.cg = in_slot / parts;
      t.row0 = uniform((int)L.row0[slot]) + part * ROWS;
      t.nrows = min(rows - part * ROWS, ROWS);
      t.expert = uniform((int)L.expert[slot]);
      if (flagged) t.seg = p.own_index ? segment_of((int)L.token[t.row0 + t.nrows - 1]) : uniform((int)L.seg[slot]);
#pragma unroll
      for (int g = 0; g < RB; g++) {
        const int r = t.row0 + min(g * 8 + (lane >> 3), t.nrows - 1);
        t.row[g] = MODE == MODE_L1 ? r : (p.own_index ? (int)L.token[r] : p.a_rows[r]);
      }
    }
    return t;
  };

  u32x4 areg[U][RB], breg[U][NBL];
  const __amdgpu_buffer_rsrc_t a_buf = buffer(p.A, kRowsEnd);
  __amdgpu_buffer_rsrc_t b_buf;
  uint32_t a_off[RB];
  const int g16 = lane >> 4, j16 = lane & 15;
  // Packed: the operand of one MFMA (32 values of K of 16 columns) is 4 pieces of 256 bytes, one per 8 values of K.
  // Plain: a load takes 8 rows of K (128-byte lines), or 16 rows (64 bytes) where the wavefront has 32 columns of a matrix.
  constexpr int kLineCols = NB * 16, kLineLanes = kLineCols / 8, kLineRows = 64 / kLineLanes;
  const uint32_t b_off = PK ? (g16 >> 1) * (kStageBytes / 2) + (g16 & 1) * 512 + j16 * 16
                            : (lane / kLineLanes) * p.ldb * 2 + (lane % kLineLanes) * 16;
  const uint32_t b_rows = p.ldb * 2 * kLineRows;
  const uint32_t b_step = PK ? 2 * kStageBytes : p.ldb * 2 * kStepK;
  auto load = [&](int u, int st) {
    const uint32_t bs = (uint32_t)st * b_step;
    auto load_a = [&]() {
#pragma unroll
      for (int g = 0; g < RB; g++) areg[u][g] = __builtin_amdgcn_raw_buffer_load_b128(a_buf, a_off[g], st * (kStepK * 2), 0);
    };
    if (kAhead) load_a();
#pragma unroll
    for (int j = 0; j < NBL; j++) {
      uint32_t at;
      if (PK) {   // (32 values of K j / NB, block j % NB)
        const int nb = j % NB;
        at = bs + (j / NB) * kStageBytes + (nb / OB) * 4096 + ((nb % OB) >> 1) * 1024 + (nb & (OB > 1 ? 1 : 0)) * 256;
      } else {
        at = bs + j * b_rows;
      }
      breg[u][j] = __builtin_amdgcn_raw_buffer_load_b128(b_buf, b_off, at, STREAM ? kNonTemporal : 0);
    }
    if (!kAhead) load_a();
  };
  // addresses of a unit and its first loads (past the last step: the last step again, it is in the caches; a load under
  // a condition would make the compiler wait for more than it has to at every use)
  auto start = [&](const Unit& t) {
    const int col = t.cg * (OB * 16);   // of C
#pragma unroll
    for (int g = 0; g < RB; g++)
      a_off[g] = g * 8 + (lane >> 3) < t.nrows ? (uint32_t)t.row[g] * p.lda_bytes + (lane & 7) * 16 : kRowsEnd;
    if (PK) {   // column tiles of 256 columns (SwiGLU: 128 gate and the 128 up columns of the same units)
      const int tile = kPair ? col >> 7 : col >> 8, in_tile = kPair ? col & 127 : col & 255;
      b_buf = buffer(p.B + ((uint64_t)t.expert * p.n_tiles_n + tile) * nk * (2 * kStageBytes) + (in_tile >> 5) * 1024 + ((in_tile >> 4) & 1) * 256);
    } else {
      b_buf = buffer(p.B + (uint64_t)t.expert * p.b_expert_bytes + ((uint64_t)(kTwoWaves ? w * p.F : 0) + col) * 2);
    }
#pragma unroll
    for (int u = 0; u < U; u++) load(u, min(u, nk - 1));
  };

  // LDS positions: A rows of 128 bytes, the 16-byte chunks swizzled by row; plain B rows of 64 columns
  const uint32_t lds_a = (uint32_t)(uintptr_t)operands + w * kWaveBytes, lds_b = lds_a + kABytes;
  const int row8 = lane >> 3, c8 = lane & 7;
  const uint32_t a_wr = lds_a + row8 * 128 + ((c8 ^ ((row8 >> 1) & 3)) << 4);   // + 1 KiB per 8-row group, chunks ^ 4 in odd ones
  const uint32_t a_rd = lds_a + j16 * 128;
  const int s = (j16 >> 1) & 7;
  const uint32_t tr_wr = lds_b + (lane / kLineLanes) * kPlainPitch + (lane % kLineLanes) * 16;
  const uint32_t tr_rd = lds_b + (8 * g16 + (j16 >> 2)) * kPlainPitch + (j16 & 3) * 8;
  f32x4 acc[RR][NB];
  bf16x8 af[kAhead ? 2 : 1][2][RR];
  auto through_lds = [&](int u, int set) {   // the rows of A of ring slot u, as fragments
#pragma unroll
    for (int g = 0; g < RB; g++)
      *(u32x4 __attribute__((address_space(3)))*)(uintptr_t)((a_wr ^ ((g & 1) << 6)) + g * 1024) = areg[u][g];
#pragma unroll
    for (int kk = 0; kk < 2; kk++)
#pragma unroll
      for (int r = 0; r < RR; r++)
        af[set][kk][r] = *(const bf16x8 __attribute__((address_space(3)))*)(uintptr_t)(a_rd + r * 2048 + (((kk * 4 + g16) ^ s) << 4));
  };
  auto multiply = [&](int u, int rows_now) {
    if (kAhead) through_lds((u + 1) % U, (u + 1) & 1);
    else through_lds(u, 0);
    bf16x8 b[2][NB];
#pragma unroll
    for (int kk = 0; kk < 2; kk++) {
      if (!PK) {   // 32 rows of K
#pragma unroll
        for (int j = 0; j < NBL / 2; j++)
          *(u32x4 __attribute__((address_space(3)))*)(uintptr_t)(tr_wr + j * kLineRows * kPlainPitch) = breg[u][kk * (NBL / 2) + j];
      }
#pragma unroll
      for (int nb = 0; nb < NB; nb++) {
        if (PK) {
          b[kk][nb] = __builtin_bit_cast(bf16x8, breg[u][kk * NB + nb]);
        } else {
          const uint32_t at = tr_rd + nb * 32;
          b[kk][nb] = lds_read_b(at, at + 4 * kPlainPitch);
        }
      }
    }
#pragma unroll
    for (int r = 0; r < RR; r++) {
      if (r > 0 && rows_now <= 16 * r) break;
#pragma unroll
      for (int kk = 0; kk < 2; kk++)
#pragma unroll
        for (int nb = 0; nb < NB; nb++)
          acc[r][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[kk][nb], af[kAhead ? u & 1 : 0][kk][r], acc[r][nb], 0, 0, 0);
    }
  };

  auto arrived = [&](const Unit& t) { return MODE == MODE_L1 || ((there >> t.seg) & 1); };
  // waits for the rows of a unit and starts it; false: they have not come
  auto start_when_there = [&](const Unit& t) {
    if (!arrived(t)) {
      if (patient && !spin_until_ge(&p.seg_ready[t.seg], p.ready_epoch, p.spin_limit)) {
        patient = false;
        // (a launch that makes its index clears the status word itself: layer1 moves this one there)
        if (lane == 0) atomicExch(p.own_index ? p.status + kTimedOutAt : p.status, p.own_index ? p.forward_serial : (int)MOE_ERR_TIMEOUT);
      }
      look();
      if (!arrived(t)) return false;
    }
    start(t);
    return true;
  };

  const int first = kTwoWaves ? block / kXcds : block / kXcds * kDecodeWaves + w;
  Unit cur = find(first);
  bool started = cur.nrows > 0 && start_when_there(cur);
  int turn = 0;
  while (cur.nrows > 0) {
#pragma unroll
    for (int r = 0; r < RR; r++)
#pragma unroll
      for (int nb = 0; nb < NB; nb++) acc[r][nb] = (f32x4){0};
    const Unit next = find(cur.turn + stride);   // asked for now: its table entries are back when they are needed
    if (started) {
      if (kAhead) through_lds(0, 0);
      int st = 0;
#pragma unroll 1
      do {
#pragma unroll
        for (int u = 0; u < U; u++) {
          __builtin_amdgcn_sched_barrier(0);   // a step's loads reuse the registers just consumed
          if (st + u < nk) multiply(u, cur.nrows);
          __builtin_amdgcn_sched_barrier(0);
          load(u, min(st + u + U, nk - 1));
        }
        st += U;
      } while (st < nk);
    }
    // the next unit's first loads are under way while this one is written
    bool next_started = next.nrows > 0 && arrived(next);
    if (next_started) start(next);

    // SwiGLU of plain weights: wavefront 0 gives the gate columns of the upper blocks away and gets the up columns of the
    // lower ones, wavefront 1 the reverse.
    if constexpr (kTwoWaves) {
#pragma unroll
      for (int r = 0; r < RR; r++)
#pragma unroll
        for (int i = 0; i < 2; i++) swap_lds[turn][w][r * 2 + i][lane] = w == 0 ? acc[r][2 + i] : acc[r][i];
      given_up[turn][w] = !started;
      __syncthreads();   // (this turn's buffer is written again two units on, behind the next unit's barrier)
      started = started && !given_up[turn][w ^ 1];
    }
    // a lane holds, of row lane % 16 of a block, the 4 columns from 4 (lane / 16) on
#pragma unroll
    for (int r = 0; r < RR; r++) {
      const int row = r * 16 + j16;
      uint16_t* dst = p.C + (size_t)(cur.row0 + row) * p.ldc + cur.cg * (OB * 16) + (kTwoWaves ? w * 32 : 0) + g16 * 4;
#pragma unroll
      for (int nb = 0; nb < (kTwoWaves ? 2 : OB); nb++) {
        f32x4 v = acc[r][nb], up = v;
        if constexpr (kInWave) up = acc[r][nb + OB];
        if constexpr (kTwoWaves) {
          const f32x4 other = swap_lds[turn][w ^ 1][r * 2 + nb][lane];
          up = w == 0 ? other : acc[r][2 + nb];
          v = w == 0 ? v : other;
        }
#pragma unroll
        for (int i = 0; i < 4; i++) {
          if (kPair) v[i] = silu(v[i]) * up[i];
          else if (MODE == MODE_L0_GELU) v[i] = gelu_erf(v[i]);
        }
        const bf16x2 lo = {(__bf16)v[0], (__bf16)v[1]}, hi = {(__bf16)v[2], (__bf16)v[3]};
        const u32x2 pk = {__builtin_bit_cast(uint32_t, lo), __builtin_bit_cast(uint32_t, hi)};
        if (started && row < cur.nrows) *(u32x2*)(dst + nb * 16) = pk;
      }
    }
    if (next.nrows > 0 && !next_started) next_started = start_when_there(next);
    turn ^= 1;
    cur = next;
    started = next_started;
  }
}

template <int MODE, bool PK, int NB, int RB, int U, int EU>
static hipError_t launch_decode(const DecodeParams& p, const IndexParams& ip, hipStream_t st) {
  constexpr bool kTwoWaves = MODE == MODE_L0_SWIGLU && !PK, kInWave = MODE == MODE_L0_SWIGLU && PK;
  constexpr int kUnitWaves = kTwoWaves ? kDecodeWaves : 1;   // wavefronts per unit
  const int64_t n_groups = p.N / (NB * 16 / (kInWave ? 2 : 1));
  // no more wavefronts than can be resident, or than there can be units (an expert's last part is not full)
  const int64_t most = ((int64_t)p.R / (8 * RB) + p.n_slots) * n_groups, resident = (int64_t)p.n_cu * 4 * EU / kUnitWaves;
  const int64_t per_xcd = ((most < resident ? most : resident) + kXcds * kUnitChunk - 1) / (kXcds * kUnitChunk) * kUnitChunk;
  const unsigned grid = (unsigned)(per_xcd * kUnitWaves / kDecodeWaves) * kXcds + (MODE != MODE_L1 && p.own_index ? kXcds : 0);
  // (64-byte pieces of plain weights: the other half of a line is another wavefront's and should still be there)
  if (p.b_stream && (PK || NB == 4)) hipLaunchKernelGGL((k_decode_gemm<MODE, PK, NB, RB, U, EU, (PK || NB == 4)>), dim3(grid), dim3(kDecodeWaves * 64), 0, st, p, ip);
  else hipLaunchKernelGGL((k_decode_gemm<MODE, PK, NB, RB, U, EU, false>), dim3(grid), dim3(kDecodeWaves * 64), 0, st, p, ip);
  return hipGetLastError();
}

// Columns of a wavefront, ring depth and wavefronts per SIMD by what fits the registers and measured best, us per launch:
//   packed, up to 8 rows    SwiGLU 4 steps x 4 wavefronts 86, 6 x 2 87, 3 x 4 87; layer1 (512 wavefronts in all for one token) 16 columns
//                           each, 8 x 2 44, 4 x 4 52; 32 columns 4 x 4 66   (1 token, Mixtral-shaped)
//   packed, 9 to 16 rows    4 x 3 / 4 x 4, 2 x 4 3 % and 3 x 4 0.4 % longer (16 tokens, Mixtral-shaped)
//   packed, more            layer0 + layer1 of 48 tokens of 64 experts of F = 2560, gate and index build in it: SwiGLU 2 x 4 with layer1 3 x 3
//                           611, 3 x 3 with 2 x 4 620, 4 x 2 with 4 x 2 615, 4 x 3 with 3 x 4 (spills) 694
//   plain, SwiGLU           3 x 2 25, 2 x 2 33 (4 tokens); 4 x 1 47, 3 x 2 50 (33 tokens, 8 experts of F = 1792)
// Plain weights without SwiGLU: 64 columns, whole lines (12 tokens, F = 2560, weights from HBM: layer1 33 us against 46 in
// 64-byte pieces), but 32 where the wavefronts of 64 would leave compute units idle (one token, 120 wavefronts of 64 columns: layer1
// of F = 1792 19 -> 16; 4 tokens of GELU layer0, 147: 33 -> 26, 210: 37 / 37, 252 and cold: 44 -> 67).
template <int MODE, int RB>
static hipError_t launch_decode_depth(const DecodeParams& p, const IndexParams& ip, int packed, hipStream_t st) {
  constexpr bool kPair = MODE == MODE_L0_SWIGLU;
  if (packed) {
    if constexpr (RB == 1) return launch_decode<MODE, true, (kPair ? 2 : 1), 1, (kPair ? 4 : 8), (kPair ? 4 : 2)>(p, ip, st);
    else if constexpr (RB == 2) return launch_decode<MODE, true, (MODE == MODE_L1 ? 1 : 2), 2, 4, (MODE == MODE_L1 ? 4 : 3)>(p, ip, st);
    else return launch_decode<MODE, true, 2, 4, (kPair ? 2 : 3), (kPair ? 4 : 3)>(p, ip, st);
  }
  if constexpr (!kPair) {
    if (p.experts * (p.N / 64) < 0.75f * p.n_cu) return launch_decode<MODE, false, 2, RB, (RB == 1 ? 6 : 4), 2>(p, ip, st);
  }
  return launch_decode<MODE, false, 4, RB, (RB == 1 ? 3 : 4), (RB == 4 ? 1 : 2)>(p, ip, st);
}

template <int MODE>
static hipError_t launch_decode_rows(const DecodeParams& p, const IndexParams& ip, int packed, hipStream_t st) {
  // rows a unit holds: what most experts of the batch stay under
  if (p.T <= 8) return launch_decode_depth<MODE, 1>(p, ip, packed, st);
  if (p.T <= 16) return launch_decode_depth<MODE, 2>(p, ip, packed, st);
  return launch_decode_depth<MODE, 4>(p, ip, packed, st);
}

hipError_t launch_decode_gemm(const DecodeParams& p, const IndexParams& ip, int layer1, int act, int packed, hipStream_t st) {
  if (p.n_slots == 0) return hipSuccess;
  if (layer1) return launch_decode_rows<MODE_L1>(p, ip, packed, st);
  if (act == MOE_ACT_SWIGLU) return launch_decode_rows<MODE_L0_SWIGLU>(p, ip, packed, st);
  return launch_decode_rows<MODE_L0_GELU>(p, ip, packed, st);
}

}  // namespace moe
