// GroupGEMM of small batches (a few rows per expert: decoding), for gfx950.
//
// What bounds it is the stream of weights from HBM: every expert that some token picked is read once for a handful of
// rows.  The persistent tile kernel (grouped_gemm.hip) keeps that stream going only while it has a 64 x 256 tile or two
// per compute unit; with few rows there are few tiles (layer1 of one token of 8 experts, H = 4096: 32), and the rest of
// the chip idles.  Here the unit is 32 columns (plain weights: 64) of one expert by up to 32 rows:
//  * a workgroup is 8 wavefronts that share the columns and split K, so that even one token's layer1 is 256 units; the
//    parts of K meet in LDS at the end, in a fixed order;
//  * a wavefront keeps a ring of operands in registers, loaded two or three 64-deep steps ahead, and meets the others
//    only at the end of a unit; its rows of A go through a private piece of LDS (8 whole lines per load instruction, then
//    one ds_read_b128 per fragment: read as fragments from memory, 32 rows apart, they took a third longer at 8 rows);
//  * the first loads of the next unit are issued before the parts of this one meet, and two workgroups share a compute
//    unit (128 registers a wavefront), so that the stream does not stop at the ends of units;
//  * packed weights arrive in MFMA operand order (one 1 KiB load is one fragment).  Plain weights are loaded as they lie
//    (rows of K, whole 128-byte lines) and transposed through LDS with ds_read_b64_tr_b16;
//  * there is no schedule: workgroups walk the units with a fixed stride.  (A workgroup per unit cost 220 us on layer0 +
//    layer1 of 32 tokens of the Mixtral-shaped layer, where every other workgroup finds no rows and returns: those keep
//    waiting ones from starting.)
// Measured on that shape with packed weights, both layers, tile kernel -> this one: 1 token 259 -> 128 us (704 MB: 5.5
// TB/s), 16 tokens 531 -> 482 us (2.8 GB: 5.8 TB/s; a copy of 1 GiB moves 4.4 TB/s, half of it writes).
#include "moe_device.h"

namespace moe {

constexpr int kDecodeWaves = 8;
constexpr int kStageBytes = kTileK * kTileN * 2;   // packed weights: one K step of one column tile
constexpr int kPlainPitch = 144;                   // bytes between rows of K in the transposing buffer (64 columns + padding)
constexpr int kStepK = 64;                         // K of one ring slot: a whole 128-byte line of every row of A
constexpr int kABytes = 32 * kStepK * 2;           // a wavefront's rows of A for one step, in LDS

// The memory from ptr on (the same in every lane) as a buffer: loads then take one 32-bit offset per lane and one scalar
// offset, and no 64-bit address per load sits in vector registers.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer(const char* ptr) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)uniform(ptr), 0, -1, 0x00020000);
}

// NB: 32-column blocks of a wavefront; RB: 8-row groups of A that are loaded (a unit is up to 8 RB rows); U: steps in flight.
template <int MODE, bool PK, int NB, int RB, int U>
__global__ __launch_bounds__(kDecodeWaves * 64) __attribute__((amdgpu_waves_per_eu(PK ? 4 : 2))) void k_decode_gemm(DecodeParams p) {
  static_assert(PK || NB == 2, "plain weights are loaded in whole 128-byte lines: 64 columns");
  constexpr bool kPair = MODE == MODE_L0_SWIGLU;       // gate and up columns of the same hidden units meet in the workgroup
  constexpr int ROWS = 8 * RB;
  constexpr int CW = NB * 32;                          // columns of a wavefront
  constexpr int PITCH = CW + 4;                        // floats between rows of a partial result
  constexpr int NBL = NB * 4;                          // 16-byte loads of B per lane and step
  constexpr int kWaveBytes = kABytes + (PK ? 0 : kTileK * kPlainPitch);   // operands on their way through LDS
  __shared__ __attribute__((aligned(16))) float part[kDecodeWaves * ROWS * PITCH];
  __shared__ __attribute__((aligned(128))) char operands[kDecodeWaves * kWaveBytes];
  __shared__ int ok_lds;

  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n_tiles = *p.n_tiles;
  if (MODE != MODE_L1 && p.seg_ready != nullptr) {
    // a small batch waits for every segment its tiles need before it starts on the first
    if (tid == 0) ok_lds = 1;
    __syncthreads();
    for (int i = tid; i < n_tiles; i += kDecodeWaves * 64)
      if (!spin_until_ge(&p.seg_ready[p.tile_ready[i]], p.ready_epoch, p.spin_limit)) ok_lds = 0;
    __syncthreads();
    if (!ok_lds) {
      if (tid == 0) atomicExch(p.status, (int)MOE_ERR_TIMEOUT);
      return;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "");
  }

  // this wavefront's part of K and its columns
  const int ks = 1 << p.k_split_log2;
  const int kw = w & (ks - 1), cw = w >> p.k_split_log2;
  const int n_cw = kDecodeWaves >> p.k_split_log2;       // column groups of the workgroup
  const int n_units = kPair ? n_cw / 2 : n_cw;           // ... of its output
  const int half = kPair && cw >= n_units;               // 1: up columns
  const int nk = p.K / kStepK;
  const int k_lo = kw * nk >> p.k_split_log2, k_hi = (kw + 1) * nk >> p.k_split_log2;
  const int wave_col = (half ? cw - n_units : cw) * CW;

  // Units: (row part, tile, columns), the parts slowest and the columns fastest.  Workgroups take them in turn.
  const int n_parts = (*p.tallest + ROWS - 1) / ROWS;
  const int per_part = n_tiles * p.n_groups, n_wg_units = per_part * n_parts;
  struct Unit {
    int index, cg, row0, nrows, expert;
    uint32_t a_off[RB];          // per lane: rows 8 g + lane / 8 of A, 16 bytes at lane % 8 of a line
  };
  auto find = [&](int index) {   // the first unit with rows from this one on
    Unit t;
    t.nrows = 0;
    for (; index < n_wg_units; index += gridDim.x) {
      const int sub = index / per_part, in_part = index % per_part;
      const int slot = in_part / p.n_groups;
      const int rows = p.tile_rows[slot] - sub * ROWS;
      if (rows <= 0) continue;
      t.cg = in_part % p.n_groups;
      t.row0 = p.tile_row0[slot] + sub * ROWS;
      t.nrows = rows < ROWS ? rows : ROWS;
      t.expert = p.tile_expert[slot];
      break;
    }
    t.index = index;
    if (t.nrows > 0) {
#pragma unroll
      for (int g = 0; g < RB; g++) {
        const int r = t.row0 + min(g * 8 + (lane >> 3), t.nrows - 1);   // rows past the end: the last row again
        t.a_off[g] = (uint32_t)(MODE != MODE_L1 ? p.a_rows[r] : r) * p.lda_bytes + (lane & 7) * 16;
      }
    }
    return t;
  };

  u32x4 areg[U][RB], breg[U][NBL];
  __amdgpu_buffer_rsrc_t a_buf, b_buf;
  uint32_t a_off[RB];
  int n = 0;                                             // steps of this wavefront
  const uint32_t b_off = PK ? lane * 16 : (lane >> 3) * p.ldb * 2 + (lane & 7) * 16;
  const uint32_t b_row8 = p.ldb * 2 * 8;                 // plain: 8 rows of K
  const uint32_t b_step = PK ? 2 * kStageBytes : p.ldb * 2 * kStepK;
  auto load = [&](int u, int st) {
    const uint32_t bs = (uint32_t)st * b_step;
    // packed: fragment (K 16 kk .. + 15, block nb) at kk * NB + nb; plain: rows 8 j .. + 7 of K at j
#pragma unroll
    for (int j = 0; j < NBL; j++) {
      const uint32_t at = PK ? bs + (j / NB) * (kStageBytes / 2) + (j % NB) * 1024 : bs + j * b_row8;
      breg[u][j] = __builtin_amdgcn_raw_buffer_load_b128(b_buf, b_off, at, 0);
    }
#pragma unroll
    for (int g = 0; g < RB; g++) areg[u][g] = __builtin_amdgcn_raw_buffer_load_b128(a_buf, a_off[g], st * (kStepK * 2), 0);
  };
  // addresses of a unit and its first loads (past the last step: the last step again, it is in the caches; a load under
  // a condition would make the compiler wait for more than it has to at every use)
  auto start = [&](const Unit& t) {
    const int out_col = t.cg * n_units * CW + wave_col;
    n = out_col < p.N ? k_hi - k_lo : 0;
    if (n == 0) return;
#pragma unroll
    for (int g = 0; g < RB; g++) a_off[g] = t.a_off[g];
    a_buf = buffer(p.A + (size_t)k_lo * (kStepK * 2));
    if (PK) {
      const int blk = out_col / 32;
      const int tile = kPair ? blk >> 2 : blk >> 3;
      const int c = kPair ? (blk & 3) + half * 4 : blk & 7;
      b_buf = buffer(p.B + (((uint64_t)t.expert * p.n_tiles_n + tile) * nk + k_lo) * (2 * kStageBytes) + c * 1024);
    } else {
      b_buf = buffer(p.B + (uint64_t)t.expert * p.b_expert_bytes + ((uint64_t)k_lo * kStepK * p.ldb + half * p.F + out_col) * 2);
    }
#pragma unroll
    for (int u = 0; u < U; u++) load(u, min(u, n - 1));
  };

  // LDS positions: A rows of 128 bytes, the 16-byte chunks swizzled by row; plain B rows of 64 columns
  const uint32_t lds_a = (uint32_t)(uintptr_t)operands + w * kWaveBytes, lds_b = lds_a + kABytes;
  const int row8 = lane >> 3, c8 = lane & 7, g16 = lane >> 4, j16 = lane & 15;
  const uint32_t a_wr = lds_a + row8 * 128 + ((c8 ^ ((row8 >> 1) & 3)) << 4);   // + 1 KiB per 8-row group, chunks ^ 4 in odd ones
  const uint32_t a_rd = lds_a + (lane & 31) * 128;
  const int s = ((lane & 31) >> 1) & 7;
  const uint32_t tr_wr = lds_b + row8 * kPlainPitch + c8 * 16;
  const uint32_t tr_rd = lds_b + (8 * (g16 >> 1) + (j16 >> 2)) * kPlainPitch + (16 * (g16 & 1) + 4 * (j16 & 3)) * 2;
  f32x16 acc[NB];
  auto multiply = [&](int u) {
#pragma unroll
    for (int g = 0; g < RB; g++)
      *(u32x4 __attribute__((address_space(3)))*)(uintptr_t)((a_wr ^ ((g & 1) << 6)) + g * 1024) = areg[u][g];
#pragma unroll
    for (int kk = 0; kk < 4; kk++) {
      if (!PK && (kk & 1) == 0) {
#pragma unroll
        for (int j = 0; j < 4; j++)
          *(u32x4 __attribute__((address_space(3)))*)(uintptr_t)(tr_wr + j * 8 * kPlainPitch) = breg[u][kk * 2 + j];
      }
      const bf16x8 a = *(const bf16x8 __attribute__((address_space(3)))*)(uintptr_t)(a_rd + (((kk * 2 + (lane >> 5)) ^ s) << 4));
#pragma unroll
      for (int nb = 0; nb < NB; nb++) {
        bf16x8 b;
        if (PK) {
          b = __builtin_bit_cast(bf16x8, breg[u][kk * NB + nb]);
        } else {
          const uint32_t at = tr_rd + (kk & 1) * 16 * kPlainPitch + nb * 64;
          b = lds_read_b(at, at + 4 * kPlainPitch);
        }
        acc[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b, a, acc[nb], 0, 0, 0);
      }
    }
  };

  Unit cur = find(blockIdx.x);
  if (cur.index < n_wg_units) start(cur);
  while (cur.index < n_wg_units) {
#pragma unroll
    for (int nb = 0; nb < NB; nb++) acc[nb] = (f32x16){0};
    const Unit next = find(cur.index + gridDim.x);   // asked for now: its table entries are back when they are needed
    if (n > 0) {
      int st = 0;
#pragma unroll 1
      do {
#pragma unroll
        for (int u = 0; u < U; u++) {
          __builtin_amdgcn_sched_barrier(0);   // a step's loads reuse the registers just consumed
          if (st + u < n) multiply(u);
          __builtin_amdgcn_sched_barrier(0);
          load(u, min(st + u + U, n - 1));
        }
        st += U;
      } while (st < n);
    }
    // the next unit's first loads are under way while this one's parts meet
    if (next.index < n_wg_units) start(next);

    // the parts of K meet in LDS; a lane holds, of row lane & 31, the columns 8*(i/4) + 4*(lane/32) + i%4 of each block
    __syncthreads();   // the partial results of the unit before are read out
    if ((lane & 31) < cur.nrows) {
      float* dst = part + (w * ROWS + (lane & 31)) * PITCH + (lane >> 5) * 4;
#pragma unroll
      for (int nb = 0; nb < NB; nb++)
#pragma unroll
        for (int i = 0; i < 4; i++)
          *(float4*)(dst + nb * 32 + i * 8) = make_float4(acc[nb][4 * i], acc[nb][4 * i + 1], acc[nb][4 * i + 2], acc[nb][4 * i + 3]);
    }
    __syncthreads();
    const int total = n_units * cur.nrows * (CW / 4);
    for (int v = tid; v < total; v += kDecodeWaves * 64) {
      const int c4 = v % (CW / 4), ur = v / (CW / 4), rr = ur % cur.nrows, u = ur / cur.nrows;
      const int col = (cur.cg * n_units + u) * CW + c4 * 4;
      if (col >= p.N) continue;
      auto sum = [&](int column_group) {
        const float* src = part + ((column_group << p.k_split_log2) * ROWS + rr) * PITCH + c4 * 4;
        float4 t = *(const float4*)src;
        for (int i = 1; i < ks; i++) {
          const float4 o = *(const float4*)(src + i * ROWS * PITCH);
          t.x += o.x; t.y += o.y; t.z += o.z; t.w += o.w;
        }
        return t;
      };
      const float4 t = sum(u);
      float o[4] = {t.x, t.y, t.z, t.w};
      if (kPair) {
        const float4 t2 = sum(u + n_units);
        const float up[4] = {t2.x, t2.y, t2.z, t2.w};
#pragma unroll
        for (int i = 0; i < 4; i++) o[i] = silu(o[i]) * up[i];
      } else if (MODE == MODE_L0_GELU) {
#pragma unroll
        for (int i = 0; i < 4; i++) o[i] = gelu_erf(o[i]);
      }
      const bf16x2 lo = {(__bf16)o[0], (__bf16)o[1]}, hi = {(__bf16)o[2], (__bf16)o[3]};
      const u32x2 pk = {__builtin_bit_cast(uint32_t, lo), __builtin_bit_cast(uint32_t, hi)};
      *(u32x2*)(p.C + (size_t)(cur.row0 + rr) * p.ldc + col) = pk;
    }
    cur = next;
  }
}

template <int MODE, bool PK, int RB>
static hipError_t launch_decode(DecodeParams p, hipStream_t st) {
  constexpr int NB = PK ? 1 : 2, U = PK ? (RB == 4 ? 2 : 3) : 2;
  const int units_per_wg = (kDecodeWaves >> p.k_split_log2) / (MODE == MODE_L0_SWIGLU ? 2 : 1);
  p.n_groups = (p.N + units_per_wg * NB * 32 - 1) / (units_per_wg * NB * 32);
  const int64_t units = (int64_t)p.n_slots * p.n_groups * ((p.tile_m + 8 * RB - 1) / (8 * RB));
  const int64_t resident = (int64_t)p.n_cu * (PK ? 2 : 1);
  hipLaunchKernelGGL((k_decode_gemm<MODE, PK, NB, RB, U>), dim3((unsigned)(units < resident ? units : resident)),
                     dim3(kDecodeWaves * 64), 0, st, p);
  return hipGetLastError();
}

template <int MODE>
static hipError_t launch_decode_rows(const DecodeParams& p, int packed, hipStream_t st) {
  // rows a unit holds: what most experts of the batch stay under
  if (p.T <= 8) return packed ? launch_decode<MODE, true, 1>(p, st) : launch_decode<MODE, false, 1>(p, st);
  if (p.T <= 16) return packed ? launch_decode<MODE, true, 2>(p, st) : launch_decode<MODE, false, 2>(p, st);
  return packed ? launch_decode<MODE, true, 4>(p, st) : launch_decode<MODE, false, 4>(p, st);
}

hipError_t launch_decode_gemm(const DecodeParams& p, int layer1, int act, int packed, hipStream_t st) {
  if (p.n_slots == 0) return hipSuccess;
  if (layer1) return launch_decode_rows<MODE_L1>(p, packed, st);
  if (act == MOE_ACT_SWIGLU) return launch_decode_rows<MODE_L0_SWIGLU>(p, packed, st);
  return launch_decode_rows<MODE_L0_GELU>(p, packed, st);
}

}  // namespace moe
