// Gate, shared-tensor row order, tile tables and tile schedules (integer work, bit-exact).
//
// Row order (paper Section 3.1.2, Fig. 5): rows of the shared tensor are grouped by expert and, inside an
// expert, sorted by source rank.  Source segment s owns a contiguous token range, so a stable counting sort of
// the pair ids q = t*k + j by expert id gives exactly that order.
#include "moe_device.h"

namespace moe {

// ---------------------------------------------------------------------------------------------
// Gate (Section 2.1): softmax over E logits, top-k, renormalise.  One wavefront per token.
// ---------------------------------------------------------------------------------------------
// What it costs is latency: k rounds of an argmax over the wavefront, one behind the other.  By lane exchange through LDS on (value, expert)
// pairs a round is 12 dependent exchanges, 8192 tokens of 64 experts with k = 4 took 10.2 us and 48 with k = 8 7.1; by the maximum of keys that sort like the
// logits, in DPP instructions, and a ballot for who has it, 6.9 and 4.7.  Rows with a NaN, which has no place in the order, keep the exchange.
// Largest key of the wavefront, in every lane.
__device__ __forceinline__ uint32_t wave_max(uint32_t v) {
  auto step = [&](auto ctrl) {   // lanes the control does not reach keep their own
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, decltype(ctrl)::value, 0xf, 0xf, false));
  };
  step(std::integral_constant<int, 0x111>{});   // row_shr 1, 2, 4, 8: the last lane of every 16 has their maximum
  step(std::integral_constant<int, 0x112>{});
  step(std::integral_constant<int, 0x114>{});
  step(std::integral_constant<int, 0x118>{});
  step(std::integral_constant<int, 0x142>{});   // row_bcast 15, 31: the last lane of all
  step(std::integral_constant<int, 0x143>{});
  return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

__global__ __launch_bounds__(256) void k_route_topk(const float* __restrict__ logits, int T, int E, int k,
                                                    int32_t* __restrict__ ids, float* __restrict__ w) {
  const int lane = threadIdx.x & 63;
  const int t = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (t >= T) return;
  // each lane holds up to 4 experts: e = lane + 64*i
  float v[4];
  bool taken[4];
#pragma unroll
  for (int i = 0; i < 4; i++) {
    int e = lane + 64 * i;
    v[i] = e < E ? logits[(size_t)t * E + e] : -INFINITY;
    taken[i] = e >= E;
  }
  float sel_logit = 0.f;  // lane j keeps the logit of slot j
  float top = 0.f;
  bool nan = false;
#pragma unroll
  for (int i = 0; i < 4; i++) nan = nan || v[i] != v[i];
  if (__ballot(nan) == 0) {
    uint32_t key[4];   // in the order of the logits, 0: taken
#pragma unroll
    for (int i = 0; i < 4; i++) {
      const uint32_t bits = __float_as_uint(v[i] + 0.f);   // (-0 and 0 are equal)
      key[i] = taken[i] ? 0u : bits ^ ((bits >> 31) ? 0xffffffffu : 0x80000000u);
    }
    int my_id = 0;
    for (int j = 0; j < k; j++) {
      uint32_t best = key[0];
#pragma unroll
      for (int i = 1; i < 4; i++) best = max(best, key[i]);
      best = wave_max(best);
      int be = -1;   // the lowest expert that has it
#pragma unroll
      for (int i = 0; i < 4; i++) {
        const uint64_t has = __ballot(key[i] == best);
        if (be < 0 && has) be = 64 * i + __ffsll((unsigned long long)has) - 1;
      }
#pragma unroll
      for (int i = 0; i < 4; i++)
        if (be == lane + 64 * i) key[i] = 0;
      const float logit = __uint_as_float(best ^ ((best >> 31) ? 0x80000000u : 0xffffffffu));
      if (j == 0) top = logit;
      if (lane == j) {
        sel_logit = logit;
        my_id = be;
      }
    }
    if (lane < k) ids[(size_t)t * k + lane] = my_id;
  } else for (int j = 0; j < k; j++) {
    // lane-local best among untaken (lowest expert id wins ties: i ascending, strict >)
    float bv = -INFINITY;
    int be = 0x7fffffff;
#pragma unroll
    for (int i = 0; i < 4; i++) {
      if (!taken[i] && (be == 0x7fffffff || v[i] > bv)) { bv = v[i]; be = lane + 64 * i; }
    }
    // wave argmax with ties to the lower expert id
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
      float ov = __shfl_xor(bv, off);
      int oe = __shfl_xor(be, off);
      bool better = (oe != 0x7fffffff) && (be == 0x7fffffff || ov > bv || (ov == bv && oe < be));
      if (better) { bv = ov; be = oe; }
    }
#pragma unroll
    for (int i = 0; i < 4; i++) taken[i] = taken[i] || (be == lane + 64 * i);
    if (j == 0) top = bv;
    if (lane == j) sel_logit = bv;
    if (lane == 0) ids[(size_t)t * k + j] = be;
  }
  // weights: softmax restricted to the kept logits (equal to softmax over all E followed by renormalisation)
  float p = lane < k ? expf(sel_logit - top) : 0.f;
  float sum = p;
  for (int off = k > 16 ? 32 : 8; off >= 1; off >>= 1) sum += __shfl_xor(sum, off);   // (lanes beyond k hold zeros)
  if (lane < k) w[(size_t)t * k + lane] = p / sum;
}

hipError_t launch_route_topk(const float* logits, int T, int E, int k, int32_t* ids, float* w, hipStream_t st) {
  if (T == 0) return hipSuccess;
  hipLaunchKernelGGL(k_route_topk, dim3((T + 3) / 4), dim3(256), 0, st, logits, T, E, k, ids, w);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// Index build, step 1: per-workgroup histogram of expert ids.
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_index_hist(IndexParams p) {
  __shared__ int32_t hist[kMaxExperts];
  const int E = p.s.E, R = p.s.R;
  for (int e = threadIdx.x; e < E; e += 256) hist[e] = 0;
  __syncthreads();
  const int base = blockIdx.x * kIndexChunk;
#pragma unroll
  for (int i = 0; i < kIndexChunk / 256; i++) {
    int q = base + i * 256 + threadIdx.x;
    if (q < R) {
      int e = p.topk_ids[q];
      if ((unsigned)e >= (unsigned)E) {   // not an expert: reported through the status word, counted as the last expert
        p.ws.status[5] = p.forward_serial;
        e = E - 1;
      }
      atomicAdd(&hist[e], 1);
    }
  }
  __syncthreads();
  for (int e = threadIdx.x; e < E; e += 256) p.ws.block_hist[blockIdx.x * E + e] = hist[e];
}

// Exclusive prefix sum over 256 values, one per thread of the workgroup, left in LDS; returns the total.
__device__ inline int exclusive_scan_256(int32_t* buf, int v) {
  __shared__ int32_t wave_sum[4];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  int incl = v;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int o = __shfl_up(incl, d);
    if (lane >= d) incl += o;
  }
  if (lane == 63) wave_sum[wave] = incl;
  __syncthreads();
  int before = 0, total = 0;
#pragma unroll
  for (int w = 0; w < 4; w++) {
    const int c = wave_sum[w];
    if (w < wave) before += c;
    total += c;
  }
  buf[t] = before + incl - v;
  __syncthreads();
  return total;
}

// ---------------------------------------------------------------------------------------------
// Step 2: stable scatter.  A workgroup owns kIndexChunk consecutive pair ids, cut into runs of 64
// (one per wavefront pass); a pair's position is
//   offsets[e] + rows of e in earlier workgroups + rows of e in earlier runs + rows of e earlier in its run.
// Every workgroup derives the expert offsets and its own bases from the per-workgroup histograms (a few
// thousand values at most), which saves a kernel between the histogram and the scatter; workgroup 0 also
// writes the counts, the offsets, the M-tile table and the zeroed counters of this forward.
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_index_scatter(IndexParams p) {
  constexpr int kRuns = kIndexChunk / 64;
  __shared__ int32_t run_cnt[kRuns][kMaxExperts];
  __shared__ int32_t off[kMaxExperts];     // first row of each expert
  __shared__ int32_t before[kMaxExperts];  // rows of each expert owned by earlier workgroups
  __shared__ int32_t tbase[kMaxExperts];   // first M-tile of each expert (workgroup 0)
  const int E = p.s.E, R = p.s.R, k = p.s.k;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int my_cnt = 0;
  {
    const int e = threadIdx.x;   // E <= 256 = threads
    int mine = 0;
    constexpr int kHistLds = kRuns * kMaxExperts;   // run_cnt doubles as the landing area of the histograms
    const int n_hist = p.n_blocks * E;
    if (n_hist <= kHistLds) {
      // all histograms in one coalesced sweep, then summed out of LDS (a per-thread walk over the workgroups would
      // be a chain of dependent global loads)
      int32_t* hist = &run_cnt[0][0];
      for (int i = threadIdx.x; i < n_hist; i += 256) hist[i] = p.ws.block_hist[i];
      __syncthreads();
      if (e < E) {
        for (int b = 0; b < p.n_blocks; b++) {
          const int c = hist[b * E + e];
          if (b < (int)blockIdx.x) mine += c;
          my_cnt += c;
        }
      }
      __syncthreads();
    } else if (e < E) {
      for (int b = 0; b < p.n_blocks; b++) {
        const int c = p.ws.block_hist[b * E + e];
        if (b < (int)blockIdx.x) mine += c;
        my_cnt += c;
      }
    }
    before[threadIdx.x] = mine;
  }
  for (int i = threadIdx.x; i < kRuns * kMaxExperts; i += 256) (&run_cnt[0][0])[i] = 0;
  const int total_rows = exclusive_scan_256(off, my_cnt);
  if (blockIdx.x == 0) {
    const int e = threadIdx.x;
    const int tail = my_cnt % p.tile_m;
    const int my_tiles = e < E ? my_cnt / p.tile_m + (tail > 0) : 0;
    const int n_tiles = exclusive_scan_256(tbase, my_tiles);
    const int waves = wave == 0 ? waves_now(p, lane) : 0;
    if (threadIdx.x == 0) {
      p.ws.status[0] = 0;
      p.ws.status[1] = n_tiles;
      p.ws.status[7] = waves;
      p.ws.status[2] = n_tiles * p.n_tiles_n0;
      p.ws.status[3] = n_tiles * p.n_tiles_n1;
      p.ws.status[4] = 0;
      p.ws.status[6] = 0;
      p.ws.offsets[E] = total_rows;
    }
    if (threadIdx.x < 2 * kXcds) p.ws.queue_heads[threadIdx.x * p.ws.head_stride] = 0;
    for (int i = threadIdx.x; i < p.n_tiles_n1; i += 256) p.ws.panel_done[i] = 0;
    for (int i = threadIdx.x; i < p.max_tiles + 1; i += 256) p.ws.tile_done[i] = 0;
    if (e < E) {
      p.ws.counts[e] = my_cnt;
      p.ws.offsets[e] = off[e];
      const int nfull = my_cnt / p.tile_m;
      int ti = tbase[e], row = off[e];
      for (int i = 0; i < nfull; i++, ti++, row += p.tile_m) {
        p.ws.tile_expert[ti] = e;
        p.ws.tile_row0[ti] = row;
        p.ws.tile_rows[ti] = p.tile_m;
        p.ws.tile_kind[ti] = height_class(p.tile_m);
      }
      if (tail > 0) {
        p.ws.tile_expert[ti] = e;
        p.ws.tile_row0[ti] = row;
        p.ws.tile_rows[ti] = tail;
        p.ws.tile_kind[ti] = height_class(tail);
      }
    }
  }
  __syncthreads();
  int key[kRuns / 4], rank[kRuns / 4];
  const int base = blockIdx.x * kIndexChunk;
#pragma unroll
  for (int s = 0; s < kRuns / 4; s++) {
    const int run = wave * (kRuns / 4) + s;
    const int q = base + run * 64 + lane;
    const bool valid = q < R;
    int e = valid ? p.topk_ids[q] : -1;
    if (valid && (unsigned)e >= (unsigned)E) e = E - 1;   // as in the histogram
    // lanes of this run holding the same expert
    uint64_t same = __ballot(valid);
#pragma unroll
    for (int bit = 0; bit < 8; bit++) {
      const uint64_t b = __ballot((e >> bit) & 1);
      same &= ((e >> bit) & 1) ? b : ~b;
    }
    const uint64_t below = same & ((1ull << lane) - 1ull);
    key[s] = e;
    rank[s] = __popcll(below);
    if (valid && below == 0) run_cnt[run][e] = __popcll(same);
  }
  __syncthreads();
  for (int e = threadIdx.x; e < E; e += 256) {
    int acc = 0;
#pragma unroll
    for (int r = 0; r < kRuns; r++) {
      int c = run_cnt[r][e];
      run_cnt[r][e] = acc;
      acc += c;
    }
  }
  __syncthreads();
#pragma unroll
  for (int s = 0; s < kRuns / 4; s++) {
    const int run = wave * (kRuns / 4) + s;
    const int q = base + run * 64 + lane;
    const int e = key[s];
    if (e >= 0) {
      const int pos = off[e] + before[e] + run_cnt[run][e] + rank[s];
      p.ws.perm[pos] = q;
      p.ws.inv_perm[q] = pos;
      p.ws.row_token[pos] = q / k;
    }
  }
}

// ---------------------------------------------------------------------------------------------
// Step 3: the source segment each M-tile waits for, and the tile schedules.
//
// A tile can start once all its rows have arrived (Section 2.2.1); its rows are in source order, so that is
// the segment of its last row.
//
// A schedule is a list of (M-tile, column tile) items.  Position i of the list belongs to XCD i % 8 (a
// workgroup takes the next position of its own XCD's share and, when that is used up, of the others'), so
// consecutive positions should differ in the column tile and keep the M-tile: the workgroups of one XCD then
// work on few column tiles of many M-tiles and share weight panels in their L2.  Tall tiles come first and the
// short tiles last, so that the short ones fill the gaps at the end of the kernel.
// The orders (k_index_schedule, for up to 2048 M-tiles; see there for the locality order):
// Layer0, order 0: locality order (blocks of an expert's M-tiles per XCD, column tiles ascending inside a block).
// Order 1: per tile height, M-tiles by the segment they wait for (Fig. 5: rows that are local or arrive early first),
// all column tiles of an M-tile in a row.  Order 2: the locality order inside waves of source segments, the waves in
// arrival order.  Layer1: the locality order, or (in-kernel panel reduction) per tile height the M-tiles are dealt to
// the XCDs in contiguous chunks and every XCD sweeps its chunk column-panel-major, 4 panels at a time (Fig. 6).
// The one-workgroup builder below (any number of M-tiles) knows simpler versions of orders 0 and 1.
// ---------------------------------------------------------------------------------------------
constexpr int kTileCap = kScheduleTileCap;  // tiles whose table fits the LDS copies of the schedule builder

__device__ inline ItemRec make_item(const Workspace& ws, int m, int n) {
  ItemRec r;
  r.m_tile = m;
  r.n_tile = n;
  r.expert = ws.tile_expert[m];
  r.row0 = ws.tile_row0[m];
  r.nrows = ws.tile_rows[m];
  r.kind = ws.tile_kind[m];
  r.ready_seg = ws.tile_ready[m];
  r.pad = 0;
  return r;
}

// Layer0 items of the tiles order[lo..hi) (one height, expert-major), written from position base on.
// ord / exp_of: LDS copies (or the global arrays when the table is too large).
template <typename OrdT, typename ExpT>
__device__ inline void emit_expert_major(const Workspace& ws, ItemRec* items, const OrdT* ord, const ExpT* exp_of, int lo,
                                         int hi, int base, int n_tiles_n, int tid, int nthreads) {
  // one (tile, group of 8 column tiles) pair per thread step
  const int n_groups = (n_tiles_n + 7) >> 3;
  for (int w = tid; w < (hi - lo) * n_groups; w += nthreads) {
    const int i = lo + w / n_groups, g = w % n_groups;
    const int e = exp_of[ord[i]];
    int a = i, b = i + 1;
    while (a > lo && exp_of[ord[a - 1]] == e) a--;
    while (b < hi && exp_of[ord[b]] == e) b++;
    const int cnt = b - a;
    const int gw = min(8, n_tiles_n - g * 8);
    const int pos = base + (a - lo) * n_tiles_n + g * 8 * cnt + (i - a) * gw;
    ItemRec r = make_item(ws, ord[i], 0);
    for (int n = 0; n < gw; n++) {
      r.n_tile = g * 8 + n;
      items[pos + n] = r;
    }
  }
}

// Layer1 items of the tiles order[lo..hi): the tiles are dealt to the XCDs in contiguous chunks (an XCD then
// keeps to few experts); XCD x's queue continues, from position queue_pos[x] on, with its chunk swept per group of
// 4 column panels: the chunk's tiles, each with the 4 panels.  Panel groups ascend, so all M-tiles of the chunk
// finish panel group g before g + 1 (Fig. 6).
template <typename OrdT>
__device__ inline void emit_chunked(const Workspace& ws, ItemRec* items, const OrdT* ord, int lo, int hi,
                                    const int32_t* queue_pos, int n_tiles_n, int tid, int nthreads) {
  const int nt = hi - lo;
  if (nt == 0) return;
  const int chunk = (nt + kXcds - 1) / kXcds;
  const int n_groups = (n_tiles_n + 3) >> 2;
  for (int w = tid; w < nt * n_groups; w += nthreads) {
    const int i = w / n_groups, g = w % n_groups;
    const int x = i / chunk, j = i % chunk;
    const int cnt = min(chunk, nt - x * chunk);
    const int gw = min(4, n_tiles_n - g * 4);
    const int pos = queue_pos[x] + g * 4 * cnt + j * gw;
    ItemRec r = make_item(ws, ord[lo + i], 0);
    for (int n = 0; n < gw; n++) {
      r.n_tile = g * 4 + n;
      items[pos + n] = r;
    }
  }
}

__global__ __launch_bounds__(1024) void k_index_schedule_large(IndexParams p) {
  __shared__ int32_t cls_first[4];  // first position in order[] of the tiles of kind 2, 1, 0, and the end
  __shared__ int32_t key_pos[3 * kMaxSegments];
  __shared__ uint8_t keys[kTileCap];
  __shared__ uint8_t exp_lds[kTileCap];
  __shared__ uint16_t ord_lds[kTileCap];
  if (p.only_if_owed && p.ws.status[6] != kScheduleOwed) return;
  const int n_tiles = p.ws.status[1];
  const int tid = threadIdx.x;
  const int S = p.s.S;
  const bool in_lds = n_tiles <= kTileCap;
  const int nseg = p.layer0_order == 1 ? S : 1;
  const int nkeys = 3 * nseg;
  // the source segment each tile waits for; sort key = (height class, segment) or the height class alone
  for (int m = tid; m < n_tiles; m += 1024) {
    const int last = p.ws.tile_row0[m] + p.ws.tile_rows[m] - 1;
    const int t = p.ws.row_token[last];
    int s = 0;
    while (s + 1 < S && p.seg_offsets[s + 1] <= t) s++;
    p.ws.tile_ready[m] = s;
    if (in_lds) {
      keys[m] = (uint8_t)((2 - p.ws.tile_kind[m]) * nseg + (nseg > 1 ? s : 0));
      exp_lds[m] = (uint8_t)p.ws.tile_expert[m];
    }
  }
  __syncthreads();
  auto key_of = [&](int m) {
    return in_lds ? (int)keys[m] : (2 - p.ws.tile_kind[m]) * nseg + (nseg > 1 ? p.ws.tile_ready[m] : 0);
  };
  // stable counting sort: one thread per key value walks the keys twice, first counting, then placing
  if (tid < nkeys) {
    int c = 0;
    for (int m = 0; m < n_tiles; m++) c += (key_of(m) == tid);
    key_pos[tid] = c;
  }
  __syncthreads();
  if (tid == 0) {
    int pos = 0;
    for (int i = 0; i < nkeys; i++) {
      if (i % nseg == 0) cls_first[i / nseg] = pos;
      const int c = key_pos[i];
      key_pos[i] = pos;
      pos += c;
    }
    cls_first[3] = pos;
  }
  __syncthreads();
  if (tid < nkeys) {
    int pos = key_pos[tid];
    for (int m = 0; m < n_tiles; m++)
      if (key_of(m) == tid) {
        if (in_lds) ord_lds[pos] = (uint16_t)m; else p.ws.tile_order[pos] = m;
        pos++;
      }
  }
  __syncthreads();
  for (int c = 0; c < 3; c++) {
    const int lo = cls_first[c], hi = cls_first[c + 1];
    if (p.layer0_order == 0) {
      if (in_lds) emit_expert_major(p.ws, p.ws.items0, ord_lds, exp_lds, lo, hi, lo * p.n_tiles_n0, p.n_tiles_n0, tid, 1024);
      else emit_expert_major(p.ws, p.ws.items0, p.ws.tile_order, p.ws.tile_expert, lo, hi, lo * p.n_tiles_n0, p.n_tiles_n0, tid, 1024);
    } else {
      for (int i = tid; i < (hi - lo) * p.n_tiles_n0; i += 1024) {
        const int m = in_lds ? (int)ord_lds[lo + i / p.n_tiles_n0] : p.ws.tile_order[lo + i / p.n_tiles_n0];
        p.ws.items0[lo * p.n_tiles_n0 + i] = make_item(p.ws, m, i % p.n_tiles_n0);
      }
    }
  }
  if (p.layer0_order == 1) {
    // layer1 wants table order inside a height: rebuild order[] (the layer0 list is complete by now)
    __syncthreads();
    if (tid < 3) {
      int pos = cls_first[tid];
      for (int m = 0; m < n_tiles; m++)
        if (key_of(m) / nseg == tid) {
          if (in_lds) ord_lds[pos] = (uint16_t)m; else p.ws.tile_order[pos] = m;
          pos++;
        }
    }
    __syncthreads();
  }
  // layer1: one contiguous queue per XCD; queue x holds its chunk of every height class, tallest first
  __shared__ int32_t queue_pos[kXcds];
  const int cap = (n_tiles + 3 * kXcds) / kXcds * p.n_tiles_n1;   // room per queue
  if (tid < kXcds) queue_pos[tid] = tid * cap;
  __syncthreads();
  for (int c = 0; c < 3; c++) {
    const int lo = cls_first[c], hi = cls_first[c + 1];
    if (in_lds) emit_chunked(p.ws, p.ws.items1, ord_lds, lo, hi, queue_pos, p.n_tiles_n1, tid, 1024);
    else emit_chunked(p.ws, p.ws.items1, p.ws.tile_order, lo, hi, queue_pos, p.n_tiles_n1, tid, 1024);
    __syncthreads();
    if (tid < kXcds) {
      const int nt = hi - lo, chunk = (nt + kXcds - 1) / kXcds;
      const int cnt = nt == 0 ? 0 : max(0, min(chunk, nt - tid * chunk));
      queue_pos[tid] += cnt * p.n_tiles_n1;
    }
    __syncthreads();
  }
  if (tid < kXcds) {
    const int n0 = n_tiles * p.n_tiles_n0;
    p.ws.status[24 + tid] = tid < n0 ? (n0 - tid + kXcds - 1) / kXcds : 0;   // layer0: positions tid, tid + 8, ...
    p.ws.status[32 + tid] = queue_pos[tid] - tid * cap;
    p.ws.status[40 + tid] = tid * cap;
  }
}

// The schedule builder for tables of up to kTileCap tiles (anything but very large batches): a few workgroups, each
// of which copies the tile table into LDS, sorts it there (every tile finds its own rank, all in parallel) and
// then writes its share of the item records.  k_index_schedule_large above is the one-workgroup version without
// the size limit (and with simpler orders).
//
// Locality order (layer0 with order 0, layer1 with the separate combine kernel): per tile height, an expert's
// M-tiles are cut into blocks of up to block_m (4 by default, a light tile beside them not counted); the blocks are dealt to the XCDs, whose queues hold
// their blocks one after the other, tallest first.  Inside a block of G M-tiles the column tiles ascend and the block's M-tiles are the inner
// loop.  The 32 workgroups of an XCD, taking consecutive items, then work on G M-tiles x about 32/G column tiles of
// one expert wherever in the block they are, and share both operands in their L2; an expert with few rows is
// streamed through one XCD only (its weight panels are fetched once).
constexpr int kRankTiles = 96;       // M-tiles up to which they are ranked against each other
constexpr int kBesideItems = 128;    // light items of a layer, of experts of one block, from which on light tiles lie beside full ones
constexpr int kFewItems = 128;       // items of a layer up to which they are dealt out without blocks
constexpr int kScheduleWgs = 64;   // at most; one per 1024 items up to there (8 for 35 k items: 44 us)

struct ScheduleLds {
  int32_t row0[kTileCap];
  int32_t blk_off[kTileCap];   // M-tiles ahead of block b in its XCD's queue
  uint16_t rows[kTileCap];
  uint16_t ord0[kTileCap];     // layer0 order: position -> tile
  uint16_t ord1[kTileCap];     // layer1 order (height class, then table order)
  uint16_t blk_g[kTileCap];    // M-tiles of block b
  uint16_t blk_first[kTileCap];   // position in the order of block b's first tile
  uint16_t blk_ord[kTileCap];  // blocks in dealing order: height class, then larger blocks first
  uint8_t blk_q[kTileCap];     // XCD queue of block b
  uint8_t blk_key[kTileCap + 4];
  uint8_t expert[kTileCap];
  uint8_t kind[kTileCap];
  uint8_t ready[kTileCap];
  uint8_t key0[kTileCap + 4];   // (height class, segment) or the height class alone; padded with 0xff
  uint8_t key1[kTileCap + 4];   // height class, tallest first
  uint8_t key2[kTileCap + 4];   // the same with the light tiles in the class of their expert's full ones
  uint16_t blk_of[kTileCap];          // block of the tile at position i of ord1
  int32_t scan_buf[16];               // scratch of the prefix scans
  int32_t cls_first[4];
  int32_t cls_count[3], beside_count[3];   // tiles by key1 and by key2
  int32_t n_light_near;   // light tiles of experts of one block
  int32_t queue_pos[3][kXcds];
  int32_t q_len_t[kXcds], q_base_t[kXcds];   // locality order: M-tiles per XCD queue, and ahead of it
  int32_t n_blocks;
};

__device__ inline ItemRec make_item_lds(const ScheduleLds& L, int m, int n) {
  ItemRec r;
  r.m_tile = m;
  r.n_tile = n;
  r.expert = L.expert[m];
  r.row0 = L.row0[m];
  r.nrows = L.rows[m];
  r.kind = L.kind[m];
  r.ready_seg = L.ready[m];
  r.pad = 0;
  return r;
}

// ord[rank of tile m] = m for the stable order by key (keys < 0xff, so that the padding never counts).
__device__ inline void rank_sort(const uint8_t* key, uint16_t* ord, int n, int tid) {
  const uint32_t* words = (const uint32_t*)key;
  const int nw = (n + 3) >> 2;
  for (int m = tid; m < n; m += 1024) {
    const int km = key[m];
    int rank = 0;
    for (int j4 = 0; j4 < nw; j4++) {
      const uint32_t w = words[j4];
#pragma unroll
      for (int b = 0; b < 4; b++) {
        const int kj = (w >> (8 * b)) & 0xff, j = j4 * 4 + b;
        rank += (kj < km || (kj == km && j < m)) ? 1 : 0;
      }
    }
    ord[rank] = (uint16_t)m;
  }
}

// Inclusive prefix scan over up to 2048 values, two per thread (thread t holds elements 2t and 2t+1), running maximum
// (MAX) or running sum: inside the wavefronts by lane exchange, across them through 16 values of LDS (buf).
template <bool MAX>
__device__ inline void scan_pairs(int32_t* buf, int& v0, int& v1) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  constexpr int kNeutral = MAX ? -0x7fffffff : 0;
  auto join = [](int a, int b) { return MAX ? max(a, b) : a + b; };
  v1 = join(v0, v1);
  int incl = v1;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int o = __shfl_up(incl, d);
    if (lane >= d) incl = join(incl, o);
  }
  const int prev = __shfl_up(incl, 1);
  int before = lane > 0 ? prev : kNeutral;
  if (lane == 63) buf[wave] = incl;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < 15; w++)
    if (w < wave) before = join(before, buf[w]);
  __syncthreads();
  v0 = join(before, v0);
  v1 = join(before, v1);
}

// rank_sort for the three height classes alone, up to kTileCap tiles: two counts in one scan instead of a pass over all keys
// per tile (the schedule kernel for 250 tiles of 64 experts: 21.6 us with that, 17.4 so; up to kRankTiles tiles the pass is the shorter).  count: tiles of each class.
__device__ inline void class_sort(const uint8_t* key, uint16_t* ord, int n, const int32_t* count, int32_t* buf) {
  static_assert(kTileCap <= 2048, "counts of 16 bits, two tiles per thread");
  const int n0 = count[0], n1 = count[1];
  const int i0 = 2 * threadIdx.x, i1 = i0 + 1;
  const int k0 = i0 < n ? key[i0] : 2, k1 = i1 < n ? key[i1] : 2;
  auto one = [](int k) { return k == 0 ? 1 : (k == 1 ? 1 << 16 : 0); };
  int s0 = one(k0), s1 = one(k1);
  scan_pairs<false>(buf, s0, s1);   // of the first and second class up to and including this tile
  auto place = [&](int i, int k, int s) {
    const int a = s & 0xffff, b = s >> 16;
    ord[k == 0 ? a - 1 : (k == 1 ? n0 + b - 1 : n0 + n1 + i - a - b)] = (uint16_t)i;
  };
  if (i0 < n) place(i0, k0, s0);
  if (i1 < n) place(i1, k1, s1);
}

// Items of one layer in the locality order (see above); n_tiles_n column tiles.
__device__ inline void emit_blocks(const ScheduleLds& L, const uint16_t* ord, ItemRec* items, int n_tiles, int n_tiles_n,
                                   int block_m, int gtid, int gthreads) {
  for (int w = gtid; w < n_tiles * n_tiles_n; w += gthreads) {
    const int i = w / n_tiles_n, n = w % n_tiles_n;
    const int b = L.blk_of[i], g = L.blk_g[b], jm = i - L.blk_first[b];
    const int pos = (L.q_base_t[L.blk_q[b]] + L.blk_off[b]) * n_tiles_n + n * g + jm;
    items[pos] = make_item_lds(L, ord[i], n);
  }
}

// Blocks of the locality order and their XCD queues.  The tiles (in ord1's order: height class, expert, source order)
// fall into runs of the same height class, expert and wave -- a wave being a group of consecutive source segments,
// n_waves of them over the S segments (1: no waves) -- and every run is cut into blocks of up to block_m M-tiles.  beside: a
// light tile is in its expert's last block; otherwise it is in the runs of its own height class.
// The blocks are sorted by (wave, height class, larger first) and dealt to the XCD queues back and forth (0..7,
// 7..0, ...): with the sizes descending this keeps the queues level even when the experts' loads differ a lot, which
// round-robin does not (what is left uneven, the workgroups even out by taking from other XCDs' queues at the end).
// With waves the queues are segment-major across waves (tiles whose rows arrive early come first, Fig. 5) and
// weight-panel-major inside a wave (a block's M-tiles share every weight panel they sweep).
__device__ inline void build_blocks(ScheduleLds& L, const uint16_t* ord1, int n_tiles, int block_m, int n_waves, int S, bool beside) {
  const int tid = threadIdx.x;
  auto run_key = [&](int i) {
    const int m = ord1[i];
    const int wave = n_waves > 1 ? (int)L.ready[m] * n_waves / S : 0;
    return ((int)(beside ? L.key2[m] : L.key1[m]) << 16) | ((int)L.expert[m] << 8) | wave;
  };
  if (tid < kXcds) L.q_len_t[tid] = 0;
  const int i0 = 2 * tid, i1 = 2 * tid + 1;
  int f0 = -1, f1 = -1;
  if (i0 < n_tiles && (i0 == 0 || run_key(i0) != run_key(i0 - 1))) f0 = i0;
  if (i1 < n_tiles && run_key(i1) != run_key(i1 - 1)) f1 = i1;
  scan_pairs<true>(L.scan_buf, f0, f1);
  int s0 = 0, s1 = 0;
  auto starts = [&](int i, int f) { return (i - f) % block_m == 0 && !(i > f && beside && L.key2[ord1[i]] != L.key1[ord1[i]]); };
  if (i0 < n_tiles) s0 = starts(i0, f0);
  if (i1 < n_tiles) s1 = starts(i1, f1);
  const int start0 = s0, start1 = s1;
  scan_pairs<false>(L.scan_buf, s0, s1);
  if (i0 < n_tiles) L.blk_of[i0] = (uint16_t)(s0 - 1);
  if (i1 < n_tiles) L.blk_of[i1] = (uint16_t)(s1 - 1);
  if (i0 == n_tiles - 1) L.n_blocks = s0;
  if (i1 == n_tiles - 1) L.n_blocks = s1;
  __syncthreads();
  auto describe = [&](int i, int b) {   // tile i starts block b
    int g = 1;
    while (i + g < n_tiles && L.blk_of[i + g] == b) g++;
    const int key = run_key(i);
    L.blk_g[b] = (uint16_t)g;
    L.blk_first[b] = (uint16_t)i;
    L.blk_key[b] = (uint8_t)((key & 0xff) * 24 + (key >> 16) * 8 + (8 - min(g, 8)));   // wave, class, larger blocks first
  };
  if (i0 < n_tiles && start0) describe(i0, s0 - 1);
  if (i1 < n_tiles && start1) describe(i1, s1 - 1);
  const int n_blocks = L.n_blocks;
  for (int b = n_blocks + tid; b < n_blocks + 4; b += 1024) L.blk_key[b] = 0xff;
  __syncthreads();
  rank_sort(L.blk_key, L.blk_ord, n_blocks, tid);
  __syncthreads();
  for (int pos = tid; pos < n_blocks; pos += 1024) {
    const int r = pos / kXcds, i = pos % kXcds;
    const int x = (r & 1) ? kXcds - 1 - i : i;
    int off = 0;
    for (int r2 = 0; r2 < r; r2++) off += L.blk_g[L.blk_ord[r2 * kXcds + ((r2 & 1) ? kXcds - 1 - x : x)]];
    const int b = L.blk_ord[pos];
    L.blk_off[b] = off;
    L.blk_q[b] = (uint8_t)x;
    // the queue's last block: no later round has a block for this queue
    const int next = (r + 1) * kXcds + (((r + 1) & 1) ? kXcds - 1 - x : x);
    if (next >= n_blocks) L.q_len_t[x] = off + L.blk_g[b];
  }
  __syncthreads();
  if (tid == 0) {
    int pos = 0;
    for (int x = 0; x < kXcds; x++) {
      L.q_base_t[x] = pos;
      pos += L.q_len_t[x];
    }
  }
  __syncthreads();
}

// M-tile m as the schedule builder sees it: its table row and the segment of its last row (of token `last_token`).  ragged: it is the
// remainder beside full tiles of its expert, light where its class is a lower one.
__device__ inline void note_tile(ScheduleLds& L, const IndexParams& p, const int32_t* seg_lds, int m, int expert, int row0,
                                 int nrows, int kind, bool ragged, int last_token, bool publish) {
  const int S = p.s.S, nseg = p.layer0_order == 1 ? S : 1;
  int s = 0;
  while (s + 1 < S && seg_lds[s + 1] <= last_token) s++;
  L.row0[m] = row0;
  L.rows[m] = (uint16_t)nrows;
  L.kind[m] = (uint8_t)kind;
  L.expert[m] = (uint8_t)expert;
  L.ready[m] = (uint8_t)s;
  const int beside = 2 - (ragged ? height_class(p.tile_m) : kind);
  L.key0[m] = (uint8_t)((2 - kind) * nseg + (nseg > 1 ? s : 0));
  L.key1[m] = (uint8_t)(2 - kind);
  L.key2[m] = (uint8_t)beside;
  atomicAdd(&L.cls_count[2 - kind], 1);
  atomicAdd(&L.beside_count[beside], 1);
  if (publish) p.ws.tile_ready[m] = s;
}

// The schedules of both layers from the noted tiles.  The workgroups that share the work (gtid of gthreads) all build the
// tables; the one with first set writes the queues.  waves: of layer0_order 2.  Entered with the tiles noted and a barrier behind them.
__device__ inline void build_schedules(ScheduleLds& L, const IndexParams& p, int n_tiles, int waves, bool first, int gtid, int gthreads) {
  const int tid = threadIdx.x;
  const int S = p.s.S, nseg = p.layer0_order == 1 ? S : 1;
  // layer0: 0 expert-major (locality order), 1 by source segment, 2 locality order inside waves of source segments
  const bool local0 = p.layer0_order != 1, local1 = p.layer1_order == 0;
  const int n_waves0 = p.layer0_order == 2 ? max(1, min(waves, min(S, 8))) : 1;
  const int block_m = p.block_m;   // M-tiles per block of the locality order (1..8)
  // Where the light tiles lie in the locality order of a layer: in the block of their expert's full tiles (beside), with which
  // they then share the weights in the L2 instead of streaming them again, or behind all full tiles, where they fill the gaps at the
  // end of the launch.  The first pays where there are enough of them, the second where a launch is few rounds of long tiles; and an
  // expert of several blocks saves the least.  us per layer, behind / beside: 2 full tiles and a light one for each of 64 experts (9000
  // tokens, top-4, F = 1408; 704 and 512 light items) 731 / 630, for half of them (8192 tokens; 319 and 232) 607 / 567, (4096 tokens, top-8, F =
  // 2560; 580 and 406) 1707 / 1641; one full tile (1060 tokens of 8 experts of F = 7168) 545 / 497; 112 and 64 items (2047 tokens of 8 experts)
  // 381 / 414; 8 full tiles (8192 tokens of 8 experts of F = 14336, 448 items in layer0) 4045 / 4088.
  // Other orders keep to the tiles' own classes (4096 tokens of 8 experts of F = 14336, light
  // tiles among the full ones / behind: panel-major 2345 / 2257, large builder 2305 / 2230).
  for (int m = tid; m < n_tiles; m += 1024)
    if (L.key2[m] != L.key1[m] && !(m > block_m && L.expert[m - block_m - 1] == L.expert[m])) atomicAdd(&L.n_light_near, 1);
  __syncthreads();
  const bool beside0 = local0 && L.n_light_near * p.n_tiles_n0 >= kBesideItems;
  const bool beside1 = local1 && L.n_light_near * p.n_tiles_n1 >= kBesideItems;
  auto sort_tiles = [&](uint16_t* ord, bool beside) {   // tallest class first, then table order
    if (n_tiles <= kRankTiles) rank_sort(beside ? L.key2 : L.key1, ord, n_tiles, tid);
    else class_sort(beside ? L.key2 : L.key1, ord, n_tiles, beside ? L.beside_count : L.cls_count, L.scan_buf);
  };
  if (nseg > 1) rank_sort(L.key0, L.ord0, n_tiles, tid);
  else sort_tiles(L.ord0, beside0);
  const bool two_orders = nseg > 1 || beside0 != beside1;
  if (two_orders) sort_tiles(L.ord1, beside1);
  if (tid == 0) {
    int pos = 0;
    for (int c = 0; c < 3; c++) {
      L.cls_first[c] = pos;
      pos += L.cls_count[c];
    }
    L.cls_first[3] = pos;
  }
  // layer1 in panel-major order (in-kernel combine): XCD x gets a contiguous chunk of every height class
  const int cap = (n_tiles + 3 * kXcds) / kXcds * p.n_tiles_n1;   // room per queue
  if (tid < kXcds) {
    int pos = tid * cap;
    for (int c = 0; c < 3; c++) {
      L.queue_pos[c][tid] = pos;
      const int nt = L.cls_count[c], chunk = (nt + kXcds - 1) / kXcds;
      const int cnt = nt == 0 ? 0 : max(0, min(chunk, nt - tid * chunk));
      pos += cnt * p.n_tiles_n1;
    }
    if (first && !local1) {
      p.ws.status[32 + tid] = pos - tid * cap;
      p.ws.status[40 + tid] = tid * cap;
    }
    if (first && !local0) {
      const int n0 = n_tiles * p.n_tiles_n0;
      p.ws.status[24 + tid] = tid < n0 ? (n0 - tid + kXcds - 1) / kXcds : 0;   // positions tid, tid + 8, ...
    }
  }
  __syncthreads();
  const uint16_t* ord1 = two_orders ? L.ord1 : L.ord0;   // height class, then table order (expert-major)
  // So few items that most workgroups get none and none gets a second: there is no locality to arrange, the items are
  // dealt out one by one (the block tables cost 4 us, of 38 us for a layer of 128 tokens and H = 256).
  if (local0 && local1 && n_waves0 == 1 && n_tiles * max(p.n_tiles_n0, p.n_tiles_n1) <= kFewItems) {
    auto deal = [&](ItemRec* items, int n_tiles_n, int len_at, int base_at) {
      const int n = n_tiles * n_tiles_n;
      auto base = [&](int x) { return x * (n / kXcds) + min(x, n % kXcds); };
      for (int i = gtid; i < n; i += gthreads)
        items[base(i % kXcds) + i / kXcds] = make_item_lds(L, ord1[i / n_tiles_n], i % n_tiles_n);
      if (first && tid < kXcds) {
        p.ws.status[len_at + tid] = base(tid + 1) - base(tid);
        p.ws.status[base_at + tid] = base(tid);
      }
    };
    deal(p.ws.items0, p.n_tiles_n0, 24, 48);
    deal(p.ws.items1, p.n_tiles_n1, 32, 40);
    return;
  }
  if (local0) {
    build_blocks(L, L.ord0, n_tiles, block_m, n_waves0, S, beside0);
    if (first && tid < kXcds) {
      p.ws.status[24 + tid] = L.q_len_t[tid] * p.n_tiles_n0;
      p.ws.status[48 + tid] = L.q_base_t[tid] * p.n_tiles_n0;
    }
    emit_blocks(L, L.ord0, p.ws.items0, n_tiles, p.n_tiles_n0, block_m, gtid, gthreads);
  } else {
    // by source segment (Fig. 5): all column tiles of an M-tile in a row; list position i belongs to XCD i % 8
    for (int i = gtid; i < n_tiles * p.n_tiles_n0; i += gthreads)
      p.ws.items0[i] = make_item_lds(L, L.ord0[i / p.n_tiles_n0], i % p.n_tiles_n0);
  }
  if (local1) {
    if (!local0 || n_waves0 > 1 || two_orders) {
      __syncthreads();   // the layer0 items are out: the block tables can be rebuilt without waves
      build_blocks(L, ord1, n_tiles, block_m, 1, S, beside1);
    }
    if (first && tid < kXcds) {
      p.ws.status[32 + tid] = L.q_len_t[tid] * p.n_tiles_n1;
      p.ws.status[40 + tid] = L.q_base_t[tid] * p.n_tiles_n1;
    }
  }
  if (local1) {
    emit_blocks(L, ord1, p.ws.items1, n_tiles, p.n_tiles_n1, block_m, gtid, gthreads);
  } else {
    // panel-major (Fig. 6): every XCD sweeps its chunk of a height class per group of 4 column panels: the chunk's
    // tiles, each with the 4 panels; panel groups ascend, so all M-tiles of the chunk finish group g before g + 1
    const int n_groups1 = (p.n_tiles_n1 + 3) >> 2;
    for (int w = gtid; w < n_tiles * n_groups1; w += gthreads) {
      const int ig = w / n_groups1, g = w % n_groups1;
      const int m = ord1[ig], c = 2 - L.kind[m];
      const int i = ig - L.cls_first[c], nt = L.cls_count[c];
      const int chunk = (nt + kXcds - 1) / kXcds;
      const int x = i / chunk, j = i % chunk;
      const int cnt = min(chunk, nt - x * chunk);
      const int gw = min(4, p.n_tiles_n1 - g * 4);
      const int pos = L.queue_pos[c][x] + g * 4 * cnt + j * gw;
      ItemRec r = make_item_lds(L, m, 0);
      for (int n = 0; n < gw; n++) {
        r.n_tile = g * 4 + n;
        p.ws.items1[pos + n] = r;
      }
    }
  }
}

__global__ __launch_bounds__(1024) void k_index_schedule(IndexParams p) {
  __shared__ __attribute__((aligned(16))) ScheduleLds L;
  __shared__ int32_t seg_lds[kMaxSegments + 1];
  if (p.only_if_owed && p.ws.status[6] != kScheduleOwed) return;
  const int n_tiles = max(0, min(p.ws.status[1], p.max_tiles));
  const int tid = threadIdx.x;
  if (tid <= p.s.S) seg_lds[tid] = p.seg_offsets[tid];
  if (tid < 3) L.cls_count[tid] = L.beside_count[tid] = 0;
  if (tid == 3) L.n_light_near = 0;
  __syncthreads();
  for (int m = tid; m < n_tiles + 4; m += 1024) {
    if (m >= n_tiles) {
      L.key0[m] = 0xff;
      L.key1[m] = 0xff;
      L.key2[m] = 0xff;
      continue;
    }
    const int r0 = p.ws.tile_row0[m], nr = p.ws.tile_rows[m], kd = p.ws.tile_kind[m];
    const int e = p.ws.tile_expert[m];
    const bool ragged = nr < p.tile_m && m > 0 && p.ws.tile_expert[m - 1] == e;
    note_tile(L, p, seg_lds, m, e, r0, nr, kd, ragged, p.ws.row_token[max(0, min(r0 + nr, p.s.R) - 1)], blockIdx.x == 0);
  }
  __syncthreads();
  build_schedules(L, p, n_tiles, p.ws.status[7], blockIdx.x == 0, blockIdx.x * 1024 + tid, gridDim.x * 1024);
}

// ---------------------------------------------------------------------------------------------
// The whole index build of a small batch in one workgroup: the three kernels above it are 5 us each of launch and
// start, whatever the batch (with 128 tokens, 21 us of a 43 us forward).  Wavefronts rank their runs of 64 pair ids as
// k_index_scatter does; the runs' counts, the row order and the tile table stay in LDS.  schedule: 0 leaves the tile
// schedules out (a forward whose GroupGEMMs do not use them).
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(1024) void k_index_small(IndexParams p, int schedule) {
  constexpr int kRuns = kIndexSmallRows / 64, kPerWave = kRuns / 16;
  __shared__ __attribute__((aligned(16))) ScheduleLds L;
  __shared__ int32_t seg_lds[kMaxSegments + 1];
  __shared__ uint16_t run_cnt[kRuns * kMaxExperts];   // [run][expert]: rows of the expert in the run, then in the runs before it
  __shared__ int32_t token_of[kIndexSmallRows];       // row -> token
  __shared__ int32_t cnt[kMaxExperts], off[kMaxExperts], tbase[kMaxExperts + 1];
  __shared__ int32_t waves;
  const int E = p.s.E, R = p.s.R, k = p.s.k;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n_runs = (R + 63) / 64;
  int key[kPerWave], rank[kPerWave];
#pragma unroll
  for (int i = 0; i < kPerWave; i++) {
    const int q = (i * 16 + wave) * 64 + lane;
    key[i] = q < R ? p.topk_ids[q] : -1;
  }
  for (int i = tid; i < n_runs * E; i += 1024) run_cnt[i] = 0;
  if (tid <= p.s.S) seg_lds[tid] = p.seg_offsets[tid];
  if (tid < 3) L.cls_count[tid] = L.beside_count[tid] = 0;
  if (tid == 3) L.n_light_near = 0;
  if (tid < kMaxExperts) cnt[tid] = 0;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < kPerWave; i++) {
    const int run = i * 16 + wave;
    if (run >= n_runs) break;
    const bool valid = run * 64 + lane < R;
    int e = key[i];
    if (valid && (unsigned)e >= (unsigned)E) {   // not an expert: reported through the status word, counted as the last expert
      p.ws.status[5] = p.forward_serial;
      e = E - 1;
    }
    uint64_t same = __ballot(valid);
#pragma unroll
    for (int bit = 0; bit < 8; bit++) {
      const uint64_t b = __ballot((e >> bit) & 1);
      same &= ((e >> bit) & 1) ? b : ~b;
    }
    const uint64_t below = same & ((1ull << lane) - 1ull);
    key[i] = e;
    rank[i] = __popcll(below);
    if (valid && below == 0) run_cnt[run * E + e] = (uint16_t)__popcll(same);
  }
  __syncthreads();
  if (tid < E) {
    int acc = 0;
    for (int r = 0; r < n_runs; r++) {
      const int c = run_cnt[r * E + tid];
      run_cnt[r * E + tid] = (uint16_t)acc;
      acc += c;
    }
    cnt[tid] = acc;
  }
  __syncthreads();
  // offsets and first tiles of the experts: four experts per lane of the first wavefront
  if (wave == 0) {
    int c[4], t[4], rows = 0, tiles = 0;
#pragma unroll
    for (int i = 0; i < 4; i++) {
      c[i] = cnt[lane * 4 + i];
      t[i] = c[i] / p.tile_m + (c[i] % p.tile_m > 0);
      rows += c[i];
      tiles += t[i];
    }
    int rows_incl = rows, tiles_incl = tiles;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const int ro = __shfl_up(rows_incl, d), to = __shfl_up(tiles_incl, d);
      if (lane >= d) {
        rows_incl += ro;
        tiles_incl += to;
      }
    }
    int ro = rows_incl - rows, to = tiles_incl - tiles;
#pragma unroll
    for (int i = 0; i < 4; i++) {
      off[lane * 4 + i] = ro;
      tbase[lane * 4 + i] = to;
      ro += c[i];
      to += t[i];
    }
    if (lane == 63) {
      tbase[kMaxExperts] = tiles_incl;
      p.ws.status[0] = 0;
      p.ws.status[1] = tiles_incl;
      p.ws.status[2] = tiles_incl * p.n_tiles_n0;
      p.ws.status[3] = tiles_incl * p.n_tiles_n1;
      p.ws.status[4] = 0;
      p.ws.status[6] = schedule ? 0 : kScheduleOwed;
      p.ws.offsets[E] = rows_incl;
    }
  } else if (wave == 1) {
    if (lane < 2 * kXcds) p.ws.queue_heads[lane * p.ws.head_stride] = 0;
    const int now = waves_now(p, lane);
    if (lane == 0) p.ws.status[7] = waves = now;
  } else if (wave < 4) {
    for (int i = tid - 128; i < p.n_tiles_n1; i += 128) p.ws.panel_done[i] = 0;
  } else {
    for (int i = tid - 256; i < p.max_tiles + 1; i += 768) p.ws.tile_done[i] = 0;
  }
  __syncthreads();
  if (tid < E) {
    p.ws.counts[tid] = cnt[tid];
    p.ws.offsets[tid] = off[tid];
  }
#pragma unroll
  for (int i = 0; i < kPerWave; i++) {
    const int run = i * 16 + wave, q = run * 64 + lane;
    if (q < R) {
      const int e = key[i], pos = off[e] + run_cnt[run * E + e] + rank[i], t = q / k;
      p.ws.perm[pos] = q;
      p.ws.inv_perm[q] = pos;
      p.ws.row_token[pos] = t;
      token_of[pos] = t;
    }
  }
  __syncthreads();
  const int n_tiles = tbase[kMaxExperts];
  for (int m = tid; m < n_tiles + 4; m += 1024) {
    if (m >= n_tiles) {
      L.key0[m] = 0xff;
      L.key1[m] = 0xff;
      L.key2[m] = 0xff;
      continue;
    }
    int lo = 0, hi = E - 1;   // the last expert whose first tile is at most m (experts without tiles share the next one's)
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (tbase[mid] <= m) lo = mid;
      else hi = mid - 1;
    }
    const int i = m - tbase[lo], full = cnt[lo] / p.tile_m;
    const int row0 = off[lo] + i * p.tile_m;
    const int rows = i < full ? p.tile_m : cnt[lo] % p.tile_m, kind = height_class(rows);
    p.ws.tile_expert[m] = lo;
    p.ws.tile_row0[m] = row0;
    p.ws.tile_rows[m] = rows;
    p.ws.tile_kind[m] = kind;
    note_tile(L, p, seg_lds, m, lo, row0, rows, kind, i >= full && full > 0, token_of[row0 + rows - 1], true);
  }
  if (!schedule) return;
  __syncthreads();
  build_schedules(L, p, n_tiles, waves, true, tid, 1024);
}

__global__ void k_tile_heights(const int32_t* __restrict__ rows, int32_t* __restrict__ height, int n) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < n) height[i] = variant_rows(rows[i]);
}

hipError_t launch_tile_heights(const int32_t* rows, int32_t* height, int n, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_tile_heights, dim3((n + 255) / 256), dim3(256), 0, st, rows, height, n);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// Stand-in for the peers of Section 3.1.2 on one GPU: a few workgroups play all sources in turn, copying each source's
// segment of token rows from a staging buffer into the receive buffer at a paced rate and then raising the
// segment's ready flag (data first, system-scope release, then the flag), the way a peer's one-sided stores would.
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(1024) void k_arrival_producer(const uint4* __restrict__ staging, uint4* __restrict__ x,
                                                           ArrivalParams a) {
  const long long t_start = wall_clock64();   // 100 MHz
  long long sent = 0;                          // bytes (of all workgroups together) before the current chunk
  const int nwg = gridDim.x, wg = blockIdx.x;
  for (int s = 0; s < a.S; s++) {
    const size_t lo = (size_t)a.seg_offsets[s] * a.row_bytes / 16, hi = (size_t)a.seg_offsets[s + 1] * a.row_bytes / 16;
    for (size_t c = lo; c < hi; c += a.chunk16) {
      const size_t end = c + a.chunk16 < hi ? c + a.chunk16 : hi;
      // pace: this chunk may start once the bytes before it have had their time at the requested rate
      if (a.bytes_per_us > 0) {
        const long long due = t_start + (long long)((double)sent / a.bytes_per_us * 100.0);
        while (wall_clock64() < due) __builtin_amdgcn_s_sleep(16);
      }
      for (size_t i = c + (size_t)wg * 1024 + threadIdx.x; i < end; i += (size_t)nwg * 1024) x[i] = staging[i];
      sent += (long long)(end - c) * 16;
    }
    // the segment is there once every workgroup has written its share: the last one to arrive raises the flag
    __threadfence_system();
    __syncthreads();
    if (threadIdx.x == 0) {
      const uint32_t arrived = __hip_atomic_fetch_add(&a.seg_arrived[s], 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
      if (arrived + 1 == (uint32_t)nwg) {
        __hip_atomic_store(&a.seg_arrived[s], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // ready for the next call
        __hip_atomic_store(&a.seg_ready[s], a.epoch, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
      }
    }
  }
}

hipError_t launch_arrival_producer(const void* staging, void* x, const ArrivalParams& a, int n_wg, hipStream_t st) {
  hipLaunchKernelGGL(k_arrival_producer, dim3(n_wg), dim3(1024), 0, st, (const uint4*)staging, (uint4*)x, a);
  return hipGetLastError();
}

// Queue heads, combine counter, panel counters and the status word back to zero: what the scatter kernel does at the
// start of a forward, for a forward that runs the schedules of an earlier index build again.
__global__ void k_reset_counters(Workspace ws, int n_tiles_n1, int max_tiles, int schedule_built) {
  const int t = threadIdx.x;
  for (int i = t; i < max_tiles + 1; i += 256) ws.tile_done[i] = 0;
  if (t == 0) {
    ws.status[0] = 0;
    ws.status[4] = 0;
    if (schedule_built) ws.status[6] = 0;
  }
  if (t < 2 * kXcds) ws.queue_heads[t * ws.head_stride] = 0;
  for (int i = t; i < n_tiles_n1; i += 256) ws.panel_done[i] = 0;
}

hipError_t launch_reset_counters(const Workspace& ws, int n_tiles_n1, int max_tiles, bool schedule_built, hipStream_t st) {
  hipLaunchKernelGGL(k_reset_counters, dim3(1), dim3(256), 0, st, ws, n_tiles_n1, max_tiles, schedule_built ? 1 : 0);
  return hipGetLastError();
}

hipError_t launch_index_schedule(const IndexParams& p, hipStream_t st) {
  if (!uses_large_schedule(p.max_tiles, p.force_large_schedule)) {
    const int64_t items = (int64_t)(p.s.R / p.tile_m + p.s.E) * (p.n_tiles_n0 + p.n_tiles_n1);
    const int wgs = (int)(items / 1024 < 1 ? 1 : (items / 1024 > kScheduleWgs ? kScheduleWgs : items / 1024));
    hipLaunchKernelGGL(k_index_schedule, dim3(wgs), dim3(1024), 0, st, p);
  } else {
    hipLaunchKernelGGL(k_index_schedule_large, dim3(1), dim3(1024), 0, st, p);
  }
  return hipGetLastError();
}

hipError_t launch_index_build(const IndexParams& p, bool schedule, hipStream_t st) {
  if (p.s.R == 0) return hipSuccess;
  // one workgroup while it ends before the three kernels would (it then writes the item records alone)
  const bool large = uses_large_schedule(p.max_tiles, p.force_large_schedule);
  if (p.s.R <= kIndexSmallRows && !large &&
      (!schedule || (int64_t)p.max_tiles * (p.n_tiles_n0 + p.n_tiles_n1) <= kIndexSmallItems)) {
    hipLaunchKernelGGL(k_index_small, dim3(1), dim3(1024), 0, st, p, schedule ? 1 : 0);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(k_index_hist, dim3(p.n_blocks), dim3(256), 0, st, p);
  hipLaunchKernelGGL(k_index_scatter, dim3(p.n_blocks), dim3(256), 0, st, p);
  return launch_index_schedule(p, st);
}

}  // namespace moe
