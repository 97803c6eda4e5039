// Device-side planning: turns ctx_lens / q_lens into compact work lists without a host
// round trip, so a call never synchronises.  The partition depends on the lengths only,
// never on physical page ids.
#include "rollattn_internal.h"

namespace rollattn {

namespace {

constexpr int kPlanThreads = 1024;

constexpr int kLdsPrefix = 8192;   // batches up to this size keep the scan in LDS for the searches

// Inclusive scan over the wave in six cross-lane steps of the vector ALU (rows of 16, then their last lanes broadcast).
__device__ __forceinline__ int wave_inclusive_scan(int x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);   // row_shr:1
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);   // row_shr:2
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);   // row_shr:4
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);   // row_shr:8
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);   // row_bcast:15 into rows 1 and 3
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);   // row_bcast:31 into rows 2 and 3
  return x;
}

__device__ __forceinline__ int wave_sum(int x) { return __builtin_amdgcn_readlane(wave_inclusive_scan(x), 63); }

// Largest of one unsigned per lane, by the same steps (a step that has no source lane contributes zero).
__device__ __forceinline__ unsigned wave_max(unsigned v) {
  int x = (int)v;
  auto step = [&](int other) { x = (int)max((unsigned)x, (unsigned)other); };
  step(__builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false));
  step(__builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false));
  step(__builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false));
  step(__builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false));
  step(__builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false));
  step(__builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false));
  return (unsigned)__builtin_amdgcn_readlane(x, 63);
}

// Exclusive scan of one int per thread across the workgroup; returns this thread's prefix
// and leaves the workgroup total in *total.  A plan kernel is one workgroup that every CU waits for, so its barriers
// and LDS round trips count: two barriers, four reads.
__device__ int block_exclusive_scan(int v, int4* wave_tot /*[kPlanThreads / 256]*/, int* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int incl = wave_inclusive_scan(v);
  if (lane == 63) ((int*)wave_tot)[wave] = incl;
  __syncthreads();
  int base = 0, tot = 0;
#pragma unroll
  for (int i = 0; i < kPlanThreads / 256; ++i) {
    const int4 t = wave_tot[i];
    base += (4 * i < wave ? t.x : 0) + (4 * i + 1 < wave ? t.y : 0) + (4 * i + 2 < wave ? t.z : 0) + (4 * i + 3 < wave ? t.w : 0);
    tot += t.x + t.y + t.z + t.w;
  }
  *total = tot;
  __syncthreads();
  return base + incl - v;
}

// Decode partition.  Every trajectory is cut into blocks of kBlockTokens tokens; the rows
// (trajectory b, row r in [0, rows_per_b)) are laid end to end, b outermost, each with
// n_b = ceil(L_b / kBlockTokens) blocks; the resulting sequence of T blocks is dealt to the W
// workers in equal contiguous runs of per = ceil(T / W) blocks.  Written out: the exclusive
// scan of n_b, the run length, T, and for every worker one 16-byte record with all it needs to
// start: (b, r << 20 | block, L_b, blocks in its run), or b = -1 for a worker without blocks.
// len_of(b): tokens of trajectory b that take part.
template <class L>
__device__ __forceinline__ void plan_decode(const DecodePlanArgs& a, L&& len_of) {
  __shared__ int4 wave_tot[kPlanThreads / 256];
  __shared__ int prefix_s[kLdsPrefix + 1];
  const int tid = threadIdx.x;
  const int32_t batch = a.batch, rows_per_b = a.rows_per_b, workers = a.workers, slots = a.slots;
  int32_t* const header = a.header;
  int32_t* const prefix = a.prefix;
  int32_t* const wstart = a.wstart;
  const bool in_lds = batch <= kLdsPrefix;
  __shared__ int len_s[kLdsPrefix];
  int running = 0;
  for (int b0 = 0; b0 < batch; b0 += kPlanThreads) {
    const int b = b0 + tid;
    const int len = b < batch ? len_of(b) : 0;
    const int count = (len + kBlockTokens - 1) / kBlockTokens;
    int tile_total;
    const int first = running + block_exclusive_scan(count, wave_tot, &tile_total);
    if (b < batch) {
      prefix[b] = first;
      if (in_lds) {
        prefix_s[b] = first;
        len_s[b] = len;
      }
    }
    running += tile_total;
  }
  if (tid == 0) {
    prefix[batch] = running;
    if (in_lds) prefix_s[batch] = running;
  }
  const int total = running * rows_per_b;
  const int per = max(1, (total + workers - 1) / workers);
  if (tid == 0) {
    header[kPlanPer] = per;
    header[kPlanTotal] = total;
    header[kPlanWorkers] = workers;
    header[kPlanRowsPerB] = rows_per_b;
  }
  __threadfence_block();
  __syncthreads();   // prefix[] written above is read below by other threads of this workgroup
  for (int w = tid; w < slots; w += kPlanThreads) {
    const long x = (long)w * per;
    int4 st = make_int4(-1, 0, 0, 0);
    if (w < workers && x < total) {
      // largest b with rows_per_b * prefix[b] <= x (rows without blocks can never be the answer
      // because the next row then starts at the same position)
      const int* pf = in_lds ? prefix_s : prefix;
      int lo = 0, hi = batch;
      while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if ((long)rows_per_b * pf[mid] <= x) lo = mid; else hi = mid;
      }
      const int n = pf[lo + 1] - pf[lo];
      const int rem = (int)(x - (long)rows_per_b * pf[lo]);
      const int mine = (int)min((long)per, (long)total - x);
      st = make_int4(lo, ((rem / n) << 20) | (rem % n), in_lds ? len_s[lo] : len_of(lo), mine);
    }
    *(int4*)(wstart + 4 * w) = st;
  }
}

// With q_lens given (mixed step) only the trajectories with q_lens[b] == 1 take part; the others count as empty.
__device__ __forceinline__ void plan_decode(const DecodePlanArgs& a) {
  plan_decode(a, [&](int b) { return (!a.q_lens || a.q_lens[b] == 1) ? a.ctx_lens[b] : 0; });
}

__global__ __launch_bounds__(kPlanThreads) void plan_decode_kernel(const DecodePlanArgs a) { plan_decode(a); }

// Append work list: each chunk cut into tiles of tile_tokens query tokens.  A tile's cost grows
// with its trajectory's context, and workgroups are dispatched in list order, so (for batches that
// fit the ranking in LDS) trajectories are listed longest context first: the long tiles start
// early and the short ones fill the tail.  For the same reason a chunk's tiles are listed last
// tile first.
//
// Pieces.  A tile walks its visible context block by block, so a call ends no earlier than its longest tile, however
// many CUs have nothing to do: a few observations behind long prefixes, or one 64k history among short ones, leave
// most of the chip idle.  When the list is short enough to be looked at as a whole (kSplitTiles), the kernel asks
// whether cutting the tiles into pieces of at most P blocks would end sooner: 64 values of P around the mean
// load of a CU are tried side by side, each priced in blocks as
//   max(P + kPieceCost, load + u (P + kPieceCost) (ceil(w) - w)),   w = pieces / CUs, load = (blocks + kPieceCost pieces) / CUs,
// u = mean piece / P: with equal pieces that is the number of full rounds over the CUs, with unequal ones the later,
// shorter pieces fill the gaps.  kPieceCost is what a workgroup costs besides its blocks (start, first tiles from HBM,
// epilogue, hand-over of the CU: 22,000 cycles against 2,500 per block when measured), kMergeCost the merge launch and
// the float partials' way to memory and back.  The split is taken only where the price drops by a tenth.
// Measured: three observations of 16 .. 512 tokens behind 2k .. 16k (32/8/128, bf16, one of every four CUs idle before)
// 275 -> 208 us with plan and merge; 33 of 3 .. 96 tokens behind up to 64k (64/4/128, FP8) 1410 -> 652 us.  The decision
// adds 3 us to the plan of a short list, the merge takes 12 us where tiles were cut and 3 us where none was; lists too
// long to be cut skip both (the host knows a lower bound of the number of tiles).
constexpr int kRankBatch = 4096;
constexpr int kSplitTiles = 1024;
constexpr float kPieceCost = 8.f;
constexpr float kMergeCost = 8.f;

__device__ __forceinline__ float split_price(float p, float blocks, float pieces, float cus) {
  const float w = pieces / cus, load = (blocks + kPieceCost * pieces) / cus;
  const float u = fminf(1.f, blocks / (pieces * p));
  return fmaxf(p + kPieceCost, load + u * (p + kPieceCost) * (ceilf(w) - w));
}

// What the append plan asks about a chunk: its context, its rows, where they start in the packed query.
struct ChunkLens {
  const int32_t *ctx_lens, *q_lens, *q_offsets;
  __device__ __forceinline__ int ctx(int b) const { return ctx_lens[b]; }
  __device__ __forceinline__ int rows(int b) const { return q_lens[b]; }
  __device__ __forceinline__ int offset(int b) const { return q_offsets[b]; }
};

template <class C>
__device__ __forceinline__ void plan_append(const AppendPlanArgs& a, const C& chunk) {
  __shared__ int4 wave_tot[kPlanThreads / 256];
  __shared__ int len_s[kRankBatch];
  __shared__ int order_s[kRankBatch];
  const int tid = threadIdx.x;
  const int batch = a.batch, tile_tokens = a.tile_tokens;
  const bool ranked = batch <= kRankBatch;
  if (ranked) {
    for (int b = tid; b < batch; b += kPlanThreads) len_s[b] = chunk.ctx(b);
    __syncthreads();
    for (int b = tid; b < batch; b += kPlanThreads) {
      const int mine = len_s[b];
      int rank = 0;
      for (int o = 0; o < batch; ++o) {
        const int other = len_s[o];
        rank += (other > mine || (other == mine && o < b)) ? 1 : 0;
      }
      order_s[rank] = b;
    }
    __syncthreads();
  }
  __shared__ int first_s[kPlanThreads], count_s[kPlanThreads], b_s[kPlanThreads], qlen_s[kPlanThreads], ctx_s[kPlanThreads],
      qoff_s[kPlanThreads];
  // the first kSplitTiles tiles of the list, for the decision about pieces: record and number of blocks
  __shared__ int4 tile_s[kSplitTiles];
  __shared__ int tile_qoff_s[kSplitTiles], blocks_s[kSplitTiles];
  int running = 0;
  for (int p0 = 0; p0 < batch; p0 += kPlanThreads) {
    const int p = p0 + tid;
    int b = 0, count = 0, q_len = 0;
    if (p < batch) {
      b = ranked ? order_s[p] : p;
      q_len = chunk.rows(b);
      count = (q_len + tile_tokens - 1) / tile_tokens;
      if (a.skip_unit_chunks && q_len == 1) count = 0;   // mixed step: the decode kernel takes these
    }
    int tile_total;
    const int first = running + block_exclusive_scan(count, wave_tot, &tile_total);
    first_s[tid] = first;
    count_s[tid] = count;
    b_s[tid] = b;
    qlen_s[tid] = q_len;
    ctx_s[tid] = p < batch ? chunk.ctx(b) : 0;
    qoff_s[tid] = p < batch ? chunk.offset(b) : 0;
    __syncthreads();
    // One 32-byte record per tile with everything the tile's workgroup needs to start, so that it gets there with
    // one dependent load instead of a chain of them: (b, first row, n_b, L_b, q_offsets[b], first block, blocks, slot).
    // The tiles of these trajectories are dealt to the threads one by one (a trajectory may have hundreds): a tile
    // finds its trajectory as the last one of the group that starts at or before it (those without tiles start where
    // the next one starts, and are never the last such).
    const int end = min(running + tile_total, a.cap);
    for (int t = running + tid; t < end; t += kPlanThreads) {
      int lo = 0, hi = kPlanThreads;
      while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (first_s[mid] <= t) lo = mid; else hi = mid;
      }
      const int s = t - first_s[lo];
      const int q0 = (count_s[lo] - 1 - s) * tile_tokens;   // a chunk's last tile sees the most context
      const int seen = a.noncausal ? ctx_s[lo] : ctx_s[lo] - qlen_s[lo] + min(q0 + tile_tokens, qlen_s[lo]);
      const int blocks = (seen + kAppendBlockTokens - 1) / kAppendBlockTokens;
      int4* rec = (int4*)(a.tile_rec + (size_t)t * kTileRecWords);
      rec[0] = make_int4(b_s[lo], q0, qlen_s[lo], ctx_s[lo]);
      rec[1] = make_int4(qoff_s[lo], 0, blocks, -1);
      if (t < kSplitTiles) {
        tile_s[t] = make_int4(b_s[lo], q0, qlen_s[lo], ctx_s[lo]);
        tile_qoff_s[t] = qoff_s[lo];
        blocks_s[t] = blocks;
      }
    }
    __syncthreads();
    running += tile_total;
  }
  const int tiles = min(running, a.cap);
  if (tid == 0) {
    a.header[kPlanTiles] = tiles;
    a.header[kPlanMerges] = 0;
  }
  if (a.max_pieces == 0 || tiles == 0 || tiles > min(kSplitTiles, a.max_pieces)) return;

  // ---- pieces: 64 limits P tried side by side, four per wave.  Two barriers to here: every wave totals the whole list.
  __shared__ int pieces_s[64];
  const int lane = tid & 63, wave = tid >> 6;
  int blocks_total = 0;
  unsigned longest_seen = 0;
  for (int t = lane; t < tiles; t += 64) {
    blocks_total += blocks_s[t];
    longest_seen = max(longest_seen, (unsigned)blocks_s[t]);
  }
  blocks_total = wave_sum(blocks_total);
  const int longest = (int)wave_max(longest_seen);
  if (longest < 2 * kMinPieceBlocks) return;
  const float cus = (float)kNumCUs / (float)a.hkv;      // a list entry is one workgroup per KV head
  const float mean = fmaxf((float)blocks_total / cus, 1.f);
  auto limit_of = [&](int i) { return fmaxf((float)kMinPieceBlocks, ceilf(mean * (0.3f + 0.04f * (float)i))); };
  float per_limit[4];                                    // (a count off by one where the product rounds: the limits are checked again below)
  int pieces[4] = {0, 0, 0, 0};
#pragma unroll
  for (int c = 0; c < 4; ++c) per_limit[c] = __builtin_amdgcn_rcpf(limit_of(wave * 4 + c));
  for (int t = lane; t < tiles; t += 64) {
    const float n = (float)blocks_s[t];
#pragma unroll
    for (int c = 0; c < 4; ++c) pieces[c] += max(1, (int)ceilf(n * per_limit[c]));
  }
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const int n = wave_sum(pieces[c]);
    if (lane == 0) pieces_s[wave * 4 + c] = n;
  }
  __syncthreads();
  // prices as integers (a sixteenth of a block), complemented, so that the cheapest is the largest
  const int n_lane = pieces_s[lane];
  const float price_lane = split_price(limit_of(lane), (float)blocks_total, (float)n_lane, cus) + kMergeCost;
  const unsigned key = (n_lane > tiles && n_lane <= a.max_pieces) ? ~(unsigned)fminf(16.f * price_lane, 6e7f) : 0u;
  const unsigned cheapest = wave_max(key);
  const int at = __builtin_ctzll(__builtin_amdgcn_ballot_w64(key == cheapest));
  const float best = cheapest ? (float)~cheapest * (1.f / 16.f) : INFINITY;
  const float whole = split_price((float)longest, (float)blocks_total, (float)tiles, cus);
  if (!(best < 0.9f * whole)) return;                    // the same in every thread
  const int p_max = (int)limit_of(at);
  const int mine = tid < tiles ? blocks_s[tid] : 0;
  const int k = tid < tiles ? max(1, (mine + p_max - 1) / p_max) : 0;   // pieces of this thread's tile (one without blocks has zero rows to write)
  const bool cut = k > 1;
  // pieces and cut tiles in one scan: at most 2 * kSplitTiles of the first (the price counted them, give or take a rounding
  // per tile), kSplitTiles of the second
  int both;
  const int before = block_exclusive_scan(k | (cut ? 1 << 16 : 0), wave_tot, &both);
  const int piece0 = before & 0xffff, merge0 = before >> 16, n_pieces = both & 0xffff, n_merges = both >> 16;
  const int slot0 = piece0 - (tid - merge0), n_slots = n_pieces - (tiles - n_merges);   // every uncut tile is one piece without a slot
  if (n_pieces > a.max_pieces || n_slots > a.max_slots) return;
  if (cut) {
    int4* m = (int4*)(a.merge_rec + (size_t)merge0 * kTileRecWords);
    m[0] = make_int4(tile_s[tid].y, tile_s[tid].z, tile_qoff_s[tid], slot0);   // (first row, n_b, q_offsets[b], first slot, pieces)
    m[1] = make_int4(k, 0, 0, 0);
  }
  first_s[tid] = piece0;                                  // threads past the tiles hold n_pieces
  count_s[tid] = k;
  b_s[tid] = cut ? slot0 : -1;
  __syncthreads();
  for (int t = tid; t < n_pieces; t += kPlanThreads) {
    int lo = 0, hi = tiles;
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (first_s[mid] <= t) lo = mid; else hi = mid;
    }
    // a tile's blocks are dealt to its pieces as evenly as they go
    const int kk = count_s[lo], i = t - first_s[lo], n = blocks_s[lo];
    const int each = n / kk, more = n % kk;
    const int blk0 = each * i + min(i, more), blk1 = blk0 + each + (i < more ? 1 : 0);
    int4* rec = (int4*)(a.tile_rec + (size_t)t * kTileRecWords);
    rec[0] = tile_s[lo];
    rec[1] = make_int4(tile_qoff_s[lo], blk0, blk1 - blk0, b_s[lo] < 0 ? -1 : b_s[lo] + i);
  }
  if (tid == 0) {
    a.header[kPlanTiles] = n_pieces;
    a.header[kPlanMerges] = n_merges;
  }
}

__global__ __launch_bounds__(kPlanThreads) void plan_append_kernel(const AppendPlanArgs a) {
  plan_append(a, ChunkLens{a.ctx_lens, a.q_lens, a.q_offsets});
}

// Both plans of a mixed step side by side.
__global__ __launch_bounds__(kPlanThreads) void plan_step_kernel(const AppendPlanArgs a, const DecodePlanArgs d) {
  if (blockIdx.x == 0) plan_append(a, ChunkLens{a.ctx_lens, a.q_lens, a.q_offsets});
  else plan_decode(d);
}

// Decode of groups that share a prompt: per group the shared length actually used, S = floor32(min(shared_lens[group],
// min over the group of L_b - 1)), so that every trajectory keeps at least its current token for itself and the private
// part starts on a block boundary.  One workgroup plans the shared half (a chunk per group, its members' query rows, over
// the group's first S tokens), the other one the private half (every trajectory from token S on), whose lengths and
// first table entries it writes out for the decode kernel.  Each works S out for itself: a launch that did, and
// copied the table shifted by S, took 5 us, and the plans one after the other 12 where this launch takes 8 (64 groups of 8).
constexpr int kSharedGroups = 2048;   // up to this many groups their lengths are settled in LDS

__global__ __launch_bounds__(kPlanThreads) void plan_shared_kernel(const SharedPlanArgs sh, const AppendPlanArgs a, const DecodePlanArgs d) {
  __shared__ int used_s[kSharedGroups];
  const int groups = sh.batch / sh.group_size;
  const bool in_lds = groups <= kSharedGroups;
  if (in_lds) {
    for (int g = threadIdx.x; g < groups; g += kPlanThreads) used_s[g] = max(0, sh.shared_lens[g]);
    __syncthreads();
    for (int b = threadIdx.x; b < sh.batch; b += kPlanThreads) atomicMin(&used_s[b / sh.group_size], max(0, sh.ctx_lens[b] - 1));
    __syncthreads();
  }
  auto used = [&](int g) -> int {
    int s;
    if (in_lds) {
      s = used_s[g];
    } else {
      s = sh.shared_lens[g];
      for (int m = 0; m < sh.group_size; ++m) s = min(s, sh.ctx_lens[(size_t)g * sh.group_size + m] - 1);
      s = max(s, 0);
    }
    return s & ~(kBlockTokens - 1);
  };
  if (blockIdx.x == 0) {
    struct Groups {
      decltype(used)& len;
      int size;
      __device__ __forceinline__ int ctx(int g) const { return len(g); }
      __device__ __forceinline__ int rows(int) const { return size; }
      __device__ __forceinline__ int offset(int g) const { return g * size; }
    };
    plan_append(a, Groups{used, sh.group_size});
  } else {
    for (int b = threadIdx.x; b < sh.batch; b += kPlanThreads) {
      const int s = used(b / sh.group_size);
      sh.own_ctx[b] = sh.ctx_lens[b] - s;
      sh.own_page[b] = s / kPageSize;
    }
    plan_decode(d, [&](int b) { return sh.ctx_lens[b] - used(b / sh.group_size); });
  }
}

}  // namespace

hipError_t launch_plan_decode(const DecodePlanArgs& d, hipStream_t s) {
  hipLaunchKernelGGL(plan_decode_kernel, dim3(1), dim3(kPlanThreads), 0, s, d);
  return hipGetLastError();
}

hipError_t launch_plan_append(const AppendPlanArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(plan_append_kernel, dim3(1), dim3(kPlanThreads), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_plan_step(const AppendPlanArgs& a, const DecodePlanArgs& d, hipStream_t s) {
  hipLaunchKernelGGL(plan_step_kernel, dim3(2), dim3(kPlanThreads), 0, s, a, d);
  return hipGetLastError();
}

hipError_t launch_plan_shared(const SharedPlanArgs& sh, const AppendPlanArgs& a, const DecodePlanArgs& d, hipStream_t s) {
  hipLaunchKernelGGL(plan_shared_kernel, dim3(2), dim3(kPlanThreads), 0, s, sh, a, d);
  return hipGetLastError();
}

}  // namespace rollattn
