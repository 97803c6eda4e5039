// Device-side planning: turns ctx_lens / q_lens into compact work lists without a host
// round trip, so a call never synchronises.  The partition depends on the lengths only,
// never on physical page ids (which only say how the decode kernel's loads treat the caches).
#include "plan_device.h"

namespace rollattn {

namespace {

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

// With q_lens given (mixed step) only the trajectories with q_lens[b] == 1 take part; the others count as empty.
__device__ __forceinline__ int decode_len(const DecodePlanArgs& a, int b) { return (!a.q_lens || a.q_lens[b] == 1) ? a.ctx_lens[b] : 0; }
__device__ __forceinline__ void plan_decode(const DecodePlanArgs& a, DecodePlanLds& lds) {
  plan_decode(a, lds, [&](int b) { return decode_len(a, b); });
}

// Whether the pages of this call are read by several workers.  Trajectories that share a prefix of their contexts have its
// pages in common (grouped rollouts, a system prompt in front of all of them), wherever they stand in the batch.  Told by the
// second page (a single shared page is not worth it): equal ids meet in a hash table in LDS.  The call's pages count as read
// again where the trajectories that have met have a quarter of all blocks: with so many in groups of 8 that share nine tenths
// the hint still takes 0.91 to 0.99 of the plain loads' time (256 contexts of 8k over FP8 pools 290 against 317 us, 72 over
// bf16 384 against 389), with half of them 0.97 to 1.04, with all 1.09 to 1.64 (bf16, 256 of 4k: 459 against 282 us).
// A workgroup of its own beside the plan's: both wait for the lengths, and this one then for the tables (in one workgroup
// the plan of 200 trajectories took 2 us longer).
struct ReadAgainLds {
  int key[2 * kLdsPrefix], blocks[2 * kLdsPrefix];   // twice as many slots as trajectories, or more
  unsigned int twice[2 * kLdsPrefix / 32];
  int sum[2];
};
// len_of(b): tokens of trajectory b that take part; second_page(b): entry of the second page of those.
template <class L, class P>
__device__ __forceinline__ void plan_read_again(const DecodePlanArgs& a, ReadAgainLds& lds, L&& len_of, P&& second_page) {
  const int tid = threadIdx.x;
  if (a.head_tiles || a.batch > kLdsPrefix) {
    if (tid == 0) a.header[kPlanReadAgain] = 1;
    return;
  }
  const int mask = (1 << (32 - __builtin_clz(2 * max(a.batch, 16) - 1))) - 1;
  for (int i = tid; i <= mask; i += kPlanThreads) {
    lds.key[i] = -1;
    lds.blocks[i] = 0;
  }
  for (int i = tid; i <= mask / 32; i += kPlanThreads) lds.twice[i] = 0;
  if (tid < 2) lds.sum[tid] = 0;
  __syncthreads();
  int all = 0, met = 0;
  for (int b = tid; b < a.batch; b += kPlanThreads) {
    const int len = len_of(b), blocks = (len + kBlockTokens - 1) / kBlockTokens;
    all += blocks;
    const int page = len > kPageSize ? a.page_table[(size_t)b * a.max_pages + second_page(b)] : -1;
    if (page < 0) continue;
    int h = (int)(((unsigned int)page * 0x9e3779b1u) >> 15) & mask;
    for (;; h = (h + 1) & mask) {                      // (a free slot is always found)
      const int before = atomicCAS(&lds.key[h], -1, page);
      if (before == page) atomicOr(&lds.twice[h / 32], 1u << (h % 32));
      if (before == -1 || before == page) break;
    }
    atomicAdd(&lds.blocks[h], blocks);
  }
  __syncthreads();
  for (int i = tid; i <= mask; i += kPlanThreads) met += (lds.twice[i / 32] >> (i % 32) & 1) ? lds.blocks[i] : 0;
  all = wave_sum(all);
  met = wave_sum(met);
  if ((tid & 63) == 0) {
    atomicAdd(&lds.sum[0], all);
    atomicAdd(&lds.sum[1], met);
  }
  __syncthreads();
  if (tid == 0) a.header[kPlanReadAgain] = all_read_again(a, lds.sum[0]) || (long)lds.sum[1] * 4 >= max(lds.sum[0], 1);
}

__device__ __forceinline__ void plan_read_again(const DecodePlanArgs& a, ReadAgainLds& lds) {
  plan_read_again(a, lds, [&](int b) { return decode_len(a, b); }, [](int) { return 1; });
}

// Whole rows (kPlanWhole).  A run that starts or ends inside a row leaves a float partial to be written, read and folded: of 16
// query heads per KV head, twice that is four blocks of FP8 codes or two of bf16 values.  Instead every row may be taken whole,
// by one wave (the records then only tell what the runs would have been).  What that costs is that long rows go on by themselves
// when the others have ended: memory is busy with about `whole_busy` waves, and every block that fewer are left for costs a
// wave's own time, 0.6 us or so at D = 128.  So rows stay whole where
//   sum over i = 1 .. longest of max(0, 1 - n_i / busy)  -  the same of the runs  <=  1.2 + cuts * whole_gain (+ 4),
// n_i: rows of i blocks or more, as a share of the waves where there are more rows than those (the longest could come
// last; 4 because their sums even out and neighbours read neighbouring pages); 1.2: a merge that finds nothing to do; cuts:
// boundaries of runs that fall inside rows.  n_i is counted at 32 lengths.  busy, 900 waves over FP8 pools and 450 over bf16 pools, whose blocks are twice the
// bytes, and whole_gain, a block's time for 130 cuts of 16 heads of 128, are fitted to 250 calls of 65 to 200000 contexts of 1
// to 8 KV heads, uniform, lognormal, of two lengths, and short ones with one or four long ones among them.  Over these the
// choice takes 0.7 % more than the better of the two on average, and never more than 1 % where it is whole rows.  (The longest
// row's lateness alone, up to 16 blocks or 10, let one row of 17 blocks decide for 520 of one: 12.9 -> 29.8 us.)
// us per call, runs against whole rows, the choice first; 16 query heads per KV head over FP8 pools, 4 over bf16 pools, D = 128,
// contexts uniform in the range:
//   FP8, 512 x 4 KV heads: 256-512 whole 50.3, 63.4; 64-1024 whole 67.3, 80.7; 1024-2048 whole 145, 169; 512-4096 runs 239, 233
//   FP8, 512 x 4, 256 and one of 800: runs 50.2, 47.5; 210 x 4: 33-64 whole 15.6, 23.3; 64-1024 runs 42.4, 46.8; 512-4096 runs 106, 142
//   FP8, 65 x 1, 256-512: runs 15.9, 22.2; 65 x 8 (4 heads each), 32 and one of 544: runs 13.3, 23.5
//   bf16, 256 x 8: 256-512 whole 72.7, 79.2; 1024-2048 whole 265, 270; 512-4096 runs 396, 424; 512 x 8: 256-512 whole 138, 151
//   bf16, 128 x 8: 64-1024 runs 58.6, 59.1; 65 x 1 (16 heads), 256-320: runs 15.6, 17.6
// Not for batches that the decode waves plan for themselves, nor for a mixed step with as few decode rows, so that a
// step's rows are bit for bit those of a call of their own.  A workgroup of its own, like the look at the pages.
constexpr int kWholeLevels = 32;
struct WholeLds {
  int4 of_wave[kPlanThreads / 64];
  int at_least[kWholeLevels];
};
template <class L>
__device__ __forceinline__ void plan_whole(const DecodePlanArgs& a, WholeLds& lds, L&& len_of) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (tid < kWholeLevels) lds.at_least[tid] = 0;
  auto blocks_of = [&](int b) { return b < a.batch ? (len_of(b) + kBlockTokens - 1) / kBlockTokens : 0; };
  const int mine = blocks_of(tid);
  int blocks = 0, longest = 0, part = 0, live = 0;
  for (int b = tid; b < a.batch; b += kPlanThreads) {
    const int n = b == tid ? mine : blocks_of(b);
    blocks += n;
    longest = max(longest, n);
    part += !a.q_lens || a.q_lens[b] == 1;
    live += n > 0;
  }
  blocks = wave_sum(blocks);
  longest = (int)wave_max((unsigned)longest);
  part = wave_sum(part);
  live = wave_sum(live);
  if (lane == 0) lds.of_wave[wave] = make_int4(blocks, longest, part, live);
  __syncthreads();
  blocks = longest = part = live = 0;
  for (int w = 0; w < kPlanThreads / 64; ++w) {
    const int4 x = lds.of_wave[w];
    blocks += x.x;
    longest = max(longest, x.y);
    part += x.z;
    live += x.w;
  }
  if (part <= kWavePlanBatch || longest == 0) {
    if (tid == 0) a.header[kPlanWhole] = 0;
    return;
  }
  // level j stands for the lengths (j * step, (j + 1) * step]
  const int step = (longest + kWholeLevels - 1) / kWholeLevels;
  int at_least = 0;                                    // of level `lane`
  for (int b0 = wave * 64; b0 < a.batch; b0 += kPlanThreads) {
    const int n = b0 == wave * 64 ? mine : blocks_of(b0 + lane);
    int level = (step - 1) / 2;
#pragma unroll 4
    for (int j = 0; j < kWholeLevels; ++j, level += step) {
      const int hits = __builtin_popcountll(__builtin_amdgcn_ballot_w64(n > level));
      at_least += lane == j ? hits : 0;
    }
  }
  if (lane < kWholeLevels && at_least) atomicAdd(&lds.at_least[lane], at_least);
  __syncthreads();
  if (wave != 0) return;
  const float rows = (float)live * (float)a.rows_per_b, workers = (float)a.workers;
  const float share = rows > workers ? workers / rows : 1.f;
  auto idle = [&](float n) { return fmaxf(0.f, 1.f - n / a.whole_busy); };
  float late = 0.f;
  if (lane < kWholeLevels) late = (float)max(0, min(step, longest - lane * step)) * idle((float)lds.at_least[lane] * (float)a.rows_per_b * share);
#pragma unroll
  for (int i = 1; i < kWholeLevels; i *= 2) late += __shfl_xor(late, i);
  const int total = blocks * a.rows_per_b, per = max(1, (total + a.workers - 1) / a.workers), used = (total + per - 1) / per;
  const float cuts = (float)(used - 1) * (1.f - rows / (float)total);
  if (lane == 0) a.header[kPlanWhole] = late - (float)per * idle((float)used) <= 1.2f + cuts * a.whole_gain + (rows > workers ? 4.f : 0.f);
}

union DecodeLds {
  DecodePlanLds plan;
  ReadAgainLds pages;
  WholeLds whole;
};

// The second workgroup looks at the pages and the third decides on whole rows, where there are such.
__global__ __launch_bounds__(kPlanThreads) void plan_decode_kernel(const DecodePlanArgs a) {
  __shared__ DecodeLds lds;
  if (blockIdx.x == 0) plan_decode(a, lds.plan);
  else if (blockIdx.x == 1) plan_read_again(a, lds.pages);
  else plan_whole(a, lds.whole, [&](int b) { return decode_len(a, b); });
}

// Append work list: each chunk cut into tiles of tile_tokens query tokens.  A tile's cost grows
// with its trajectory's context, and workgroups are dispatched in list order, so (for batches that
// fit the ranking in LDS) trajectories are listed longest context first: the long tiles start
// early and the short ones fill the tail.  For the same reason a chunk's tiles are listed last
// tile first.
//
// Pieces.  A tile walks its visible context block by block, so a call ends no earlier than its longest tile, however
// many CUs have nothing to do: a few observations behind long prefixes, or one 64k history among short ones, leave
// most of the chip idle.  When the list is short enough to be looked at as a whole (kSplitTiles), the kernel asks
// whether cutting the tiles into pieces of at most P blocks would end sooner: 63 values of P around the mean
// load of a CU are tried side by side, each priced in us as
//   m (alone + (full - alone) (load / m)^3),   m = max(P + start, load + u (P + start) (ceil(w) - w)),
//   w = pieces / CUs, load = (blocks + start pieces) / CUs, u = mean piece / P:
// m is the length in blocks: with equal pieces the number of full rounds over the CUs, with unequal ones the later, shorter
// pieces fill the gaps.  A block's time grows with the share of the CUs that are busy (memory, power), from `alone` to
// `full`, which the host passes for the kernel that will run: 1.05 and 1.75 us for whole tiles of bf16 at D = 128, 0.76 and
// 1.42 for half tiles, where it is memory that a full chip waits for and cutting gains nothing any more.  start: what a
// workgroup costs besides its blocks (kPieceUs).  Cutting adds the partials' way to memory and back (us_per_unit) and the
// folding.  It is done where that is a twentieth and 1.5 us shorter, fixed costs of the call (kCallUs) included.  Limits whose pieces or
// partials there is no room for are left out (13 chunks of 64 tokens behind 16k, 32/8/128, bf16: the cheapest would need 91
// pieces of 256 rows per head), and those of more than two rounds above the tiles, so that the launch need not have room
// for them: an empty workgroup waits for a CU's LDS like any other.
// Against the times of 193 calls, whole and cut, the price is off by 6 and 8 % (standard deviation).
// Measured: three observations of 16 .. 512 tokens behind 2k .. 16k (32/8/128, bf16, one of every four CUs idle before)
// 275 -> 207 us with plan and merge; 33 of 3 .. 96 tokens behind up to 64k (64/4/128, FP8) 1410 -> 650 us; 13 of 64 behind
// 12k 281 -> 215 us.  40 chunks of 2 tokens behind 9000 (64/4/128, bf16) read at the memory's rate as they are, 135 us, and
// stay whole; cut they took 152.  What the offer costs a call that stays whole: 1 us of plan where the list is priced, and
// the start of a merge launch that finds nothing to do, 1.7 us.  The host makes none of it where the table is too narrow for
// a context that could be cut, or the list too long.
constexpr int kRankBatch = 4096;
constexpr int kSplitTiles = kSplitPieces;
static_assert(kSplitTiles <= kPlanThreads, "a thread per tile");

constexpr int kMaxCutBlocks = 1 << 19;   // 33 million tokens

struct SplitPrice {
  float alone, full, per_cu, start;                      // per_cu: list entries (one workgroup per KV head) that a CU gets of each
  __device__ SplitPrice(const AppendPlanArgs& a) : alone(a.us_alone), full(a.us_full), per_cu((float)a.hkv * (1.f / kNumCUs)), start(kPieceUs * __builtin_amdgcn_rcpf(a.us_full)) {}
  __device__ __forceinline__ float operator()(float p, float blocks, float pieces) const {
    const float w = pieces * per_cu, load = (blocks + start * pieces) * per_cu;
    const float u = fminf(1.f, blocks * __builtin_amdgcn_rcpf(pieces * p));
    const float m = fmaxf(p + start, load + u * (p + start) * (ceilf(w) - w));
    const float busy = load * __builtin_amdgcn_rcpf(m);
    return m * (alone + (full - alone) * busy * busy * busy);
  }
};

// What the append plan asks about a chunk: its context, its rows, where they start in the packed query.
struct ChunkLens {
  const int32_t *ctx_lens, *q_lens, *q_offsets;
  __device__ __forceinline__ int ctx(int b) const { return ctx_lens[b]; }
  __device__ __forceinline__ int rows(int b) const { return q_lens[b]; }
  __device__ __forceinline__ int offset(int b) const { return q_offsets[b]; }
};

struct AppendPlanLds {
  int4 wave_tot[kPlanThreads / 256];
  int4 tile_s[kSplitTiles];            // the first kSplitTiles tiles of the list, for the decision about pieces: record ...
  int len_s[kRankBatch], order_s[kRankBatch];
  int2 chunk_s[kRankBatch];            // rows and offset of a chunk
  int first_s[kPlanThreads], count_s[kPlanThreads], b_s[kPlanThreads], qlen_s[kPlanThreads], ctx_s[kPlanThreads], qoff_s[kPlanThreads];
  int tile_qoff_s[kSplitTiles], blocks_s[kSplitTiles], units_s[kSplitTiles];   // ... number of blocks, units of rows
  int pieces_s[64], merges_s[64], piece_units_s[64];
};

template <class C>
__device__ __forceinline__ void plan_append(const AppendPlanArgs& a, AppendPlanLds& lds, const C& chunk) {
  auto& [wave_tot, tile_s, len_s, order_s, chunk_s, first_s, count_s, b_s, qlen_s, ctx_s, qoff_s, tile_qoff_s, blocks_s, units_s, pieces_s, merges_s,
         piece_units_s] = lds;
  const int tid = threadIdx.x;
  const int batch = a.batch, tile_tokens = a.tile_tokens;
  const bool ranked = batch <= kRankBatch;
  if (ranked) {
    // everything the plan reads, in one round trip to memory
    const int padded = (batch + 3) & ~3;
    for (int b = tid; b < padded; b += kPlanThreads) {
      len_s[b] = b < batch ? chunk.ctx(b) : INT32_MIN;   // (the padding ranks behind everything)
      if (b < batch) chunk_s[b] = make_int2(chunk.rows(b), chunk.offset(b));
    }
    __syncthreads();
    for (int b = tid; b < batch; b += kPlanThreads) {
      const int mine = len_s[b];
      int rank = 0;
      for (int o = 0; o < padded; o += 4) {
        const int4 other = *(const int4*)(len_s + o);
        rank += (other.x > mine || (other.x == mine && o < b)) ? 1 : 0;
        rank += (other.y > mine || (other.y == mine && o + 1 < b)) ? 1 : 0;
        rank += (other.z > mine || (other.z == mine && o + 2 < b)) ? 1 : 0;
        rank += (other.w > mine || (other.w == mine && o + 3 < b)) ? 1 : 0;
      }
      order_s[rank] = b;
    }
    __syncthreads();
  }
  int running = 0;
  for (int p0 = 0; p0 < batch; p0 += kPlanThreads) {
    const int p = p0 + tid;
    int b = 0, count = 0, q_len = 0, q_off = 0, ctx = 0;
    if (p < batch) {
      b = ranked ? order_s[p] : p;
      q_len = ranked ? chunk_s[b].x : chunk.rows(b);
      q_off = ranked ? chunk_s[b].y : chunk.offset(b);
      ctx = ranked ? len_s[b] : chunk.ctx(b);
      count = (q_len + tile_tokens - 1) / tile_tokens;
      if (a.skip_unit_chunks && q_len == 1) count = 0;   // mixed step: the decode kernel takes these
    }
    int tile_total;
    const int first = running + block_exclusive_scan(count, wave_tot, &tile_total);
    first_s[tid] = first;
    count_s[tid] = count;
    b_s[tid] = b;
    qlen_s[tid] = q_len;
    ctx_s[tid] = ctx;
    qoff_s[tid] = q_off;
    __syncthreads();
    // One 32-byte record per tile with everything the tile's workgroup needs to start, so that it gets there with
    // one dependent load instead of a chain of them: (b, first row, n_b, L_b, q_offsets[b], first block, blocks, unit).
    // The tiles of these trajectories are dealt to the threads one by one (a trajectory may have hundreds): a tile
    // finds its trajectory as the last one of the group that starts at or before it (those without tiles start where
    // the next one starts, and are never the last such).
    const int end = min(running + tile_total, a.cap);
    for (int t = running + tid; t < end; t += kPlanThreads) {
      int lo = 0, hi = min(kPlanThreads, batch - p0);
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
      if (a.max_pieces && t < kSplitTiles) {
        tile_s[t] = make_int4(b_s[lo], q0, qlen_s[lo], ctx_s[lo]);
        tile_qoff_s[t] = qoff_s[lo];
        blocks_s[t] = blocks;
        units_s[t] = (min(tile_tokens, qlen_s[lo] - q0) * a.group + kUnitRows - 1) / kUnitRows;
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

  // ---- pieces.  Two barriers to the decision: every wave totals the whole list; then a lane per limit P, the tiles dealt
  // to the waves.  (Code that runs once costs its fetch: this is kept short.)
  const int lane = tid & 63, wave = tid >> 6;
  int blocks_total = 0;
  unsigned longest_seen = 0;
  for (int t = lane; t < tiles; t += 64) {
    blocks_total += blocks_s[t];
    longest_seen = max(longest_seen, (unsigned)blocks_s[t]);
  }
  const int longest = (int)wave_max(longest_seen);
  if (longest < a.min_longest || longest >= kMaxCutBlocks) return;
  if (wave == 0) pieces_s[lane] = merges_s[lane] = piece_units_s[lane] = 0;
  __syncthreads();
  blocks_total = wave_sum(blocks_total);
  const SplitPrice price(a);
  const float limit = fmaxf((float)kMinPieceBlocks, ceilf((float)blocks_total * price.per_cu * (0.3f + 0.04f * (float)lane)));
  const float per_limit = __builtin_amdgcn_rcpf(limit), below = limit - 0.5f;
  int pieces = 0, merges = 0, units = 0;
  for (int t = wave; t < tiles; t += kPlanThreads / 64) {
    // n / p rounded up, exactly: (n + p - 1/2) / p lies half a block away from every whole number, more than its rounding
    // below kMaxCutBlocks
    const int k = max(1, (int)(((float)blocks_s[t] + below) * per_limit));
    pieces += k;
    merges += k > 1 ? 1 : 0;
    units += k > 1 ? k * units_s[t] : 0;
  }
  atomicAdd(&pieces_s[lane], pieces);
  atomicAdd(&merges_s[lane], merges);
  atomicAdd(&piece_units_s[lane], units);
  __syncthreads();
  pieces = pieces_s[lane];
  merges = merges_s[lane];
  units = piece_units_s[lane];
  // prices as integers (a sixteenth of a us), complemented, so that the cheapest is the largest; the last lane prices the
  // whole tiles
  const float cost = price(lane == 63 ? (float)longest : limit, (float)blocks_total, (float)(lane == 63 ? tiles : pieces)) + kCallUs +
                     (lane == 63 ? 0.f : kMergeUs + a.us_per_unit * (float)units * (float)a.hkv);
  const unsigned ticks = (unsigned)fminf(16.f * cost, 6e7f);
  const bool fits = lane != 63 && pieces > tiles && pieces <= min(a.max_pieces, tiles + split_extra_pieces(a.hkv)) && merges <= a.max_merges && units <= a.max_units;
  const unsigned key = fits ? ~ticks : 0u;
  const unsigned cheapest = wave_max(key);
  const unsigned whole = (unsigned)__builtin_amdgcn_readlane((int)ticks, 63);
  if (cheapest == 0u || !((float)~cheapest < kSplitGain * (float)whole - 16.f * kSplitGainUs)) return;   // the same in every thread
  const int at = __builtin_ctzll(__builtin_amdgcn_ballot_w64(key == cheapest));
  const int p_max = __builtin_amdgcn_readlane((int)limit, at);
  const int mine = tid < tiles ? blocks_s[tid] : 0;
  const int k = tid < tiles ? max(1, (mine + p_max - 1) / p_max) : 0;   // pieces of this thread's tile (one without blocks has zero rows to write)
  const bool cut = k > 1;
  // pieces, cut tiles and units of partials in one scan: 10, 9 and 12 bits
  static_assert(kSplitPieces < 1024 && kSplitMerges < 512 && kSplitUnits <= 4096, "one scan");
  const int my_units = cut ? units_s[tid] : 0;
  int all;
  const int before = block_exclusive_scan(k | (cut ? 1 << 10 : 0) | (k * my_units) << 19, wave_tot, &all);
  const int piece0 = before & 1023, merge0 = (before >> 10) & 511, unit0 = (int)((unsigned)before >> 19), n_pieces = all & 1023, n_merges = (all >> 10) & 511;
  if (cut) {
    int4* m = (int4*)(a.merge_rec + (size_t)merge0 * kTileRecWords);
    m[0] = make_int4(tile_s[tid].y, tile_s[tid].z, tile_qoff_s[tid], unit0);   // (first row, n_b, q_offsets[b], first unit, pieces)
    m[1] = make_int4(k, 0, 0, 0);
  }
  first_s[tid] = piece0;                                  // threads past the tiles hold n_pieces
  count_s[tid] = k;
  b_s[tid] = cut ? unit0 : -1;
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
    rec[1] = make_int4(tile_qoff_s[lo], blk0, blk1 - blk0, b_s[lo] < 0 ? -1 : b_s[lo] + i * units_s[lo]);
  }
  if (tid == 0) {
    a.header[kPlanTiles] = n_pieces;
    a.header[kPlanMerges] = n_merges;
  }
}

__global__ __launch_bounds__(kPlanThreads) void plan_append_kernel(const AppendPlanArgs a) {
  __shared__ AppendPlanLds lds;
  plan_append(a, lds, ChunkLens{a.ctx_lens, a.q_lens, a.q_offsets});
}

// Plans side by side, a workgroup each.
union PlanLds {
  AppendPlanLds append;
  DecodeLds decode;
  __device__ PlanLds() {}
};

// Both plans of a mixed step, its decode rows' pages, and whether they stay whole.
__global__ __launch_bounds__(kPlanThreads) void plan_step_kernel(const AppendPlanArgs a, const DecodePlanArgs d) {
  __shared__ PlanLds lds;
  if (blockIdx.x == 0) plan_append(a, lds.append, ChunkLens{a.ctx_lens, a.q_lens, a.q_offsets});
  else if (blockIdx.x == 1) plan_decode(d, lds.decode.plan);
  else if (blockIdx.x == 2) plan_read_again(d, lds.decode.pages);
  else plan_whole(d, lds.decode.whole, [&](int b) { return decode_len(d, b); });
}

// Decode of groups that share a prompt: per group the shared length actually used, S = floor32(min(shared_lens[group],
// min over the group of L_b - 1)), so that every trajectory keeps at least its current token for itself and the private
// part starts on a block boundary.  One workgroup plans the shared half (a chunk per group, its members' query rows, over
// the group's first S tokens), another one the private half (every trajectory from token S on), whose lengths and
// first table entries it writes out for the decode kernel, a third looks at the private half's pages, a
// fourth decides on whole rows.  Each works S out for itself: a launch that did, and
// copied the table shifted by S, took 5 us, and the plans one after the other 12 where this launch takes 8 (64 groups of 8).
constexpr int kSharedGroups = 4096;   // up to this many groups their lengths are settled in LDS

__global__ __launch_bounds__(kPlanThreads) void plan_shared_kernel(const SharedPlanArgs sh, const AppendPlanArgs a, const DecodePlanArgs d) {
  __shared__ PlanLds lds;
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
  auto own_len = [&](int b) { return sh.ctx_lens[b] - used(b / sh.group_size); };
  if (blockIdx.x == 0) {
    struct Groups {
      decltype(used)& len;
      int size;
      __device__ __forceinline__ int ctx(int g) const { return len(g); }
      __device__ __forceinline__ int rows(int) const { return size; }
      __device__ __forceinline__ int offset(int g) const { return g * size; }
    };
    plan_append(a, lds.append, Groups{used, sh.group_size});
  } else if (blockIdx.x == 2) {
    // (the private parts have pages in common where a short member leaves some of the prompt to the others, or where the
    // caller says less than there is)
    plan_read_again(d, lds.decode.pages, own_len, [&](int b) { return used(b / sh.group_size) / kPageSize + 1; });
  } else if (blockIdx.x == 3) {
    plan_whole(d, lds.decode.whole, own_len);
  } else {
    for (int b = threadIdx.x; b < sh.batch; b += kPlanThreads) {
      const int s = used(b / sh.group_size);
      sh.own_ctx[b] = sh.ctx_lens[b] - s;
      sh.own_page[b] = s / kPageSize;
    }
    plan_decode(d, lds.decode.plan, own_len);
  }
}

}  // namespace

hipError_t launch_plan_decode(const DecodePlanArgs& d, hipStream_t s) {
  hipLaunchKernelGGL(plan_decode_kernel, dim3(d.page_table ? 3 : 1), dim3(kPlanThreads), 0, s, d);
  return hipGetLastError();
}

hipError_t launch_plan_append(const AppendPlanArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(plan_append_kernel, dim3(1), dim3(kPlanThreads), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_plan_step(const AppendPlanArgs& a, const DecodePlanArgs& d, hipStream_t s) {
  hipLaunchKernelGGL(plan_step_kernel, dim3(4), dim3(kPlanThreads), 0, s, a, d);
  return hipGetLastError();
}

hipError_t launch_plan_shared(const SharedPlanArgs& sh, const AppendPlanArgs& a, const DecodePlanArgs& d, hipStream_t s) {
  hipLaunchKernelGGL(plan_shared_kernel, dim3(4), dim3(kPlanThreads), 0, s, sh, a, d);
  return hipGetLastError();
}

}  // namespace rollattn
