// Internal declarations shared by the host entry points and the HIP kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "rollattn.h"

namespace rollattn {

constexpr int kPageSize = 16;
constexpr int kNumCUs = 256;            // MI355X
constexpr int kBlockTokens = 32;        // unit of the decode partition: two pages
constexpr int kMfmaDecodeWgs = 2 * kNumCUs;   // 4 wave-workers each
constexpr int kMfmaHeadTile = 16;       // query heads per MFMA decode row
constexpr int kF32DecodeWgs = 4 * kNumCUs;    // one workgroup-worker each
constexpr int kF32HeadTile = 4;         // query heads per float32 decode row
constexpr int kWavePlanBatch = 64;      // batches up to this size are planned by every decode wave for itself
constexpr float kWholeBusyFp8 = 900.f, kWholeBusy = 450.f, kWholeGain = 1.f / 130;   // MFMA decode: what rows that stay whole are priced with (plan_whole)
constexpr int kMfmaDecodeWgsD64 = 3 * kNumCUs;   // MFMA decode, D = 64: workgroups that run at once, all of them where rows stay whole
constexpr int kDirectPages = 32;        // float32 contexts of at most this many pages are not cut
constexpr int kAppendTileRows = 256;    // query rows (token, head-in-group pairs) per append workgroup
constexpr int kXcds = 8;                // accelerator dies, each with its own L2; workgroups are dealt to them round-robin
constexpr int kAppendBlockTokens = 64;  // KV tokens staged per step of the append kernel
constexpr int kTileRecWords = 8;       // append: int32 per tile record (32 bytes: one scalar load)
constexpr int kSplitPieces = 768;       // append: a list whose tiles are cut into pieces has at most this many workgroups
constexpr int kSplitMerges = 256;       // append: ... from at most this many tiles
constexpr int kSplitUnits = 4096;       // append: ... whose pieces leave at most this many partials of kUnitRows rows each,
constexpr int kLentUnits = 2048;        // ... or as many as there is room for decode partials, where the workspace has no more
constexpr int kUnitRows = 32;           // append: query rows per wave, and per unit of the partials of a tile's piece
constexpr int kMinPieceBlocks = 8;      // append: shorter pieces cost more in their start and end than they save
constexpr float kPieceUs = 8.f;         // append, price of a cut in us: what a workgroup costs besides its blocks,
constexpr float kMergeUs = 2.f;         // ... folding pieces, besides the way of the partials,
constexpr float kCallUs = 7.f;          // ... the rest of the call;
constexpr float kSplitGain = 0.95f, kSplitGainUs = 1.5f;   // ... a list is cut where that ends the call sooner by both shares
constexpr int split_extra_pieces(int hkv) { return 2 * kNumCUs / hkv; }   // append: cutting makes a list at most this much longer (two rounds)
constexpr int kAppendXcdRun = 16;       // append: consecutive tiles of the list that one XCD takes in a row (one per CU)

// Header words of the plan, at the start of the workspace.
enum PlanWord { kPlanPer = 0, kPlanTotal = 1, kPlanWorkers = 2, kPlanRowsPerB = 3, kPlanTiles = 4, kPlanMerges = 5, kPlanWhole = 6,
                kPlanReadAgain = 32,   // (this word and kPlanWhole are each written by another workgroup than the rest)
                kPlanWords = 64 };

// Byte offsets of the workspace regions (all multiples of 256).
struct WorkspaceLayout {
  int32_t workers;        // decode: number of workers W; append: capacity in query tiles
  int32_t max_pieces, max_merges, max_units;   // append: limits per KV head of a list whose tiles are cut (0: none can be)
  int32_t head_tile;      // decode: query heads per row (16 or 4)
  int32_t rows_per_b;     // decode: rows per trajectory = Hkv * ceil(G / head_tile)
  size_t header;          // int32[kPlanWords]
  size_t prefix;          // decode: int32[B + 1] exclusive scan of per-trajectory block counts
  size_t wstart;          // decode: int32[W][4] first (b, row, block) of every worker; append: int32[workers][8] tile records
  size_t merge_rec;       // append: int32[max_merges][8], one record per tile that was cut into pieces
  size_t partial_ml;      // float[2 W][head_tile][2]   (max in log2 units, sum); append: float[max_units][Hkv][32][2]
  size_t partial_o;       // float[2 W][head_tile][D]   un-normalised; append: float[max_units][Hkv][D / 8][64][4], as the accumulators lie
  size_t total;           // what the call needs
  // append: what it needs to cut tiles, without the partials and with them.  The list of a call that cuts is short, so
  // merge_rec and the partials lie where a long list's tail would.
  size_t cut_list, cut_total;
};

WorkspaceLayout decode_layout(const rollattn_desc& d);
WorkspaceLayout append_layout(const rollattn_desc& d, int32_t total_q, int32_t units = kSplitUnits);

// Inputs and outputs of the decode partition.
struct DecodePlanArgs {
  const int32_t* ctx_lens;
  const int32_t* q_lens;           // mixed step, else null
  int32_t batch, rows_per_b;
  int32_t workers, slots;          // how many the partition is cut for; records written (those past `workers` say "no blocks")
  // What tells whether pages are read by several workers (kPlanReadAgain); page_table null: nobody asks.
  const int32_t* page_table;
  int64_t num_pages;
  int32_t max_pages;
  bool head_tiles;                 // several rows per KV head: each reads its K and V
  float whole_busy, whole_gain;    // whether rows stay whole: waves that keep memory busy; blocks' time that a cut is worth
  int32_t* header;
  int32_t* prefix;
  int32_t* wstart;
};

// The shared half's result, which the private half's rows are folded into (attn_decode_shared; all null otherwise).
struct SharedHalf {
  const void* out;      // bf16 [B][Hq][D], normalised
  const float* lse;     // [B][Hq]
  void* result;         // where the whole rows go
};

// Kernel arguments (passed by value).
struct DecodeArgs {
  const void* q;
  const void* k_pages;
  const void* v_pages;
  const int32_t* page_table;
  const int32_t* ctx_lens;
  void* out;
  const float* k_scale;
  const float* v_scale;
  const int32_t* header;
  const int32_t* prefix;
  const int32_t* wstart;
  float* partial_ml;
  float* partial_o;
  int32_t batch, hq, hkv, group, max_pages, head_tile, rows_per_b;
  float scale_log2;     // sm_scale * log2(e)
  int32_t whole_rows;   // 1: the plan may say that every row is one worker's (kPlanWhole); with the first of the arguments, whose cache lines are read first
  float* lse;           // optional [B][Hq]: log2 of each row's softmax denominator (reference included)
  // Mixed step (both null otherwise): only trajectories with q_lens[b] == 1 are decode rows, the others count
  // as empty here; the query and output row of trajectory b is q_offsets[b] instead of b.
  const int32_t* q_lens;
  const int32_t* q_offsets;
  // Private half of attn_decode_shared (null otherwise): the context of trajectory b starts at this entry of its table row.
  const int32_t* first_page;
  SharedHalf shared;
  // Set (batch > 0) where no plan was launched: the decode kernel plans for itself.
  DecodePlanArgs plan;
};

struct AppendArgs {
  const void* q;
  const void* k_pages;
  const void* v_pages;
  const int32_t* page_table;
  const int32_t* ctx_lens;
  const int32_t* q_lens;
  const int32_t* q_offsets;
  void* out;
  const float* k_scale;
  const float* v_scale;
  int32_t* header;
  // [tile_cap][kTileRecWords]: (b, first row of the tile in its chunk, n_b, L_b, q_offsets[b], first block, number of
  // blocks, unit); unit: -1 for a whole tile, else where the partial results of this piece of one start
  const int32_t* tile_rec;
  int32_t tile_cap;
  const int32_t* merge_rec;  // (first row of the tile, n_b, q_offsets[b], first unit, pieces, 0, 0, 0) of every tile that was cut
  float* partial_ml;
  float* partial_o;
  int32_t batch, hq, hkv, group, max_pages, tile_tokens, total_q;
  float scale_log2;
  float* lse;           // optional [total_q][Hq], as in DecodeArgs
  int32_t noncausal;    // every row sees all of [0, L_b); the rows' own tokens are not in that range
  // Optional (profiling): two sums over the launch's tiles as wave 0 sees them, shader-clock cycles and ticks of the
  // constant-rate counter; their ratio is the clock the kernel ran at.
  unsigned long long* clock_sums;
};

// Inputs and outputs of the shared lengths of attn_decode_shared.
struct SharedPlanArgs {
  const int32_t* ctx_lens;
  const int32_t* shared_lens;
  int32_t batch, group_size;
  int32_t* own_ctx;                // [B] tokens past the shared ones
  int32_t* own_page;               // [B] table entry they start at
};

// Inputs and outputs of the append work list.
struct AppendPlanArgs {
  const int32_t* q_lens;
  const int32_t* q_offsets;
  const int32_t* ctx_lens;
  int32_t batch, hkv, group, tile_tokens;
  int32_t cap;                     // room in the list
  int32_t max_pieces, max_merges, max_units;   // cut tiles into pieces only within these (0: never)
  float us_alone, us_full;         // a block of the kernel that will run: on a chip with nothing else to do, on a full one
  float us_per_unit;               // a unit of partials on its way to memory and back
  int32_t min_longest;             // blocks: where the longest tile is shorter, no cut can pay
  bool skip_unit_chunks;           // mixed step: chunks of one token are decode rows
  bool noncausal;
  int32_t* header;
  int32_t* tile_rec;
  int32_t* merge_rec;
};

// Launchers (defined in the .hip files).  Each returns the hipError_t of its launch.
hipError_t launch_plan_decode(const DecodePlanArgs& d, hipStream_t s);
hipError_t launch_plan_append(const AppendPlanArgs& a, hipStream_t s);
// two plans at once; launch_plan_shared reads the lengths of both from `sh` (those in a and d are not used)
hipError_t launch_plan_step(const AppendPlanArgs& a, const DecodePlanArgs& d, hipStream_t s);
hipError_t launch_plan_shared(const SharedPlanArgs& sh, const AppendPlanArgs& a, const DecodePlanArgs& d, hipStream_t s);
hipError_t launch_decode_f32(const DecodeArgs& a, int head_dim, int grid, hipStream_t s);
// float32, one launch for plan, attention and output: a workgroup per row, for tables of at most kDirectPages pages and no more rows than CUs
hipError_t launch_decode_f32_direct(const DecodeArgs& a, int head_dim, hipStream_t s);
hipError_t launch_decode_mfma(const DecodeArgs& a, int head_dim, bool fp8, int grid, hipStream_t s);
hipError_t launch_combine(const DecodeArgs& a, int head_dim, bool out_bf16, hipStream_t s);
// the same for bf16 rows of which a.shared holds another part of the context: every row is written, to a.shared.result
hipError_t launch_combine_shared(const DecodeArgs& a, int head_dim, hipStream_t s);
// half_tiles: every tile has at most kAppendTileRows / 2 rows (a.tile_tokens is set accordingly) and the
// two waves of a SIMD split each block of a tile between them instead of owning different rows
hipError_t launch_append_mfma(const AppendArgs& a, int head_dim, bool fp8, bool half_tiles, int grid, hipStream_t s);
// folds the pieces of the tiles that were cut (max_merges: at most this many tiles)
hipError_t launch_append_merge(const AppendArgs& a, int head_dim, int max_merges, hipStream_t s);
hipError_t launch_append_f32(const AppendArgs& a, int head_dim, int grid, hipStream_t s);
hipError_t launch_kv_write(const void* k_new, const void* v_new, const int32_t* q_lens, const int32_t* q_offsets,
                           void* k_pages, void* v_pages, const int32_t* page_table, const int32_t* ctx_lens,
                           float* k_scale, float* v_scale, int32_t batch, int32_t hkv, int32_t max_pages,
                           int32_t max_q_len, int head_dim, int src_bytes, bool fp8, hipStream_t s);
hipError_t launch_merge_states(const void* o1, const float* d1, const void* o2, const float* d2, void* out, float* d_out,
                               long rows, int head_dim, bool f32, hipStream_t s);
hipError_t launch_check_inputs(const int32_t* page_table, const int32_t* ctx_lens, const int32_t* q_lens,
                               const int32_t* q_offsets, int32_t batch, int32_t max_pages, int64_t num_pages,
                               int32_t* counts, hipStream_t s);
hipError_t launch_gather(const void* pages, const int32_t* page_table, const int32_t* ctx_lens, int32_t b,
                         int32_t kv_head, int32_t hkv, int32_t max_pages, int32_t row_bytes, void* dst,
                         hipStream_t s);

}  // namespace rollattn
