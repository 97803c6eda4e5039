// Observation-append attention (chunked causal prefill on a cached prefix) for bf16 queries
// over bf16 or FP8-E4M3 paged KV, on the gfx950 matrix cores.
//
// One workgroup = 256 query rows of one (trajectory, KV head): a row is a (chunk token, query
// head of the group) pair, token-major, so the G heads that share the KV head reuse every K/V
// tile.  Eight waves of 32 rows each walk the visible KV range in 64-token blocks (four pages)
// that the workgroup stages once in LDS, always as bf16: bf16 pools are copied from HBM into LDS
// directly (no register stop, ring of four tiles per pool), FP8 pools pass through registers to
// be widened (two tiles per pool, loads two blocks ahead of the LDS write).  Per block a wave
// computes
//   S^T = K Q^T        tokens x rows, v_mfma_f32_32x32x16_bf16, K rows as A operand
//   O^T += V^T P^T     dims x rows, V read transposed with ds_read_b64_tr_b16
// The transposed products keep "row" on the lane axis in both accumulators: the softmax
// state is one scalar per lane (shared by two lanes) and P goes from accumulator registers
// straight into the B operand of the second product.
//
// Schedule.  A SIMD holds two of the workgroup's waves (w and w + 4).  Left alone they run in
// step, both in their MFMAs and then both in their softmax, and the matrix and vector pipelines
// take turns.  Here every block is cut into a matrix phase (the second product of the previous
// block, then the first product of this one) and a vector phase (this block's softmax), each
// closed by a workgroup barrier, and waves 4-7 enter the sequence one barrier late: on every SIMD
// one wave feeds the matrix core while the other does the exponentials.  A wave in its matrix
// phase has no partner to hide its latencies, so it reads its LDS operands several steps ahead in
// a fixed source-order schedule and issues as little else as possible: measured with per-phase
// cycle counters, a vector-memory instruction issued between the MFMAs costs the phase 70-90
// cycles (four of them stretched 32 MFMAs from 1270 to 1400 cycles), while the same instruction
// costs the vector phase little more than its issue slot.  All tile loads and the scalar loads of
// page ids therefore belong to the vector phase; only the widening of FP8 tiles
// (conversions and LDS writes of registers loaded two blocks earlier) stays between the MFMAs, spread over the
// phase (stage_widen), where it was measured to cost less than in the vector phase (all of it there, the two halves a unit
// apart: the mixed step 12.91 -> 13.9 ms; behind the softmax, or V alone: no difference).
// A wave issues one instruction per 4 cycles whatever its kind (vector instructions 6 beside a partner's MFMAs, exponentials
// 4 more), so the scalar instructions of a vector phase count like the others: page ids by running offsets, page scales once
// for 64 pages (fill_scales), LDS offsets as immediates and no maximum of the row to look at took it from about 150 vector
// and 95 scalar instructions to 121 and 20 over FP8 pools, and with waits for the tile loads by their true count the
// calls from 4.217 to 4.117 ms (64 chunks of 64 .. 1024 tokens behind 2k .. 16k, 32/8/128, bf16), 5.824 to 5.753 (without
// a prefix, 512 .. 8k tokens), 13.08 to 12.91 (mixed step of 512 trajectories, 64/4/128, FP8), all on one box: the clock gives most of the cycles
// back over bf16 pools, where the part is at its power limit, and some over FP8 pools.  The vector phase keeps its VALU work short in turn:
//   bf16 pools: the query is multiplied by sm_scale * log2(e) once, when it is loaded (one extra
//     bf16 rounding of q, far below the rounding of P), and the score accumulators start from
//     minus the row's reference instead of zero, so the MFMA result already is the exponent and
//     the softmax is one v_exp_f32 per element with nothing in front of it;
//   FP8 pools: the score needs its page's K scale anyway (one fused multiply-add per element,
//     whose addend carries minus the reference), and the V scale of the page is folded into that
//     addend as log2(vs), so P comes out of the exponential already weighted for the second
//     product; the row sum divides each page's share by vs again (four multiplies per block).
//
// Half tiles.  A call whose chunks all fit into 128 rows gets tiles of 128 rows: waves w and w + 4 then own the
// same 32 rows and split every step, and their two running states are merged when the tile ends.  Over FP8 pools a
// step of a long tile is two blocks, 64 tokens to each wave (see the template parameter HALF below).
#include <type_traits>
#include <utility>

#include "rollattn_internal.h"

namespace rollattn {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef short shortx4 __attribute__((ext_vector_type(4)));
typedef unsigned int uintx2 __attribute__((ext_vector_type(2)));
typedef unsigned int uintx4 __attribute__((ext_vector_type(4)));

constexpr int kThreads = 512;
constexpr int kWaves = kThreads / 64;
constexpr int kRowsPerWave = kUnitRows;
static_assert(kWaves * kRowsPerWave == kAppendTileRows, "tile rows");
constexpr int kBlockTokens = kAppendBlockTokens;   // KV tokens staged per step
constexpr int kLongTileBlocks = 20;                // half tiles over FP8 pools: from this many blocks on a step is two of them
constexpr int kScaleWindow = 64;                   // FP8: pages whose scales are fetched at a time, a lane each
constexpr float kSumLimit = 16384.f;               // a lane's 32 probabilities of a block may add up to this much before the row's reference moves

// Row t of an S^T tile holds this token of its 16-token group: the middle two quads are
// swapped so that the 8 scores a lane ends up with are 8 consecutive tokens.
__device__ __forceinline__ int tau(int r) { return (r & ~12) | ((r & 4) << 1) | ((r & 8) >> 1); }

__device__ __forceinline__ float xor32_max(float x) {
  uintx2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float xor32_add(float x) {
  uintx2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Pair PAIR of sixteen E4M3 codes to bf16, exactly (every E4M3 value is a bf16 value): the hardware's scaled
// conversion with a scale of one turns two codes into a packed pair per instruction.
template <int PAIR>
__device__ __forceinline__ uint32_t fp8_pair(const uintx4 codes) {
  return __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(codes[PAIR / 2], 1.0f, PAIR % 2 != 0));
}

// 16 bytes of a pool; once: nobody reads them again, so they go past the caches' care (see load16 in decode_mfma.hip).
template <bool ONCE>
__device__ __forceinline__ uintx4 load16(const unsigned char* p) {
  return ONCE ? __builtin_nontemporal_load((const uintx4*)p) : *(const uintx4*)p;
}

// Normalises and stores one 32-wide accumulator tile: lane (row n32, half h2) owns dims (i/4)*8 + h2*4 + i%4 of it, four
// at a time (o(i4, e): dim e of group i4).  The two lanes of a row first trade every other group of four, so that each
// holds runs of eight dims and stores 16 bytes at a time: half as many store instructions, each of which touches 32 rows.
// dst: the tile's dims in the row's output, + 8 for the upper lane of the row.
template <class O>
__device__ __forceinline__ void store_row_dims(__bf16* dst, bool row_ok, float inv, O&& o) {
  uintx2 g[4];
#pragma unroll
  for (int i4 = 0; i4 < 4; ++i4) {
    bf16x4 pk;
#pragma unroll
    for (int e = 0; e < 4; ++e) pk[e] = (__bf16)(o(i4, e) * inv);
    g[i4] = __builtin_bit_cast(uintx2, pk);
  }
#pragma unroll
  for (int pr = 0; pr < 2; ++pr) {
    // h2 = 0 keeps its group 2 pr (dims 8 pr .. + 3 of the 16) and gets the other lane's; h2 = 1 gets this lane's group
    // 2 pr + 1 and keeps its own: lower lane dims 16 pr + 0 .. 7, upper lane dims 16 pr + 8 .. 15
    const uintx2 w0 = __builtin_amdgcn_permlane32_swap(g[2 * pr][0], g[2 * pr + 1][0], false, false);
    const uintx2 w1 = __builtin_amdgcn_permlane32_swap(g[2 * pr][1], g[2 * pr + 1][1], false, false);
    if (row_ok) *(uintx4*)(dst + pr * 16) = uintx4{w0[0], w1[0], w0[1], w1[1]};
  }
}

// The operand reads and tile writes of the block loop: a lane's part of the LDS address is a pointer of its own that stays in a
// register over the whole loop, and everything else is the instruction's immediate offset.
typedef __attribute__((address_space(3))) unsigned char* lds_p;
template <class T>
__device__ __forceinline__ __attribute__((address_space(3))) T* lds_at(lds_p base, int offset) {
  return (__attribute__((address_space(3))) T*)(base + offset);
}

// The pointer with one bit of its address the other way round.
__device__ __forceinline__ lds_p flip(lds_p p, unsigned int bit) { return (lds_p)((unsigned int)(uintptr_t)p ^ bit); }

template <class F, int... I>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// HALF: for tiles of at most 128 rows.  With the plain layout such a tile keeps only the leading four waves busy
// and the two pipelines of a SIMD take turns.  Here waves w and w + 4 both own rows 32 (w % 4) .. and split every
// step between them: the leading wave takes its first half, the trailing wave the other one, each with a
// running reference, sum and accumulator of its own, merged through LDS when the tile ends.
// What a phase costs besides its scores (tile loads, page ids and scales, their waits, the barrier) does not shrink with
// them.  FP8 pools: two tiles of 128 tokens per pool fit the LDS, so a step may be two blocks and each wave's share a whole
// one (decode of 64 groups of 8 with prompts of 8192 tokens, 64/4/128: 253 -> 242 us in all, with steps of one block and
// of two).  A tile or piece of few blocks is mostly padding then, and takes steps of one: each workgroup picks by its own
// blocks (kLongTileBlocks: 64 chunks of 4 tokens behind 200, 32/8/128, 23.9 us with steps of one and 25.0 of two, of 2 behind
// 300 25.2 and 29.2, of 4 behind 900 47.7 and 48.4, of 4 behind 4000 142 and 126).  The choice costs 1 us at a tile's start,
// so calls whose table is too narrow for a long tile run a kernel without it.  bf16 pools: a ring of four tiles is all
// the LDS there is, a step stays one block, 32 tokens to each wave.
// ONCE: the pools are read with the streaming hint.  For the shared half of attn_decode_shared, where a group is one tile and
// no other reads its pages (64 groups of 8 behind 8192 tokens, 64/4/128, FP8: 242 -> 236 us in all).  Chunks of a few tokens
// are one tile each as well, but their prompts may be shared: 256 of 4 tokens in groups behind a common prompt would take
// 590 instead of 530 us over bf16 pools, against 516 instead of 557 us with prompts of their own.
// STEP: KV tokens staged per step of the loop.
template <int D, bool FP8, bool HALF, int STEP>
struct AppendGeo {
  // bf16 pools go from HBM straight into LDS (no register stop): a ring of four tiles per pool gives
  // every load a whole block period to land.  FP8 pools pass through registers to be widened: their
  // LDS writes are immediate, two tiles are enough.
  static constexpr int kRing = FP8 ? 2 : 4;
  static constexpr int kTileBytes = STEP * D * 2;
  // HALF: where the trailing waves leave their result for the leading ones: per wave pair the accumulators
  // [D / 32][4][64 lanes] as 16-byte quads, and reference and sum.  The accumulators of the four pairs go into the K ring,
  // which nobody reads, loads into or widens into any more by then (bf16: every wave has waited for its last loads; FP8: the
  // last tile is widened in a wave's last matrix phase but one; the last read of a K tile lies before the trailing waves'
  // last barrier); two FP8 tiles of one block are too small, there the accumulators get LDS of their own.
  static constexpr int kMergeAcc = (D / 32) * 16 * 64;      // floats per wave pair
  static constexpr bool kMergeInRing = (size_t)kRing * kTileBytes >= (size_t)(kWaves / 2) * kMergeAcc * sizeof(float);
  static constexpr bool kMergeApart = HALF && !kMergeInRing;
  // FP8: what the softmax needs of a page's scales, for two windows of kScaleWindow pages (see fill_scales below)
  static constexpr int kScales = FP8 ? 2 * kScaleWindow : 4;
};
// The LDS of a kernel with two instances, as one of them sees it.
template <int D, bool FP8, bool HALF, int STEP>
struct AppendLds {
  typedef AppendGeo<D, FP8, HALF, STEP> Geo;
  __attribute__((aligned(1024))) unsigned char k[Geo::kRing][Geo::kTileBytes], v[Geo::kRing][Geo::kTileBytes];
  __attribute__((aligned(16))) float merge_acc[Geo::kMergeApart ? kWaves / 2 : 1][Geo::kMergeApart ? Geo::kMergeAcc : 4];
  float merge_ml[HALF ? kWaves / 2 : 1][HALF ? 128 : 1];
  __attribute__((aligned(16))) float scales[3][Geo::kScales];
  long clock[2];
};

// Workgroup -> (tile, KV head).  Workgroups go to the 8 XCDs round-robin and every XCD has an L2 of its
// own; tiles of one trajectory and KV head walk the same K/V stream and should share one L2.  With the
// plain order (head fastest) that holds when the head count is a multiple of 8: XCD x then only ever sees
// heads x, x + 8, ...  With 1, 2 or 4 KV heads a head's tiles would be dealt to 8, 4 or 2 XCDs and each of
// them would fetch the whole stream; there the 8 / Hkv XCDs that serve a head take turns by runs of
// kAppendXcdRun consecutive tiles of the list (the list keeps a trajectory's tiles together).
__device__ __forceinline__ int tile_of(int block, int hkv, int& g) {
  if (hkv < kXcds && kXcds % hkv == 0) {
    const int x = block % kXcds, slot = block / kXcds;
    const int parts = kXcds / hkv;
    g = x % hkv;
    return (slot / kAppendXcdRun) * (parts * kAppendXcdRun) + (x / hkv) * kAppendXcdRun + slot % kAppendXcdRun;
  }
  const int tile = block / hkv;
  g = block - tile * hkv;
  return tile;
}

// The kernel's arguments, from its argument segment; ANEW: not shared with what other code has read of them.
typedef const __attribute__((address_space(4))) AppendArgs* const_args_p;
template <bool ANEW>
__device__ __forceinline__ decltype(auto) args_of(const AppendArgs& a) {
  if constexpr (ANEW) {
    const_args_p p = (const_args_p)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return (*p);
  } else {
    return (a);
  }
}

template <bool FIRST, class A, class B>
__device__ __forceinline__ decltype(auto) choose(A& a, B& b) {
  if constexpr (FIRST) return (a); else return (b);
}

// kOneOfTwo: another instance in the same kernel, both in `shared`; what is worked out in one stays in it, behind the branch.
template <int D, bool FP8, bool HALF, bool ONCE, int STEP, bool kOneOfTwo>
__device__ __forceinline__ void append_tile(const AppendArgs& kernel_args, AppendLds<D, FP8, HALF, STEP>* shared) {
  auto& a = args_of<kOneOfTwo>(kernel_args);
  typedef AppendGeo<D, FP8, HALF, STEP> Geo;
  constexpr int kStepTokens = STEP;
  constexpr int kRowBytes = D * 2;                 // bf16 rows in LDS
  constexpr int kChunks = kRowBytes / 16;          // 16-byte chunks per LDS row
  constexpr int kTileBytes = kStepTokens * kRowBytes;
  constexpr int kSrcRowBytes = D * (FP8 ? 1 : 2);  // row bytes in HBM
  constexpr int kSrcChunks = kSrcRowBytes / 16;
  constexpr int kLoads = (kStepTokens * kSrcChunks + kThreads - 1) / kThreads;   // per pool, per thread
  constexpr int kKK = D / 16;                      // 16-deep steps of the QK product
  constexpr int kDT = D / 32;                      // 32-wide output tiles along D
  static_assert((kStepTokens * kSrcChunks) % kThreads == 0 || kStepTokens * kSrcChunks < kThreads, "staging shape");

  constexpr int kRing = Geo::kRing;
  constexpr int kMergeAcc = Geo::kMergeAcc;
  constexpr bool kApart = Geo::kMergeApart && !kOneOfTwo;
  __shared__ __attribute__((aligned(1024))) unsigned char k_own[kOneOfTwo ? 1 : kRing][kOneOfTwo ? 16 : kTileBytes];
  __shared__ __attribute__((aligned(1024))) unsigned char v_own[kOneOfTwo ? 1 : kRing][kOneOfTwo ? 16 : kTileBytes];
  __shared__ __attribute__((aligned(16))) float merge_acc_own[kApart ? kWaves / 2 : 1][kApart ? kMergeAcc : 4];
  __shared__ float merge_ml_own[HALF && !kOneOfTwo ? kWaves / 2 : 1][HALF && !kOneOfTwo ? 128 : 1];
  __shared__ __attribute__((aligned(16))) float scales_own[3][kOneOfTwo ? 4 : Geo::kScales];
  __shared__ long clock_own[2];
  auto& k_lds = choose<kOneOfTwo>(shared->k, k_own);
  auto& v_lds = choose<kOneOfTwo>(shared->v, v_own);
  auto& merge_acc_s = choose<kOneOfTwo>(shared->merge_acc, merge_acc_own);
  auto& merge_ml_s = choose<kOneOfTwo>(shared->merge_ml, merge_ml_own);
  auto& scales_s = choose<kOneOfTwo>(shared->scales, scales_own);
  auto& clock_s = choose<kOneOfTwo>(shared->clock, clock_own);

  int tid = threadIdx.x, block = blockIdx.x;
  if constexpr (kOneOfTwo) asm volatile("" : "+v"(tid), "+s"(block));
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n32 = lane & 31;   // row (B column) / K token row (A row) carried by this lane
  const int h2 = lane >> 5;    // half of the contraction this lane feeds

  // Everything a tile's start hangs off comes in three trips to memory: the arguments, then the tile's record, then page ids
  // (and behind them the tiles and the query rows): 637.4 -> 634.5 us for 33 chunks of 3 .. 96 tokens behind up to 64k (64/4/128,
  // FP8), 12.31 -> 12.28 ms for the mixed step of 512; no difference over bf16 pools.
  const int group = a.group;
  const int hkv = a.hkv;
  const int tile_tokens = a.tile_tokens;
  const int tile_cap = a.tile_cap, max_pages = a.max_pages, hq = a.hq, noncausal = a.noncausal;
  const int32_t *tile_recs = a.tile_rec, *header = a.header, *page_table = a.page_table;
  const void *q = a.q, *k_pages = a.k_pages, *v_pages = a.v_pages;
  asm volatile("" ::"s"(group), "s"(hkv), "s"(tile_tokens), "s"(tile_cap), "s"(max_pages), "s"(hq), "s"(noncausal), "s"(tile_recs), "s"(header), "s"(page_table), "s"(q),
               "s"(k_pages), "s"(v_pages));
  int g;
  const int tile = tile_of(block, hkv, g);
  // The tile's record does not wait for the tile count (the index is clamped to the list's capacity): both loads
  // leave together, and everything else the workgroup needs to start hangs off the record alone.
  typedef const __attribute__((address_space(4))) int32_t* const_rec_p;
  const const_rec_p rec = (const_rec_p)(tile_recs + (size_t)min(tile, tile_cap - 1) * kTileRecWords);
  // A record is a whole tile, or a piece of one: blocks [blk0, blk0 + n_blocks) of the context.  The piece sees the
  // context as if it started there (table, length and positions shifted), so nothing below differs; rows whose last
  // token lies before it have negative positions and see nothing.
  const int b = rec[0], q0 = rec[1], n_b = rec[2], ctx_all = rec[3], q_off = rec[4], blk0 = rec[5], blocks = rec[6];
  const int n_tiles = *(const __attribute__((address_space(4))) int32_t*)(header + kPlanTiles);
  asm volatile("" ::"s"(b), "s"(q0), "s"(n_b), "s"(ctx_all), "s"(q_off), "s"(blk0), "s"(blocks), "s"(n_tiles));
  const int n_blocks = kStepTokens == kBlockTokens ? blocks : (blocks + 1) / 2;   // (the latter in steps of the loop)
  const int ctx = ctx_all - blk0 * kBlockTokens;
  if (tile >= n_tiles) return;
  if (a.clock_sums && threadIdx.x == 0) {
    clock_s[0] = __builtin_amdgcn_s_memtime();
    clock_s[1] = __builtin_amdgcn_s_memrealtime();
  }
  const int tokens_here = min(tile_tokens, n_b - q0);
  const int rows_here = tokens_here * group;
  // Causal mode: row i of the chunk sits at position L_b - n_b + i and sees tokens up to itself.
  // Non-causal mode (the shared part of a decode step for a group of trajectories): every row sees
  // all of [0, L_b), the rows' own tokens lie outside this range.
  const bool causal = noncausal == 0;
  const int pos0 = causal ? ctx - n_b + q0 : ctx - 1;    // position of the tile's first token
  // Page ids are an input nobody writes during the call: reading them through the constant address space lets the loads of
  // those behind the tile loads (all uniform) take the scalar path.
  typedef const __attribute__((address_space(4))) int32_t* const_i32_p;
  const const_i32_p table = (const_i32_p)(page_table + (size_t)b * max_pages + blk0 * (kBlockTokens / kPageSize));
  const size_t tile_stride = (size_t)kPageSize * kSrcRowBytes;

  // ---- this lane's query row
  const int grp = wave >> 2;   // 0: leading half of the workgroup, 1: the half that runs one phase behind (waves w and w + 4 share a SIMD)
  const int row_wave = HALF ? (wave & 3) : wave;         // which 32 rows of the tile this wave owns
  const int tok_wave = HALF ? grp * (kStepTokens / 2) : 0;   // HALF: where this wave's half of every step starts
  const int row = row_wave * kRowsPerWave + n32;
  const bool row_ok = row < rows_here;
  const int tok_in_tile = row / group;
  const int head = g * group + (row - tok_in_tile * group);
  int my_pos = row_ok ? (causal ? pos0 + tok_in_tile : pos0) : -1;   // last visible token of this row
  // blocks that end at or before this position are fully visible to every row of the wave
  const bool wave_active = row_wave * kRowsPerWave < rows_here;
  int wave_min_pos = wave_active ? (causal ? pos0 + (row_wave * kRowsPerWave) / group : pos0) : -1;
  if constexpr (kStepTokens != kBlockTokens) {
    // a piece of an odd number of blocks ends inside its last step: what follows is another piece's
    my_pos = min(my_pos, blocks * kBlockTokens - 1);
    wave_min_pos = min(wave_min_pos, blocks * kBlockTokens - 1);
  }

  if (n_blocks <= 0) {                                   // nothing to attend to (non-causal mode with L_b = 0): zero rows
    int tid_z = threadIdx.x;
    asm volatile("" : "+v"(tid_z));                      // (worked out again: kept for here, it would take registers in the loop)
    const int row_z = row_wave * kRowsPerWave + (tid_z & 31), half_z = (tid_z >> 5) & 1;
    const int tok_z = row_z / group;
    if (row_z < rows_here) {
      const size_t at_z = (size_t)(q_off + q0 + tok_z) * hq + g * group + (row_z - tok_z * group);
      __bf16* orow = (__bf16*)a.out + at_z * D;
#pragma unroll
      for (int d0 = half_z * (D / 2); d0 < (half_z + 1) * (D / 2); d0 += 4) *(bf16x4*)(orow + d0) = bf16x4{0, 0, 0, 0};
      if (a.lse && half_z == 0) a.lse[at_z] = -INFINITY;
    }
    return;
  }

  const int live_pages = (ctx + kPageSize - 1) / kPageSize;
  const int last_blk = n_blocks - 1;
  constexpr int kPagesPerBlock = kStepTokens / kPageSize;
  // The 64 chunks a wave fetches with one instruction lie in one page, so its id is a scalar.  Block after block the entries
  // behind a load lie kPagesPerBlock apart: their byte offset in the table runs along, no further than to the page of the last
  // block (page_end) or the last live page (page_live), whose rows are clamped too.
  int page_run[kLoads], page_end[kLoads];
  const int page_live = (live_pages - 1) * 4;
#pragma unroll
  for (int j = 0; j < kLoads; ++j) {
    page_run[j] = ((j * kThreads + wave * 64) / kSrcChunks) / kPageSize * 4;
    page_end[j] = min(last_blk * kPagesPerBlock * 4 + page_run[j], page_live);
  }
  // the page ids behind this wave's kLoads loads of one block, and whether that is the last live page; the blocks in order
  auto fetch_pids = [&](int* dst, int* at) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < kLoads; ++j) {
      at[j] = min(page_run[j], page_end[j]);
      dst[j] = *(const_i32_p)((const __attribute__((address_space(4))) char*)table + (unsigned int)at[j]);
      page_run[j] += kPagesPerBlock * 4;
    }
  };
  // those of the first four blocks, on their way while the query rows' addresses are worked out
  int first_ids[4][kLoads], first_at[4][kLoads];
#pragma unroll
  for (int d = 0; d < 4; ++d) fetch_pids(first_ids[d], first_at[d]);

  // Rows past the tile's last read that one again: what becomes of them is neither stored nor looked at.  (A branch around each
  // load had one of them waited for before the next was sent.)
  bf16x8 qop[kKK];
  {
    const int qtok = row_ok ? tok_in_tile : tokens_here - 1, qhead = row_ok ? head : g * group;
    const __bf16* qrow = (const __bf16*)q + ((size_t)(q_off + q0 + qtok) * hq + qhead) * D;
#pragma unroll
    for (int kk = 0; kk < kKK; ++kk) qop[kk] = *(const bf16x8*)(qrow + kk * 16 + h2 * 8);   // bf16 pools: scaled further down
  }

  floatx16 acc[kDT];
#pragma unroll
  for (int dt = 0; dt < kDT; ++dt)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[dt][i] = 0.f;
  float m_ref = 0.f, l_run = 0.f;               // the row's reference, zero as long as it has seen nothing, and its sum
  float sum_limit = row_ok ? -1.f : INFINITY;   // a lane's probabilities of a block may add up to this much; below zero: no reference yet
  auto seen_max = [&]() __attribute__((always_inline)) { return sum_limit < 0.f ? -INFINITY : m_ref; };
  floatx16 negm;            // bf16 pools: minus the row's reference in every element, the value the score accumulators start from
#pragma unroll
  for (int i = 0; i < 16; ++i) negm[i] = 0.f;
  const bool positive_scale = __float_as_int(a.scale_log2) > 0;   // the usual case (compared as an integer, in a scalar register); FP8 page scales are positive too

  // ---- staging.  Unit u = (K block u + 1, V block u): the two tiles that the matrix phase of
  // block u + 1 reads; block j lives in ring slot j % kRing of its pool.  Per thread and load, the
  // byte offset inside a (page, head) tile never changes: only the page does, and that is a scalar.
  // Every wave stages its share of a unit in its vector phase; branch-free on purpose (loads can
  // then be waited on by count).  Rows at or past L_b (ragged
  // last block, or a block index clamped at the end of the loop) re-read the trajectory's last
  // token instead: finite data that the causal / length mask never lets through.
  const int last_slot = (ctx - 1) % kPageSize;
  constexpr bool kAllThreadsLoad = kStepTokens * kSrcChunks >= kThreads;
  // Chunk idx = j * kThreads + tid of a block sits in LDS row idx / kChunks at chunk position
  // (idx % kChunks), holding the row's chunk (position ^ key): key = row & 15 for K, v_key for V.  The
  // register path (FP8) applies the swizzle when it writes LDS; the direct path has to apply it on the
  // global side, because there the LDS position of a lane's chunk is fixed.
  // V: the four rows of a transposing read lie a quarter of a row apart.
  // FP8: a chunk becomes two, so that one write has every other position of a row.  Eight lanes write 128 bytes at once: with
  // four chunks of each of two rows, one in even positions and the other (both keys have the row's last bit) in odd ones, they
  // meet all banks; with a row's eight they meet half of them twice: 8.5 M conflicts in 35.5 M busy cycles of the LDS over the
  // shared half of 64 groups of 8 behind 8192 tokens (64/4/128), none in 27.0 M this way; 64 chunks of 8 tokens behind 8k 195 -> 186 us.
  auto v_key = [](int row) __attribute__((always_inline)) { return (row & 3) << 2 | (FP8 ? row & 1 : 0); };
  unsigned int goff[kLoads][2], goff_last[kLoads][2];   // [][0]: K, [][1]: V
  lds_p wptr[kLoads][3];                                // FP8: where a widened chunk goes, K's two halves and V
#pragma unroll
  for (int j = 0; j < kLoads; ++j) {
    const int idx = j * kThreads + tid;
    // (FP8, D = 128: lanes 0-3 and 8-11 the first of two rows, the others the second)
    constexpr bool kPairs = FP8 && kSrcChunks == 8;
    const int trow = kPairs ? idx / 16 * 2 + (idx >> 2 & 1) : idx / kSrcChunks;
    const int tslot = trow % kPageSize;               // token slot within its page
    const int c = kPairs ? (idx >> 3 & 1) * 4 + (idx & 3) : idx % kSrcChunks;
    const int kkey = trow & 15, vkey = v_key(trow);
    const int ck = FP8 ? c : ((c ^ kkey) & (kChunks - 1)), cv = FP8 ? c : ((c ^ vkey) & (kChunks - 1));
    goff[j][0] = tslot * kSrcRowBytes + ck * 16;
    goff[j][1] = tslot * kSrcRowBytes + cv * 16;
    goff_last[j][0] = min(tslot, last_slot) * kSrcRowBytes + ck * 16;
    goff_last[j][1] = min(tslot, last_slot) * kSrcRowBytes + cv * 16;
    if constexpr (FP8) {
      // the two 16-byte halves of the widened chunk sit in chunks 2c and 2c + 1: 16 bytes apart after the swizzle, one behind the
      // other or in front of it
      const int kat = trow * kRowBytes + (((2 * c) ^ kkey) & (kChunks - 1)) * 16;
      wptr[j][0] = (lds_p)(k_lds[0] + kat);
      wptr[j][1] = (lds_p)(k_lds[0] + (kat ^ 16));
      wptr[j][2] = (lds_p)(v_lds[0] + trow * kRowBytes + (((2 * c) ^ vkey) & (kChunks - 1)) * 16);
    }
  }
  // byte offset of the (page, KV head) tile in either pool
  auto tile_off_of = [&](int pid) __attribute__((always_inline)) -> size_t {
    return (size_t)(unsigned int)(pid * hkv + g) * tile_stride;
  };
  // one wave-wide 16-byte load: scalar tile base, per-lane offset
  struct TileAddr { const unsigned char* base; unsigned int off; };
  auto tile_addr = [&](const void* pool, int pool_i, size_t toff, bool last, int j) __attribute__((always_inline)) -> TileAddr {
    return TileAddr{(const unsigned char*)pool + toff, last ? goff_last[j][FP8 ? 0 : pool_i] : goff[j][FP8 ? 0 : pool_i]};   // (FP8: the same for both pools)
  };
  // -- register path (FP8)
  uintx4 kreg[2][kLoads], vreg[2][kLoads];   // two units in flight
  auto put = [&](lds_p lo_at, lds_p hi_at, int offset, const uintx4 codes) __attribute__((always_inline)) {
    *lds_at<uintx4>(lo_at, offset) = uintx4{fp8_pair<0>(codes), fp8_pair<1>(codes), fp8_pair<2>(codes), fp8_pair<3>(codes)};
    *lds_at<uintx4>(hi_at, offset) = uintx4{fp8_pair<4>(codes), fp8_pair<5>(codes), fp8_pair<6>(codes), fp8_pair<7>(codes)};
  };
  // -- direct path (bf16): HBM -> LDS without a register stop.  Lane l's 16 bytes land at
  // M0 + 16 l.  The compiler does not see these loads as loads: completion is awaited by count
  // below, which is sound only as long as nothing else in the loop uses the vector-memory counter,
  // register spills to scratch memory included (the build checks that this kernel has none).  M0 is
  // a reserved register for this compiler (it refuses it in a clobber list) and is never live
  // across statements in the code it generates, so it is simply overwritten.
  auto dma = [&](const TileAddr& t, unsigned char* lds_dst) __attribute__((always_inline)) {
    const unsigned int m0 = __builtin_amdgcn_readfirstlane((unsigned int)(uintptr_t)lds_dst);
    if constexpr (ONCE) asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt" ::"s"(m0), "v"(t.off), "s"(t.base) : "memory");
    else asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(m0), "v"(t.off), "s"(t.base) : "memory");
  };
#define DMA_WAIT(n) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(n))

  // FP8: per page, K scale times softmax scale, log2 of the V scale, and its reciprocal.  Worked out by wave 0 for kScaleWindow
  // pages at a time, a lane each, and left in LDS: scalar loads in every wave and block (page ids, then scales, then two
  // transcendentals per page that all lanes compute alike) took a quarter of the instructions of a vector phase, which is bound
  // by how fast one wave issues.
  constexpr int kPg = HALF ? kPagesPerBlock / 2 : kPagesPerBlock;   // pages of a block that this wave's tokens lie in
  constexpr int kWindowBlocks = kScaleWindow / kPagesPerBlock;
  float ksc_cur[kPg], lvs_cur[kPg], ivs_cur[kPg];
  unsigned int window_k = 0;      // the page's id, then its K scale
  float window_v = 1.f;
  auto window_ids = [&](int blk) __attribute__((always_inline)) {      // of the window that starts at block blk
    window_k = *(const unsigned int*)((const char*)(const int32_t*)table + (unsigned int)min((blk * kPagesPerBlock + lane) * 4, page_live));
  };
  auto window_scales = [&]() __attribute__((always_inline)) {
    window_v = a.v_scale[window_k];
    window_k = __float_as_uint(a.k_scale[window_k]);
  };
  auto window_write = [&](int blk) __attribute__((always_inline)) {
    const int at = (blk * kPagesPerBlock + lane) % (2 * kScaleWindow);
    scales_s[0][at] = __uint_as_float(window_k) * a.scale_log2;
    scales_s[1][at] = __builtin_amdgcn_logf(window_v);
    scales_s[2][at] = __builtin_amdgcn_rcpf(window_v);
  };
  // this wave's pages of block blk
  auto read_scales = [&](int blk) __attribute__((always_inline)) {
    const int at = (blk * kPagesPerBlock) % (2 * kScaleWindow) + (HALF ? grp * kPg : 0);
#pragma unroll
    for (int p = 0; p < kPg; ++p) { ksc_cur[p] = scales_s[0][at + p]; lvs_cur[p] = scales_s[1][at + p]; ivs_cur[p] = scales_s[2][at + p]; }
  };

  // Per-lane LDS pointers that do not change over the loop: the K row this lane feeds as an A
  // operand for each 16-dim step, and the V row / column pair it addresses in each transposed
  // read.  Everything else (buffer, sub-block, token group) is a compile-time immediate.
  lds_p kptr[kKK], vptr[kDT];
  const int sub_bytes = tok_wave * kRowBytes;           // HALF: where this wave's tokens start in a K or V tile
  {
    const int t = (n32 & 16) + tau(n32 & 15);
#pragma unroll
    for (int kk = 0; kk < kKK; ++kk) kptr[kk] = (lds_p)(k_lds[0] + sub_bytes + t * kRowBytes + (((kk * 2 + h2) ^ (t & 15)) & (kChunks - 1)) * 16);
    const int j = lane & 15;
    const int tv = h2 * 8 + (j >> 2);
#pragma unroll
    for (int dt = 0; dt < kDT; ++dt)
      vptr[dt] = (lds_p)(v_lds[0] + sub_bytes + tv * kRowBytes +
                 (((dt * 4 + ((lane >> 4) & 1) * 2 + ((j & 3) >> 1)) ^ v_key(tv)) & (kChunks - 1)) * 16 + (j & 1) * 8);
  }

  constexpr int kSubs = kStepTokens / (HALF ? 64 : 32);   // 32-token sub-blocks of a step that this wave works on
  constexpr int kPvSteps = 8 * kSubs, kSteps = 16 * kSubs;
  floatx16 s[kSubs];        // scores of the block between its two phases
  bf16x8 pop[kSubs][2];     // its probabilities, as B operands of the second product

  // ---- matrix phase: up to kSteps (32; HALF over bf16 pools: 16) MFMA steps, O^T += V^T P^T for the previous block (the
  // first kPvSteps, V buffer at vbo) and S^T = K Q^T for this one (the others, K buffer at kbo).  Every step
  // needs one 32x16 operand from LDS; the reads run kAhead steps in front of the MFMAs that consume them,
  // because during this phase no second wave hides the LDS latency.  The phase has 32 schedule positions
  // spread evenly over its steps; after a step the caller's piece(pos) runs for the positions that belong to
  // it: the FP8 path threads its LDS writes between the MFMAs there.
  // (how far ahead, measured with everything else alike.  bf16: 1, 2, 3, 4, 5 steps: 5.33, 4.13, 4.02, 4.05, 4.11 ms on 64 chunks
  // of 64 .. 1024 tokens behind 2k .. 16k, 32/8/128; 7.20, 5.74, 5.64, 5.66, 5.75 ms without a prefix, 512 .. 8k tokens.
  // FP8: 3, 4: 1701, 1701 us on 32 chunks of 256 tokens behind 8k, 64/4/128)
  constexpr int kAhead = 3;
  // bf16 pools: the operands of the first kAhead steps of a phase that starts with the second product are
  // read at the end of the vector phase before it, in front of the barrier (the V tile they come from was
  // complete one phase earlier), so that the phase does not open with an LDS round trip.
  constexpr bool kEarly = !FP8;
  bf16x8 early[kAhead];
  auto read_v_operand = [&](int vbo, auto t_c, bf16x8& dst) __attribute__((always_inline)) {
    constexpr int t = decltype(t_c)::value;
    constexpr int sub = t >> 3, ks = (t >> 2) & 1, dt = t & 3;
    if constexpr (dt < kDT) {
#pragma unroll
      for (int hf = 0; hf < 2; ++hf) {
        const shortx4 raw = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            lds_at<shortx4>(vptr[dt], vbo + (sub * 32 + ks * 16 + hf * 4) * kRowBytes));
        const bf16x4 h4 = __builtin_bit_cast(bf16x4, raw);
        dst[hf * 4 + 0] = h4[0]; dst[hf * 4 + 1] = h4[1]; dst[hf * 4 + 2] = h4[2]; dst[hf * 4 + 3] = h4[3];
      }
    }
  };
  auto read_early = [&](int vbo) __attribute__((always_inline)) {
    static_for<kAhead>([&](auto t_c) __attribute__((always_inline)) { read_v_operand(vbo, t_c, early[decltype(t_c)::value]); });
  };
  auto matrix_phase = [&](auto first_c, auto last_c, int kbo, int vbo, auto&& piece) __attribute__((always_inline)) {
    constexpr int T0 = decltype(first_c)::value, T1 = decltype(last_c)::value;
    bf16x8 ops[kSteps];
    auto fetch = [&](auto t_c) __attribute__((always_inline)) {
      constexpr int t = decltype(t_c)::value;
      if constexpr (t < kPvSteps) {
        read_v_operand(vbo, t_c, ops[t]);
      } else {
        constexpr int u = t - kPvSteps, kk = u / kSubs, sub = u % kSubs;
        if constexpr (kk < kKK) ops[t] = *lds_at<const bf16x8>(kptr[kk], kbo + sub * 32 * kRowBytes);
      }
    };
    auto fire = [&](auto t_c) __attribute__((always_inline)) {
      constexpr int t = decltype(t_c)::value;
      if constexpr (t < kPvSteps) {
        constexpr int sub = t >> 3, ks = (t >> 2) & 1, dt = t & 3;
        if constexpr (dt < kDT) acc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ops[t], pop[sub][ks], acc[dt], 0, 0, 0);
      } else {
        constexpr int u = t - kPvSteps, kk = u / kSubs, sub = u % kSubs;
        if constexpr (kk < kKK) {
          if constexpr (kk == 0) {
            if constexpr (FP8) {
#pragma unroll
              for (int i = 0; i < 16; ++i) s[sub][i] = 0.f;
              s[sub] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ops[t], qop[kk], s[sub], 0, 0, 0);
            } else {
              s[sub] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ops[t], qop[kk], negm, 0, 0, 0);
            }
          } else {
            s[sub] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ops[t], qop[kk], s[sub], 0, 0, 0);
          }
        }
      }
    };
    static_for<kAhead>([&](auto d_c) __attribute__((always_inline)) {
      constexpr int t = T0 + decltype(d_c)::value;
      if constexpr (kEarly && T0 == 0) ops[t] = early[t];
      else if constexpr (t < T1) fetch(std::integral_constant<int, t>{});
    });
    __builtin_amdgcn_sched_barrier(0);
    static_for<kSteps>([&](auto t_c) __attribute__((always_inline)) {
      constexpr int t = decltype(t_c)::value;
      if constexpr (t >= T0 && t < T1) {
        if constexpr (t + kAhead < T1) fetch(std::integral_constant<int, t + kAhead>{});
        fire(t_c);
        constexpr int P0 = (t - T0) * 32 / (T1 - T0), P1 = (t + 1 - T0) * 32 / (T1 - T0);
        static_for<P1 - P0>([&](auto d_c) __attribute__((always_inline)) { piece(std::integral_constant<int, P0 + decltype(d_c)::value>{}); });
        __builtin_amdgcn_sched_barrier(0);           // the source order of the steps is the schedule
      }
    });
  };
  constexpr std::integral_constant<int, 0> c0{};
  // ---- vector phase: online softmax of block blk.  Register i of s[sub] is token
  // blk*64 + sub*32 + (i/8)*16 + h2*8 + (i%8) of row n32.
  //   bf16 pools: s already is the exponent (scaled query, accumulators started from minus the reference).
  //   FP8 pools:  s is the raw product with the codes; per page sc = K scale times the softmax scale and
  //               ad = log2(V scale) - reference, so p' = 2^(s * sc + ad) = p * vs is the weight the second
  //               product needs, and the row sum takes each page's share divided by vs again.
  // The reference of a row only moves when it has to.  The exponentials are taken against the
  // reference as it stands, without looking for the block's maximum first, and may exceed one: float
  // sums and bf16 P hold large values with the same relative precision as small ones.  Only when the p
  // of one lane add up to more than kSumLimit (so that no single p ever exceeds it), or when a row has no
  // reference yet, does the wave find the true maxima, move the references there, rescale the
  // accumulators and redo the block's exponentials.  In all other blocks the maximum, a chain of
  // dependent steps across the row, is never computed.
  static_assert(kPg == 2 * kSubs, "two pages per 32-token sub-block");
  auto softmax = [&](int blk) __attribute__((always_inline)) {
    float sc[kPg], lvs[kPg], ivs[kPg];                 // this wave's pages: K scale times softmax scale, log2 of the V scale, its reciprocal
    if constexpr (FP8) {
#pragma unroll
      for (int p = 0; p < kPg; ++p) { sc[p] = ksc_cur[p]; lvs[p] = lvs_cur[p]; ivs[p] = ivs_cur[p]; }
      if (!positive_scale) {                           // rare: scale the scores themselves instead
#pragma unroll
        for (int sub = 0; sub < kSubs; ++sub)
#pragma unroll
          for (int i = 0; i < 16; ++i) s[sub][i] *= sc[sub * 2 + (i >> 3)];
#pragma unroll
        for (int p = 0; p < kPg; ++p) sc[p] = 1.f;
      }
    }
    const int tok0 = blk * kStepTokens + tok_wave;     // first token of this wave's share of the block
    if (tok0 + kSubs * 32 - 1 > wave_min_pos) {        // causal edge or ragged end inside this block
#pragma unroll
      for (int sub = 0; sub < kSubs; ++sub)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int tok = tok0 + sub * 32 + (i >> 3) * 16 + h2 * 8 + (i & 7);
          if (tok > my_pos) s[sub][i] = -INFINITY;
        }
    }
    const float m_old = m_ref;                         // what the exponents in s (bf16 pools) are relative to
    float p[kSubs][16];
    // exponentials of the block against reference m_old + shift, and this lane's share of the row sums
    auto exponentials = [&](auto first_c, float shift) __attribute__((always_inline)) -> float {
      float ad[kPg], psum[kPg];
      if constexpr (FP8) {
#pragma unroll
        for (int pg = 0; pg < kPg; ++pg) ad[pg] = lvs[pg] - (decltype(first_c)::value ? m_old : m_old + shift);
      }
#pragma unroll
      for (int sub = 0; sub < kSubs; ++sub)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int pg = sub * 2 + (i >> 3);
          float x;
          if constexpr (FP8) x = __builtin_fmaf(s[sub][i], sc[pg], ad[pg]);
          else if constexpr (decltype(first_c)::value) x = s[sub][i];
          else x = s[sub][i] - shift;
          p[sub][i] = __builtin_amdgcn_exp2f(x);
          if ((i & 7) == 0) psum[pg] = p[sub][i];
          else psum[pg] += p[sub][i];
        }
      if constexpr (kPg == 2) return FP8 ? psum[0] * ivs[0] + psum[1] * ivs[1] : psum[0] + psum[1];
      else if constexpr (FP8) return (psum[0] * ivs[0] + psum[1] * ivs[1]) + (psum[2] * ivs[2] + psum[3] * ivs[3]);
      else return (psum[0] + psum[1]) + (psum[2] + psum[3]);
    };
    float lane_sum = exponentials(std::true_type{}, 0.f);
    // (an infinite or undefined sum also fails the comparison and takes the slow path)
    if (__builtin_amdgcn_ballot_w64(!(lane_sum <= sum_limit))) {
      // largest exponent of the block: FP8 page scales and the softmax scale are positive here, so the maximum
      // can be taken on the raw products of each page
      float pm[kPg];
#pragma unroll
      for (int q = 0; q < kPg; ++q) {
        const int sub = q >> 1, o = (q & 1) * 8;
        float x = fmaxf(fmaxf(s[sub][o], s[sub][o + 1]), s[sub][o + 2]);
        x = fmaxf(fmaxf(x, s[sub][o + 3]), s[sub][o + 4]);
        x = fmaxf(fmaxf(x, s[sub][o + 5]), s[sub][o + 6]);
        pm[q] = fmaxf(x, s[sub][o + 7]);
      }
      float mloc;
      if constexpr (kPg == 2) mloc = FP8 ? fmaxf(pm[0] * sc[0], pm[1] * sc[1]) : fmaxf(pm[0], pm[1]) + m_old;
      else if constexpr (FP8) mloc = fmaxf(fmaxf(pm[0] * sc[0], pm[1] * sc[1]), fmaxf(pm[2] * sc[2], pm[3] * sc[3]));
      else mloc = fmaxf(fmaxf(pm[0], pm[1]), fmaxf(pm[2], pm[3])) + m_old;
      const float m_run = seen_max();
      const float m_new = fmaxf(m_run, xor32_max(mloc));           // the same in both lanes of a row
      const float m_safe = (m_new == -INFINITY) ? 0.f : m_new;     // rows that see nothing yet
      const float alpha = __builtin_amdgcn_exp2f(m_run - m_safe);
      l_run *= alpha;
#pragma unroll
      for (int dt = 0; dt < kDT; ++dt)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[dt][i] *= alpha;
      m_ref = m_safe;
      if (row_ok && m_new != -INFINITY) sum_limit = kSumLimit;
      if constexpr (!FP8) {
#pragma unroll
        for (int i = 0; i < 16; ++i) negm[i] = -m_safe;
      }
      lane_sum = exponentials(std::false_type{}, m_safe - m_old);
    }
    l_run += lane_sum;
#pragma unroll
    for (int sub = 0; sub < kSubs; ++sub)
#pragma unroll
      for (int i = 0; i < 16; ++i) pop[sub][i >> 3][i & 7] = (__bf16)p[sub][i];
    // the probabilities are finished here, in this phase, not wherever the compiler would like to sink them
#pragma unroll
    for (int sub = 0; sub < kSubs; ++sub)
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        uintx4 t = __builtin_bit_cast(uintx4, pop[sub][ks]);
        asm volatile("" : "+v"(t));
        pop[sub][ks] = __builtin_bit_cast(bf16x8, t);
      }
  };

  // Two phases per block, a matrix phase (O += V P of the previous block, then S = K Q^T of this
  // one: MFMAs and their LDS operand reads, nothing else) and a vector phase (softmax of this block and
  // the wave's share of the staging), each closed by a workgroup barrier.  The trailing half of the
  // waves entered the sequence one barrier late, so on every SIMD one wave is in its matrix phase
  // while the other is in its vector phase and the two pipelines run side by side instead of taking
  // turns.  Phases are numbered by barriers: the leading half has its matrix phase of block i in phase
  // 2i and its vector phase in 2i + 1, the trailing half in 2i + 1 and 2i + 2.  K block i and V block
  // i - 1 are read in phases 2i and 2i + 1 and their ring slots are free from phase 2i + 2 on.
  //   bf16: in its vector phase of block i a wave starts the loads of unit i + 2 (K block i + 3 into
  //         the slot K block i - 1 left in phase 2i - 1 at the latest, V block i + 2 into the slot of
  //         V block i - 2) and then waits until all but those newest loads have landed: unit i + 1,
  //         a whole block period after it was started, and two barriers before phase 2i + 4 reads it.
  //   FP8:  in its matrix phase of block i (phase 2i or 2i + 1) a wave widens its share of unit i
  //         (K block i + 1, V block i; first read in phase 2i + 2) from registers into the tiles that
  //         are not being read, and in the vector phase that follows it reloads those registers
  //         with unit i + 2.
  // FP8: the wave's LDS writes must be complete before the barrier, but its tile loads for later units
  // must stay in flight across it (a full fence would wait for them too).  bf16: a bare barrier; the
  // direct loads are awaited by count where they are issued.
#define BARRIER_RAW() do { if (FP8) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); else asm volatile("s_barrier" ::: "memory"); } while (0)
#define PHASE_END() do { __builtin_amdgcn_sched_barrier(0); BARRIER_RAW(); __builtin_amdgcn_sched_barrier(0); } while (0)
  constexpr std::integral_constant<int, kPvSteps> c_pv{};   // first step of the first product
  constexpr std::integral_constant<int, kSteps> c_end{};     // end of the phase
  // Page ids run ahead of the tile loads, so that no load ever waits for an address: U = i + kLead being
  // the unit whose loads a wave starts in its vector phase of block i, toff holds (on entry to that
  // phase) the tile offsets of block U and pid_new the page ids of block U + 1.
  constexpr int kLead = 2;
  size_t toff[2][kLoads];      // rotated at the start of the staging step: then [0] is K block U + 1, [1] V block U
  bool is_last[2][kLoads];     // ... whose page is the last live one
  int pid_new[kLoads], at_new[kLoads];   // not yet turned into an offset
  {
    auto& h = first_ids;
    auto& at = first_at;
    size_t off[4][kLoads];
    bool end[4][kLoads];
    if constexpr (FP8) {
      if (wave == 0) window_ids(0);
    }
#pragma unroll
    for (int d = 0; d < 4; ++d)
#pragma unroll
      for (int j = 0; j < kLoads; ++j) { off[d][j] = tile_off_of(h[d][j]); end[d][j] = at[d][j] == page_live; }
    if constexpr (FP8) {
      // K block 0 goes to LDS here; units 0 and 1 wait in registers
      uintx4 k0[kLoads];
#pragma unroll
      for (int j = 0; j < kLoads; ++j)
        if (kAllThreadsLoad || (j * kThreads + tid) / kSrcChunks < kStepTokens) {
          const TileAddr ka = tile_addr(a.k_pages, 0, off[0][j], end[0][j], j);
          k0[j] = load16<ONCE>(ka.base + ka.off);
        }
#pragma unroll
      for (int u = 0; u < kLead; ++u)
#pragma unroll
        for (int j = 0; j < kLoads; ++j)
          if (kAllThreadsLoad || (j * kThreads + tid) / kSrcChunks < kStepTokens) {
            const TileAddr ka = tile_addr(a.k_pages, 0, off[u + 1][j], end[u + 1][j], j), va = tile_addr(a.v_pages, 1, off[u][j], end[u][j], j);
            kreg[u][j] = load16<ONCE>(ka.base + ka.off);
            vreg[u][j] = load16<ONCE>(va.base + va.off);
          }
      if (wave == 0) {
        window_scales();
        window_write(0);
      }
#pragma unroll
      for (int j = 0; j < kLoads; ++j)
        if (kAllThreadsLoad || (j * kThreads + tid) / kSrcChunks < kStepTokens) put(wptr[j][0], wptr[j][1], 0, k0[j]);
    } else {
      // The query rows have been under way as long as the page ids; their scaling (bf16 pools: the scores then leave the
      // matrix core as exponents) waits for them in front of the tile loads.  Those are no loads to the compiler: behind them,
      // its wait for the rows would be one for all of them, unit 1 included (4096 tiles of 1, 2 and 6 blocks, 32/8/128: 216.9,
      // 244.2 and 359.5 us that way, 207.6, 235.5 and 352.1 this way).
#pragma unroll
      for (int kk = 0; kk < kKK; ++kk) {
#pragma unroll
        for (int e = 0; e < 8; ++e) qop[kk][e] = (__bf16)((float)qop[kk][e] * a.scale_log2);
        asm volatile("" : "+v"(qop[kk]));
      }
#pragma unroll
      for (int j = 0; j < kLoads; ++j)
        dma(tile_addr(a.k_pages, 0, off[0][j], end[0][j], j), k_lds[0] + wave * 1024 + j * kThreads * 16);
#pragma unroll
      for (int u = 0; u < kLead; ++u)                // units 0 .. kLead - 1
#pragma unroll
        for (int j = 0; j < kLoads; ++j) {
          dma(tile_addr(a.k_pages, 0, off[u + 1][j], end[u + 1][j], j), k_lds[0] + (u + 1) * kTileBytes + wave * 1024 + j * kThreads * 16);
          dma(tile_addr(a.v_pages, 1, off[u][j], end[u][j], j), v_lds[0] + u * kTileBytes + wave * 1024 + j * kThreads * 16);
        }
      DMA_WAIT((kLead - 1) * 2 * kLoads);            // K block 0 and unit 0 have landed (unit 0 is read early, one barrier from now)
    }
    PHASE_END();
    if (grp == 1) {                                  // the trailing half starts one phase late
      PHASE_END();
    }
#pragma unroll
    for (int j = 0; j < kLoads; ++j) {
      pid_new[j] = h[3][j];
      at_new[j] = at[3][j];
      toff[0][j] = off[2][j];
      is_last[0][j] = end[2][j];
    }
  }
  // Staging.  The tile addresses of the unit whose loads start in this vector phase:
  auto stage_addresses = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < kLoads; ++j) {
      toff[1][j] = toff[0][j];
      is_last[1][j] = is_last[0][j];
      toff[0][j] = tile_off_of(pid_new[j]);
      is_last[0][j] = at_new[j] == page_live;
    }
  };
  // Byte offset of the ring slot of block i + d, block i - 1 sharing that of block i + kRing - 1.  The loop is unrolled twice
  // (slot_c: i % 2 from here on): a ring of two needs no variable, the offset goes into the LDS instructions as it is.
  int ko[kRing];
#pragma unroll
  for (int d = 0; d < kRing; ++d) ko[d] = d * kTileBytes;
  auto ring = [&](auto slot_c, auto d_c) __attribute__((always_inline)) -> int {
    constexpr int slot = decltype(slot_c)::value, d = (decltype(d_c)::value + kRing) % kRing;
    if constexpr (kRing == 2) return (slot + d) % 2 * kTileBytes;
    else return ko[d];
  };
  constexpr std::integral_constant<int, 1> c1{};
  constexpr std::integral_constant<int, 2> c2{};
  constexpr std::integral_constant<int, -1> cm1{};
  // ... those loads, in the vector phase of block i (FP8: into the register slot that the matrix phase of block
  // i has just drained) ...
  auto stage_loads = [&](int i, auto slot_c) __attribute__((always_inline)) {
    constexpr int slot = decltype(slot_c)::value;
    if constexpr (FP8) {
      // (units past the tile's last block are loaded as well, the last block once more, and widened into tiles nobody reads:
      // a branch around them would have every wait for an earlier unit wait for this one too, since on the other way round
      // the branch nothing follows the earlier unit)
#pragma unroll
      for (int j = 0; j < kLoads; ++j)
        if (kAllThreadsLoad || (j * kThreads + tid) / kSrcChunks < kStepTokens) {
          const TileAddr ka = tile_addr(a.k_pages, 0, toff[0][j], is_last[0][j], j), va = tile_addr(a.v_pages, 1, toff[1][j], is_last[1][j], j);
          kreg[slot][j] = load16<ONCE>(ka.base + ka.off);
          vreg[slot][j] = load16<ONCE>(va.base + va.off);
        }
    } else if (i + kLead <= last_blk) {
#pragma unroll
      for (int j = 0; j < kLoads; ++j) {
        dma(tile_addr(a.k_pages, 0, toff[0][j], is_last[0][j], j), k_lds[0] + ring(slot_c, cm1) + wave * 1024 + j * kThreads * 16);
        dma(tile_addr(a.v_pages, 1, toff[1][j], is_last[1][j], j), v_lds[0] + ring(slot_c, c2) + wave * 1024 + j * kThreads * 16);
      }
      DMA_WAIT(2 * kLoads);                          // everything but the unit just started has landed
    } else {
      DMA_WAIT(0);                                   // past the tile's last block nothing is started: the units still on their way are real ones
    }
  };
  // ... and, FP8 only, the widening of unit i (K block i + 1, V block i) from registers into LDS during the matrix phase of
  // block i: 16 conversions and 4 writes per load, spread over the first 31 of the phase's 32 positions.  Whole tiles at D = 128
  // have 20 of them for 32 MFMAs, at most one behind each; a tile's first block, without the second product, 20 for 16.  Half
  // tiles have 40 for 32 in steps of two blocks and 20 for 16 in steps of one, up to two behind an MFMA; at D = 64 half of the
  // steps have no MFMA.  A wave issues in order, an MFMA takes the matrix core 33 cycles and its own issue 10, the operand read
  // in front of it 12: one or two instructions more per MFMA cost nothing, ten in one place keep the core waiting for 40
  // cycles.  With a chunk's ten instructions behind one MFMA a block of a whole tile took
  // 3300 cycles, so 3003; 32 chunks of 256 tokens behind 8k (64/4/128), back to back, 1840 -> 1797 us, the rest went into the clock
  // (1.81 -> 1.68 GHz); with pauses between the launches 1770 -> 1701 us.
  // All of it in front of the 20th or 26th of 32 MFMAs instead of the 31st: 1 to 2 % slower.
  uintx4 wide[kLoads];
  auto stage_widen = [&](auto slot_c, auto pos_c) __attribute__((always_inline)) {
    if constexpr (FP8) {
      constexpr int slot = decltype(slot_c)::value, pos = decltype(pos_c)::value;
      constexpr int kItems = 20 * kLoads;
      static_for<kItems>([&](auto item_c) __attribute__((always_inline)) {
        constexpr int item = decltype(item_c)::value;
        if constexpr (item * 31 / kItems == pos) {
          constexpr int j = item % kLoads, part = item / kLoads / 5, m = item / kLoads % 5;   // the halves of K's chunk, then V's
          if constexpr (m < 4) {
            wide[j][m] = fp8_pair<(part & 1) * 4 + m>((part < 2 ? kreg : vreg)[slot][j]);
          } else if (kAllThreadsLoad || (j * kThreads + tid) / kSrcChunks < kStepTokens) {
            if constexpr (part < 2) *lds_at<uintx4>(wptr[j][part], ring(slot_c, c1)) = wide[j];
            else *lds_at<uintx4>(part == 2 ? wptr[j][2] : flip(wptr[j][2], 16), ring(slot_c, c0)) = wide[j];
          }
        }
      });
    }
  };
  // The page ids of the unit started two vector phases from now go out before the softmax and are awaited after it.
  auto ids_await = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < kLoads; ++j) { pid_new[j] = __builtin_amdgcn_readfirstlane(pid_new[j]); asm volatile("" : "+s"(pid_new[j])); }   // arrived here, not wherever it is used next
  };
  // FP8: the next window's page scales, in three steps a few blocks apart, in wave 0 (whose rows are never all past the end).
  // A window is written two blocks before its first use at the latest, and a whole window after the last read of what was
  // in its place.
  auto fill_scales = [&](int i) __attribute__((always_inline)) {
    if (wave == 0) {
      const int step = i % kWindowBlocks, next = i - step + kWindowBlocks;
      if (step == 2) window_ids(next);
      else if (step == 2 + kWindowBlocks / 4) window_scales();
      else if (step == 2 + kWindowBlocks / 2) window_write(next);
    }
  };
  // A wave whose 32 rows all lie past the tile's last row (ragged last tile of a chunk, or a group
  // call with few rows) keeps its share of the staging and every barrier but skips the products and
  // the softmax: it would only compete with the wave it shares a SIMD with.
  auto run = [&](auto active_c) __attribute__((always_inline)) {
    constexpr bool kActive = decltype(active_c)::value;
    auto block = [&](int i, auto first_c, auto slot_c) __attribute__((always_inline)) {
      constexpr int slot = decltype(slot_c)::value;
      // the pointers could be others in every block, as far as the compiler can tell: it would keep each sum of one and an
      // offset in a register of its own, two hundred of them, instead of using the offset as it is
#pragma unroll
      for (int kk = 0; kk < kKK; ++kk) asm volatile("" : "+v"(kptr[kk]));
#pragma unroll
      for (int dt = 0; dt < kDT; ++dt) asm volatile("" : "+v"(vptr[dt]));
      if constexpr (FP8) {
#pragma unroll
        for (int j = 0; j < kLoads; ++j) {
          asm volatile("" : "+v"(wptr[j][0]), "+v"(wptr[j][1]), "+v"(wptr[j][2]));
          asm volatile("" : "+v"(goff[j][0]), "+v"(goff_last[j][0]));   // (nor widened to 64 bits)
        }
      }
      auto piece = [&](auto pos_c) __attribute__((always_inline)) {
        stage_widen(slot_c, pos_c);
        if constexpr (FP8 && kActive && decltype(pos_c)::value == 24) read_scales(i);
      };
      if constexpr (kActive) {
        __builtin_amdgcn_s_setprio(1);
        matrix_phase(first_c, c_end, ring(slot_c, c0), ring(slot_c, cm1), piece);
        __builtin_amdgcn_s_setprio(0);
      } else {
        static_for<32>(piece);
      }
      PHASE_END();
      stage_addresses();
      if constexpr (FP8 && kActive && slot == 0) fill_scales(i);
      stage_loads(i, slot_c);
      fetch_pids(pid_new, at_new);
      if constexpr (kActive) softmax(i);
      ids_await();
      if constexpr (kEarly && kActive) read_early(ring(slot_c, c0));   // V block i, for the matrix phase that follows
      PHASE_END();
      const int t = ko[0];
#pragma unroll
      for (int d = 0; d + 1 < kRing; ++d) ko[d] = ko[d + 1];
      ko[kRing - 1] = t;
    };
    if constexpr (FP8 && !kActive) {
      // nothing of this side is worked out in front of the branch and kept in registers over the other side's loop
#pragma unroll
      for (int j = 0; j < kLoads; ++j) {
        asm volatile("" : "+v"(kreg[0][j]), "+v"(vreg[0][j]), "+v"(kreg[1][j]), "+v"(vreg[1][j]));
        asm volatile("" : "+v"(goff[j][0]), "+v"(goff_last[j][0]));
      }
    }
    block(0, c_pv, c0);                                 // block 0 has no predecessor: scores only
    // (two blocks at a time and the odd one behind the loop: on a way through the loop from an odd block to the next odd one,
    // the loads of the even block between them would be missing, and the waits by count would have to do with fewer)
    int i = 1;
    for (; i + 1 < n_blocks; i += 2) {
      block(i, c0, c1);
      block(i + 1, c0, c0);
    }
    if (i < n_blocks) block(i, c0, c1);
    if constexpr (kActive) {
      __builtin_amdgcn_s_setprio(1);
      matrix_phase(c0, c_pv, 0, ko[kRing - 1], [](auto) {});
      __builtin_amdgcn_s_setprio(0);
    }
  };
  if (wave_active) run(std::true_type{}); else run(std::false_type{});
  float m_run = seen_max();
  float* const mine = Geo::kMergeApart ? merge_acc_s[Geo::kMergeApart ? (wave & 3) : 0] : (float*)&k_lds[0][0] + (wave & 3) * kMergeAcc;   // HALF only
  float* const mine_ml = merge_ml_s[HALF ? (wave & 3) : 0];
  if constexpr (HALF) {
    // The trailing wave of a pair hands over its half of the tile: accumulators, reference and (per-lane) sum.
    if (grp == 1 && wave_active) {
#pragma unroll
      for (int dt = 0; dt < kDT; ++dt)
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4)
          *(floatx4*)(mine + ((dt * 4 + i4) * 64 + lane) * 4) = floatx4{acc[dt][i4 * 4], acc[dt][i4 * 4 + 1], acc[dt][i4 * 4 + 2], acc[dt][i4 * 4 + 3]};
      mine_ml[lane] = m_run;
      mine_ml[64 + lane] = l_run;
    }
  }
  if (grp == 0) PHASE_END();
  if constexpr (!FP8) DMA_WAIT(0);                   // nothing may still be landing in LDS when the workgroup retires
  if constexpr (HALF) {
    __syncthreads();                                   // the trailing waves' results are in LDS
    if (grp == 1) return;
    if (wave_active) {
      const float* theirs = mine;
      const float m2 = mine_ml[lane], l2 = mine_ml[64 + lane];
      const float m_new = fmaxf(m_run, m2);
      const float m_safe = (m_new == -INFINITY) ? 0.f : m_new;
      const float a1 = __builtin_amdgcn_exp2f(m_run - m_safe), a2 = __builtin_amdgcn_exp2f(m2 - m_safe);
      l_run = l_run * a1 + l2 * a2;
      m_run = m_new;
#pragma unroll
      for (int dt = 0; dt < kDT; ++dt)
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4) {
          const floatx4 o = *(const floatx4*)(theirs + ((dt * 4 + i4) * 64 + lane) * 4);
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[dt][i4 * 4 + e] = acc[dt][i4 * 4 + e] * a1 + o[e] * a2;
        }
    }
  }
#undef PHASE_END
#undef BARRIER_RAW
#undef DMA_WAIT

  // ---- normalise and store.  Where the rows go is worked out again here, from the thread and workgroup numbers, the
  // kernel's arguments and the tile's record, all read anew: what only the end of a tile needs occupies no register
  // during the loop (FP8, D = 128: 256 vector registers of 256 otherwise, and scalar ones that spill).
  const_args_p args_e = (const_args_p)__builtin_amdgcn_kernarg_segment_ptr();
  int block_e = blockIdx.x, tid_e = threadIdx.x;
  asm volatile("" : "+s"(args_e), "+s"(block_e), "+v"(tid_e));
  const int hkv_e = args_e->hkv, group_e = args_e->group;
  int g_e;
  const int tile_e = tile_of(block_e, hkv_e, g_e);
  const const_rec_p rec_e = (const_rec_p)(args_e->tile_rec + (size_t)tile_e * kTileRecWords);
  const int q0_e = rec_e[1], n_e = rec_e[2], qoff_e = rec_e[4], unit = rec_e[7];
  const int lane_e = tid_e & 63, wave_e = __builtin_amdgcn_readfirstlane(tid_e >> 6), row_wave_e = HALF ? (wave_e & 3) : wave_e;
  const int rows_e = min(args_e->tile_tokens, n_e - q0_e) * group_e;
  const int row_e = row_wave_e * kRowsPerWave + (lane_e & 31);
  const bool upper = lane_e >= 32;
  const bool ok = row_e < rows_e;
  l_run = xor32_add(l_run);
  if (unit >= 0) {
    // a piece of a tile: accumulators as they lie, 16 bytes per lane and store, reference and sum of each row
    if (row_wave_e * kRowsPerWave < rows_e) {
      const size_t part = (size_t)(unit + row_wave_e) * hkv_e + g_e;
      float* po = args_e->partial_o + part * (kRowsPerWave * D) + lane_e * 4;
#pragma unroll
      for (int dt = 0; dt < kDT; ++dt)
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4)
          *(floatx4*)(po + (dt * 4 + i4) * 256) = floatx4{acc[dt][i4 * 4], acc[dt][i4 * 4 + 1], acc[dt][i4 * 4 + 2], acc[dt][i4 * 4 + 3]};
      if (!upper) *(floatx2*)(args_e->partial_ml + (part * kRowsPerWave + lane_e) * 2) = floatx2{m_run, l_run};
    }
  } else {
    const int tok_e = row_e / group_e;
    const size_t orow = (size_t)(qoff_e + q0_e + tok_e) * args_e->hq + g_e * group_e + (row_e - tok_e * group_e);
    const float inv = 1.f / l_run;
    // log2 of the row's softmax denominator, for callers that merge this result with another range's
    if (ok && args_e->lse && !upper) args_e->lse[orow] = m_run + __builtin_amdgcn_logf(l_run);
    __bf16* dst = (__bf16*)args_e->out + orow * D + (upper ? 8 : 0);
#pragma unroll
    for (int dt = 0; dt < kDT; ++dt)
      store_row_dims(dst + dt * 32, ok, inv, [&](int i4, int e) __attribute__((always_inline)) { return acc[dt][i4 * 4 + e]; });
  }
  if (args_e->clock_sums && tid_e == 0) {
    atomicAdd(args_e->clock_sums, (unsigned long long)(__builtin_amdgcn_s_memtime() - clock_s[0]));
    atomicAdd(args_e->clock_sums + 1, (unsigned long long)(__builtin_amdgcn_s_memrealtime() - clock_s[1]));
  }
}

template <int D, bool FP8, bool HALF, bool ONCE, int STEP>
__global__ __launch_bounds__(kThreads, HALF && D == 64 && STEP == kBlockTokens ? 4 : 2) void append_mfma_kernel(const AppendArgs a) {
  if constexpr (STEP == 0) {
    __shared__ union {
      AppendLds<D, FP8, HALF, kBlockTokens> one;
      AppendLds<D, FP8, HALF, 2 * kBlockTokens> two;
    } lds;
    int g;
    const int tile = tile_of(blockIdx.x, a.hkv, g);
    const int blocks = ((const __attribute__((address_space(4))) int32_t*)(a.tile_rec + (size_t)min(tile, a.tile_cap - 1) * kTileRecWords))[6];
    if (blocks < kLongTileBlocks) append_tile<D, FP8, HALF, ONCE, kBlockTokens, true>(a, &lds.one);
    else append_tile<D, FP8, HALF, ONCE, 2 * kBlockTokens, true>(a, &lds.two);
  } else {
    append_tile<D, FP8, HALF, ONCE, STEP, false>(a, nullptr);
  }
}

// Merge of the pieces of a tile: one wave per (cut tile, KV head, 32 rows, 32 dims), lanes as in the append kernel's
// accumulators.  M = max_s m_s; out = sum_s 2^(m_s - M) o_s / sum_s 2^(m_s - M) l_s.  A piece that a row did not see has
// m = -inf and weight zero; some piece has seen the row (its own token is in the last one it sees).
// Bound by the latency of the partials' loads (a few hundred kilobytes per tile out of L2 and the memory-side cache):
// four waves of different dims per row group keep each wave's chain to one 4 KB load per piece, and four pieces are
// under way at a time.
template <int D>
__global__ __launch_bounds__(256) void append_merge_kernel(const AppendArgs a) {
  constexpr int kDT = D / 32;
  const int lane = threadIdx.x & 63;
  const int n32 = lane & 31, h2 = lane >> 5;
  const int wave = threadIdx.x >> 6;
  constexpr int kWgsPerTile = kWaves * kDT / 4;
  // Where no tile was cut the launch costs its start, so nothing is worked out before the count is there.
  const int n_merges = a.header[kPlanMerges];
  const int sub = blockIdx.x / a.hkv, g = blockIdx.x - sub * a.hkv;    // head fastest, as in the append kernel: with 8 heads the XCD that wrote the partials reads them
  const int m = sub / kWgsPerTile, unit = (sub - m * kWgsPerTile) * 4 + wave;
  const int dt = unit % kDT, row_wave = unit / kDT;
  if (m >= n_merges) return;
  const int32_t* rec = a.merge_rec + (size_t)m * kTileRecWords;
  const int q0 = rec[0], n_b = rec[1], q_off = rec[2], unit0 = rec[3], pieces = rec[4];
  const int rows_here = min(a.tile_tokens, n_b - q0) * a.group;
  if (row_wave * kRowsPerWave >= rows_here) return;
  const size_t stride = (size_t)((rows_here + kRowsPerWave - 1) / kRowsPerWave) * a.hkv;   // parts from one piece to the next
  const size_t part0 = (size_t)(unit0 + row_wave) * a.hkv + g;
  const floatx2* ml = (const floatx2*)a.partial_ml + part0 * kRowsPerWave + n32;
  const float* po = a.partial_o + part0 * (kRowsPerWave * D) + (dt * 4 * 64 + lane) * 4;
  floatx4 o[4];
#pragma unroll
  for (int i4 = 0; i4 < 4; ++i4) o[i4] = floatx4{0.f, 0.f, 0.f, 0.f};
  float ref = -INFINITY, l = 0.f;
  // folds kN pieces from s0 on (past the last one: the last one again, with weight zero)
  auto fold = [&](int s0, auto n_c) __attribute__((always_inline)) {
    constexpr int kN = decltype(n_c)::value;
    floatx2 x[kN];
    floatx4 y[kN][4];
#pragma unroll
    for (int i = 0; i < kN; ++i) {
      const size_t s = min(s0 + i, pieces - 1) * stride;
      x[i] = ml[s * kRowsPerWave];
#pragma unroll
      for (int i4 = 0; i4 < 4; ++i4) y[i][i4] = *(const floatx4*)(po + s * (kRowsPerWave * D) + i4 * 256);
    }
    float top = ref;
#pragma unroll
    for (int i = 0; i < kN; ++i) {
      if (s0 + i >= pieces) {                              // (zero times an infinity would not be zero)
        x[i][0] = -INFINITY;
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4) y[i][i4] = floatx4{0.f, 0.f, 0.f, 0.f};
      }
      top = fmaxf(top, x[i][0]);
    }
    const float base = (top == -INFINITY) ? 0.f : top;
    const float keep = __builtin_amdgcn_exp2f(ref - base);
    ref = top;
    l *= keep;
#pragma unroll
    for (int i4 = 0; i4 < 4; ++i4) o[i4] *= keep;
#pragma unroll
    for (int i = 0; i < kN; ++i) {
      const float f = __builtin_amdgcn_exp2f(x[i][0] - base);
      l += f * x[i][1];
#pragma unroll
      for (int i4 = 0; i4 < 4; ++i4) o[i4] += f * y[i][i4];
    }
  };
  // four pieces under way at a time; loading one twice is as slow as loading another, so the usual two and three have
  // folds of their own
  if (pieces == 2) fold(0, std::integral_constant<int, 2>{});
  else if (pieces == 3) fold(0, std::integral_constant<int, 3>{});
  else for (int s0 = 0; s0 < pieces; s0 += 4) fold(s0, std::integral_constant<int, 4>{});
  const int row = row_wave * kRowsPerWave + n32;
  const bool row_ok = row < rows_here;
  const int tok = row / a.group;
  const size_t orow = (size_t)(q_off + q0 + tok) * a.hq + g * a.group + (row - tok * a.group);
  if (row_ok && a.lse && dt == 0 && h2 == 0) a.lse[orow] = ref + __builtin_amdgcn_logf(l);
  const float inv = 1.f / l;
  store_row_dims((__bf16*)a.out + orow * D + dt * 32 + h2 * 8, row_ok, inv, [&](int i4, int e) { return o[i4][e]; });
}

}  // namespace

hipError_t launch_append_merge(const AppendArgs& a, int head_dim, int max_merges, hipStream_t s) {
  const dim3 grid((unsigned)((max_merges * kWaves * (head_dim / 32) + 3) / 4 * a.hkv));
  if (head_dim == 128) {
    hipLaunchKernelGGL((append_merge_kernel<128>), grid, dim3(256), 0, s, a);
  } else {
    hipLaunchKernelGGL((append_merge_kernel<64>), grid, dim3(256), 0, s, a);
  }
  return hipGetLastError();
}

hipError_t launch_append_mfma(const AppendArgs& a, int head_dim, bool fp8, bool half_tiles, int grid, hipStream_t s) {
  if (head_dim != 128 && head_dim != 64) return hipErrorInvalidValue;
  const bool once = half_tiles && a.noncausal;
  const bool short_tiles = a.max_pages < kLongTileBlocks * (kAppendBlockTokens / kPageSize);   // no context reaches a long tile
  auto launch = [&](auto d, auto f) {
    constexpr int D = decltype(d)::value;
    constexpr bool F = decltype(f)::value;
    if (once) {
      hipLaunchKernelGGL((append_mfma_kernel<D, F, true, true, F ? 2 * kAppendBlockTokens : kAppendBlockTokens>), dim3(grid), dim3(kThreads), 0, s, a);
    } else if (half_tiles && F && !short_tiles) {
      hipLaunchKernelGGL((append_mfma_kernel<D, F, true, false, F ? 0 : kAppendBlockTokens>), dim3(grid), dim3(kThreads), 0, s, a);
    } else if (half_tiles) {
      hipLaunchKernelGGL((append_mfma_kernel<D, F, true, false, kAppendBlockTokens>), dim3(grid), dim3(kThreads), 0, s, a);
    } else {
      hipLaunchKernelGGL((append_mfma_kernel<D, F, false, false, kAppendBlockTokens>), dim3(grid), dim3(kThreads), 0, s, a);
    }
  };
  std::integral_constant<int, 128> d128;
  std::integral_constant<int, 64> d64;
  if (head_dim == 128 && fp8) launch(d128, std::true_type{});
  else if (head_dim == 128) launch(d128, std::false_type{});
  else if (fp8) launch(d64, std::true_type{});
  else launch(d64, std::false_type{});
  return hipGetLastError();
}

}  // namespace rollattn
