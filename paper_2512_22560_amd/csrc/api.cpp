// Host side of librollattn: argument checks, workspace layout, the host twin of the
// partition rule, and the launch sequence of each entry point.  Nothing here touches the
// GPU before every argument check has passed.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

#include "host_plan.h"
#include "rollattn_internal.h"

// Scratch memory of attn_decode_static, the decode call for callers that cannot allocate: one array per GPU,
// part of the library's code object, alive until the process ends.  In host code this name is only a handle for
// hipGetSymbolAddress; the device address it stands for is looked up once per device (static_scratch_ptr).
constexpr size_t kStaticScratchBytes = (size_t)36 << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];
// Profiling only: what the append kernel adds up while profiling is on (shader-clock cycles, constant-rate ticks).
static __device__ unsigned long long clock_sums[2];

namespace rollattn {

namespace {

std::mutex g_mu;
std::string g_hip_error;
bool g_profile = false;
struct EventPair {
  hipEvent_t a, b;
};
constexpr size_t kMaxEvents = 1024;

size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

int fail_hip(hipError_t e) {
  std::lock_guard<std::mutex> lk(g_mu);
  g_hip_error = hipGetErrorString(e);
  return ROLLATTN_EHIP;
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

int dtype_bytes(int dt) { return dt == ROLLATTN_F32 ? 4 : dt == ROLLATTN_BF16 ? 2 : 1; }

// Descriptor checks shared by every entry point.
int check_desc(const rollattn_desc* d, bool need_scales = true) {
  if (!d) return ROLLATTN_EINVAL;
  if (d->batch < 0 || d->num_pages < 0 || d->max_pages_per_seq < 1) return ROLLATTN_EINVAL;
  if (d->num_q_heads < 1 || d->num_kv_heads < 1 || d->num_q_heads % d->num_kv_heads) return ROLLATTN_ESHAPE;
  if (d->head_dim != 64 && d->head_dim != 128) return ROLLATTN_ESHAPE;
  if (d->page_size != kPageSize) return ROLLATTN_ESHAPE;
  if (d->num_pages * (int64_t)d->num_kv_heads > INT32_MAX) return ROLLATTN_ESHAPE;   // (page, head) tiles are counted in 32 bits
  const bool f32 = d->q_dtype == ROLLATTN_F32 && d->kv_dtype == ROLLATTN_F32;
  const bool bf = d->q_dtype == ROLLATTN_BF16 && (d->kv_dtype == ROLLATTN_BF16 || d->kv_dtype == ROLLATTN_FP8_E4M3);
  if (!f32 && !bf) return ROLLATTN_EDTYPE;
  if (d->kv_dtype == ROLLATTN_FP8_E4M3 && need_scales) {
    if (!d->k_scale || !d->v_scale) return ROLLATTN_EDTYPE;
    if (!aligned16(d->k_scale) || !aligned16(d->v_scale)) return ROLLATTN_EALIGN;
  }
  if (!(d->sm_scale == d->sm_scale) || std::isinf(d->sm_scale)) return ROLLATTN_EINVAL;
  return ROLLATTN_OK;
}

// Timing events are created when profiling is switched on, never inside an attention call: a call only
// records a pair from the pool, and records nothing on a stream that is being captured into a graph
// (events recorded during capture cannot be read back).
std::vector<EventPair> g_pool;
size_t g_used = 0;
int32_t g_debug_workers = 0;                  // testing: decode plans are cut for this many workers (0: all of them)
unsigned long long* g_clock_sums = nullptr;   // device address of clock_sums on the device profiling was switched on for
int g_clock_dev = -1;                         // ... and that device: launches on other devices do not count

struct ProfileScope {
  hipStream_t s;
  bool on = false;
  EventPair ev{};
  explicit ProfileScope(hipStream_t stream) : s(stream) {
    std::lock_guard<std::mutex> lk(g_mu);
    if (!g_profile || g_used >= g_pool.size()) return;
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &st) != hipSuccess || st != hipStreamCaptureStatusNone) return;
    ev = g_pool[g_used++];
    on = true;
    (void)hipEventRecord(ev.a, s);
  }
  void stop() {
    if (!on) return;
    (void)hipEventRecord(ev.b, s);
    on = false;
  }
};

}  // namespace

WorkspaceLayout decode_layout(const rollattn_desc& d) {
  WorkspaceLayout w{};
  const int group = d.num_q_heads / d.num_kv_heads;
  const bool f32 = d.q_dtype == ROLLATTN_F32;
  w.head_tile = f32 ? kF32HeadTile : kMfmaHeadTile;
  w.rows_per_b = d.num_kv_heads * ((group + w.head_tile - 1) / w.head_tile);
  w.workers = f32 ? kF32DecodeWgs : kMfmaDecodeWgs * 4;
  size_t off = 0;
  w.header = off;      off += align256(sizeof(int32_t) * kPlanWords);
  w.prefix = off;      off += align256(sizeof(int32_t) * ((size_t)d.batch + 1));
  w.wstart = off;      off += align256(sizeof(int32_t) * 4 * (size_t)w.workers);
  w.partial_ml = off;  off += align256(sizeof(float) * 2 * (size_t)w.workers * w.head_tile * 2);
  w.partial_o = off;   off += align256(sizeof(float) * 2 * (size_t)w.workers * w.head_tile * d.head_dim);
  w.total = off;
  return w;
}

// Workers the decode partition is cut for: all of them, unless rollattn_debug_set_decode_workers says fewer.
static int32_t plan_workers(const WorkspaceLayout& w) {
  std::lock_guard<std::mutex> lk(g_mu);
  return (g_debug_workers > 0 && g_debug_workers < w.workers) ? g_debug_workers : w.workers;
}

WorkspaceLayout append_layout(const rollattn_desc& d, int32_t total_q, int32_t units) {
  WorkspaceLayout w{};
  const int group = d.num_q_heads / d.num_kv_heads;
  // room for the list of half-size tiles too (a call whose chunks are all short chooses them)
  const int tile_tokens = std::max(1, kAppendTileRows / 2 / group);
  w.workers = (int32_t)std::min<int64_t>((int64_t)total_q / tile_tokens + d.batch + 1, INT32_MAX);
  // Tiles may be cut into pieces, within limits on the whole launch
  if (d.q_dtype != ROLLATTN_F32 && d.num_kv_heads <= kSplitMerges) {
    w.max_pieces = kSplitPieces / d.num_kv_heads;
    w.max_merges = kSplitMerges / d.num_kv_heads;
    w.max_units = units / d.num_kv_heads;
  }
  const size_t rec = sizeof(int32_t) * kTileRecWords, parts = (size_t)w.max_units * d.num_kv_heads;
  size_t off = 0;
  w.header = off;      off += align256(sizeof(int32_t) * kPlanWords);
  w.wstart = off;
  w.prefix = off;
  w.total = off + align256(rec * (size_t)w.workers);
  off += align256(rec * (size_t)w.max_pieces);
  w.merge_rec = off;   off += align256(rec * (size_t)w.max_merges);
  w.cut_list = std::max(w.total, off);
  w.partial_ml = off;  off += align256(sizeof(float) * 2 * kUnitRows * parts);
  w.partial_o = off;   off += align256(sizeof(float) * kUnitRows * d.head_dim * parts);
  w.cut_total = std::max(w.total, off);
  return w;
}

}  // namespace rollattn

using namespace rollattn;

static_assert(kPlanBlockTokens == kBlockTokens, "the host twin and the kernels cut rows into the same blocks");
// kLentUnits partials of an append call's pieces take the room that the decode partials of the same descriptor take, and its
// list no more than the start records: a workspace that is large enough for the decode call lets an append call cut its
// tiles, and attn_decode_shared, and attn_step where the workspace has no more, lend the one region to both halves in turn.
static_assert(kLentUnits * kUnitRows == 2 * kMfmaDecodeWgs * 4 * kMfmaHeadTile, "partials of append and decode");
static_assert(kTileRecWords * (kSplitPieces + kSplitMerges) <= 4 * kMfmaDecodeWgs * 4, "records of append and decode");

// What an append call is told to bring: room for all the pieces its tiles may be cut into, unless it has more tiles than
// are ever cut (it has rows / 256 at least, counted with a group's heads).
static size_t append_bytes(const rollattn_desc& d, int32_t total_q, int64_t rows) {
  const WorkspaceLayout w = append_layout(d, total_q);
  return rows / std::max(1, kAppendTileRows / (d.num_q_heads / d.num_kv_heads)) <= w.max_pieces ? w.cut_total : w.total;
}

extern "C" {

size_t rollattn_workspace_bytes(const rollattn_desc* desc, int32_t total_q) {
  if (check_desc(desc) != ROLLATTN_OK || total_q < 0) return 0;
  return std::max(decode_layout(*desc).total, append_bytes(*desc, total_q, total_q > desc->batch ? total_q : INT32_MAX));
}

int32_t rollattn_plan_capacity(const rollattn_desc* desc) {
  if (check_desc(desc, false) != ROLLATTN_OK) return 0;
  const WorkspaceLayout w = decode_layout(*desc);
  // every worker boundary and every row end closes one segment
  const int64_t cap = (int64_t)w.workers + (int64_t)desc->batch * w.rows_per_b;
  return (int32_t)std::min<int64_t>(cap, INT32_MAX);
}

int rollattn_debug_plan(const rollattn_desc* desc, const int32_t* ctx_lens_host, int32_t* per_out,
                        int32_t* total_out, int32_t* segments_out, int32_t* n_segments) {
  int rc = check_desc(desc, false);
  if (rc) return rc;
  if ((!ctx_lens_host && desc->batch > 0) || !per_out || !total_out || !n_segments) return ROLLATTN_EINVAL;
  const WorkspaceLayout w = decode_layout(*desc);
  const int32_t workers = plan_workers(w);
  const HostPlan p = host_plan(ctx_lens_host, desc->batch, w.rows_per_b, workers);
  *per_out = p.per;
  *total_out = p.total;
  *n_segments = expand_segments(p, desc->batch, w.rows_per_b, workers, segments_out, rollattn_plan_capacity(desc));
  return ROLLATTN_OK;
}

int rollattn_debug_read_plan(const rollattn_desc* desc, const void* workspace, int32_t* per_out,
                             int32_t* total_out, int32_t* starts_out, void* hip_stream) {
  int rc = check_desc(desc, false);
  if (rc) return rc;
  if (!workspace || !per_out || !total_out || !starts_out) return ROLLATTN_EINVAL;
  const WorkspaceLayout w = decode_layout(*desc);
  hipStream_t s = (hipStream_t)hip_stream;
  hipError_t e = hipStreamSynchronize(s);
  if (e != hipSuccess) return fail_hip(e);
  const char* base = (const char*)workspace;
  int32_t header[kPlanWords];
  e = hipMemcpy(header, base + w.header, sizeof(header), hipMemcpyDeviceToHost);
  if (e == hipSuccess)
    e = hipMemcpy(starts_out, base + w.wstart, sizeof(int32_t) * 4 * (size_t)plan_workers(w), hipMemcpyDeviceToHost);
  if (e != hipSuccess) return fail_hip(e);
  *per_out = header[kPlanPer];
  *total_out = header[kPlanTotal];
  return ROLLATTN_OK;
}

int32_t rollattn_append_plan_capacity(const rollattn_desc* desc, int32_t total_q) {
  if (check_desc(desc, false) != ROLLATTN_OK || total_q < 0) return 0;
  return append_layout(*desc, total_q).workers;
}

int rollattn_debug_read_append_plan(const rollattn_desc* desc, const void* workspace, int32_t total_q, int32_t* n_tiles_out,
                                    int32_t* tiles_out, void* hip_stream) {
  int rc = check_desc(desc, false);
  if (rc) return rc;
  if (!workspace || !n_tiles_out || !tiles_out || total_q < 0) return ROLLATTN_EINVAL;
  const WorkspaceLayout w = append_layout(*desc, total_q);
  hipStream_t s = (hipStream_t)hip_stream;
  hipError_t e = hipStreamSynchronize(s);
  if (e != hipSuccess) return fail_hip(e);
  const char* base = (const char*)workspace;
  int32_t header[kPlanWords];
  e = hipMemcpy(header, base + w.header, sizeof(header), hipMemcpyDeviceToHost);
  if (e != hipSuccess) return fail_hip(e);
  const int32_t n = std::max(0, std::min(header[kPlanTiles], header[kPlanMerges] > 0 ? w.max_pieces : w.workers));
  std::vector<int32_t> rec((size_t)n * kTileRecWords);
  if (n) e = hipMemcpy(rec.data(), base + w.wstart, sizeof(int32_t) * rec.size(), hipMemcpyDeviceToHost);
  if (e != hipSuccess) return fail_hip(e);
  int32_t tiles = 0;
  for (int32_t i = 0; i < n && tiles < w.workers; ++i) {
    const int32_t* r = rec.data() + (size_t)i * kTileRecWords;
    if (r[5] != 0) continue;                     // a later piece of the tile before it
    tiles_out[2 * tiles] = r[0];
    tiles_out[2 * tiles + 1] = r[1];
    ++tiles;
  }
  *n_tiles_out = tiles;
  return ROLLATTN_OK;
}

int32_t rollattn_plan_workers(const rollattn_desc* desc) {
  if (check_desc(desc, false) != ROLLATTN_OK) return 0;
  return plan_workers(decode_layout(*desc));
}

int32_t rollattn_debug_set_decode_workers(int32_t workers) {
  std::lock_guard<std::mutex> lk(g_mu);
  const int32_t before = g_debug_workers;
  g_debug_workers = workers > 0 ? workers : 0;
  return before;
}

// Shape limits of the decode path and of the append path beyond the descriptor checks; the entry points that
// chain several launches check both before the first one.
static int decode_limits(const rollattn_desc& d) {
  const WorkspaceLayout w = decode_layout(d);
  // the block sequence is indexed with 32-bit integers
  if ((int64_t)d.batch * w.rows_per_b * ((int64_t)d.max_pages_per_seq / 2 + 1) > INT32_MAX) return ROLLATTN_ESHAPE;
  // a worker's start record packs the row index into 11 bits and the block index into 20
  if (w.rows_per_b > 2047 || d.max_pages_per_seq / 2 + 1 > (1 << 20)) return ROLLATTN_ESHAPE;
  return ROLLATTN_OK;
}
static int append_limits(const rollattn_desc& d) {
  if (d.q_dtype != ROLLATTN_F32 && d.num_q_heads / d.num_kv_heads > kAppendTileRows) return ROLLATTN_ESHAPE;
  return ROLLATTN_OK;
}

// A decode call whose arguments have been checked: its plan's inputs and its kernels' arguments.
struct DecodeCall {
  DecodePlanArgs plan;
  DecodeArgs args;
};

// Argument checks of attn_decode and the arguments of its launches; lse (optional, device [B][Hq]) receives log2 of every
// row's softmax denominator.  q_lens / q_offsets (both or neither): the mixed step, see DecodeArgs.  call stays untouched,
// with an empty batch, where there is nothing to launch.
static int decode_prepare(const rollattn_desc* desc, const void* q, const void* k_pages, const void* v_pages,
                          const int32_t* page_table, const int32_t* ctx_lens, void* out, void* workspace,
                          size_t workspace_bytes, float* lse, const int32_t* q_lens, const int32_t* q_offsets, DecodeCall* call) {
  int rc = check_desc(desc);
  if (rc) return rc;
  if (desc->batch == 0) return ROLLATTN_OK;
  if (!q || !k_pages || !v_pages || !page_table || !ctx_lens || !out || !workspace) return ROLLATTN_EINVAL;
  if (!aligned16(q) || !aligned16(k_pages) || !aligned16(v_pages) || !aligned16(page_table) ||
      !aligned16(ctx_lens) || !aligned16(out) || !aligned16(workspace))
    return ROLLATTN_EALIGN;
  const WorkspaceLayout w = decode_layout(*desc);
  if (workspace_bytes < w.total) return ROLLATTN_EWORKSPACE;
  rc = decode_limits(*desc);
  if (rc) return rc;

  char* base = (char*)workspace;
  DecodeArgs& a = call->args;
  a.q = q; a.k_pages = k_pages; a.v_pages = v_pages; a.page_table = page_table; a.ctx_lens = ctx_lens;
  a.out = out; a.k_scale = desc->k_scale; a.v_scale = desc->v_scale;
  a.header = (const int32_t*)(base + w.header);
  a.prefix = (const int32_t*)(base + w.prefix);
  a.wstart = (const int32_t*)(base + w.wstart);
  a.partial_ml = (float*)(base + w.partial_ml);
  a.partial_o = (float*)(base + w.partial_o);
  a.batch = desc->batch; a.hq = desc->num_q_heads; a.hkv = desc->num_kv_heads;
  a.group = desc->num_q_heads / desc->num_kv_heads; a.max_pages = desc->max_pages_per_seq;
  a.head_tile = w.head_tile; a.rows_per_b = w.rows_per_b;
  a.scale_log2 = desc->sm_scale * 1.4426950408889634f;
  a.lse = lse;
  a.q_lens = q_lens;
  a.q_offsets = q_offsets;
  DecodePlanArgs& d = call->plan;
  d.ctx_lens = ctx_lens; d.q_lens = q_lens; d.batch = desc->batch; d.rows_per_b = w.rows_per_b;
  // (the launch has w.workers workers whatever the partition is cut for: the others get a record without blocks)
  d.workers = plan_workers(w); d.slots = w.workers;
  // (whole rows instead, where the plan says so: not where the number of workers is forced)
  const int n_ht = w.rows_per_b / desc->num_kv_heads;
  d.whole_busy = (desc->kv_dtype == ROLLATTN_FP8_E4M3 ? kWholeBusyFp8 : kWholeBusy) * n_ht;   // (several rows read the same K and V)
  d.whole_gain = kWholeGain * (a.group * desc->head_dim) / (float)(n_ht * kMfmaHeadTile * 128);   // (as large as its partials)
  a.whole_rows = desc->q_dtype != ROLLATTN_F32 && d.workers == w.workers;
  if (desc->q_dtype != ROLLATTN_F32) d.page_table = page_table;
  d.max_pages = desc->max_pages_per_seq; d.num_pages = desc->num_pages; d.head_tiles = w.rows_per_b > desc->num_kv_heads;
  d.header = (int32_t*)(base + w.header); d.prefix = (int32_t*)(base + w.prefix); d.wstart = (int32_t*)(base + w.wstart);
  return ROLLATTN_OK;
}

// The launches behind the plan.
static int decode_launch(const rollattn_desc* desc, const DecodeArgs& a, hipStream_t s) {
  const bool f32 = desc->q_dtype == ROLLATTN_F32;
  hipError_t e;
  {
    ProfileScope prof(s);
    if (f32) {
      e = launch_decode_f32(a, desc->head_dim, kF32DecodeWgs, s);
    } else {
      e = launch_decode_mfma(a, desc->head_dim, desc->kv_dtype == ROLLATTN_FP8_E4M3, a.whole_rows && desc->head_dim == 64 ? kMfmaDecodeWgsD64 : kMfmaDecodeWgs, s);
    }
    prof.stop();
  }
  if (e != hipSuccess) return fail_hip(e);
  e = a.shared.result ? launch_combine_shared(a, desc->head_dim, s) : launch_combine(a, desc->head_dim, !f32, s);
  if (e != hipSuccess) return fail_hip(e);
  return ROLLATTN_OK;
}

static int decode_impl(const rollattn_desc* desc, const void* q, const void* k_pages, const void* v_pages,
                       const int32_t* page_table, const int32_t* ctx_lens, void* out, void* workspace,
                       size_t workspace_bytes, void* hip_stream, float* lse) {
  DecodeCall call{};
  const int rc = decode_prepare(desc, q, k_pages, v_pages, page_table, ctx_lens, out, workspace, workspace_bytes, lse, nullptr,
                                nullptr, &call);
  if (rc || call.args.batch == 0) return rc;
  hipStream_t s = (hipStream_t)hip_stream;
  const bool f32 = desc->q_dtype == ROLLATTN_F32;
  // A launch of its own for the plan costs its 3 to 5 us and the gap behind it.  Small batches do without.  Over MFMA every
  // wave finds its own start, a lane per trajectory (64 contexts of 512 .. 8k, 32/8/128, bf16: 159.6 -> 155.0 us; with more
  // trajectories the step is long enough not to notice).  Short float32 contexts are not cut at all while their rows fit the
  // chip at once (8/2/64, one launch against three: 4 contexts of 256 tokens 4.2 against 10.5 us, 64 of 512 tokens 11.3
  // against 16.3; but 256 of 16 tokens 13.2 against 10.5).
  const bool alone = f32 ? desc->max_pages_per_seq <= kDirectPages && (int64_t)desc->batch * call.args.rows_per_b <= kNumCUs
                         : desc->batch <= kWavePlanBatch;
  if (alone) {
    call.args.plan = call.plan;
    call.args.whole_rows = 0;
  } else {
    const hipError_t e = launch_plan_decode(call.plan, s);
    if (e != hipSuccess) return fail_hip(e);
  }
  if (f32 && call.args.plan.batch) {
    ProfileScope prof(s);
    const hipError_t e = launch_decode_f32_direct(call.args, desc->head_dim, s);
    prof.stop();
    return e == hipSuccess ? ROLLATTN_OK : fail_hip(e);
  }
  return decode_launch(desc, call.args, s);
}

int attn_decode(const rollattn_desc* desc, const void* q, const void* k_pages, const void* v_pages,
                const int32_t* page_table, const int32_t* ctx_lens, void* out, void* workspace,
                size_t workspace_bytes, void* hip_stream) {
  return decode_impl(desc, q, k_pages, v_pages, page_table, ctx_lens, out, workspace, workspace_bytes, hip_stream, nullptr);
}

namespace {
constexpr int kMaxDevices = 64;
void* g_static_ptr[kMaxDevices] = {};   // device address of `scratch` on each GPU, null until looked up

// Address of the current device's copy of `scratch`; the lookup runs once per device, with that device current.
int static_scratch_ptr(void** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return fail_hip(e);
  if (dev < 0 || dev >= kMaxDevices) return fail_hip(hipErrorInvalidDevice);
  {
    std::lock_guard<std::mutex> lk(g_mu);
    if (g_static_ptr[dev]) {
      *out = g_static_ptr[dev];
      return ROLLATTN_OK;
    }
  }
  void* p = nullptr;
  e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
  if (e != hipSuccess) return fail_hip(e);
  if (!p) return fail_hip(hipErrorInvalidSymbol);
  std::lock_guard<std::mutex> lk(g_mu);
  g_static_ptr[dev] = p;
  *out = p;
  return ROLLATTN_OK;
}
}  // namespace

size_t rollattn_static_scratch_bytes(void) { return kStaticScratchBytes; }

int rollattn_static_init(void) {
  void* p = nullptr;
  return static_scratch_ptr(&p);
}

int attn_decode_static(const rollattn_desc* desc, const void* q, const void* k_pages, const void* v_pages,
                       const int32_t* page_table, const int32_t* ctx_lens, void* out, void* hip_stream) {
  int rc = check_desc(desc);
  if (rc) return rc;
  if (desc->batch == 0) return ROLLATTN_OK;
  if (decode_layout(*desc).total > kStaticScratchBytes) return ROLLATTN_ELIMIT;
  void* ws = nullptr;
  rc = static_scratch_ptr(&ws);
  if (rc) return rc;
  return decode_impl(desc, q, k_pages, v_pages, page_table, ctx_lens, out, ws, kStaticScratchBytes, hip_stream, nullptr);
}

// attn_append proper.  table_stride: int32 entries between the page-table rows of consecutive
// trajectories; noncausal: every row sees all of [0, L_b) (then n_b <= L_b is not required);
// lse as in decode_impl, [total_q][Hq].  table_stride and noncausal are for the bf16 kernels only.  lender: the decode half
// of the same call, launched behind this one, whose room for partials this one may use first (null: a call of its own).
// Time in us of a block (64 tokens) of an append tile with few CUs busy and with all of them, from the slope over contexts
// of 1k to 8k with 8 and 256 workgroups: what the plan prices pieces with.
struct BlockTime {
  float alone, full;
};
static BlockTime block_time(const rollattn_desc& d, bool half_tiles) {
  const bool fp8 = d.kv_dtype == ROLLATTN_FP8_E4M3;
  if (d.head_dim == 128) return half_tiles ? (fp8 ? BlockTime{0.85f, 1.10f} : BlockTime{0.76f, 1.42f}) : (fp8 ? BlockTime{1.28f, 1.82f} : BlockTime{1.05f, 1.75f});
  return half_tiles ? (fp8 ? BlockTime{0.74f, 0.79f} : BlockTime{0.60f, 0.82f}) : (fp8 ? BlockTime{1.21f, 1.32f} : BlockTime{0.89f, 1.07f});
}

struct AppendCall {
  AppendPlanArgs plan;
  AppendArgs args;
  bool half_tiles;
  int32_t tile_cap, max_merges;    // room in the list; tiles that may have been cut (0: no merge)
};

static int append_prepare(const rollattn_desc* desc, const void* q_chunk, const int32_t* q_lens, const int32_t* q_offsets,
                          int32_t total_q, int32_t max_q_len, const void* k_pages, const void* v_pages,
                          const int32_t* page_table, const int32_t* ctx_lens, void* out, void* workspace,
                          size_t workspace_bytes, int32_t table_stride, bool noncausal, float* lse, bool skip_unit_chunks,
                          const DecodeArgs* lender, AppendCall* call) {
  int rc = check_desc(desc);
  if (rc) return rc;
  if (total_q < 0 || max_q_len < 0) return ROLLATTN_EINVAL;
  rc = append_limits(*desc);
  if (rc) return rc;
  if (desc->batch == 0 || total_q == 0) return ROLLATTN_OK;
  // (the lengths of a non-causal call's chunks are the plan's own)
  if (!q_chunk || !k_pages || !v_pages || !page_table || !out || !workspace) return ROLLATTN_EINVAL;
  if (!noncausal && (!q_lens || !q_offsets || !ctx_lens)) return ROLLATTN_EINVAL;
  if (!aligned16(q_chunk) || !aligned16(q_lens) || !aligned16(q_offsets) || !aligned16(k_pages) ||
      !aligned16(v_pages) || !aligned16(page_table) || !aligned16(ctx_lens) || !aligned16(out) ||
      !aligned16(workspace))
    return ROLLATTN_EALIGN;
  WorkspaceLayout w = append_layout(*desc, total_q);
  if (workspace_bytes < w.total) return ROLLATTN_EWORKSPACE;
  const bool lent = lender && workspace_bytes < w.cut_total;
  if (lent || workspace_bytes < w.cut_total) w = append_layout(*desc, total_q, kLentUnits);

  char* base = (char*)workspace;
  AppendArgs& a = call->args;
  a.q = q_chunk; a.k_pages = k_pages; a.v_pages = v_pages; a.page_table = page_table; a.ctx_lens = ctx_lens;
  a.q_lens = q_lens; a.q_offsets = q_offsets; a.out = out; a.k_scale = desc->k_scale; a.v_scale = desc->v_scale;
  a.header = (int32_t*)(base + w.header);
  a.tile_rec = (const int32_t*)(base + w.wstart);
  a.batch = desc->batch; a.hq = desc->num_q_heads; a.hkv = desc->num_kv_heads;
  a.group = desc->num_q_heads / desc->num_kv_heads; a.max_pages = table_stride;
  a.tile_tokens = std::max(1, kAppendTileRows / a.group);
  // No chunk longer than half a tile (a few new tokens per trajectory; the members of a group in attn_decode_shared):
  // half tiles, whose blocks the two waves of a SIMD share
  const bool half_tiles = call->half_tiles = desc->q_dtype != ROLLATTN_F32 && (int64_t)max_q_len * a.group <= kAppendTileRows / 2;
  if (half_tiles) a.tile_tokens = std::max(1, kAppendTileRows / 2 / a.group);
  // tiles this call can have at most (<= the capacity of the workspace, which is laid out for half tiles), or pieces
  const int32_t max_tiles = (int32_t)std::min<int64_t>((int64_t)total_q / a.tile_tokens + desc->batch + 1, w.workers);
  // ... and at least (every group of attn_decode_shared is one; in a mixed step up to B rows are not chunk rows): a list
  // that is too long to be cut, or as good as even already, needs neither the decision nor the merge launch
  const int64_t min_tiles = noncausal ? desc->batch : ((int64_t)total_q - (skip_unit_chunks ? desc->batch : 0)) / a.tile_tokens;
  // ... as does a table whose contexts are all too short: the least that pays is a lone tile cut into shortest pieces.
  // Whether the workspace has room is told from its size alone: one as large as the call is told to bring has, one that is
  // large enough for a decode call has for kLentUnits.
  const BlockTime t = block_time(*desc, half_tiles);
  const float start = kPieceUs / t.full;
  const int32_t min_longest = std::max(2 * kMinPieceBlocks, (int32_t)std::ceil(((t.alone * (kMinPieceBlocks + start) + kMergeUs + kCallUs + kSplitGainUs) / kSplitGain - kCallUs) / t.alone - start));
  const bool may_cut = min_tiles <= w.max_pieces && !(noncausal && min_tiles * a.hkv >= kNumCUs) &&
                       desc->max_pages_per_seq > (min_longest - 1) * (kAppendBlockTokens / kPageSize) &&
                       workspace_bytes >= (lent ? w.cut_list : w.cut_total);
  const int32_t max_pieces = may_cut ? w.max_pieces : 0;
  // (the launch has room for no more pieces than the plan may choose: two rounds above the tiles, none shorter than it may be)
  const int64_t per_tile = (desc->max_pages_per_seq + (int64_t)kMinPieceBlocks * (kAppendBlockTokens / kPageSize) - 1) / (kMinPieceBlocks * (kAppendBlockTokens / kPageSize));
  const int32_t tile_cap = (int32_t)std::max<int64_t>(max_tiles, std::min<int64_t>({max_pieces, (int64_t)max_tiles + split_extra_pieces(a.hkv), max_tiles * per_tile}));
  a.tile_cap = tile_cap;
  a.merge_rec = (const int32_t*)(base + w.merge_rec);
  a.partial_ml = lent ? lender->partial_ml : (float*)(base + w.partial_ml);
  a.partial_o = lent ? lender->partial_o : (float*)(base + w.partial_o);
  a.total_q = total_q;
  a.scale_log2 = desc->sm_scale * 1.4426950408889634f;
  a.lse = lse;
  a.noncausal = noncausal ? 1 : 0;

  AppendPlanArgs& pa = call->plan;
  pa.q_lens = q_lens; pa.q_offsets = q_offsets; pa.ctx_lens = ctx_lens;
  pa.batch = desc->batch; pa.hkv = a.hkv; pa.group = a.group; pa.tile_tokens = a.tile_tokens;
  pa.cap = tile_cap; pa.max_pieces = max_pieces; pa.max_merges = w.max_merges; pa.max_units = w.max_units;
  pa.skip_unit_chunks = skip_unit_chunks; pa.noncausal = noncausal;
  pa.us_alone = t.alone; pa.us_full = t.full;
  pa.min_longest = min_longest;
  pa.us_per_unit = 0.004f * desc->head_dim / 128.f;
  pa.header = a.header; pa.tile_rec = (int32_t*)(base + w.wstart); pa.merge_rec = (int32_t*)(base + w.merge_rec);
  call->tile_cap = tile_cap;
  call->max_merges = max_pieces ? std::min(max_tiles, w.max_merges) : 0;
  return ROLLATTN_OK;
}

// The launches behind the plan (float32 has no plan: rows are enumerated directly).
static int append_launch(const rollattn_desc* desc, AppendCall& call, hipStream_t s) {
  AppendArgs& a = call.args;
  hipError_t e;
  if (desc->q_dtype == ROLLATTN_F32) {
    const int tiles = (a.group + 3) / 4;
    const int grid = (int)std::min<int64_t>((int64_t)a.total_q * a.hkv * tiles, 1 << 20);
    ProfileScope prof(s);
    e = launch_append_f32(a, desc->head_dim, grid, s);
    prof.stop();
    if (e != hipSuccess) return fail_hip(e);
    return ROLLATTN_OK;
  }
  {
    ProfileScope prof(s);
    // one workgroup per (tile, KV head); with fewer than 8 heads the kernel deals runs of tiles to the XCDs
    // of a head, which needs up to one run of slack per XCD (see the kernel's index mapping)
    int64_t grid64 = (int64_t)call.tile_cap * a.hkv;
    if (a.hkv < kXcds && kXcds % a.hkv == 0) {
      const int64_t parts = kXcds / a.hkv;
      grid64 = kXcds * (((int64_t)call.tile_cap + parts - 1) / parts + kAppendXcdRun);
    }
    const int grid = (int)std::min<int64_t>(grid64, INT32_MAX);
    int dev = -1;
    if (prof.on && hipGetDevice(&dev) == hipSuccess && dev == g_clock_dev) a.clock_sums = g_clock_sums;
    e = launch_append_mfma(a, desc->head_dim, desc->kv_dtype == ROLLATTN_FP8_E4M3, call.half_tiles, grid, s);
    prof.stop();
  }
  if (e != hipSuccess) return fail_hip(e);
  if (call.max_merges) {
    e = launch_append_merge(a, desc->head_dim, call.max_merges, s);
    if (e != hipSuccess) return fail_hip(e);
  }
  return ROLLATTN_OK;
}

static int append_impl(const rollattn_desc* desc, const void* q_chunk, const int32_t* q_lens, const int32_t* q_offsets,
                       int32_t total_q, int32_t max_q_len, const void* k_pages, const void* v_pages,
                       const int32_t* page_table, const int32_t* ctx_lens, void* out, void* workspace,
                       size_t workspace_bytes, void* hip_stream, float* lse) {
  if (!desc) return ROLLATTN_EINVAL;
  AppendCall call{};
  const int rc = append_prepare(desc, q_chunk, q_lens, q_offsets, total_q, max_q_len, k_pages, v_pages, page_table, ctx_lens, out,
                                workspace, workspace_bytes, desc->max_pages_per_seq, false, lse, false, nullptr, &call);
  if (rc || call.args.batch == 0) return rc;
  hipStream_t s = (hipStream_t)hip_stream;
  if (desc->q_dtype != ROLLATTN_F32) {
    const hipError_t e = launch_plan_append(call.plan, s);
    if (e != hipSuccess) return fail_hip(e);
  }
  return append_launch(desc, call, s);
}

int attn_append(const rollattn_desc* desc, const void* q_chunk, const int32_t* q_lens, const int32_t* q_offsets,
                int32_t total_q, int32_t max_q_len, const void* k_pages, const void* v_pages,
                const int32_t* page_table, const int32_t* ctx_lens, void* out, void* workspace,
                size_t workspace_bytes, void* hip_stream) {
  if (!desc) return ROLLATTN_EINVAL;
  return append_impl(desc, q_chunk, q_lens, q_offsets, total_q, max_q_len, k_pages, v_pages, page_table, ctx_lens, out,
                     workspace, workspace_bytes, hip_stream, nullptr);
}

int attn_decode_lse(const rollattn_desc* desc, const void* q, const void* k_pages, const void* v_pages,
                    const int32_t* page_table, const int32_t* ctx_lens, void* out, float* lse, void* workspace,
                    size_t workspace_bytes, void* hip_stream) {
  if (desc && desc->batch > 0 && !lse) return ROLLATTN_EINVAL;
  if (lse && !aligned16(lse)) return ROLLATTN_EALIGN;
  return decode_impl(desc, q, k_pages, v_pages, page_table, ctx_lens, out, workspace, workspace_bytes, hip_stream, lse);
}

int attn_append_lse(const rollattn_desc* desc, const void* q_chunk, const int32_t* q_lens, const int32_t* q_offsets,
                    int32_t total_q, int32_t max_q_len, const void* k_pages, const void* v_pages,
                    const int32_t* page_table, const int32_t* ctx_lens, void* out, float* lse, void* workspace,
                    size_t workspace_bytes, void* hip_stream) {
  if (!desc) return ROLLATTN_EINVAL;
  if (desc->batch > 0 && total_q > 0 && !lse) return ROLLATTN_EINVAL;
  if (lse && !aligned16(lse)) return ROLLATTN_EALIGN;
  return append_impl(desc, q_chunk, q_lens, q_offsets, total_q, max_q_len, k_pages, v_pages, page_table, ctx_lens, out,
                     workspace, workspace_bytes, hip_stream, lse);
}

int attn_merge(const rollattn_desc* desc, int64_t rows, const void* o1, const float* lse1, const void* o2,
               const float* lse2, void* out, float* lse_out, void* hip_stream) {
  int rc = check_desc(desc, /*need_scales=*/false);
  if (rc) return rc;
  if (rows < 0) return ROLLATTN_EINVAL;
  if (rows == 0) return ROLLATTN_OK;
  if (!o1 || !lse1 || !o2 || !lse2 || !out) return ROLLATTN_EINVAL;
  if (!aligned16(o1) || !aligned16(lse1) || !aligned16(o2) || !aligned16(lse2) || !aligned16(out) ||
      (lse_out && !aligned16(lse_out)))
    return ROLLATTN_EALIGN;
  if (rows * (int64_t)desc->num_q_heads > (int64_t)INT32_MAX * 4) return ROLLATTN_ESHAPE;   // one wave per (row, head), four per workgroup
  const hipError_t e = launch_merge_states(o1, lse1, o2, lse2, out, lse_out, (long)rows * desc->num_q_heads, desc->head_dim,
                                           desc->q_dtype == ROLLATTN_F32, (hipStream_t)hip_stream);
  if (e != hipSuccess) return fail_hip(e);
  return ROLLATTN_OK;
}

size_t rollattn_step_workspace_bytes(const rollattn_desc* desc, int32_t total_q) {
  if (check_desc(desc) != ROLLATTN_OK || total_q < 0) return 0;
  return align256(decode_layout(*desc).total) + std::max(append_layout(*desc, total_q).cut_list, append_bytes(*desc, total_q, std::max(0, total_q - desc->batch)));
}

size_t rollattn_step_append_offset(const rollattn_desc* desc) {
  if (check_desc(desc, false) != ROLLATTN_OK) return 0;
  return align256(decode_layout(*desc).total);
}

int attn_step(const rollattn_desc* desc, const void* q, const int32_t* q_lens, const int32_t* q_offsets, int32_t total_q,
              int32_t max_q_len, const void* k_pages, const void* v_pages, const int32_t* page_table,
              const int32_t* ctx_lens, void* out, void* workspace, size_t workspace_bytes, void* hip_stream) {
  int rc = check_desc(desc);
  if (rc) return rc;
  if (total_q < 0 || max_q_len < 0) return ROLLATTN_EINVAL;
  if (desc->batch == 0 || total_q == 0) return ROLLATTN_OK;
  if (!workspace) return ROLLATTN_EINVAL;
  if (!aligned16(workspace)) return ROLLATTN_EALIGN;
  if (workspace_bytes < align256(decode_layout(*desc).total) + append_layout(*desc, total_q).total) return ROLLATTN_EWORKSPACE;
  if (desc->q_dtype == ROLLATTN_F32) {
    // the float32 path has one kernel for chunks of any length, one token included
    return append_impl(desc, q, q_lens, q_offsets, total_q, max_q_len, k_pages, v_pages, page_table, ctx_lens, out,
                       workspace, workspace_bytes, hip_stream, nullptr);
  }
  if (!q || !q_lens || !q_offsets || !k_pages || !v_pages || !page_table || !ctx_lens || !out) return ROLLATTN_EINVAL;
  if (!aligned16(q) || !aligned16(q_lens) || !aligned16(q_offsets) || !aligned16(k_pages) || !aligned16(v_pages) ||
      !aligned16(page_table) || !aligned16(ctx_lens) || !aligned16(out))
    return ROLLATTN_EALIGN;
  rc = append_limits(*desc);                       // everything either half could object to, before the first launch
  if (!rc) rc = decode_limits(*desc);
  if (rc) return rc;
  const size_t dec_bytes = align256(decode_layout(*desc).total);
  AppendCall app{};
  DecodeCall dec{};
  rc = decode_prepare(desc, q, k_pages, v_pages, page_table, ctx_lens, out, workspace, dec_bytes, nullptr, q_lens, q_offsets, &dec);
  if (!rc) rc = append_prepare(desc, q, q_lens, q_offsets, total_q, max_q_len, k_pages, v_pages, page_table, ctx_lens, out,
                               (char*)workspace + dec_bytes, workspace_bytes - dec_bytes, desc->max_pages_per_seq, false, nullptr,
                               /*skip_unit_chunks=*/true, &dec.args, &app);
  if (rc) return rc;
  // both plans in one launch, then the long tiles of the chunks first, then the decode rows and their merge; all on one
  // stream, disjoint output rows (the partials of cut tiles are merged before the decode rows' partials take their place)
  hipStream_t s = (hipStream_t)hip_stream;
  const hipError_t e = launch_plan_step(app.plan, dec.plan, s);
  if (e != hipSuccess) return fail_hip(e);
  rc = append_launch(desc, app, s);
  if (rc) return rc;
  return decode_launch(desc, dec.args, s);
}

namespace {
// Workspace of attn_decode_shared: the two inner workspaces, the two halves' rows and denominators, and where every
// trajectory's private part starts.
struct SharedLayout {
  rollattn_desc grp;      // descriptor of the shared half: one "trajectory" per group
  size_t dec_ws, app_ws, o1, o2, d1, d2, own_ctx, own_page, total;
  size_t dec_bytes, app_bytes;
};
SharedLayout shared_layout(const rollattn_desc& d, int32_t group_size) {
  SharedLayout L{};
  L.grp = d;
  L.grp.batch = d.batch / group_size;
  const size_t rows = (size_t)d.batch * d.num_q_heads;
  L.dec_bytes = decode_layout(d).total;
  L.app_bytes = append_layout(L.grp, d.batch).cut_list;
  size_t off = 0;
  L.dec_ws = off;    off += align256(L.dec_bytes);
  L.app_ws = off;    off += align256(L.app_bytes);
  L.o1 = off;        off += align256(rows * d.head_dim * 2);
  L.o2 = off;        off += align256(rows * d.head_dim * 2);
  L.d1 = off;        off += align256(rows * sizeof(float));
  L.d2 = off;        off += align256(rows * sizeof(float));
  L.own_ctx = off;   off += align256((size_t)d.batch * sizeof(int32_t));
  L.own_page = off;  off += align256((size_t)d.batch * sizeof(int32_t));
  L.total = off;
  return L;
}
int check_shared(const rollattn_desc* desc, int32_t group_size) {
  int rc = check_desc(desc);
  if (rc) return rc;
  if (desc->q_dtype != ROLLATTN_BF16) return ROLLATTN_EDTYPE;
  if (group_size < 1 || desc->batch % group_size) return ROLLATTN_EINVAL;
  if ((int64_t)group_size * desc->max_pages_per_seq > INT32_MAX) return ROLLATTN_ESHAPE;
  return ROLLATTN_OK;
}
}  // namespace

size_t rollattn_shared_workspace_bytes(const rollattn_desc* desc, int32_t group_size) {
  if (check_shared(desc, group_size) != ROLLATTN_OK) return 0;
  return shared_layout(*desc, group_size).total;
}

int attn_decode_shared(const rollattn_desc* desc, const void* q, const void* k_pages, const void* v_pages,
                       const int32_t* page_table, const int32_t* ctx_lens, int32_t group_size, const int32_t* shared_lens,
                       void* out, void* workspace, size_t workspace_bytes, void* hip_stream) {
  int rc = check_shared(desc, group_size);
  if (rc) return rc;
  if (desc->batch == 0) return ROLLATTN_OK;
  if (!q || !k_pages || !v_pages || !page_table || !ctx_lens || !shared_lens || !out || !workspace) return ROLLATTN_EINVAL;
  if (!aligned16(q) || !aligned16(k_pages) || !aligned16(v_pages) || !aligned16(page_table) || !aligned16(ctx_lens) ||
      !aligned16(shared_lens) || !aligned16(out) || !aligned16(workspace))
    return ROLLATTN_EALIGN;
  const SharedLayout L = shared_layout(*desc, group_size);
  if (workspace_bytes < L.total) return ROLLATTN_EWORKSPACE;
  rc = append_limits(L.grp);                       // everything either half could object to, before the first launch
  if (!rc) rc = decode_limits(*desc);
  if (rc) return rc;
  hipStream_t s = (hipStream_t)hip_stream;
  char* base = (char*)workspace;
  SharedPlanArgs sh{};
  sh.ctx_lens = ctx_lens; sh.shared_lens = shared_lens; sh.batch = desc->batch; sh.group_size = group_size;
  sh.own_ctx = (int32_t*)(base + L.own_ctx);
  sh.own_page = (int32_t*)(base + L.own_page);
  // shared half: the members' query rows of a group as one chunk over the group's first S tokens, behind its first
  // member's table; private half: every trajectory from token S on
  AppendCall app{};
  DecodeCall dec{};
  rc = decode_prepare(desc, q, k_pages, v_pages, page_table, sh.own_ctx, base + L.o2, base + L.dec_ws, L.dec_bytes,
                      (float*)(base + L.d2), nullptr, nullptr, &dec);
  if (!rc) rc = append_prepare(&L.grp, q, nullptr, nullptr, desc->batch, group_size, k_pages, v_pages, page_table, nullptr,
                               base + L.o1, base + L.app_ws, L.app_bytes, group_size * desc->max_pages_per_seq, true,
                               (float*)(base + L.d1), false, &dec.args, &app);
  if (rc) return rc;
  dec.args.first_page = sh.own_page;
  const hipError_t e = launch_plan_shared(sh, app.plan, dec.plan, s);
  if (e != hipSuccess) return fail_hip(e);
  rc = append_launch(&L.grp, app, s);
  if (rc) return rc;
  dec.args.shared = SharedHalf{base + L.o1, (const float*)(base + L.d1), out};
  return decode_launch(desc, dec.args, s);
}

int kv_write(const rollattn_desc* desc, const void* k_new, const void* v_new, const int32_t* q_lens,
             const int32_t* q_offsets, int32_t total_q, int32_t max_q_len, void* k_pages, void* v_pages,
             const int32_t* page_table, const int32_t* ctx_lens, float* k_scale, float* v_scale, void* hip_stream) {
  int rc = check_desc(desc, /*need_scales=*/false);
  if (rc) return rc;
  if (total_q < 0 || max_q_len < 0) return ROLLATTN_EINVAL;
  if (desc->batch == 0 || total_q == 0) return ROLLATTN_OK;
  const bool fp8 = desc->kv_dtype == ROLLATTN_FP8_E4M3;
  if (!k_new || !v_new || !q_lens || !q_offsets || !k_pages || !v_pages || !page_table || !ctx_lens) return ROLLATTN_EINVAL;
  if (fp8 && (!k_scale || !v_scale)) return ROLLATTN_EDTYPE;
  if (!aligned16(k_new) || !aligned16(v_new) || !aligned16(q_lens) || !aligned16(q_offsets) || !aligned16(k_pages) ||
      !aligned16(v_pages) || !aligned16(page_table) || !aligned16(ctx_lens) || (fp8 && (!aligned16(k_scale) || !aligned16(v_scale))))
    return ROLLATTN_EALIGN;
  if (desc->batch > 65535) return ROLLATTN_ESHAPE;     // one grid row per trajectory
  hipStream_t s = (hipStream_t)hip_stream;
  ProfileScope prof(s);
  const hipError_t e = launch_kv_write(k_new, v_new, q_lens, q_offsets, k_pages, v_pages, page_table, ctx_lens, k_scale,
                                       v_scale, desc->batch, desc->num_kv_heads, desc->max_pages_per_seq, max_q_len,
                                       desc->head_dim, desc->q_dtype == ROLLATTN_F32 ? 4 : 2, fp8, s);
  prof.stop();
  if (e != hipSuccess) return fail_hip(e);
  return ROLLATTN_OK;
}

int rollattn_debug_gather(const rollattn_desc* desc, const void* pages, const int32_t* page_table,
                          const int32_t* ctx_lens, int32_t b, int32_t kv_head, void* dst, void* hip_stream) {
  int rc = check_desc(desc, /*need_scales=*/false);
  if (rc) return rc;
  if (!pages || !page_table || !ctx_lens || !dst) return ROLLATTN_EINVAL;
  if (b < 0 || b >= desc->batch || kv_head < 0 || kv_head >= desc->num_kv_heads) return ROLLATTN_EINVAL;
  if (!aligned16(pages) || !aligned16(page_table) || !aligned16(dst)) return ROLLATTN_EALIGN;
  hipError_t e = launch_gather(pages, page_table, ctx_lens, b, kv_head, desc->num_kv_heads, desc->max_pages_per_seq,
                               desc->head_dim * dtype_bytes(desc->kv_dtype), dst, (hipStream_t)hip_stream);
  if (e != hipSuccess) return fail_hip(e);
  return ROLLATTN_OK;
}

int rollattn_debug_check_inputs(const rollattn_desc* desc, const int32_t* page_table, const int32_t* ctx_lens,
                                const int32_t* q_lens, const int32_t* q_offsets, int32_t* counts_dev,
                                int32_t* counts_out, void* hip_stream) {
  int rc = check_desc(desc, /*need_scales=*/false);
  if (rc) return rc;
  if (!counts_out) return ROLLATTN_EINVAL;
  for (int i = 0; i < 4; ++i) counts_out[i] = 0;
  if (desc->batch == 0) return ROLLATTN_OK;
  if (!page_table || !ctx_lens || !counts_dev) return ROLLATTN_EINVAL;
  if (!aligned16(page_table) || !aligned16(ctx_lens) || !aligned16(counts_dev) || (q_lens && !aligned16(q_lens)) ||
      (q_offsets && !aligned16(q_offsets)))
    return ROLLATTN_EALIGN;
  hipStream_t s = (hipStream_t)hip_stream;
  hipError_t e = launch_check_inputs(page_table, ctx_lens, q_lens, q_offsets, desc->batch, desc->max_pages_per_seq,
                                     desc->num_pages, counts_dev, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  if (e == hipSuccess) e = hipMemcpy(counts_out, counts_dev, 4 * sizeof(int32_t), hipMemcpyDeviceToHost);
  if (e != hipSuccess) return fail_hip(e);
  return ROLLATTN_OK;
}

int rollattn_profile_enable(int on) {
  std::lock_guard<std::mutex> lk(g_mu);
  if (on && g_pool.empty()) {
    g_pool.reserve(kMaxEvents);
    for (size_t i = 0; i < kMaxEvents; ++i) {
      EventPair ev{};
      hipError_t e = hipEventCreate(&ev.a);
      if (e == hipSuccess) {
        e = hipEventCreate(&ev.b);
        if (e != hipSuccess) (void)hipEventDestroy(ev.a);
      }
      if (e != hipSuccess) {
        g_hip_error = hipGetErrorString(e);
        for (auto& p : g_pool) { (void)hipEventDestroy(p.a); (void)hipEventDestroy(p.b); }
        g_pool.clear();
        return ROLLATTN_EHIP;
      }
      g_pool.push_back(ev);
    }
  }
  if (on && !g_clock_sums) {
    void* p = nullptr;
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipGetSymbolAddress(&p, HIP_SYMBOL(clock_sums));
    if (e == hipSuccess) e = hipMemset(p, 0, 2 * sizeof(unsigned long long));
    if (e != hipSuccess) {
      g_hip_error = hipGetErrorString(e);
      return ROLLATTN_EHIP;
    }
    g_clock_sums = (unsigned long long*)p;
    g_clock_dev = dev;
  }
  g_profile = on != 0;
  return ROLLATTN_OK;
}

int rollattn_profile_append_clock(double* mhz_out) {
  if (!mhz_out) return ROLLATTN_EINVAL;
  *mhz_out = 0.0;
  unsigned long long* p;
  {
    std::lock_guard<std::mutex> lk(g_mu);
    p = g_clock_sums;
  }
  if (!p) return ROLLATTN_OK;
  unsigned long long sums[2] = {0, 0};
  hipError_t e = hipDeviceSynchronize();
  if (e == hipSuccess) e = hipMemcpy(sums, p, sizeof(sums), hipMemcpyDeviceToHost);
  if (e == hipSuccess) e = hipMemset(p, 0, sizeof(sums));
  if (e != hipSuccess) return fail_hip(e);
  if (sums[1]) *mhz_out = 100.0 * (double)sums[0] / (double)sums[1];
  return ROLLATTN_OK;
}

int rollattn_profile_read(float* ms_out, int cap) {
  std::vector<EventPair> evs;
  {
    std::lock_guard<std::mutex> lk(g_mu);
    evs.assign(g_pool.begin(), g_pool.begin() + g_used);
    g_used = 0;
  }
  int n = 0;
  for (auto& ev : evs) {
    float ms = 0.f;
    hipError_t e = hipEventSynchronize(ev.b);
    if (e == hipSuccess) e = hipEventElapsedTime(&ms, ev.a, ev.b);
    if (e == hipSuccess && ms_out && n < cap) ms_out[n++] = ms;
  }
  return n;
}

const char* rollattn_status_string(int status) {
  switch (status) {
    case ROLLATTN_OK: return "ok";
    case ROLLATTN_EINVAL: return "invalid argument (null pointer or negative size)";
    case ROLLATTN_ESHAPE: return "unsupported shape (Hq % Hkv != 0, head_dim not 64/128, page_size not 16)";
    case ROLLATTN_EDTYPE: return "unsupported q/kv dtype pair, or FP8 pools without scales";
    case ROLLATTN_EALIGN: return "device pointer not 16-byte aligned";
    case ROLLATTN_EWORKSPACE: return "workspace smaller than rollattn_workspace_bytes()";
    case ROLLATTN_EHIP: return "HIP call failed (see rollattn_last_hip_error)";
    case ROLLATTN_ELIMIT: return "the call needs more scratch memory than the library's built-in array holds (rollattn_static_scratch_bytes)";
    default: return "unknown status";
  }
}

const char* rollattn_last_hip_error(void) {
  std::lock_guard<std::mutex> lk(g_mu);
  static thread_local std::string copy;
  copy = g_hip_error;
  return copy.c_str();
}

int rollattn_version(void) { return 101; }

}  // extern "C"
