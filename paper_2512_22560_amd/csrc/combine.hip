// Split-K merge: folds the partial results that the decode workers left for rows they did not cover alone (max m_s in
// log2 units, sum l_s, un-normalised o_s) into the final row:
//   M = max_s m_s ;  out = sum_s 2^(m_s - M) o_s / sum_s 2^(m_s - M) l_s
// which equals the softmax over the whole context.  Which workers touched a row follows from
// the plan alone: the row occupies blocks [R0, R1) of the global sequence and worker w owns
// [w * per, (w + 1) * per).  A worker keeps at most two partials, slot 0 for the first row
// segment of its run and slot 1 for the last; the only segment that lands in slot 1 is the one
// of the worker whose run began before this row.  Rows covered by a single worker were already
// written by it; rows without tokens are zero-filled here.
//
// A row here is a decode row, (trajectory, KV head, tile of query heads): its heads lie side by side in every partial.
// They are folded in chunks of 256 floats (four per lane, two heads at D = 128).  Bound by the latency of the partials'
// loads, so up to eight pieces are under way at a time; a row of up to sixteen is one wave's work per chunk.  A row of more
// pieces (few trajectories, cut for all workers) has its pieces dealt to four sums that are folded in their order: four
// waves make them where a workgroup has one chunk, which it has while those are few enough to be resident at once; with
// more chunks each wave has one of its own and makes the four in turn.  So a row's result depends on its pieces alone, not on
// what else is in the batch.  Against one wave per (trajectory, head) and one piece at a time:
// 13.4 -> 5.2 us for 40 rows of about 50 pieces (5 trajectories, 8 KV heads), 15.5 -> 10.6 us for 1536 rows of two or
// three (FP8, 384 trajectories, 64/4/128), 6.2 -> 5.5 us for 512 rows of about five.
#include <algorithm>
#include <type_traits>

#include "rollattn_internal.h"

namespace rollattn {

namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;
constexpr int kChunkFloats = 256;      // of a row's partial, per wave: four per lane
constexpr int kBatch = 8;              // pieces under way at a time
constexpr int kAlone = 2 * kBatch;
constexpr int kCombineResident = 8 * kNumCUs;
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ floatx4 widen(const bf16x4 x) { return floatx4{(float)x[0], (float)x[1], (float)x[2], (float)x[3]}; }

// TOGETHER: a workgroup per chunk, whose waves share the pieces of a row of many; else a chunk per wave.
// SHARED (attn_decode_shared): another result over the first part of every context is folded in as one more piece, with
// the weight 2^d of its denominator, and every row is written: one that a single worker finished is read back as a piece.
// The merge of the two halves as a launch of its own cost 8 us of a 268 us step and rounded split rows to bf16 in between.
template <int D, bool OUT_BF16, bool SHARED, bool TOGETHER>
__global__ __launch_bounds__(kThreads) void combine_kernel(const DecodeArgs a, int chunks_per_row) {
  __shared__ __attribute__((aligned(16))) float sum_s[TOGETHER ? kWaves : 1][64][4];
  __shared__ float ml_s[TOGETHER ? kWaves : 1][64][2];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int unit = TOGETHER ? (int)blockIdx.x : __builtin_amdgcn_readfirstlane(blockIdx.x * kWaves + wave);
  // What decides whether there is anything to do comes in two trips to memory, the arguments and then what they point to, and not
  // in one trip per question.
  const int32_t* q_lens = a.q_lens;
  const int32_t* q_offsets = a.q_offsets;
  const int32_t *header = a.header, *prefix = a.prefix;
  const float *partial_ml = a.partial_ml, *partial_o = a.partial_o;
  const int batch = a.batch, rows_per_b = a.rows_per_b, hkv = a.hkv, hq = a.hq, ht = a.head_tile, group = a.group, may_be_whole = a.whole_rows;
  asm volatile("" ::"s"(q_lens), "s"(q_offsets), "s"(header), "s"(prefix), "s"(partial_ml), "s"(partial_o), "s"(batch), "s"(rows_per_b), "s"(hkv), "s"(hq), "s"(ht),
               "s"(group), "s"(may_be_whole), "s"(chunks_per_row));
  const int row = unit / chunks_per_row, c = unit - row * chunks_per_row;
  const int b = row / rows_per_b, r = row - b * rows_per_b;
  if (b >= batch) return;
  const int per = header[kPlanPer], whole = may_be_whole & header[kPlanWhole];
  const int first = prefix[b], end = prefix[b + 1];
  const int new_rows = q_lens ? q_lens[b] : 1, row0 = q_offsets ? q_offsets[b] : b;
  asm volatile("" ::"s"(per), "s"(whole), "s"(first), "s"(end), "s"(new_rows), "s"(row0));
  if (new_rows != 1) return;                                // mixed step: not a decode row, nothing of ours to write
  const int n_ht = rows_per_b / hkv;
  const int g = r / n_ht, h0 = (r - g * n_ht) * ht;
  const int heads = min(ht, group - h0);
  if (c * kChunkFloats >= heads * D) return;                // (a row's last tile of heads may have fewer chunks)
  const SharedHalf& other = a.shared;
  const int n = end - first;
  if (whole && n) return;                                   // its worker has written it
  const long r0 = (long)rows_per_b * first + (long)r * n;
  const int wf = n ? (int)(r0 / per) : 0;
  const int wl = n ? (int)((r0 + n - 1) / per) : 0;
  if (!SHARED && n && wf == wl) return;                     // one worker had the whole row
  const int pieces = n ? wl - wf + 1 : 0;
  const int first_slot = ((long)wf * per < r0) ? 1 : 0;
  const size_t orow0 = (size_t)row0 * hq + (size_t)g * group + h0;   // where the row's first head goes
  const bool dealt = pieces > kAlone;                       // to four sums
  if (TOGETHER && !dealt && wave != 0) return;
  const int at = c * kChunkFloats + lane * 4;               // first of this lane's floats within a partial
  const int head = at / D;
  const bool ok = head < heads;                             // (the last chunk of an odd number of heads is not full)
  const float* po = partial_o + (ok ? at : 0);
  const float* pml = partial_ml + (ok ? head : 0) * 2;
  floatx4 o = {0.f, 0.f, 0.f, 0.f};
  float m = -INFINITY, l = 0.f;
  const int step = dealt ? kWaves : 1;
  // folds pieces s0, s0 + step, ... of one batch; past the last piece the last one is loaded again, with weight zero
  auto fold = [&](int s0, auto batch_c) __attribute__((always_inline)) {
    constexpr int kN = decltype(batch_c)::value;
    floatx4 y[kN];
    floatx2 x[kN];
#pragma unroll
    for (int i = 0; i < kN; ++i) {
      const int s = min(s0 + i * step, pieces - 1);
      const size_t slot = ((size_t)(wf + s) * 2 + (s == 0 ? first_slot : 0)) * ht;
      x[i] = *(const floatx2*)(pml + slot * 2);
      y[i] = *(const floatx4*)(po + slot * D);
    }
    float top = m;
#pragma unroll
    for (int i = 0; i < kN; ++i) {
      if (s0 + i * step >= pieces) {                      // (zero times an infinity would not be zero)
        x[i] = floatx2{-INFINITY, 0.f};
        y[i] = floatx4{0.f, 0.f, 0.f, 0.f};
      }
      top = fmaxf(top, x[i][0]);
    }
    const float keep = __builtin_amdgcn_exp2f(m - top);   // (a partial has seen at least one token: its maximum is finite)
    m = top;
    l *= keep;
    o *= keep;
#pragma unroll
    for (int i = 0; i < kN; ++i) {
      const float f = __builtin_amdgcn_exp2f(x[i][0] - top);
      l += f * x[i][1];
      o += f * y[i];
    }
  };
  const size_t dst = orow0 * D + at;
  floatx4 o1 = {0.f, 0.f, 0.f, 0.f};
  float d1 = -INFINITY;
  if constexpr (SHARED) {
    if (ok) {
      o1 = widen(*(const bf16x4*)((const __bf16*)other.out + dst));
      d1 = other.lse[orow0 + head];
      if (pieces == 1) {
        o = widen(*(const bf16x4*)((const __bf16*)a.out + dst));
        m = a.lse[orow0 + head];
        l = 1.f;
      }
    }
  }
  // weights the four sums (x(w): maximum and sum of weights, y(w): weighted values) and adds them
  auto join = [&](auto&& x, auto&& y) __attribute__((always_inline)) {
    m = x(0)[0];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) m = fmaxf(m, x(w)[0]);
    float f = __builtin_amdgcn_exp2f(x(0)[0] - m);
    l = x(0)[1] * f;
    o = y(0) * f;
#pragma unroll
    for (int w = 1; w < kWaves; ++w) {
      f = __builtin_amdgcn_exp2f(x(w)[0] - m);
      l += f * x(w)[1];
      o += f * y(w);
    }
  };
  constexpr std::integral_constant<int, kBatch> batch_c{};
  if (pieces < 2) {}                                        // nothing to fold (none: a zero row)
  else if (pieces == 2) fold(0, std::integral_constant<int, 2>{});
  else if (pieces == 3) fold(0, std::integral_constant<int, 3>{});
  else if (pieces <= 5) fold(0, std::integral_constant<int, 5>{});
  else if (!dealt) {
    for (int s0 = 0; s0 < pieces; s0 += kBatch) fold(s0, batch_c);
  } else if constexpr (TOGETHER) {
    for (int s0 = wave; s0 < pieces; s0 += kBatch * kWaves) fold(s0, batch_c);
    *(floatx4*)sum_s[wave][lane] = o;
    ml_s[wave][lane][0] = m;
    ml_s[wave][lane][1] = l;
    __syncthreads();
    if (wave != 0) return;
    join([&](int w) { return floatx2{ml_s[w][lane][0], ml_s[w][lane][1]}; }, [&](int w) { return *(const floatx4*)sum_s[w][lane]; });
  } else {
    floatx2 x[kWaves];
    floatx4 y[kWaves];
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      o = floatx4{0.f, 0.f, 0.f, 0.f};
      m = -INFINITY;
      l = 0.f;
      for (int s0 = w; s0 < pieces; s0 += kBatch * kWaves) fold(s0, batch_c);
      x[w] = floatx2{m, l};
      y[w] = o;
    }
    join([&](int w) { return x[w]; }, [&](int w) { return y[w]; });
  }
  if (!ok) return;
  if constexpr (SHARED) {
    const float top = fmaxf(m, d1), base = (top == -INFINITY) ? 0.f : top;
    const float w1 = __builtin_amdgcn_exp2f(d1 - base), w2 = __builtin_amdgcn_exp2f(m - base);   // 2^-inf = 0
    const float tot = w1 + w2 * l, inv = tot > 0.f ? 1.f / tot : tot;
    o = (w1 * o1 + w2 * o) * inv;
    bf16x4 pk;
#pragma unroll
    for (int e = 0; e < 4; ++e) pk[e] = (__bf16)o[e];
    *(bf16x4*)((__bf16*)other.result + dst) = pk;
    return;
  }
  const float inv = n ? 1.f / l : 0.f;
  if (a.lse && at % D == 0) a.lse[orow0 + head] = n ? m + __builtin_amdgcn_logf(l) : -INFINITY;
  if constexpr (OUT_BF16) {
    bf16x4 pk;
#pragma unroll
    for (int e = 0; e < 4; ++e) pk[e] = (__bf16)(o[e] * inv);
    *(bf16x4*)((__bf16*)a.out + dst) = pk;
  } else {
    *(floatx4*)((float*)a.out + dst) = o * inv;
  }
}

// Copies logical tokens of one (trajectory, KV head) out of a pool, byte for byte.
__global__ __launch_bounds__(kThreads) void gather_kernel(const unsigned char* pages, const int32_t* page_table,
                                                          const int32_t* ctx_lens, int32_t b, int32_t kv_head,
                                                          int32_t hkv, int32_t max_pages, int32_t row_bytes,
                                                          unsigned char* dst) {
  const int len = ctx_lens[b];
  const int vec_per_row = row_bytes / 16;
  const long n_vec = (long)len * vec_per_row;
  for (long i = (long)blockIdx.x * kThreads + threadIdx.x; i < n_vec; i += (long)gridDim.x * kThreads) {
    const int t = (int)(i / vec_per_row), c = (int)(i % vec_per_row);
    const int pid = page_table[(size_t)b * max_pages + t / kPageSize];
    const size_t off = (((size_t)pid * hkv + kv_head) * kPageSize + (t % kPageSize)) * row_bytes + c * 16;
    *(uint4*)(dst + (size_t)t * row_bytes + c * 16) = *(const uint4*)(pages + off);
  }
}

// Counts what the entry points take on trust (see rollattn_debug_check_inputs): one workgroup per trajectory.
__global__ __launch_bounds__(kThreads) void check_inputs_kernel(const int32_t* page_table, const int32_t* ctx_lens,
                                                                const int32_t* q_lens, const int32_t* q_offsets,
                                                                int32_t batch, int32_t max_pages, int64_t num_pages,
                                                                int32_t* counts) {
  const int b = blockIdx.x;
  const int len = ctx_lens[b];
  const bool bad_len = len < 0 || (long)len > (long)max_pages * kPageSize;
  const int live = bad_len ? 0 : (len + kPageSize - 1) / kPageSize;
  int bad_ids = 0;
  for (int pg = threadIdx.x; pg < live; pg += kThreads) {
    const int id = page_table[(size_t)b * max_pages + pg];
    bad_ids += (id < 0 || id >= num_pages) ? 1 : 0;
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) bad_ids += __shfl_xor(bad_ids, off, 64);
  if ((threadIdx.x & 63) == 0 && bad_ids) atomicAdd(counts + 1, bad_ids);
  if (threadIdx.x == 0) {
    if (bad_len) atomicAdd(counts + 0, 1);
    if (q_lens) {
      const int n = q_lens[b];
      if (n < 0 || (!bad_len && n > len)) atomicAdd(counts + 2, 1);
      if (q_offsets && (q_offsets[b + 1] - q_offsets[b] != n || (b == 0 && q_offsets[0] != 0))) atomicAdd(counts + 3, 1);
    }
  }
}

__global__ void clear4_kernel(int32_t* counts) {
  if (threadIdx.x < 4) counts[threadIdx.x] = 0;
}

}  // namespace

hipError_t launch_check_inputs(const int32_t* page_table, const int32_t* ctx_lens, const int32_t* q_lens,
                               const int32_t* q_offsets, int32_t batch, int32_t max_pages, int64_t num_pages,
                               int32_t* counts, hipStream_t s) {
  hipLaunchKernelGGL(clear4_kernel, dim3(1), dim3(64), 0, s, counts);
  hipLaunchKernelGGL(check_inputs_kernel, dim3(batch), dim3(kThreads), 0, s, page_table, ctx_lens, q_lens, q_offsets, batch,
                     max_pages, num_pages, counts);
  return hipGetLastError();
}

namespace {
template <bool SHARED>
hipError_t launch(const DecodeArgs& a, int head_dim, bool out_bf16, hipStream_t s) {
  const int chunks = (std::min(a.head_tile, a.group) * head_dim + kChunkFloats - 1) / kChunkFloats;
  const long units = (long)a.batch * a.rows_per_b * chunks;
  // A workgroup per chunk while those are few enough to be resident at once, so that the waves of a row of many pieces
  // have one chunk to share; with more rows (of few pieces each) a chunk per wave: 1024 contexts of 16 .. 64 tokens with 8 or
  // 64 KV heads of one query head take 35.2 and 210 us with workgroups of one working wave, 29.6 and 167 with four.
  const bool together = units <= kCombineResident;
  const dim3 grid((unsigned)(together ? units : (units + kWaves - 1) / kWaves));
  auto go = [&](auto d, auto bf16, auto tog) {
    hipLaunchKernelGGL((combine_kernel<decltype(d)::value, decltype(bf16)::value, SHARED, decltype(tog)::value>), grid, dim3(kThreads), 0, s, a, chunks);
  };
  auto with_dim = [&](auto bf16, auto tog) {
    if (head_dim == 128) go(std::integral_constant<int, 128>{}, bf16, tog);
    else go(std::integral_constant<int, 64>{}, bf16, tog);
  };
  auto with_type = [&](auto tog) {
    if constexpr (SHARED) with_dim(std::true_type{}, tog);
    else if (out_bf16) with_dim(std::true_type{}, tog);
    else with_dim(std::false_type{}, tog);
  };
  if (head_dim != 128 && head_dim != 64) return hipErrorInvalidValue;
  if (together) with_type(std::true_type{});
  else with_type(std::false_type{});
  return hipGetLastError();
}
}  // namespace

hipError_t launch_combine(const DecodeArgs& a, int head_dim, bool out_bf16, hipStream_t s) {
  return launch<false>(a, head_dim, out_bf16, s);
}

hipError_t launch_combine_shared(const DecodeArgs& a, int head_dim, hipStream_t s) {
  return launch<true>(a, head_dim, /*out_bf16=*/true, s);
}

hipError_t launch_gather(const void* pages, const int32_t* page_table, const int32_t* ctx_lens, int32_t b,
                         int32_t kv_head, int32_t hkv, int32_t max_pages, int32_t row_bytes, void* dst,
                         hipStream_t s) {
  hipLaunchKernelGGL(gather_kernel, dim3(64), dim3(kThreads), 0, s, (const unsigned char*)pages, page_table,
                     ctx_lens, b, kv_head, hkv, max_pages, row_bytes, (unsigned char*)dst);
  return hipGetLastError();
}

}  // namespace rollattn
