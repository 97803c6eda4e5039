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
// loads, so up to eight pieces are under way at a time; a row of up to sixteen is one wave's work per chunk, and the four
// waves of the workgroup take different chunks.  A row of more pieces (few trajectories, cut for all workers) has its pieces
// dealt to the four waves, whose sums meet in LDS.  Which of the two a row takes depends on its pieces alone, so its
// result does not depend on what else is in the batch.  Against one wave per (trajectory, head) and one piece at a time:
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

// One workgroup per (row, run of chunks_per_wg chunks of it).
// SHARED (attn_decode_shared): another result over the first part of every context is folded in as one more piece, with
// the weight 2^d of its denominator, and every row is written: one that a single worker finished is read back as a piece.
// The merge of the two halves as a launch of its own cost 8 us of a 268 us step and rounded split rows to bf16 in between.
template <int D, bool OUT_BF16, bool SHARED>
__global__ __launch_bounds__(kThreads) void combine_kernel(const DecodeArgs a, const SharedHalf other, int wgs_per_row, int chunks_per_wg) {
  __shared__ __attribute__((aligned(16))) float sum_s[kWaves][64][4];
  __shared__ float ml_s[kWaves][64][2];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int row = blockIdx.x / wgs_per_row, part = blockIdx.x - row * wgs_per_row;
  const int b = row / a.rows_per_b, r = row - b * a.rows_per_b;
  if (a.q_lens && a.q_lens[b] != 1) return;                 // mixed step: not a decode row, nothing of ours to write
  const int ht = a.head_tile;
  const int n_ht = a.rows_per_b / a.hkv;
  const int g = r / n_ht, h0 = (r - g * n_ht) * ht;
  const int heads = min(ht, a.group - h0);
  const int chunks = (heads * D + kChunkFloats - 1) / kChunkFloats;
  const int per = a.header[kPlanPer];
  const int first = a.prefix[b];
  const int n = a.prefix[b + 1] - first;
  const long r0 = (long)a.rows_per_b * first + (long)r * n;
  const int wf = n ? (int)(r0 / per) : 0;
  const int wl = n ? (int)((r0 + n - 1) / per) : 0;
  if (!SHARED && n && wf == wl) return;                     // one worker had the whole row
  const int pieces = n ? wl - wf + 1 : 0;
  const int first_slot = ((long)wf * per < r0) ? 1 : 0;
  const size_t orow0 = (size_t)(a.q_offsets ? a.q_offsets[b] : b) * a.hq + (size_t)g * a.group + h0;   // where the row's first head goes
  const bool shared_work = pieces > kAlone;                 // the four waves share each chunk's pieces
  const int end = min(chunks, (part + 1) * chunks_per_wg);
  for (int c = part * chunks_per_wg + (shared_work ? 0 : wave); c < end; c += shared_work ? 1 : kWaves) {
    const int at = c * kChunkFloats + lane * 4;             // first of this lane's floats within a partial
    const int head = at / D;
    const bool ok = head < heads;                           // (the last chunk of an odd number of heads is not full)
    const float* po = a.partial_o + (ok ? at : 0);
    const float* pml = a.partial_ml + (ok ? head : 0) * 2;
    floatx4 o = {0.f, 0.f, 0.f, 0.f};
    float m = -INFINITY, l = 0.f;
    const int step = shared_work ? kWaves : 1;
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
    if (pieces < 2) {}                                      // nothing to fold (none: a zero row)
    else if (pieces == 2) fold(0, std::integral_constant<int, 2>{});
    else if (pieces == 3) fold(0, std::integral_constant<int, 3>{});
    else if (pieces <= 5) fold(0, std::integral_constant<int, 5>{});
    else for (int s0 = shared_work ? wave : 0; s0 < pieces; s0 += kBatch * step) fold(s0, std::integral_constant<int, kBatch>{});
    if (shared_work) {
      *(floatx4*)sum_s[wave][lane] = o;
      ml_s[wave][lane][0] = m;
      ml_s[wave][lane][1] = l;
      __syncthreads();
      if (wave == 0) {
#pragma unroll
        for (int w = 1; w < kWaves; ++w) m = fmaxf(m, ml_s[w][lane][0]);
        float f = __builtin_amdgcn_exp2f(ml_s[0][lane][0] - m);
        l *= f;
        o *= f;
#pragma unroll
        for (int w = 1; w < kWaves; ++w) {
          f = __builtin_amdgcn_exp2f(ml_s[w][lane][0] - m);
          l += f * ml_s[w][lane][1];
          o += f * *(const floatx4*)sum_s[w][lane];
        }
      }
      __syncthreads();                                      // the next chunk reuses the LDS
      if (wave != 0) continue;
    }
    if (!ok) continue;
    if constexpr (SHARED) {
      const float top = fmaxf(m, d1), base = (top == -INFINITY) ? 0.f : top;
      const float w1 = __builtin_amdgcn_exp2f(d1 - base), w2 = __builtin_amdgcn_exp2f(m - base);   // 2^-inf = 0
      const float tot = w1 + w2 * l, inv = tot > 0.f ? 1.f / tot : tot;
      o = (w1 * o1 + w2 * o) * inv;
      bf16x4 pk;
#pragma unroll
      for (int e = 0; e < 4; ++e) pk[e] = (__bf16)o[e];
      *(bf16x4*)((__bf16*)other.result + dst) = pk;
      continue;
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
struct CombineGrid {
  dim3 grid;
  int wgs_per_row, chunks_per_wg;
};
CombineGrid combine_grid(const DecodeArgs& a, int head_dim) {
  const int chunks = (std::min(a.head_tile, a.group) * head_dim + kChunkFloats - 1) / kChunkFloats;
  const long rows = (long)a.batch * a.rows_per_b;
  // A workgroup per chunk while those are few enough to be resident at once, so that the waves of a row of many pieces
  // have one chunk to share; with more rows (of few pieces each) a chunk per wave.
  const int chunks_per_wg = rows * chunks <= kCombineResident ? 1 : std::min(chunks, kWaves);
  const int wgs_per_row = (chunks + chunks_per_wg - 1) / chunks_per_wg;
  return {dim3((unsigned)(rows * wgs_per_row)), wgs_per_row, chunks_per_wg};
}
}  // namespace

hipError_t launch_combine(const DecodeArgs& a, int head_dim, bool out_bf16, hipStream_t s) {
  const CombineGrid c = combine_grid(a, head_dim);
  const SharedHalf none{};
  if (head_dim == 128 && out_bf16) {
    hipLaunchKernelGGL((combine_kernel<128, true, false>), c.grid, dim3(kThreads), 0, s, a, none, c.wgs_per_row, c.chunks_per_wg);
  } else if (head_dim == 128) {
    hipLaunchKernelGGL((combine_kernel<128, false, false>), c.grid, dim3(kThreads), 0, s, a, none, c.wgs_per_row, c.chunks_per_wg);
  } else if (head_dim == 64 && out_bf16) {
    hipLaunchKernelGGL((combine_kernel<64, true, false>), c.grid, dim3(kThreads), 0, s, a, none, c.wgs_per_row, c.chunks_per_wg);
  } else if (head_dim == 64) {
    hipLaunchKernelGGL((combine_kernel<64, false, false>), c.grid, dim3(kThreads), 0, s, a, none, c.wgs_per_row, c.chunks_per_wg);
  } else {
    return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_combine_shared(const DecodeArgs& a, const SharedHalf& shared, int head_dim, hipStream_t s) {
  const CombineGrid c = combine_grid(a, head_dim);
  if (head_dim == 128) {
    hipLaunchKernelGGL((combine_kernel<128, true, true>), c.grid, dim3(kThreads), 0, s, a, shared, c.wgs_per_row, c.chunks_per_wg);
  } else if (head_dim == 64) {
    hipLaunchKernelGGL((combine_kernel<64, true, true>), c.grid, dim3(kThreads), 0, s, a, shared, c.wgs_per_row, c.chunks_per_wg);
  } else {
    return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_gather(const void* pages, const int32_t* page_table, const int32_t* ctx_lens, int32_t b,
                         int32_t kv_head, int32_t hkv, int32_t max_pages, int32_t row_bytes, void* dst,
                         hipStream_t s) {
  hipLaunchKernelGGL(gather_kernel, dim3(64), dim3(kThreads), 0, s, (const unsigned char*)pages, page_table,
                     ctx_lens, b, kv_head, hkv, max_pages, row_bytes, (unsigned char*)dst);
  return hipGetLastError();
}

}  // namespace rollattn
