// float32 attention on the vector ALUs: decode pieces and (row-at-a-time) append.
//
// One workgroup handles one (KV piece, KV head, tile of up to 4 query heads).  Each token row
// is read by D/4 adjacent lanes with one 16-byte load each; the partial dot products are
// summed across those lanes by DPP; every lane group keeps its own online-softmax state (max, sum, weighted values);
// the groups are merged with the log-sum-exp rule at the end, across the wave in registers, across waves through LDS.
// Bound by latency (the calls are small): page id, then K and V, then the softmax chain.  Four tokens per lane group are
// under way at a time and share one step of that chain.
#include "plan_device.h"

namespace rollattn {

namespace {

constexpr int kThreads = 256;
constexpr int kDirectThreads = kPlanThreads;
constexpr int kHT = kF32HeadTile;   // query heads per row

template <int D>
struct F32Geo {
  static constexpr int kLanesPerTok = D / 4;
  static constexpr int kTokPerWave = 64 / kLanesPerTok;
};

__device__ __forceinline__ float xor16(float x, bool add) {
  typedef unsigned int uintx2 __attribute__((ext_vector_type(2)));
  const uintx2 r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return add ? __uint_as_float(r[0]) + __uint_as_float(r[1]) : fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float xor32(float x, bool add) {
  typedef unsigned int uintx2 __attribute__((ext_vector_type(2)));
  const uintx2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return add ? __uint_as_float(r[0]) + __uint_as_float(r[1]) : fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
template <int CTRL>
__device__ __forceinline__ float dpp(float x) {
  return __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), CTRL, 0xf, 0xf, true));
}
// Sum over the D/4 lanes of a token, in all of them.
template <int D>
__device__ __forceinline__ float token_sum(float x) {
  x += dpp<0xb1>(x);    // quad_perm 1 0 3 2
  x += dpp<0x4e>(x);    // quad_perm 2 3 0 1
  x += dpp<0x141>(x);   // row_half_mirror: the other quad of eight lanes
  x += dpp<0x140>(x);   // row_mirror: the other eight of sixteen
  if constexpr (D == 128) x = xor16(x, true);
  return x;
}
// Maximum or sum over the lane groups of a wave (lanes that hold the same dims).
template <int D>
__device__ __forceinline__ float across_groups(float x, bool add) {
  if constexpr (D == 64) x = xor16(x, add);
  return xor32(x, add);
}

// Attention of up to HT query rows (same KV head) over tokens [0, len), len > 0, of a paged range whose
// page ids start at table[0].  Leaves un-normalised o in o_out[h][D] (LDS), and max (log2
// units) / sum in ml_out[h][2].  All THREADS threads must call it.
template <int D, int THREADS, int HT>
__device__ void attend_f32(const float* const* qrows, int n_heads, const float* k_pages, const float* v_pages,
                           const int32_t* table, int len, int hkv, int g, float scale_log2,
                           float (*o_part)[HT][D], float (*ml_part)[HT][2], float (*o_out)[D],
                           float (*ml_out)[2]) {
  using G_ = F32Geo<D>;
  constexpr int kWaves = THREADS / 64, kGroups = kWaves * G_::kTokPerWave, kUnroll = 4;
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int sub = lane / G_::kLanesPerTok;          // token slot within the wave
  const int dl = lane % G_::kLanesPerTok;           // which 4 dims
  const int grp = wave * G_::kTokPerWave + sub;

  float4 q[HT];
#pragma unroll
  for (int h = 0; h < HT; ++h) q[h] = (h < n_heads) ? *(const float4*)(qrows[h] + dl * 4) : make_float4(0, 0, 0, 0);
  float4 acc[HT];
  float m[HT], l[HT];
#pragma unroll
  for (int h = 0; h < HT; ++h) {
    acc[h] = make_float4(0, 0, 0, 0);
    m[h] = -INFINITY;
    l[h] = 0.f;
  }
  for (int t0 = grp; t0 - grp < len; t0 += kUnroll * kGroups) {    // (the same trips for every lane)
    float4 kv[kUnroll], vv[kUnroll];
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      const int t = min(t0 + u * kGroups, len - 1);                // past the end: the last token again, weight zero
      const size_t off = (((size_t)table[t / kPageSize] * hkv + g) * kPageSize + (t % kPageSize)) * D + dl * 4;
      kv[u] = *(const float4*)(k_pages + off);
      vv[u] = *(const float4*)(v_pages + off);
    }
#pragma unroll
    for (int u = 0; u < kUnroll; ++u)                              // (zero times an infinity would not be zero)
      if (t0 + u * kGroups >= len) vv[u] = make_float4(0, 0, 0, 0);
#pragma unroll
    for (int h = 0; h < HT; ++h) {
      float s[kUnroll], m_new = m[h];
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        s[u] = q[h].x * kv[u].x + q[h].y * kv[u].y + q[h].z * kv[u].z + q[h].w * kv[u].w;
        s[u] = t0 + u * kGroups < len ? token_sum<D>(s[u]) * scale_log2 : -INFINITY;
        m_new = fmaxf(m_new, s[u]);
      }
      const float base = m_new == -INFINITY ? 0.f : m_new;         // a lane group that has seen no token yet
      const float alpha = __builtin_amdgcn_exp2f(m[h] - base);
      m[h] = m_new;
      l[h] *= alpha;
      acc[h].x *= alpha;
      acc[h].y *= alpha;
      acc[h].z *= alpha;
      acc[h].w *= alpha;
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        const float p = __builtin_amdgcn_exp2f(s[u] - base);
        l[h] += p;
        acc[h].x += p * vv[u].x;
        acc[h].y += p * vv[u].y;
        acc[h].z += p * vv[u].z;
        acc[h].w += p * vv[u].w;
      }
    }
  }
#pragma unroll
  for (int h = 0; h < HT; ++h) {
    const float top = across_groups<D>(m[h], false);
    const float f = __builtin_amdgcn_exp2f(m[h] - (top == -INFINITY ? 0.f : top));
    acc[h].x = across_groups<D>(acc[h].x * f, true);
    acc[h].y = across_groups<D>(acc[h].y * f, true);
    acc[h].z = across_groups<D>(acc[h].z * f, true);
    acc[h].w = across_groups<D>(acc[h].w * f, true);
    l[h] = across_groups<D>(l[h] * f, true);
    if (sub == 0) *(float4*)(&o_part[wave][h][dl * 4]) = acc[h];
    if (lane == 0) {
      ml_part[wave][h][0] = top;
      ml_part[wave][h][1] = l[h];
    }
  }
  __syncthreads();
  for (int e = tid; e < HT * D; e += THREADS) {
    const int h = e / D, d = e % D;
    float mmax = ml_part[0][h][0];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) mmax = fmaxf(mmax, ml_part[w][h][0]);   // finite: some wave has the first token
    float o = 0.f, ls = 0.f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      const float f = __builtin_amdgcn_exp2f(ml_part[w][h][0] - mmax);       // 2^-inf = 0
      o += f * o_part[w][h][d];
      ls += f * ml_part[w][h][1];
    }
    o_out[h][d] = o;
    if (d == 0) {
      ml_out[h][0] = mmax;
      ml_out[h][1] = ls;
    }
  }
  __syncthreads();
}

// Decode in float32 of contexts that are not worth cutting: a workgroup per row writes it, one more makes the plan that
// nobody but rollattn_debug_read_plan reads.  One launch where plan, decode and merge are three of them, each 2 to 5 us
// and most of that its start.  A row is HT heads: one while the call's heads alone do not fill the chip (its vector
// instructions are the longest stretch of a row of four), else as many as share a KV head, four at most.
template <int D, int HT>
__global__ __launch_bounds__(kDirectThreads) void decode_f32_direct_kernel(const DecodeArgs a) {
  constexpr int kWaves = kDirectThreads / 64;
  __shared__ __attribute__((aligned(16))) float o_part[kWaves][HT][D];
  __shared__ float ml_part[kWaves][HT][2];
  __shared__ __attribute__((aligned(16))) float o_out[HT][D];
  __shared__ float ml_out[HT][2];
  if (blockIdx.x == gridDim.x - 1) {
    __shared__ DecodePlanLds plan_lds;
    plan_decode(a.plan, plan_lds, [&](int b) { return a.ctx_lens[b]; });
    return;
  }
  const int n_ht = (a.group + HT - 1) / HT, rows = a.hkv * n_ht;
  const int b = blockIdx.x / rows, r = blockIdx.x - b * rows;
  const int g = r / n_ht, h0 = (r - g * n_ht) * HT;
  const int n_heads = min(HT, a.group - h0);
  const int len = a.ctx_lens[b];
  const size_t orow0 = (size_t)b * a.hq + (size_t)g * a.group + h0;
  const float* qrows[HT];
#pragma unroll
  for (int h = 0; h < HT; ++h) qrows[h] = (const float*)a.q + (orow0 + min(h, n_heads - 1)) * D;
  if (len > 0)
    attend_f32<D, kDirectThreads, HT>(qrows, n_heads, (const float*)a.k_pages, (const float*)a.v_pages,
                                  a.page_table + (size_t)b * a.max_pages, len, a.hkv, g, a.scale_log2, o_part, ml_part, o_out, ml_out);
  for (int e = threadIdx.x; e < n_heads * D; e += kDirectThreads) {
    const int h = e / D, d = e % D;
    ((float*)a.out)[(orow0 + h) * D + d] = len > 0 ? o_out[h][d] / ml_out[h][1] : 0.f;
    if (a.lse && d == 0) a.lse[orow0 + h] = len > 0 ? ml_out[h][0] + __builtin_amdgcn_logf(ml_out[h][1]) : -INFINITY;
  }
}

// Decode in float32: every workgroup is one worker of the block partition (see plan.hip) and walks
// its run of 32-token blocks one row segment at a time.
template <int D>
__global__ __launch_bounds__(kThreads) void decode_f32_kernel(const DecodeArgs a) {
  __shared__ __attribute__((aligned(16))) float o_part[kThreads / 64][kHT][D];
  __shared__ float ml_part[kThreads / 64][kHT][2];
  __shared__ __attribute__((aligned(16))) float o_out[kHT][D];
  __shared__ float ml_out[kHT][2];
  const int tid = threadIdx.x;
  const int group = a.group, hkv = a.hkv, rows_per_b = a.rows_per_b;
  const int n_ht = rows_per_b / hkv;
  const int worker = blockIdx.x;
  const int4 st = *(const int4*)(a.wstart + 4 * worker);   // (b, r << 20 | block, L_b, run length)
  if (st.x < 0) return;
  int left = st.w;
  int b = st.x, r = st.y >> 20, blk = st.y & 0xFFFFF, n = (st.z + kBlockTokens - 1) / kBlockTokens;
  bool first_segment = true;
  while (left > 0) {
    const int cnt = min(left, n - blk);                 // blocks of this row that are ours
    const int ctx = a.ctx_lens[b];
    const int tok0 = blk * kBlockTokens;
    const int len = min(ctx, (blk + cnt) * kBlockTokens) - tok0;
    const int g = r / n_ht;
    const int h0 = (r - g * n_ht) * kHT;
    const int n_heads = min(kHT, group - h0);
    const float* qrows[kHT];
#pragma unroll
    for (int h = 0; h < kHT; ++h)
      qrows[h] = (const float*)a.q + ((size_t)b * a.hq + (size_t)g * group + h0 + min(h, n_heads - 1)) * D;
    attend_f32<D, kThreads, kHT>(qrows, n_heads, (const float*)a.k_pages, (const float*)a.v_pages,
                  a.page_table + (size_t)b * a.max_pages + tok0 / kPageSize, len, hkv, g, a.scale_log2, o_part,
                  ml_part, o_out, ml_out);
    const bool whole = (blk == 0 && cnt == n);
    for (int e = tid; e < n_heads * D; e += kThreads) {
      const int h = e / D, d = e % D;
      if (whole) {
        const size_t orow = (size_t)b * a.hq + (size_t)g * group + h0 + h;
        ((float*)a.out)[orow * D + d] = o_out[h][d] / ml_out[h][1];
        if (a.lse && d == 0) a.lse[orow] = ml_out[h][0] + __builtin_amdgcn_logf(ml_out[h][1]);
      } else {
        const size_t slot = (size_t)worker * 2 + (first_segment ? 0 : 1);
        a.partial_o[(slot * kHT + h) * D + d] = o_out[h][d];
        if (d == 0) {
          a.partial_ml[(slot * kHT + h) * 2 + 0] = ml_out[h][0];
          a.partial_ml[(slot * kHT + h) * 2 + 1] = ml_out[h][1];
        }
      }
    }
    __syncthreads();
    first_segment = false;
    left -= cnt;
    if (left > 0) {                                      // next row of the sequence
      blk = 0;
      if (++r == rows_per_b) {
        r = 0;
        do {
          ++b;
          n = a.prefix[b + 1] - a.prefix[b];
        } while (n == 0);
      }
    }
  }
}

// Append in float32: one workgroup per (query row, KV head, head tile); row i of trajectory b
// sees tokens [0, L_b - n_b + i].
template <int D>
__global__ __launch_bounds__(kThreads) void append_f32_kernel(const AppendArgs a, int total_q) {
  __shared__ __attribute__((aligned(16))) float o_part[kThreads / 64][kHT][D];
  __shared__ float ml_part[kThreads / 64][kHT][2];
  __shared__ __attribute__((aligned(16))) float o_out[kHT][D];
  __shared__ float ml_out[kHT][2];
  const int tid = threadIdx.x;
  const int group = a.group, hkv = a.hkv;
  const int n_ht = (group + kHT - 1) / kHT;
  const long n_work = (long)total_q * hkv * n_ht;
  for (long work = blockIdx.x; work < n_work; work += gridDim.x) {
    const int row = (int)(work / (hkv * n_ht));
    const int g = (int)((work - (long)row * hkv * n_ht) / n_ht);
    const int h0 = (int)(work % n_ht) * kHT;
    const int n_heads = min(kHT, group - h0);
    // trajectory of this packed row: largest b with q_offsets[b] <= row
    int lo = 0, hi = a.batch;
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (a.q_offsets[mid] <= row) lo = mid; else hi = mid;
    }
    const int b = lo;
    const int i = row - a.q_offsets[b];
    const int len = a.ctx_lens[b] - a.q_lens[b] + i + 1;
    const float* qrows[kHT];
#pragma unroll
    for (int h = 0; h < kHT; ++h)
      qrows[h] = (const float*)a.q + ((size_t)row * a.hq + (size_t)g * group + h0 + min(h, n_heads - 1)) * D;
    attend_f32<D, kThreads, kHT>(qrows, n_heads, (const float*)a.k_pages, (const float*)a.v_pages,
                  a.page_table + (size_t)b * a.max_pages, len, hkv, g, a.scale_log2, o_part, ml_part, o_out,
                  ml_out);
    for (int e = tid; e < n_heads * D; e += kThreads) {
      const int h = e / D, d = e % D;
      const size_t orow = (size_t)row * a.hq + (size_t)g * group + h0 + h;
      ((float*)a.out)[orow * D + d] = o_out[h][d] / ml_out[h][1];
      if (a.lse && d == 0) a.lse[orow] = ml_out[h][0] + __builtin_amdgcn_logf(ml_out[h][1]);
    }
    __syncthreads();
  }
}

}  // namespace

hipError_t launch_decode_f32(const DecodeArgs& a, int head_dim, int grid, hipStream_t s) {
  if (head_dim == 64) {
    hipLaunchKernelGGL((decode_f32_kernel<64>), dim3(grid), dim3(kThreads), 0, s, a);
  } else if (head_dim == 128) {
    hipLaunchKernelGGL((decode_f32_kernel<128>), dim3(grid), dim3(kThreads), 0, s, a);
  } else {
    return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_decode_f32_direct(const DecodeArgs& a, int head_dim, hipStream_t s) {
  const bool single = (long)a.batch * a.hq <= kNumCUs;   // 4 contexts of 256 tokens, 8/2/64: 4.9 us a launch, with rows of four heads 8.3
  const dim3 grid((unsigned)(single ? a.batch * a.hq + 1 : a.batch * a.rows_per_b + 1));
  if (head_dim == 64 && single) {
    hipLaunchKernelGGL((decode_f32_direct_kernel<64, 1>), grid, dim3(kDirectThreads), 0, s, a);
  } else if (head_dim == 64) {
    hipLaunchKernelGGL((decode_f32_direct_kernel<64, kHT>), grid, dim3(kDirectThreads), 0, s, a);
  } else if (head_dim == 128 && single) {
    hipLaunchKernelGGL((decode_f32_direct_kernel<128, 1>), grid, dim3(kDirectThreads), 0, s, a);
  } else if (head_dim == 128) {
    hipLaunchKernelGGL((decode_f32_direct_kernel<128, kHT>), grid, dim3(kDirectThreads), 0, s, a);
  } else {
    return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_append_f32(const AppendArgs& a, int head_dim, int grid, hipStream_t s) {
  const int total_q = a.total_q;   // rows are enumerated directly, no tile list
  if (head_dim == 64) {
    hipLaunchKernelGGL((append_f32_kernel<64>), dim3(grid), dim3(kThreads), 0, s, a, total_q);
  } else if (head_dim == 128) {
    hipLaunchKernelGGL((append_f32_kernel<128>), dim3(grid), dim3(kThreads), 0, s, a, total_q);
  } else {
    return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace rollattn
