// Device code of the decode partition, shared by the kernels that plan.
#pragma once

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

// Which K and V rows are worth a place in the caches: those that another worker reads, too.  All of them where there are several
// rows per KV head, or where the contexts have more pages between them than the pool (a block is two pages, the last of a
// row one or two).
__device__ __forceinline__ bool all_read_again(const DecodePlanArgs& a, int blocks) {
  return a.head_tiles || (long)blocks * 2 - a.batch > a.num_pages;
}

// Decode partition.  Every trajectory is cut into blocks of kBlockTokens tokens; the rows
// (trajectory b, row r in [0, rows_per_b)) are laid end to end, b outermost, each with
// n_b = ceil(L_b / kBlockTokens) blocks; the resulting sequence of T blocks is dealt to the W
// workers in equal contiguous runs of per = ceil(T / W) blocks.  Written out: the exclusive
// scan of n_b, the run length, T, and for every worker one 16-byte record with all it needs to
// start: (b, r << 20 | block, L_b, blocks in its run), or b = -1 for a worker without blocks.
// len_of(b): tokens of trajectory b that take part.
struct DecodePlanLds {
  int4 wave_tot[kPlanThreads / 256];
  int prefix_s[kLdsPrefix + 1], len_s[kLdsPrefix];
};
template <class L>
__device__ __forceinline__ void plan_decode(const DecodePlanArgs& a, DecodePlanLds& lds, L&& len_of) {
  int4* const wave_tot = lds.wave_tot;
  int* const prefix_s = lds.prefix_s;
  int* const len_s = lds.len_s;
  const int tid = threadIdx.x;
  const int32_t batch = a.batch, rows_per_b = a.rows_per_b, workers = a.workers, slots = a.slots;
  int32_t* const header = a.header;
  int32_t* const prefix = a.prefix;
  int32_t* const wstart = a.wstart;
  const bool in_lds = batch <= kLdsPrefix;
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

// The same rule for a batch of at most 64 trajectories, worked out by every wave of a decode launch for itself: a lane per
// trajectory, the search for the worker's start one ballot.  Writes what the plan kernel would have written (the first
// worker the header and the scan, each worker its record), because the merge and rollattn_debug_read_plan read it.
// Returns the record (b, r << 20 | block, L_b, blocks in the run), the same in all lanes, and whether the run's pages may be read
// by another worker, too: told by a second page that another trajectory has as well (see plan_read_again).
__device__ __forceinline__ int4 plan_decode_in_wave(const DecodePlanArgs& a, int worker, bool* read_again) {
  const int lane = threadIdx.x & 63;
  const int len = lane < a.batch ? a.ctx_lens[lane] : 0;
  const int page = len > kPageSize ? a.page_table[(size_t)lane * a.max_pages + 1] : -1;
  const int count = (len + kBlockTokens - 1) / kBlockTokens;
  const int upto = wave_inclusive_scan(count), first = upto - count;
  const int blocks = __builtin_amdgcn_readlane(upto, 63);
  const int total = blocks * a.rows_per_b;
  const int per = max(1, (total + a.workers - 1) / a.workers);
  const unsigned int x = (unsigned int)worker * (unsigned int)per;
  if (worker == 0) {
    if (lane < a.batch) a.prefix[lane] = first;
    if (lane == 0) {
      a.prefix[a.batch] = blocks;
      a.header[kPlanPer] = per;
      a.header[kPlanTotal] = total;
      a.header[kPlanWorkers] = a.workers;
      a.header[kPlanRowsPerB] = a.rows_per_b;
    }
  }
  int4 st = make_int4(-1, 0, 0, 0);
  if (worker < a.workers && x < (unsigned int)total) {
    // trajectories that start at or before x: a run of lanes from 0 on, the last of them has blocks (see plan_decode)
    const unsigned long long before = __builtin_amdgcn_ballot_w64(lane < a.batch && (unsigned int)(a.rows_per_b * first) <= x);
    const int b = 63 - __builtin_clzll(before);
    const int n = __builtin_amdgcn_readlane(count, b);
    const int rem = (int)x - a.rows_per_b * __builtin_amdgcn_readlane(first, b);
    const int mine = min(per, total - (int)x);
    bool again = all_read_again(a, blocks);
    // the trajectories of the run
    const unsigned long long started = __builtin_amdgcn_ballot_w64(lane < a.batch && (unsigned int)(a.rows_per_b * first) < x + (unsigned int)mine);
    for (int i = b; i < 64 - __builtin_clzll(started) && !again; ++i) {
      const int p = __builtin_amdgcn_readlane(page, i);
      again = p >= 0 && __builtin_popcountll(__builtin_amdgcn_ballot_w64(page == p)) > 1;
    }
    st = make_int4(b, ((rem / n) << 20) | (rem % n), __builtin_amdgcn_readlane(len, b), mine);
    *read_again = again;
    if (worker == 0 && lane == 0) a.header[kPlanReadAgain] = again;   // (of the first run, for who reads the plan)
  }
  if (lane == 0) *(int4*)(a.wstart + 4 * worker) = st;
  return st;
}

}  // namespace

}  // namespace rollattn
