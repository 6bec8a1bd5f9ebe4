// Pair totals of a counted frame or batch (device), shared by the kernels
// that finish them.
#pragma once

#include "common.hpp"
#include "internal.hpp"

namespace ss {

// Pair totals after the count kernel: per frame, the sum of the one-frame
// count workgroups' totals plus what multi-frame workgroups added directly;
// then all pairs, num_pairs, the status (bad depth, over 2^32 pairs, over
// capacity) and the per-frame pair counts and first pairs.  One workgroup of
// THREADS >= 256 threads; s_fm holds kMaxFrames values.
template <int THREADS>
__device__ __forceinline__ void finish_totals(const PairTotalsArgs& a, unsigned long long* s_fm,
                                              unsigned long long* s_tmp64, uint32_t* s_tmp) {
  const uint32_t d = threadIdx.x;
  for (uint32_t f = d; f < a.n_frames; f += THREADS) s_fm[f] = a.totals[1 + f];
  __syncthreads();
  for (uint32_t b = d; b < a.count_blocks; b += THREADS) {
    const unsigned long long t = a.block_total[b];
    if (t) atomicAdd(&s_fm[a.block_frame[b]], t);
  }
  __syncthreads();
  const unsigned long long fm = d < a.n_frames ? s_fm[d] : 0ull;
  unsigned long long m;
  block_exclusive_scan<unsigned long long, THREADS>(fm, s_tmp64, m);
  if (d == 0) {
    uint32_t st = SS_OK;
    if (*a.bad) st = SS_ERR_INVALID_INPUT;
    else if (m > 0xFFFFFFFFull) st = SS_ERR_OVERFLOW;
    else if (m > a.capacity) st = SS_ERR_CAPACITY;
    *a.num_pairs = m > 0xFFFFFFFFull ? 0xFFFFFFFFu : static_cast<uint32_t>(m);
    raise_status(a.status, st);
  }
  if (a.frame_pairs == nullptr && a.seg_base == nullptr) return;
  const uint32_t f32 = fm > 0xFFFFFFFFull ? 0xFFFFFFFFu : static_cast<uint32_t>(fm);
  uint32_t all;
  const uint32_t ex = block_exclusive_scan<uint32_t, THREADS>(f32, s_tmp, all);
  if (d < a.n_frames) {
    if (a.frame_pairs) a.frame_pairs[d] = f32;
    if (a.frame_pair_base) a.frame_pair_base[d] = ex;
  }
  if (a.seg_base == nullptr) return;
  // segmented tile passes (meaningful only while the status stays SS_OK,
  // i.e. all pairs fit in 32 bits): each frame's first pair and first
  // workgroup
  const uint32_t wgs = static_cast<uint32_t>((static_cast<uint64_t>(f32) + a.seg_tile - 1) / a.seg_tile);
  uint32_t wall;
  const uint32_t wex = block_exclusive_scan<uint32_t, THREADS>(wgs, s_tmp, wall);
  if (d < a.n_frames) {
    a.seg_base[d] = ex;
    a.seg_wgs[d] = wex;
  }
  if (d == 0) {
    a.seg_base[a.n_frames] = all;
    a.seg_wgs[a.n_frames] = wall;
  }
}

}  // namespace ss
