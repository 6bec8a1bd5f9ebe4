// Small frames (at most 256 tiles and 16,384 Gaussians) in one kernel, for
// latency: the same result as the other paths -- all (tile, Gaussian) pairs
// ordered by (tile, depth, index) and the tile ranges (paper: Background,
// "Duplication with Tiles" and "Sorting") -- without a pair ever being
// exchanged between workgroups.
//
// One workgroup per tile reads every record of the frame (at most 256 KB,
// which its XCD's L2 serves after the first reader).  A Gaussian's pairs in
// lower tiles follow from its rectangle in closed form, so their sum over the
// frame is the tile's start, the sum of all rectangles is the pair count, and
// no workgroup waits for another.  The Gaussians that meet the tile are sorted
// by (depth, index) in LDS and written at the tile's start.
//
// What bounds it is one pass of loads and some 60 vector instructions per
// record, 16 waves a CU, then the sort.  Two kernels before it (one bucketing
// 512 Gaussians per workgroup, on 20 CUs for 10,000, one gathering and sorting
// the tiles) took 13.8 + 11.5 us for the 256 x 256 frame of 10,000 Gaussians,
// this one 11.4 (24.4 -> 11.4 us a call).
#include "common.hpp"
#include "internal.hpp"

namespace ss {
namespace {

constexpr uint32_t kSortThreads = 1024;
constexpr uint32_t kSortItems = kTinyMaxGaussians / kSortThreads;   // 16
constexpr uint32_t kSortWaves = kSortThreads / kWave;

__device__ __forceinline__ uint32_t tclamp(int64_t v, uint32_t n) {
  return v < 0 ? 0u : (v > static_cast<int64_t>(n) ? n : static_cast<uint32_t>(v));
}

// Workgroup t: the tile's run ordered by (depth, index), by counting when it
// fits one item per thread, else by 8-bit LSD passes (index bits, then depth
// bits) with wave-ballot ranking in LDS.
__global__ __launch_bounds__(kSortThreads) void k_tiny_frame(TinyArgs a) {
  __shared__ __align__(16) uint64_t s_buf[kTinyMaxGaussians + 2];
  __shared__ uint32_t s_wcnt[kSortWaves * 256];   // LSD passes: per-wave digit counts; counting: ranks
  __shared__ uint32_t s_dstart[256];
  __shared__ unsigned long long s_tmp64[kSortWaves];
  __shared__ uint32_t s_tmp[kSortWaves];
  __shared__ uint32_t s_bad[kSortWaves];

  const uint32_t tid = threadIdx.x, lane = lane_id(), wave = tid / kWave;
  const uint32_t t = blockIdx.x;
  const uint32_t tx = t % a.tiles_x, ty = t / a.tiles_x;
  // record j * kSortThreads + tid, eight loads at a time
  uint32_t hits = 0;                  // bit j: that record meets the tile
  uint32_t before = 0, all = 0;       // pairs in lower tiles, all pairs
  bool bad = false;
  constexpr uint32_t kLoads = 8;
  for (uint32_t j0 = 0; j0 * kSortThreads < a.n; j0 += kLoads) {
    int4 rec[kLoads];
#pragma unroll
    for (uint32_t j = 0; j < kLoads; ++j) {
      const uint32_t g = (j0 + j) * kSortThreads + tid;
      rec[j] = g < a.n ? reinterpret_cast<const int4*>(a.gaussians)[g] : make_int4(0, 0, 0, 0);
    }
#pragma unroll
    for (uint32_t j = 0; j < kLoads; ++j) {
      if ((j0 + j) * kSortThreads >= a.n) break;   // uniform: no such records
      const int4 r = rec[j];
      const uint32_t radius = static_cast<uint32_t>(r.w);   // 0: culled
      uint32_t x0, x1, y0, y1;
      // means and radii of any sensible image: 32-bit sums (|mean| < 2^29,
      // 16 radius < 2^29); the wave takes 64-bit ones if any lane must
      const bool narrow = radius < (1u << 25) && static_cast<uint32_t>(r.x) + (1u << 29) < (1u << 30) &&
                          static_cast<uint32_t>(r.y) + (1u << 29) < (1u << 30);
      if (ballot(!narrow) == 0) {
        const int R = static_cast<int>(radius << 4), nx = static_cast<int>(a.tiles_x), ny = static_cast<int>(a.tiles_y);
        x0 = static_cast<uint32_t>(min(max((r.x - R) >> 8, 0), nx));
        x1 = static_cast<uint32_t>(min(max((r.x + R + 255) >> 8, 0), nx));
        y0 = static_cast<uint32_t>(min(max((r.y - R) >> 8, 0), ny));
        y1 = static_cast<uint32_t>(min(max((r.y + R + 255) >> 8, 0), ny));
      } else {
        const int64_t R = static_cast<int64_t>(radius) << 4;
        x0 = tclamp((static_cast<int64_t>(r.x) - R) >> 8, a.tiles_x);
        x1 = tclamp((static_cast<int64_t>(r.x) + R + 255) >> 8, a.tiles_x);
        y0 = tclamp((static_cast<int64_t>(r.y) - R) >> 8, a.tiles_y);
        y1 = tclamp((static_cast<int64_t>(r.y) + R + 255) >> 8, a.tiles_y);
      }
      if (radius != 0 && x1 > x0 && y1 > y0) {
        const uint32_t w = x1 - x0;
        if (static_cast<uint32_t>(r.z) - 1u >= 0x7F7FFFFFu) bad = true;
        const bool in_row = ty >= y0 && ty < y1;
        all += w * (y1 - y0);
        before += w * (min(max(ty, y0), y1) - y0) + (in_row ? min(max(tx, x0), x1) - x0 : 0u);
        if (in_row && tx >= x0 && tx < x1) hits |= 1u << (j0 + j);
      }
    }
  }
  // one scan: hits (bits 0-14), pairs in lower tiles (15-37) and all pairs
  // (38-60), each at most 2^22
  if (lane == 0) s_bad[wave] = 0;
  if (ballot(bad) != 0 && lane == 0) s_bad[wave] = 1;
  unsigned long long sums;
  const unsigned long long ex = block_exclusive_scan<unsigned long long, kSortThreads>(
      (static_cast<unsigned long long>(all) << 38) | (static_cast<unsigned long long>(before) << 15) |
          static_cast<uint32_t>(__popc(hits)),
      s_tmp64, sums);
  // the same in every lane: scalars
  const uint32_t sums_lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(sums));
  const uint32_t sums_hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(sums >> 32));
  const uint32_t n = sums_lo & 0x7FFFu;
  const uint32_t start = (sums_lo >> 15 | sums_hi << 17) & 0x7FFFFFu;
  const uint32_t m = sums_hi >> 6;
  uint32_t any_bad = 0;
#pragma unroll
  for (uint32_t w = 0; w < kSortWaves; ++w) any_bad |= s_bad[w];
  uint32_t st = SS_OK;
  if (any_bad) st = SS_ERR_INVALID_INPUT;
  else if (m > a.capacity) st = SS_ERR_CAPACITY;
  if (t == 0 && tid == 0) {
    *a.num_pairs = m;
    *a.status = st;
  }
  if (st != SS_OK) return;
  if (tid == 0) {
    a.ranges[2 * t] = start;
    a.ranges[2 * t + 1] = start + n;
  }
  if (n == 0) return;
  // the tile's items (depth bits << 32 | index), in any order
  uint32_t at = static_cast<uint32_t>(ex) & 0x7FFFu;
  for (uint32_t bits = hits; bits != 0; bits &= bits - 1) {
    const uint32_t g = static_cast<uint32_t>(__builtin_ctz(bits)) * kSortThreads + tid;
    s_buf[at++] = (static_cast<uint64_t>(__float_as_uint(a.gaussians[g].depth)) << 32) | g;
  }
  // counting: several threads per item where there are few items, each over a
  // share of the others
  const uint32_t parts = n <= kSortThreads / 4 ? 4u : n <= kSortThreads / 2 ? 2u : 1u;
  const uint32_t n2 = (n + 2 * parts - 1) / (2 * parts) * (2 * parts);   // padded with all-ones items, above every valid one
  if (n <= kSortThreads) {
    if (tid < n2 - n) s_buf[n + tid] = ~0ull;
    s_wcnt[tid] = 0;
  }
  __syncthreads();
  uint64_t* keys = a.keys + start;
  uint32_t* vals = a.values + start;
  const uint64_t tile_hi = static_cast<uint64_t>(t) << 32;

  if (n <= kSortThreads) {
    // items are distinct, so an item's place is the number of smaller ones,
    // read two at a time; a share is whole waves.  Counted in pairs, so that
    // every read is plainly of 16 aligned bytes, one LDS access each: what this
    // loop waits for (1,000 items in a tile: 33.6 -> 23.3 us a frame)
    const uint32_t share = kSortThreads / parts, i = tid % share, len = n2 / (2 * parts);
    const uint32_t part = __builtin_amdgcn_readfirstlane(tid / share);
    const ulonglong2* two = reinterpret_cast<const ulonglong2*>(s_buf);
    const uint64_t me = i < n ? s_buf[i] : 0ull;
    uint32_t r = 0;
    if (i < n) {
#pragma unroll 4
      for (uint32_t j = part * len; j < (part + 1) * len; ++j) {
        const ulonglong2 q = two[j];
        r += (q.x < me) + (q.y < me);
      }
      if (parts != 1 && r != 0) atomicAdd(&s_wcnt[i], r);
    }
    if (parts != 1) __syncthreads();
    if (tid < n) {
      if (parts != 1) r = s_wcnt[tid];
      keys[r] = tile_hi | static_cast<uint32_t>(me >> 32);
      vals[r] = static_cast<uint32_t>(me);
    }
    return;
  }

  // stable 8-bit LSD passes over the index (bits 0-13: fewer than 2^14
  // Gaussians) and then the depth bits (32-63), items wave-striped in
  // registers (wave w holds [w * 64 * 16, (w + 1) * 64 * 16))
  uint64_t it[kSortItems];
#pragma unroll
  for (uint32_t j = 0; j < kSortItems; ++j) {
    const uint32_t q = wave * (kWave * kSortItems) + j * kWave + lane;
    it[j] = q < n ? s_buf[q] : 0ull;
  }
  constexpr uint32_t kShifts[6] = {0, 8, 32, 40, 48, 56};
  for (uint32_t sp = 0; sp < 6; ++sp) {
    const uint32_t shift = kShifts[sp];
    for (uint32_t i = tid; i < kSortWaves * 256; i += kSortThreads) s_wcnt[i] = 0;
    __syncthreads();
    uint32_t* wc = s_wcnt + wave * 256;
    uint32_t dg[kSortItems], pos[kSortItems];
#pragma unroll
    for (uint32_t j = 0; j < kSortItems; ++j) {
      const uint32_t q = wave * (kWave * kSortItems) + j * kWave + lane;
      const bool valid = q < n;
      dg[j] = valid ? static_cast<uint32_t>(it[j] >> shift) & 255u : 256u;
      const uint64_t peers = match_digit<8>(dg[j], ballot(valid));
      uint32_t r = 0;
      if (valid) {
        const uint32_t old = wc[dg[j]];
        const uint32_t below = popc_below(peers);
        r = old + below;
        __builtin_amdgcn_wave_barrier();
        if (below == 0) wc[dg[j]] = old + static_cast<uint32_t>(__popcll(peers));
      }
      __builtin_amdgcn_wave_barrier();
      pos[j] = r;
    }
    __syncthreads();
    uint32_t dcnt = 0;
    if (tid < 256) {
      for (uint32_t w = 0; w < kSortWaves; ++w) {
        const uint32_t x = s_wcnt[w * 256 + tid];
        s_wcnt[w * 256 + tid] = dcnt;
        dcnt += x;
      }
    }
    uint32_t dall;
    const uint32_t dex = block_exclusive_scan<uint32_t, kSortThreads>(dcnt, s_tmp, dall);
    if (tid < 256) s_dstart[tid] = dex;
    __syncthreads();
#pragma unroll
    for (uint32_t j = 0; j < kSortItems; ++j)
      if (dg[j] < 256) s_buf[s_dstart[dg[j]] + wc[dg[j]] + pos[j]] = it[j];
    __syncthreads();
#pragma unroll
    for (uint32_t j = 0; j < kSortItems; ++j) {
      const uint32_t q = wave * (kWave * kSortItems) + j * kWave + lane;
      it[j] = q < n ? s_buf[q] : 0ull;
    }
    __syncthreads();
  }
#pragma unroll
  for (uint32_t j = 0; j < kSortItems; ++j) {
    const uint32_t q = wave * (kWave * kSortItems) + j * kWave + lane;
    if (q < n) {
      keys[q] = tile_hi | static_cast<uint32_t>(it[j] >> 32);
      vals[q] = static_cast<uint32_t>(it[j]);
    }
  }
}

}  // namespace

hipError_t launch_tiny(const TinyArgs& a, hipStream_t s) {
  if (a.n > kTinyMaxGaussians || a.tiles_x * a.tiles_y > kTinyMaxTiles) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_tiny_frame, dim3(a.tiles_x * a.tiles_y), dim3(kSortThreads), 0, s, a);
  return hipGetLastError();
}

}  // namespace ss
