// The spread passes: from the Gaussians in depth order to the sorted pairs
// and the tile ranges in two stable partitions, by tile column and then by
// tile row, without ever writing a pair before its final place (paper:
// Background, "Duplication with Tiles" and "Sorting").
//
// A Gaussian's tiles are an interval of columns times an interval of rows,
// so duplication and sorting can share a pass per axis:
//   column pass: every Gaussian yields one item for each column of its
//     interval, and the items are partitioned stably by column;
//   row pass: every item (one column, an interval of rows) yields one pair
//     for each of its rows, partitioned stably by row.
// The input of the column pass is in (depth, index) order, so its output is
// in (column, depth, index) order and the row pass's in (row, column, depth,
// index) order, which is the order of (tile, depth, index).  Between the
// passes travel the items, about half as many as pairs (the mean height of a
// rectangle fewer), 10 bytes each; the pairs are written once, 12 bytes each.
//
// One pass, for a workgroup of some thousand consecutive items, each covering
// the digits [lo, hi):
//   1. a bit matrix in LDS, one row of a bit per item for each digit: every
//      item toggles its bit in the rows where its interval starts and ends,
//      whatever its length.  The rows are cut into blocks, each walked by
//      the lanes of one row's words; an item whose interval runs on into a
//      block sets its bit in the block's opening word.
//   2. the running XOR down a block's rows, from its opening word, is the
//      matrix of covered digits.  It is stored back, with the prefix of the
//      bit counts over a row's 64-bit words; a row's total is the workgroup's
//      count of the digit, published for the look-back.
//   3. an item's rank among a row's items is the prefix of its word plus the
//      bits below its own (the items of a wave share a word); the item writes
//      its number at that place of a list in digit order.  Each item lists
//      its first kInline digits; the rest of the wave's items' digits are
//      dealt out evenly over the lanes, so that long intervals do not hold
//      the short ones up.
//   4. decoupled look-back over the earlier workgroups of the chain (a
//      frame's) gives each digit's first output position;
//   5. the list is walked digit by digit, so that the outputs of a digit
//      leave as one run.
//
// The row pass's workgroups never straddle two columns (a column of C items
// takes max(1, ceil(C / items)) of them), so a workgroup knows its
// column, and the first workgroup of a column knows from its look-back where
// every tile of the column starts: it writes the ranges.
//
// Measured (MI355X, before: expansion into 8-byte items and two digit passes
// over them, look-back or totals and a ranges kernel beside them): the
// 6M-Gaussian full-HD frame (11.0M items, 27.6M pairs) 89 + 127 us against
// 374 us, the frame 589 -> 423 us; the 1M-Gaussian one 26 + 32 against 90,
// 162.5 -> 132.5 us; a batch of 64 frames (170M pairs) 3.41 -> 2.25 ms.  The
// row pass moves 16 B per item and pair at 3.5 TB/s; of a workgroup's 20 us
// about 5 are its loads, 5 the look-back and the rest LDS and vector work.
#include "common.hpp"
#include "internal.hpp"

namespace ss {
namespace {

constexpr uint32_t kMaxDigits = 256;
constexpr uint32_t kInline = 2;

// A workgroup of THREADS threads takes kItems = 4 * THREADS items.
template <uint32_t THREADS>
struct Shape {
  static constexpr uint32_t kThreads = THREADS;
  static constexpr uint32_t kWaves = THREADS / kWave;
  static constexpr uint32_t kPer = 4;                      // items per thread
  static constexpr uint32_t kItems = kPer * THREADS;
  static constexpr uint32_t kWords = kItems / kWave;       // 64-bit words of a matrix row
  static constexpr uint32_t kRowStride = kWords + 1;       // a column of the matrix spreads over the banks
  static constexpr uint32_t kPfxStride = kWords + 2;       // 16-bit prefixes: an odd number of 32-bit words
  static constexpr uint32_t kBlocks = THREADS / kWords;    // blocks of rows, each walked by kWords lanes
  // Outputs listed per round; a workgroup with more takes further rounds.
  static constexpr uint32_t kSlots = 3 * kItems;
  static_assert(kWords == 16 || kWords == 32 || kWords == 64, "a row's lanes are a DPP row, half a wave or a wave");
  static_assert(kBlocks == 16, "at most 16 rows a block");
  static_assert(kBlocks * kRowStride * sizeof(uint64_t) <= kSlots * sizeof(uint16_t), "opening words in the list's place");
};

// LDS, sized by the launch.  Matrix and prefixes; in their place, once the
// list is whole, the items (8 bytes, in the column pass 10).  Then the list
// (before it the blocks' opening words), and per digit its count, later its
// first output, and its first slot.
template <typename S>
struct Lds {
  uint32_t pfx, slots, cnt, off, total;
  __host__ __device__ Lds(uint32_t digits, bool rows) {
    pfx = digits * S::kRowStride * 8;
    const uint32_t m = pfx + (digits * S::kPfxStride * 2 + 15) / 16 * 16, items = S::kItems * (rows ? 8 : 10);
    slots = m > items ? m : items;
    cnt = slots + S::kSlots * 2;
    off = cnt + (digits + 3) / 4 * 16;
    total = off + (digits + 4) / 4 * 16;
  }
};

template <bool ROWS, uint32_t THREADS>
__global__ __launch_bounds__(THREADS, ROWS ? 8 : 6) void k_spread(SpreadArgs a) {
  using S = Shape<THREADS>;
  constexpr uint32_t kPer = S::kPer, kWaves = S::kWaves, kWords = S::kWords, kRowStride = S::kRowStride,
                     kPfxStride = S::kPfxStride, kBlocks = S::kBlocks, kSlots = S::kSlots;
  extern __shared__ __align__(16) unsigned char s_dyn[];
  __shared__ uint32_t s_timeout, s_exit[kWaves];
  const Lds<S> at(a.max_digits, ROWS);
  uint64_t* s_bits = reinterpret_cast<uint64_t*>(s_dyn);            // [digits][kRowStride]
  uint16_t* s_pfx = reinterpret_cast<uint16_t*>(s_dyn + at.pfx);    // [digits][kPfxStride]
  uint2* s_item = reinterpret_cast<uint2*>(s_dyn);                  // [kItems] depth bits, index
  uint16_t* s_rows = reinterpret_cast<uint16_t*>(s_item + S::kItems);  // column pass: the item's rows
  uint16_t* s_slot = reinterpret_cast<uint16_t*>(s_dyn + at.slots);
  uint64_t* s_open = reinterpret_cast<uint64_t*>(s_dyn + at.slots);       // [kBlocks][kRowStride]
  uint32_t* s_cnt = reinterpret_cast<uint32_t*>(s_dyn + at.cnt);
  uint32_t* s_off = reinterpret_cast<uint32_t*>(s_dyn + at.off);          // [digits + 1]
  const uint32_t tid = threadIdx.x;
  const uint32_t t = blockIdx.x;
  const uint32_t lane = lane_id();
  const uint32_t wave = __builtin_amdgcn_readfirstlane(tid / kWave);

  // ---- this workgroup's items ----
  // After an error the row pass's chunks are not there, and nothing is read
  // through one.  But another workgroup of this launch may raise the status
  // between two waves' reads of it, so a wave that sees an error only takes no
  // items here; the workgroup leaves as one, after the barrier below.  (The
  // rest of this part is the same in every wave.)
  const bool failed = __builtin_amdgcn_readfirstlane(*a.status) != SS_OK;
  if (lane == 0) s_exit[wave] = failed;
  const SpreadChunk ch = a.chunks[t];
  const uint32_t used = ROWS ? *a.num_chunks : ~0u;
  if (t >= used) return;
  // column pass: no live Gaussians here, nor in any later workgroup of the frame
  if (!ROWS && (ch.count & 0xFFFFu) == 0) return;
  const uint32_t base = ch.base, n = failed ? 0u : ch.count & 0xFFFFu, f = failed ? 0u : ch.frame;
  const uint32_t col = ch.count >> 16;   // row pass: the column

  // ---- loads: item i = j * THREADS + tid ----
  const FrameInfo& F = a.table[f];
  uint32_t lo[kPer], hi[kPer], rw[kPer];
  uint2 it[kPer];
  const uint32_t gauss_base = ROWS ? 0u : F.gauss_base;
#pragma unroll
  for (uint32_t j = 0; j < kPer; ++j) {
    const uint32_t i = j * THREADS + tid;
    lo[j] = hi[j] = rw[j] = 0;
    it[j] = make_uint2(0, 0);
    if (i < n) {
      if (ROWS) {
        const uint32_t r = a.item_rows[base + i];
        const uint64_t v = a.item[base + i];
        lo[j] = r & 0xFFu;
        hi[j] = lo[j] + (r >> 8) + 1u;
        it[j] = make_uint2(static_cast<uint32_t>(v), static_cast<uint32_t>(v >> 32));
      } else {
        const uint32_t g = a.val[base + i];
        const uint32_t r = a.rect[a.rect_by_index ? g : base + i];
        lo[j] = r & 0xFFu;
        hi[j] = lo[j] + ((r >> 16) & 0xFFu) + 1u;
        rw[j] = ((r >> 8) & 0xFFu) | ((r >> 24) << 8);
        it[j] = make_uint2(a.key[base + i], g - gauss_base);
      }
    }
  }
  const uint32_t digits = ROWS ? F.tiles_y : F.tiles_x;
  // cleared while the loads are on their way
  for (uint32_t i = tid; i < digits * kRowStride; i += THREADS) s_bits[i] = 0;
  for (uint32_t i = tid; i < kBlocks * kRowStride; i += THREADS) s_open[i] = 0;
  if (tid == 0) s_timeout = 0;
  __syncthreads();
  if (ballot(lane < kWaves && s_exit[lane % kWaves] != 0) != 0) return;

  // ---- 1. toggles and opening words ----
  const uint32_t per_block = (digits + kBlocks - 1) / kBlocks;
  // floor(c / per_block) for c <= 256, per_block <= 16: the product's error stays below 1 / per_block
  const uint32_t magic = (65536 + per_block - 1) / per_block;
#pragma unroll
  for (uint32_t j = 0; j < kPer; ++j) {
    const uint32_t word = j * kWaves + wave;
    uint32_t* p = reinterpret_cast<uint32_t*>(s_bits + word) + (lane >> 5);
    uint32_t* open = reinterpret_cast<uint32_t*>(s_open + word) + (lane >> 5);
    const uint32_t bit = 1u << (lane & 31);
    hi[j] = min(hi[j], digits);   // (the count kernel's rectangles end there)
    if (lo[j] < hi[j]) {
      atomicXor(&p[lo[j] * (2 * kRowStride)], bit);
      // (an interval that ends where a block starts does not open the block)
      const uint32_t end_block = (hi[j] * magic) >> 16;
      if (hi[j] < digits && end_block * per_block != hi[j]) atomicXor(&p[hi[j] * (2 * kRowStride)], bit);
      for (uint32_t b = ((lo[j] * magic) >> 16) + 1; b * per_block < hi[j]; ++b)
        atomicOr(&open[b * (2 * kRowStride)], bit);
    } else {
      lo[j] = hi[j] = 0;
    }
  }
  __syncthreads();

  // ---- 2. covered digits, prefixes, counts: kWords lanes a row ----
  {
    const uint32_t b = tid / kWords, w = tid % kWords;
    uint64_t m = s_open[b * kRowStride + w];
    for (uint32_t k = 0; k < per_block; ++k) {
      const uint32_t r = b * per_block + k;
      const bool on = r < digits;
      if (on) m ^= s_bits[r * kRowStride + w];
      const uint32_t c = on ? static_cast<uint32_t>(__popcll(m)) : 0u;
      uint32_t x = c;   // inclusive scan over the row's lanes
      x += dpp0<kDppRowShr | 1, 0xF, 0xF>(x);
      x += dpp0<kDppRowShr | 2, 0xF, 0xF>(x);
      x += dpp0<kDppRowShr | 4, 0xF, 0xF>(x);
      x += dpp0<kDppRowShr | 8, 0xF, 0xF>(x);
      if (kWords >= 32) x += dpp0<kDppRowBcast15, 0xA, 0xF>(x);
      if (kWords == kWave) x += dpp0<kDppRowBcast31, 0xC, 0xF>(x);
      if (on) {
        s_bits[r * kRowStride + w] = m;
        s_pfx[r * kPfxStride + w] = static_cast<uint16_t>(x - c);
        if (w == kWords - 1) s_cnt[r] = x;
      }
    }
  }
  __syncthreads();
  uint32_t* lb = a.lookback + static_cast<size_t>(t) * a.lb_stride;
  if (tid < digits && a.fault != SS_FAULT_WITHHOLD_BASES)
    st_agent(&lb[tid], (t == ch.first ? kLbInc32 : kLbAgg32) | s_cnt[tid]);
  // every digit's first slot; every wave writes the same values, so none
  // has to wait for another's
  uint32_t total = 0;
  for (uint32_t d0 = 0; d0 < digits; d0 += kWave) {
    const uint32_t d = d0 + lane;
    const uint32_t c = d < digits ? s_cnt[d] : 0u;
    const uint32_t x = wave_inclusive_scan<uint32_t>(c);
    if (d < digits) s_off[d] = total + x - c;
    total += static_cast<uint32_t>(__builtin_amdgcn_readlane(x, kWave - 1));
  }
  s_off[digits] = total;
  __builtin_amdgcn_wave_barrier();

  // ---- 3. the list: slots [round, round + kSlots) ----
  auto list = [&](uint32_t round) {
#pragma unroll
    for (uint32_t j = 0; j < kPer; ++j) {
      const uint32_t word = j * kWaves + wave, item0 = word * kWave;
      uint32_t s[kInline];
#pragma unroll
      for (uint32_t u = 0; u < kInline; ++u) {
        const uint32_t c = lo[j] + u < hi[j] ? lo[j] + u : lo[j];   // in bounds: lo < digits
        const uint64_t m = s_bits[c * kRowStride + word];
        s[u] = s_off[c] + s_pfx[c * kPfxStride + word] + popc_below(m) - round;
      }
#pragma unroll
      for (uint32_t u = 0; u < kInline; ++u)
        if (lo[j] + u < hi[j] && s[u] < kSlots) s_slot[s[u]] = static_cast<uint16_t>(item0 + lane);
      // the remaining digits of the wave's items, in item order, a lane each
      const uint32_t rem = hi[j] - lo[j] > kInline ? hi[j] - lo[j] - kInline : 0u;
      if (ballot(rem != 0) == 0) continue;
      const uint32_t incl = wave_inclusive_scan<uint32_t>(rem);
      const uint32_t all = static_cast<uint32_t>(__builtin_amdgcn_readlane(incl, kWave - 1));
      for (uint32_t q0 = 0; q0 < all; q0 += kWave) {
        const uint32_t q = q0 + lane;
        uint32_t own = 0;   // the first lane whose inclusive sum exceeds q
#pragma unroll
        for (uint32_t step = kWave / 2; step != 0; step >>= 1) {
          const uint32_t v = static_cast<uint32_t>(
              __builtin_amdgcn_ds_bpermute(static_cast<int>((own + step - 1) * 4), static_cast<int>(incl)));
          if (v <= q) own += step;
        }
        const uint32_t from = static_cast<uint32_t>(__builtin_amdgcn_ds_bpermute(
            static_cast<int>(own * 4), static_cast<int>(hi[j])));   // its interval's end
        const uint32_t upto = static_cast<uint32_t>(
            __builtin_amdgcn_ds_bpermute(static_cast<int>(own * 4), static_cast<int>(incl)));
        if (q < all) {
          const uint32_t c = from - (upto - q);
          const uint64_t m = s_bits[c * kRowStride + word];
          const uint32_t slot = s_off[c] + s_pfx[c * kPfxStride + word] +
                                static_cast<uint32_t>(__popcll(m & ((1ull << own) - 1))) - round;
          if (slot < kSlots) s_slot[slot] = static_cast<uint16_t>(item0 + own);
        }
      }
    }
  };
  // the opening words, in the list's place, were read before the last barrier
  list(0);
  __syncthreads();
  // the whole list at once: the matrix is done with, the items take its place
  const bool one_round = total <= kSlots;
  if (one_round) {
#pragma unroll
    for (uint32_t j = 0; j < kPer; ++j) {
      const uint32_t i = j * THREADS + tid;
      s_item[i] = it[j];
      if (!ROWS) s_rows[i] = static_cast<uint16_t>(rw[j]);
    }
  }

  // ---- 4. look-back: a lane per digit, so that a load reads one row of words
  // (two lanes per digit, 16 predecessors a round: 436 us against 426 on the
  // 6M-Gaussian frame, 137 against 133 at full HD, 2.35 ms against 2.30 for 64; four predecessors
  // a round, 2.28) ----
  constexpr uint32_t G = 1;
  if (tid < digits * G) {
    const uint32_t d = tid / G;
    const uint32_t limit = spin_limit_of(a.spin_limit);
    const uint32_t* plan = a.plan + static_cast<size_t>(f) * kPlanWords;
    const uint32_t digit_base = ROWS ? a.pair_base[f] + plan[kPlanRow + d] : a.item_base[f] + plan[d];
    uint32_t excl = 0, excl_max = 0;
    bool ok;
    if (a.fault == SS_FAULT_WITHHOLD_BASES) {
      // test hook: nobody published; every workgroup waits for a word that
      // stays empty, its own
      ok = false;
      for (uint32_t s = 0; s <= limit && !ok; ++s) {
        ok = ld_agent(&lb[d]) != 0;
        __builtin_amdgcn_s_sleep(1);
      }
      if (!ok && tid % G == 0) st_agent(a.status, static_cast<uint32_t>(SS_ERR_TIMEOUT));
    } else {
      ok = lookback_group<G, LbWords32, 4>(a.lookback, t, a.lb_stride, d, a.status, excl, excl_max, ch.first, limit);
    }
    if (!ok) {
      s_timeout = 1;
    } else if (tid % G == 0) {
      if (t != ch.first) st_agent(&lb[d], kLbInc32 | (excl + s_cnt[d]));
      const uint32_t start = digit_base + excl;   // the digit's first output here
      s_cnt[d] = start;
      if (ROWS && ch.col_first) {
        // tile (d, col) starts at `start`, where the tile before it ends
        uint32_t* rg = a.ranges + 2 * (static_cast<size_t>(F.tile_base) + static_cast<size_t>(d) * F.tiles_x + col);
        rg[0] = start;
        if (col != 0 || d != 0) rg[-1] = start;
        if (col == 0 && d == 0)
          a.ranges[2 * (static_cast<size_t>(F.tile_base) + static_cast<size_t>(F.tiles_x) * F.tiles_y) - 1] =
              a.pair_base[f + 1];
      }
    }
  }
  __syncthreads();
  if (s_timeout) return;

  // ---- 5. write the list, a digit per wave and step ----
  const uint32_t tile0 = ROWS ? F.tile_base + col : 0u, tiles_x = F.tiles_x;
  auto write = [&](uint32_t round, auto staged) {
    for (uint32_t d = wave; d < digits; d += kWaves) {
      const uint32_t s0 = max(static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(s_off[d])), round);
      const uint32_t s1 =
          min(static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(s_off[d + 1])), round + kSlots);
      // output of slot s: the digit's first output, plus s minus its first slot
      const uint32_t out = __builtin_amdgcn_readfirstlane(s_cnt[d] - s_off[d]);
      for (uint32_t s = s0 + lane; s < s1; s += kWave) {
        const uint32_t i = s_slot[s - round];
        const uint32_t o = out + s;
        if (o >= a.capacity) continue;
        uint2 v;
        uint32_t rows = 0;
        if constexpr (decltype(staged)::value) {
          v = s_item[i];
          if (!ROWS) rows = s_rows[i];
        } else if (ROWS) {
          const uint64_t w = a.item[base + i];
          v = make_uint2(static_cast<uint32_t>(w), static_cast<uint32_t>(w >> 32));
        } else {
          const uint32_t g = a.val[base + i];
          const uint32_t r = a.rect[a.rect_by_index ? g : base + i];
          v = make_uint2(a.key[base + i], g - gauss_base);
          rows = ((r >> 8) & 0xFFu) | ((r >> 24) << 8);
        }
        if (ROWS) {
          a.keys[o] = (static_cast<uint64_t>(tile0 + d * tiles_x) << 32) | v.x;
          a.values[o] = v.y;
        } else {
          a.item[o] = (static_cast<uint64_t>(v.y) << 32) | v.x;
          a.item_rows[o] = static_cast<uint16_t>(rows);
        }
      }
    }
  };
  if (one_round) {
    write(0, std::true_type{});
    return;
  }
  // more outputs than slots: the matrix stays, the items are read again
  for (uint32_t round = 0;;) {
    write(round, std::false_type{});
    round += kSlots;
    if (round >= total) break;
    __syncthreads();
    list(round);
    __syncthreads();
  }
}

template <bool ROWS, uint32_t THREADS>
hipError_t launch(const SpreadArgs& a, uint32_t nblocks, hipStream_t s) {
  if (nblocks == 0) return hipSuccess;
  if (a.max_digits == 0 || a.max_digits > kMaxDigits || a.lb_stride < a.max_digits) return hipErrorInvalidValue;
  hipLaunchKernelGGL((k_spread<ROWS, THREADS>), dim3(nblocks), dim3(THREADS),
                     Lds<Shape<THREADS>>(a.max_digits, ROWS).total, s, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_columns(const SpreadArgs& a, uint32_t nblocks, hipStream_t s) {
  static_assert(Shape<512>::kItems == kColumnItems, "the column pass's workgroups");
  return launch<false, 512>(a, nblocks, s);
}

hipError_t launch_rows(const SpreadArgs& a, uint32_t row_items, uint32_t nblocks, hipStream_t s) {
  if (row_items == Shape<256>::kItems) return launch<true, 256>(a, nblocks, s);
  if (row_items == Shape<512>::kItems) return launch<true, 512>(a, nblocks, s);
  if (row_items == Shape<1024>::kItems) return launch<true, 1024>(a, nblocks, s);
  return hipErrorInvalidValue;
}

}  // namespace ss
