// Rendering: per-tile alpha blending over the sorted tile lists (paper:
// Background, "Rendering"; Design, "Efficient Tile-Based Rendering" -- one
// workgroup per 16x16 tile, several pixels per thread, colour channels
// unrolled).  Two kernels:
// k_render_tiles, the one a caller gets for the image alone with the usual
// thresholds (described there);
// k_render, for exact compositing and for the statistics, which evaluate
// every list entry at every pixel, and for the image of a frame with fewer
// than four Gaussians per tile, whose lists are so short that a quarter of the
// workgroups counts for more (0.4 a tile at full HD: 10.2 against 15.8 us; 1.5
// a tile at 1264 x 832: 9.8 / 10.9; 2.3 at full HD: 18.7 / 19.8).  With four a
// tile and footprints of the usual kinds, k_render / k_render_tiles take 26.0 /
// 21.6 us at full HD, 17.4 / 13.5 at 1264 x 832, 10.6 / 9.9 at 640 x 360.  The
// lists are known on the GPU only: frames of nothing but round splats of 1-3 px
// would break even at eight a tile (four: 15.1 / 18.7, six: 17.7 / 19.1).
//
// In k_render one wave64 owns one tile, lane l holds the four pixels l,
// l + 64, l + 128, l + 192 of the tile (rows l/16, l/16 + 4, ...).
// Every 64 list entries the lanes load one Gaussian each (mean, conic and
// opacity, colour) and store its nine per-Gaussian values in the wave's own
// LDS slots; the wave then walks them in order, all lanes reading the same
// slot (a broadcast read, on the LDS pipe rather than the vector ALU), and
// every lane blends its four pixels.  The wave leaves the list once all 256
// pixels have stopped, tested every fourth Gaussian.
#include "common.hpp"
#include "internal.hpp"

namespace ss {
namespace {

constexpr uint32_t kRenderWaves = 4;  // tiles per workgroup
constexpr float kMaxAlpha = 0.99f;
constexpr float kMinAlpha = 1.0f / 255.0f;
constexpr float kMinT = 1e-4f;
// opacity * exp(-q / 2) = 2^(log2(opacity) - q log2(e) / 2): the factor is
// folded into the conic and log2(opacity) into the dx term once per
// Gaussian, so a pixel evaluates 2^p, p = log2(o) + a' dx^2 + 2 b' dx dy + c' dy^2
constexpr float kHalfLog2e = 0.72134752044448170f;  // log2(e) / 2

// A tile's Gaussian batch in LDS: 64 slots of nine values.
struct RenderSlots {
  float4 geo[kWave];   // mean x, mean y, -log2(e)/2 * (conic a, conic b)
  float4 mix[kWave];   // -log2(e)/2 * conic c, log2(opacity), red, green
  float blue[kWave];
};

// Gaussians blended between two tests of the wave's live pixels.  A batch's
// slots past its last entry hold a Gaussian that changes no pixel (opacity 0:
// log2 = -inf, so 2^p = 0), so every batch walks whole groups; a stopped pixel
// is left unchanged by further Gaussians, so testing once a group only adds
// work, never changes the image.
constexpr uint32_t kGroup = 4;

// Blends the Gaussian of slot j into the lane's four pixels.  `counted`
// (uniform): slot j holds a list entry, not padding (for the statistics).
template <bool EXACT, bool STATS>
__device__ __forceinline__ void blend(const RenderSlots& sl, uint32_t j, bool counted, float sx, const float (&sy)[4],
                                      float (&T)[4], float (&cr)[4], float (&cg)[4], float (&cb)[4], uint32_t (&n)[4],
                                      uint32_t& evals) {
  const float4 g0 = sl.geo[j], g1 = sl.mix[j];
  const float Gx = g0.x, Gy = g0.y, A = g0.z, B = g0.w, C = g1.x, O = g1.y;
  const float R = g1.z, Gc = g1.w, Bl = sl.blue[j];
  // p = log2(o) - q log2(e) / 2 with q = A dx^2 + 2 B dx dy + C dy^2, as
  // (log2(o) + A' dx^2) + dy (2 B' dx + C' dy): the dx terms are shared by
  // the lane's four pixels (one column); q >= 0 is p <= log2(o)
  const float dx = Gx - sx;
  const float qa = fmaf(A * dx, dx, O);
  const float qb = 2.0f * B * dx;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const float dy = Gy - sy[k];
    const float q = fmaf(dy, fmaf(C, dy, qb), qa);  // = p
    const float e = __builtin_amdgcn_exp2f(q);
    if (EXACT) {
      const float w = e * T[k];
      cr[k] = fmaf(R, w, cr[k]);
      cg[k] = fmaf(Gc, w, cg[k]);
      cb[k] = fmaf(Bl, w, cb[k]);
      T[k] = fmaf(-e, T[k], T[k]);
      if (STATS) n[k] += counted ? 1u : 0u;
    } else {
      const float alpha = fminf(kMaxAlpha, e);
      if (STATS) evals += counted && T[k] > 0.0f ? 1u : 0u;
      // a stopped pixel needs no test here: its T is negative, so is next,
      // which reads as a stop again and leaves it unchanged
      const float ae = (q <= O && alpha >= kMinAlpha) ? alpha : 0.0f;
      const float next = fmaf(-ae, T[k], T[k]);
      const bool stop = next < kMinT;  // also true for a pixel already stopped
      const float w = stop ? 0.0f : ae * T[k];
      cr[k] = fmaf(R, w, cr[k]);
      cg[k] = fmaf(Gc, w, cg[k]);
      cb[k] = fmaf(Bl, w, cb[k]);
      T[k] = stop ? -fabsf(T[k]) : next;
      if (STATS) n[k] += w != 0.0f ? 1u : 0u;
    }
  }
  if (EXACT && STATS) evals += counted ? 4u : 0u;
}

// EXACT: no thresholds.  STATS: also count the Gaussians composited per pixel
// and the evaluations per tile.  A pixel that has stopped keeps its T with the
// sign bit set (T > 0 means live), so the thresholds cost selects, not
// branches, and the lanes never diverge.  The plain exact kernel is held to 64
// VGPRs, eight waves per SIMD: a full-HD frame's 8,160 tile waves are then all
// resident at once, which beats both fewer resident waves and fewer registers
// spent on the next batch's loads.
template <bool EXACT, bool STATS>
__global__ __launch_bounds__(kRenderWaves * kWave) __attribute__((amdgpu_waves_per_eu(STATS ? 1 : 8, 8))) void k_render(RenderArgs a) {
  __shared__ RenderSlots slots[kRenderWaves];
  if (a.status && *a.status != SS_OK) return;
  const uint32_t lane = lane_id();
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  // uniform over the wave: the list bounds are scalar loads
  const uint32_t tile = blockIdx.x * kRenderWaves + wave;
  if (tile >= a.tiles_x * a.tiles_y) return;
  RenderSlots& sl = slots[wave];
  const uint32_t tx = tile % a.tiles_x, ty = tile / a.tiles_x;
  const uint32_t start = a.ranges[2 * tile], end = a.ranges[2 * tile + 1];

  // sample points of this lane's four pixels
  const float sx = static_cast<float>(tx * 16 + (lane & 15)) + 0.5f;
  float sy[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) sy[k] = static_cast<float>(ty * 16 + (lane >> 4) + 4 * k) + 0.5f;

  float T[4], cr[4], cg[4], cb[4];
  uint32_t n[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    T[k] = 1.0f;
    cr[k] = cg[k] = cb[k] = 0.0f;
    n[k] = 0;
  }
  uint32_t evals = 0;

  // The next batch's Gaussians are loaded while the wave walks the current
  // one, so the gathers' latency hides behind the blending.
  int2 m = make_int2(0, 0);
  float4 co = make_float4(0.0f, 0.0f, 0.0f, 0.0f), cl = co;
  if (start + lane < end) {
    const uint32_t gi = a.values[start + lane];
    m = *reinterpret_cast<const int2*>(a.gaussians + gi);
    co = reinterpret_cast<const float4*>(a.conic_opacity)[gi];
    cl = reinterpret_cast<const float4*>(a.rgb)[gi];
  }
  bool live = true;
  for (uint32_t b = start; b < end && live; b += kWave) {
    // one Gaussian per lane into the wave's slots; padding past the end
    const bool valid = b + lane < end;
    sl.geo[lane] = make_float4(valid ? static_cast<float>(m.x) * (1.0f / 16.0f) : 0.0f,
                               valid ? static_cast<float>(m.y) * (1.0f / 16.0f) : 0.0f,
                               valid ? -kHalfLog2e * co.x : 0.0f, valid ? -kHalfLog2e * co.y : 0.0f);
    // log2(opacity); opacity in (0, 1]
    sl.mix[lane] = make_float4(valid ? -kHalfLog2e * co.z : 0.0f,
                               valid ? __builtin_amdgcn_logf(co.w) : -__builtin_inff(), valid ? cl.x : 0.0f,
                               valid ? cl.y : 0.0f);
    sl.blue[lane] = valid ? cl.z : 0.0f;
    const uint32_t nb = b + kWave;
    if (nb + lane < end) {
      const uint32_t gi = a.values[nb + lane];
      m = *reinterpret_cast<const int2*>(a.gaussians + gi);
      co = reinterpret_cast<const float4*>(a.conic_opacity)[gi];
      cl = reinterpret_cast<const float4*>(a.rgb)[gi];
    }
    // the slots are this wave's alone and its LDS accesses complete in
    // order, so the reads below see the stores above without a barrier
    __builtin_amdgcn_wave_barrier();
    const uint32_t count = end - b < kWave ? end - b : kWave;
    for (uint32_t j = 0; j < count; j += kGroup) {
#pragma unroll
      for (uint32_t u = 0; u < kGroup; ++u)
        blend<EXACT, STATS>(sl, j + u, j + u < count, sx, sy, T, cr, cg, cb, n, evals);
      if (!EXACT) {
        live = ballot(fmaxf(fmaxf(T[0], T[1]), fmaxf(T[2], T[3])) > 0.0f) != 0;
        if (!live) break;
      }
    }
    // the next batch's stores follow this batch's reads
    __builtin_amdgcn_wave_barrier();
  }

  const uint32_t W = a.width, H = a.height;
  const size_t plane = static_cast<size_t>(W) * H;
  const uint32_t px = tx * 16 + (lane & 15);
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const uint32_t py = ty * 16 + (lane >> 4) + 4 * k;
    const float t = fabsf(T[k]);
    if (px < W && py < H) {
      const size_t o = static_cast<size_t>(py) * W + px;
      a.color[o] = cr[k] + t * a.bg[0];
      a.color[plane + o] = cg[k] + t * a.bg[1];
      a.color[2 * plane + o] = cb[k] + t * a.bg[2];
      if (a.T) a.T[o] = t;
      if (STATS && a.contrib) a.contrib[o] = n[k];
    }
  }
  if (STATS && a.tile_evals) {
    // sum over the wave of the per-lane evaluation counts
    uint32_t e = evals;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) e += __shfl_xor(e, d, kWave);
    if (lane == 0) a.tile_evals[tile] = e;
  }
}

// The image alone, with thresholds: one workgroup of four waves per tile, a
// wave per 8 x 8 block of it, a pixel per lane.
//
// A tile list holds every Gaussian whose bounding square meets the tile, but
// most reach 1/255 only in a small part of it, and an entry that stays below
// 1/255 at all 64 pixels of a block changes none of them.  Each thread loads
// one entry of a batch of 256 and bounds its exponent over the four blocks;
// the waves' ballots of the blocks that it may reach go to LDS beside the
// entry's values, and a wave then walks the set bits of its own block's mask
// only, in list order, with the arithmetic of k_render's blend().  On the
// full-HD frame of 10^6 Gaussians that leaves a third of the evaluations;
// k_render took 490 us for it (instruction issue: 71 vector instructions per
// entry and tile), this kernel takes 189: 5.2M steps of one entry and one
// block, 24 vector instructions and three LDS reads each, which keep the
// vector units about 90 % and the LDS about 75 % busy.  (Tried and slower:
// branches around the pixels an entry leaves unchanged, 348 us; one step per
// test of the live pixels, 234.)
//
// The bound.  With Q(d) = a dx^2 + 2 b dx dy + c dy^2 an entry's exponent is
// p = log2(opacity) - k Q, k = log2(e) / 2, and 2^p >= 1/255 needs
// p > -7.995.  Over a block's rectangle of offsets d the minimum of a positive
// definite Q is 0 or lies on an edge that faces the origin: at the edge's
// offset in one axis, the other axis free in the rectangle.  FP32 rounding:
// Q's terms sum to at most R = (1 + r) / (1 - r) times Q itself, r = |b| /
// sqrt(a c); for r^2 <= 0.9996, R < 10^4, and the few roundings of either
// evaluation move Q by less than 10^4 * 10 * 2^-24 < 1 % of itself.  So an
// entry is left out of a block only where 0.98 k Q > log2(opacity) + 8.
// Anything else (other conics, NaN) stays in, and so does a colour that is
// not finite, whose product with a zero weight is NaN.
constexpr uint32_t kTileThreads = 256;
constexpr float kReach = 8.0f;
// Sixteen consecutive tiles per XCD (log2): neighbours share most of their
// Gaussians, which then come from one L2 (197.5 -> 188.5 us; no workgroup
// waits on another here).
constexpr uint32_t kTileRun = 4;

// A tile of opaque splats ends after some ten entries of a list that may hold
// thousands, so nothing is loaded beyond the first batch until it is known that
// the tile goes on, and in a list of many batches, where one more costs little,
// the first is half of one (full HD, 100k splats of 60-120 px, all opaque: 77 ->
// 63 us, 66 with whole first batches, k_render 62; 50k, 75 -> 66, k_render 63;
// with opacities from 0.05 to 0.99: 99 -> 91; the frame of 10^6 Gaussians 189 ->
// 187, where half batches first everywhere took 191).
constexpr uint32_t kLongList = 6 * kTileThreads;

struct TileSlots {
  float4 geo[kTileThreads];   // mean x, mean y, -k a, -2 k b
  float4 mix[kTileThreads];   // -k c, log2(opacity), red, green
  float blue[kTileThreads];
  uint64_t mask[4][kTileThreads / kWave];   // [block][64 entries]
};

// Whether 0.98 k min Q over the block [x0, x0 + 7] x [y0, y0 + 7] of sample
// points may stay within `limit` (offsets gx - x, gy - y).
__device__ __forceinline__ bool reaches(float gx, float gy, float a, float b, float c, float nba, float nbc, float x0,
                                        float y0, float limit) {
  const float xh = gx - x0, xl = xh - 7.0f, yh = gy - y0, yl = yh - 7.0f;
  const float ex = fmaxf(xl, fminf(xh, 0.0f)), ey = fmaxf(yl, fminf(yh, 0.0f));
  const float fy = fmaxf(yl, fminf(yh, nbc * ex)), fx = fmaxf(xl, fminf(xh, nba * ey));
  const float q1 = fmaf(a * ex, ex, fy * fmaf(c, fy, 2.0f * b * ex));
  const float q2 = fmaf(c * ey, ey, fx * fmaf(a, fx, 2.0f * b * ey));
  return !(fminf(q1, q2) > limit);
}

__global__ __launch_bounds__(kTileThreads) void k_render_tiles(RenderArgs a) {
  __shared__ TileSlots sl;
  if (a.status && *a.status != SS_OK) return;
  const uint32_t tid = threadIdx.x;
  const uint32_t lane = lane_id();
  const uint32_t wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const uint32_t tile = xcd_order<kTileRun>(blockIdx.x);
  if (tile >= a.tiles_x * a.tiles_y) return;
  const uint32_t tx = tile % a.tiles_x, ty = tile / a.tiles_x;
  const uint32_t start = a.ranges[2 * tile], end = a.ranges[2 * tile + 1];
  const uint32_t px = tx * 16 + (wave & 1) * 8 + (lane & 7), py = ty * 16 + (wave >> 1) * 8 + (lane >> 3);
  const float sx = static_cast<float>(px) + 0.5f, sy = static_cast<float>(py) + 0.5f;
  const bool inside = px < a.width && py < a.height;
  const float bx = static_cast<float>(tx * 16) + 0.5f, by = static_cast<float>(ty * 16) + 0.5f;

  // a stopped pixel, and one outside the image, has T's sign bit set
  float T = inside ? 1.0f : -1.0f, cr = 0.0f, cg = 0.0f, cb = 0.0f;
  int2 m = make_int2(0, 0);
  float4 co = make_float4(0.0f, 0.0f, 0.0f, 0.0f), cl = co;
  const auto load = [&](uint32_t i) {
    const uint32_t gi = a.values[i];
    m = *reinterpret_cast<const int2*>(a.gaussians + gi);
    co = reinterpret_cast<const float4*>(a.conic_opacity)[gi];
    cl = reinterpret_cast<const float4*>(a.rgb)[gi];
  };
  const uint32_t first = end - start > kLongList ? kTileThreads / 2 : kTileThreads;
  if (tid < first && start + tid < end) load(start + tid);
  bool live = ballot(T > 0.0f) != 0;
  for (uint32_t b = start, count = first; b < end; b += count, count = kTileThreads) {
    // ---- this thread's entry: its values, and the blocks it may reach ----
    {
      const bool valid = tid < count && b + tid < end;
      const float gx = static_cast<float>(m.x) * (1.0f / 16.0f), gy = static_cast<float>(m.y) * (1.0f / 16.0f);
      const float O = __builtin_amdgcn_logf(co.w);
      sl.geo[tid] = make_float4(gx, gy, -kHalfLog2e * co.x, 2.0f * (-kHalfLog2e * co.y));
      sl.mix[tid] = make_float4(-kHalfLog2e * co.z, O, cl.x, cl.y);
      sl.blue[tid] = cl.z;
      const bool bounded = co.x > 0.0f && co.z > 0.0f && co.y * co.y <= 0.9996f * (co.x * co.z) &&
                           fabsf(cl.x) < __builtin_inff() && fabsf(cl.y) < __builtin_inff() &&
                           fabsf(cl.z) < __builtin_inff();
      const float limit = (O + kReach) * (1.0f / (0.98f * kHalfLog2e));
      const float nba = -co.y * __builtin_amdgcn_rcpf(co.x), nbc = -co.y * __builtin_amdgcn_rcpf(co.z);
#pragma unroll
      for (uint32_t k = 0; k < 4; ++k) {
        const bool hit = valid && (!bounded || reaches(gx, gy, co.x, co.y, co.z, nba, nbc, bx + 8.0f * (k & 1),
                                                       by + 8.0f * (k >> 1), limit));
        const uint64_t h = ballot(hit);
        if (lane == 0) sl.mask[k][wave] = h;
      }
    }
    // from the second batch on, the next one's entries are loaded while this
    // one is walked
    const uint32_t next = b + count + tid;
    if (b != start && next < end) load(next);
    __syncthreads();
    // ---- the entries that may reach this wave's block, in list order ----
    for (uint32_t g = 0; g < kTileThreads / kWave && live; ++g) {
      const uint64_t h = sl.mask[wave][g];
      uint64_t bits = (static_cast<uint64_t>(static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<uint32_t>(h >> 32)))) << 32) |
                      static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<uint32_t>(h)));
      while (bits != 0 && live) {
#pragma unroll
        for (uint32_t u = 0; u < kGroup; ++u) {
          if (bits == 0) break;
          const uint32_t j = g * kWave + static_cast<uint32_t>(__builtin_ctzll(bits));
          bits &= bits - 1;
          const float4 g0 = sl.geo[j], g1 = sl.mix[j];
          const float R = g1.z, Gc = g1.w, Bl = sl.blue[j], O = g1.y;
          // blend(), for one pixel
          const float dx = g0.x - sx, dy = g0.y - sy;
          const float qa = fmaf(g0.z * dx, dx, O), qb = g0.w * dx;
          const float q = fmaf(dy, fmaf(g1.x, dy, qb), qa);
          const float alpha = fminf(kMaxAlpha, __builtin_amdgcn_exp2f(q));
          const float ae = (q <= O && alpha >= kMinAlpha) ? alpha : 0.0f;
          const float next = fmaf(-ae, T, T);
          const bool stop = next < kMinT;
          const float w = stop ? 0.0f : ae * T;
          cr = fmaf(R, w, cr);
          cg = fmaf(Gc, w, cg);
          cb = fmaf(Bl, w, cb);
          T = stop ? -fabsf(T) : next;
        }
        live = ballot(T > 0.0f) != 0;
      }
    }
    if (end - b <= count) break;   // the last batch
    // every wave is done with the slots; the tile ends when all its pixels have
    if (!__syncthreads_or(live)) break;
    if (b == start && next < end) load(next);
  }
  if (inside) {
    const size_t plane = static_cast<size_t>(a.width) * a.height;
    const size_t o = static_cast<size_t>(py) * a.width + px;
    const float t = fabsf(T);
    a.color[o] = cr + t * a.bg[0];
    a.color[plane + o] = cg + t * a.bg[1];
    a.color[2 * plane + o] = cb + t * a.bg[2];
    if (a.T) a.T[o] = t;
  }
}

}  // namespace

hipError_t launch_render(const RenderArgs& a, bool exact, hipStream_t s) {
  const uint32_t tiles = a.tiles_x * a.tiles_y;
  const uint32_t blocks = (tiles + kRenderWaves - 1) / kRenderWaves;
  if (blocks == 0) return hipSuccess;
  const dim3 g(blocks), t(kRenderWaves * kWave);
  const bool stats = a.contrib != nullptr || a.tile_evals != nullptr;
  if (exact && stats) hipLaunchKernelGGL((k_render<true, true>), g, t, 0, s, a);
  else if (exact) hipLaunchKernelGGL((k_render<true, false>), g, t, 0, s, a);
  else if (stats) hipLaunchKernelGGL((k_render<false, true>), g, t, 0, s, a);
  else if (a.n < 4ull * tiles) hipLaunchKernelGGL((k_render<false, false>), g, t, 0, s, a);
  else hipLaunchKernelGGL(k_render_tiles, dim3(xcd_grid<kTileRun>(tiles)), dim3(kTileThreads), 0, s, a);
  return hipGetLastError();
}

}  // namespace ss
