// Front-to-back alpha compositing (forward) and its back-to-front
// recomputation (backward) on gfx950.  A 16x16 tile is four 8x8-pixel bands
// (quadrants); forward and backward run one band per 64-thread block (one
// wave), with no barriers between waves.
//
// Splat records of a tile's list are staged through the wave's LDS; every
// lane reads the same record (LDS broadcast), and each band walks only the
// entries that can reach it.  The forward stops a band once every pixel of it
// has terminated; the backward walks the entries that the forward composited.
#include "common.h"
#include "kernels.h"

#include <cstdlib>

namespace ls {

typedef float v4f __attribute__((ext_vector_type(4)));

struct TileCtx {
  int r;         // render
  int tile;      // global tile index
  int x, y;      // pixel of this thread
  int x0, y0;    // the tile's first pixel
  bool inside;
  int64_t pix;   // pixel index in the image arrays (if inside)
  int W, H;
};

__device__ __forceinline__ TileCtx tile_ctx(const JobDev* jobs, const int32_t* tile_off, int R, int tile) {
  TileCtx c;
  c.tile = tile;
  c.r = find_segment<int32_t>(tile_off, R, tile);
  const JobDev& J = jobs[c.r];
  const int lt = tile - J.tile_off;
  const int ty = lt / J.TX, tx = lt - ty * J.TX;
  // wave w of the block covers the 8x8 quadrant (w & 1, w >> 1); lane l its
  // pixel (l & 7, l >> 3)
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  c.x0 = tx * kTile;
  c.y0 = ty * kTile;
  c.x = c.x0 + 8 * (w & 1) + (l & 7);
  c.y = c.y0 + 8 * (w >> 1) + (l >> 3);
  c.W = J.W;
  c.H = J.H;
  c.inside = c.x < J.W && c.y < J.H;
  c.pix = J.pix_off + (int64_t)c.y * J.W + c.x;
  return c;
}

// The y-extent of the support ellipse over the column strip x0 <= x <= x1:
// from its lowest to its highest point when those lie inside the strip, else
// to the ends of the chord on the nearer strip edge (the ellipse's y-range
// over a vertical line x = xb is the root interval of a quadratic in y).
// False when the ellipse does not reach the strip.
__device__ __forceinline__ bool strip_extent(float u, float v, float A, float B, float C, float dq, float smax,
                                             float hx, float hy, float x0, float x1, float& ylo, float& yhi) {
  if (u + hx < x0 || u - hx > x1) return false;
  const float sx = B / A * hy;  // the highest point sits at x = u - sx, the lowest at u + sx
  const float top_x = u - sx, bot_x = u + sx;
  yhi = v + hy;
  ylo = v - hy;
  if (top_x < x0 || top_x > x1) {
    const float dx = (top_x < x0 ? x0 : x1) - u;
    const float D = 2.f * C * smax - dq * dx * dx;
    if (!(D >= 0.f)) return false;
    yhi = v + (-B * dx + sqrtf(D)) / C;
  }
  if (bot_x < x0 || bot_x > x1) {
    const float dx = (bot_x < x0 ? x0 : x1) - u;
    const float D = 2.f * C * smax - dq * dx * dx;
    if (!(D >= 0.f)) return false;
    ylo = v + (-B * dx - sqrtf(D)) / C;
  }
  yhi += fabsf(yhi - v) * 1e-3f + 0.02f;
  ylo -= fabsf(v - ylo) * 1e-3f + 0.02f;
  return true;
}

// Which of the tile's four 8x8-pixel wave quadrants (bit 2 qy + qx for the
// quadrant at column qx, row qy) the Gaussian can reach with alpha >= 1/255.
// The support {o exp(-sigma) >= 1/255} is the ellipse sigma <= s = ln(255 o);
// its x half-extent is sqrt(2 s Sigma_xx) (Sigma = conic^-1).  Over each of
// the two 8-pixel column strips the ellipse's y-extent (strip_extent) is
// tested against the two 8-pixel row ranges.  s is widened by 0.1% + 1e-4
// and every extent by 0.1% + 0.02 px, so FP32 rounding never drops a
// contributor.  (Against 16x4 row bands, 8x8 quadrants are reached by 7 %
// fewer (Gaussian, band) pairs on the 200k-Gaussian render loop.)
__device__ __forceinline__ uint32_t wave_mask(float4 a, float4 b, int tile_x0, int tile_y0) {
  const float o = b.y;
  if (!(o >= LS_ALPHA_MIN)) return 0u;
  const float A = a.z, B = a.w, C = b.x;
  const float dq = A * C - B * B;
  if (!(dq > 0.f)) return 0xFu;
  const float smax = __logf(o * (1.0f / LS_ALPHA_MIN)) * 1.001f + 1e-4f;
  const float hx = sqrtf(fmaxf(2.f * smax * C / dq, 0.f)) * 1.001f + 0.02f;
  const float hy = sqrtf(fmaxf(2.f * smax * A / dq, 0.f)) * 1.001f + 0.02f;
  const float xa = (float)tile_x0 + 0.5f, ya = (float)tile_y0 + 0.5f;
  uint32_t m = 0;
#pragma unroll
  for (int qx = 0; qx < 2; ++qx) {
    float ylo, yhi;
    if (!strip_extent(a.x, a.y, A, B, C, dq, smax, hx, hy, xa + 8.f * qx, xa + 8.f * qx + 7.f, ylo, yhi)) continue;
#pragma unroll
    for (int qy = 0; qy < 2; ++qy) {
      const float y0 = ya + 8.f * qy, y1 = y0 + 7.f;
      if (!(yhi < y0 || ylo > y1)) m |= 1u << (2 * qy + qx);
    }
  }
  return m;
}

// The rows of one 8x8 band (pixel centres from (bx0, by0), 1 px apart) that
// the Gaussian's alpha >= 1/255 support can reach, as a mask of whole rows
// (bit 8 r + c for every column c of a reached row r): the support's y-extent
// over the band's column strip (strip_extent, widened as in wave_mask) holds
// every pixel centre the support contains, so a row whose centre lies outside
// it holds no pixel that composites the entry.
// Reciprocals and roots are the instructions' own (1 ulp): the margins of
// 0.1 % cover them, and one such test per entry and band was a fifth of the
// forward's instructions with correctly rounded ones.
__device__ __forceinline__ uint64_t band_rows(float4 a, float4 b, float bx0, float by0) {
  const float o = b.y;
  if (!(o >= LS_ALPHA_MIN)) return 0ull;
  const float A = a.z, B = a.w, C = b.x;
  const float dq = A * C - B * B;
  if (!(dq > 1e-30f)) return ~0ull;  // (below it the reciprocal may overflow)
  const float t2 = 2.002f * __logf(o * (1.0f / LS_ALPHA_MIN)) + 2e-4f;  // 2 s, widened
  const float idq = t2 * __builtin_amdgcn_rcpf(dq), rc = __builtin_amdgcn_rcpf(C);
  const float hx = __builtin_amdgcn_sqrtf(fmaxf(C * idq, 0.f)) * 1.001f + 0.02f;
  const float hy = __builtin_amdgcn_sqrtf(fmaxf(A * idq, 0.f)) * 1.001f + 0.02f;
  const float x0 = bx0 - a.x, x1 = x0 + 7.f;  // the band's columns, from the centre
  const float sx = B * __builtin_amdgcn_rcpf(A) * hy;  // the highest point sits at -sx, the lowest at sx
  const float top = fminf(fmaxf(-sx, x0), x1), bot = fminf(fmaxf(sx, x0), x1);
  const float tc = t2 * C;
  const float dt = tc - dq * top * top, db = tc - dq * bot * bot;
  const float eh = top == -sx ? hy : (__builtin_amdgcn_sqrtf(dt) - B * top) * rc;
  const float el = bot == sx ? hy : (__builtin_amdgcn_sqrtf(db) + B * bot) * rc;
  // (a negative D makes the extent a NaN; hx decides with the same margin)
  if (!(x0 <= hx && x1 >= -hx) || !(eh == eh) || !(el == el)) return 0ull;
  const float yhi = a.y + eh + (fabsf(eh) * 1e-3f + 0.02f), ylo = a.y - el - (fabsf(el) * 1e-3f + 0.02f);
  const int r0 = (int)fmaxf(ceilf(ylo - by0), 0.f), r1 = (int)fminf(floorf(yhi - by0), 7.f);
  if (r0 > r1) return 0ull;
  return (~0ull >> (8 * (7 - r1))) & (~0ull << (8 * r0));
}

// Forward, one wave per 8x8-pixel band of a tile (a 64-thread block): no
// block barriers, and a band stops reading its tile's list as soon as all of
// its pixels have terminated.  The wave walks the list 64 entries at a time:
// each lane loads one record and tests it against the band (wave_mask, the
// test the backward uses), and the entries that can reach the band are
// compacted, in list order, into the wave's LDS.  (Measured against a
// 256-thread block per tile that staged each record once for all four bands:
// 1 % faster on the render loop and on a registration pair.)
//
// Bound by vector instruction issue (at 200k items, 1200 x 680: 43 M of them
// filled 84 % of 90 us).  A step therefore masks once, the alpha, so that one
// select covers weight and transmittance; a pixel that has stopped goes on
// with T = 0; and the four sums take one 4x4x1 matrix instruction (lane l
// supplies channel l & 3 of the entry's colour and depth, every lane its
// weight), which gives the FMA chain's bits in the time of two of its four
// FMAs and reads 4 instead of 16 bytes of LDS per lane.  With the band test
// on reciprocal and square root instructions: 34 M, 83 us; 16 renders of 150k
// and 120k items at 640 x 480 231 -> 217 us, 8 of 150k 141 -> 131 us.  Taking
// the XCDs' shares in turns (xcd_turns) made that 77, 165 and 104 us, and a
// step without branches but for stops and unused entries, which leaves T in two
// registers by turns and LDS offsets in vector registers, 74, 159 and 100 us.
// At 200k items the last waves, on half-empty SIMDs, are a fifth of the time.
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(8))) void k_composite_fwd_band(
    const JobDev* __restrict__ jobs, const int32_t* __restrict__ tile_off, int R, int T_total,
    const float4* __restrict__ rec, const int32_t* __restrict__ items, const int32_t* __restrict__ range, float bg0,
    float bg1, float bg2, float* __restrict__ out_rgb, float* __restrict__ out_depth, float* __restrict__ out_alpha,
    float* __restrict__ out_T, int32_t* __restrict__ out_n, uint64_t* __restrict__ used, int64_t ustride,
    int cover) {
  // one entry of padding: the walk takes two entries at a time and reads one ahead
  __shared__ float4 s0[65], s1[65], s2[65];
  __shared__ int32_t spos[64];
  const int unit = xcd_turns<64>(blockIdx.x, 4 * T_total);
  if (unit >= 4 * T_total) return;
  const int tile = unit >> 2, band = unit & 3;
  const int lane = threadIdx.x;
  const int r = find_segment<int32_t>(tile_off, R, tile);
  const JobDev& J = jobs[r];
  const int local = tile - J.tile_off;  // tile index within its render
  const int tile_y = local / J.TX, tile_x = local - tile_y * J.TX;
  const int tx0 = tile_x * kTile, ty0 = tile_y * kTile;
  const int x = tx0 + 8 * (band & 1) + (lane & 7), y = ty0 + 8 * (band >> 1) + (lane >> 3);
  const bool inside = x < J.W && y < J.H;
  const int start = range[2 * tile], end = range[2 * tile + 1];
  const float fx = (float)x + 0.5f, fy = (float)y + 0.5f;
  const float bx0 = (float)(tx0 + 8 * (band & 1)) + 0.5f, by0 = (float)(ty0 + 8 * (band >> 1)) + 0.5f;
  const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));

  float T = inside ? 1.f : 0.f, Tend = 1.f;  // transmittance while compositing (0 once stopped), and at the stop
  v4f acc = {0.f, 0.f, 0.f, 0.f};              // rgb and depth
  int nlast = end - start;
  uint64_t alive = __ballot(inside);  // lane l is pixel (l & 7, l >> 3) of the band: bit l of band_rows
  // chunk k of the tile's list keeps its "used" bits in slot (start / 64) +
  // tile + k of the band's row: the slots of successive tiles never overlap
  int64_t slot = (int64_t)(start >> 6) + tile;
  for (int chunk = start; chunk < end && alive != 0ull; chunk += 64, ++slot) {
    const int e = chunk + lane;
    uint64_t usedm = 0ull;  // bit j: some pixel of the band composited its j-th staged entry
    bool in = false;
    float4 r0 = make_float4(0.f, 0.f, 0.f, 0.f), r1 = r0, r2 = r0;  // this lane's record
    if (e < end) {
      const int64_t it = items[e];
      r0 = rec[it * 3 + 0];
      r1 = rec[it * 3 + 1];
      if (cover)  // some row the entry can reach holds a pixel still compositing
        in = (band_rows(r0, r1, bx0, by0) & alive) != 0ull;
      else
        in = (wave_mask(r0, r1, tx0, ty0) >> band) & 1u;
      if (in) {
        r2 = rec[it * 3 + 2];
        r2.w = r1.z;
        stage_conic(r0, r1);
      }
    }
    const uint64_t bal = __ballot(in);
    const int pos = __popcll(bal & lt);
    if (in) {
      s0[pos] = r0;
      s1[pos] = r1;
      s2[pos] = r2;
      spos[pos] = e - start;
    }
    wave_sync();
    int cw = __popcll(bal);
    if (lane == 0) {  // the walk takes two entries at a time: a last one that composites nowhere
      s0[cw] = make_float4(0.f, 0.f, 0.f, 0.f);
      s1[cw] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    wave_sync();
    // one step at staged entry j, transmittance Ti before and To after it:
    // no branch but for pixels that stop and entries that no pixel takes (whose
    // colour, should it be infinite, must not meet the weight 0)
    auto step = [&](int j, const float4& a, const float3& b, float col, float Ti, float& To) {
      const float dx = fx - a.x, dy = fy - a.y;
      const float sl = falloff_log2(a.z, a.w, b.x, dx, dy);
      const bool c = composited(sl, b.z);
      // a pixel that does not composite the entry takes alpha 0: weight 0, T as it was
      const float al = c ? fminf(LS_ALPHA_MAX, b.y * __builtin_amdgcn_exp2f(-sl)) : 0.f;
      // the weight alpha T, and T (1 - alpha) as T - alpha T in one FMA
      float w = al * Ti;
      To = __builtin_fmaf(-al, Ti, Ti);
      uint64_t use = alive & __ballot(c);
      const uint64_t stop = alive & __ballot(To < LS_T_STOP);  // (a pixel above it stays there with alpha 0)
      if (stop != 0ull) {
        if (__builtin_amdgcn_inverse_ballot_w64(stop)) {
          nlast = spos[j];
          Tend = Ti;
          w = 0.f;
          To = 0.f;
        }
        use &= ~stop;
        alive &= ~stop;
        cw = alive == 0ull ? 0 : cw;  // every pixel has stopped: the walk ends
      }
      if (use != 0ull) {
        acc = __builtin_amdgcn_mfma_f32_4x4x1f32(col, w, acc, 0, 0, 0);
        // usedm |= 1 << j in one scalar instruction (a register-only bit set)
        asm volatile("s_bitset1_b64 %0, %1" : "+s"(usedm) : "s"(j));
      }
    };
    // Records are read one entry ahead into two alternating register sets
    // (the loop unrolled by hand, so no copies), so the LDS latency of the
    // next entry overlaps the arithmetic of this one; the read past the last
    // staged entry (at most entry 64) is never used.  The offsets advance in
    // vector registers (the empty asm), as the reads want them.
    uint32_t at = 0u, atc = 4u * (lane & 3);
    asm volatile("" : "+v"(at), "+v"(atc));
    auto read = [&](int k, float4& a, float3& b, float& c) {
      a = *reinterpret_cast<const float4*>(reinterpret_cast<const char*>(s0 + k) + at);
      b = *reinterpret_cast<const float3*>(reinterpret_cast<const char*>(s1 + k) + at);
      c = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(s2 + k) + atc);
    };
    float4 aA, aB;
    float3 bA, bB;
    float cA, cB, T2;
    read(0, aA, bA, cA);
    for (int jj = 0; jj < cw; jj += 2) {
      read(1, aB, bB, cB);
      step(jj, aA, bA, cA, T, T2);
      read(2, aA, bA, cA);
      at += 32u;
      atc += 32u;
      step(jj + 1, aB, bB, cB, T2, T);
    }
    // the entries of this chunk that some pixel of the band composited
    // (bit l: entry chunk + l): exactly the (entry, band) pairs in which the
    // backward has an active lane
    const uint64_t um = __ballot(in && ((usedm >> pos) & 1ull));
    if (lane == 0) used[band * ustride + slot] = um;
    wave_sync();
  }
  if (!inside) return;
  const int64_t hw = (int64_t)J.W * J.H;
  const int64_t pix = J.pix_off + (int64_t)y * J.W + x;
  float* rgb = out_rgb + 3 * J.pix_off + (int64_t)y * J.W + x;
  const float Tf = __builtin_amdgcn_inverse_ballot_w64(alive) ? T : Tend;
  rgb[0] = acc[0] + Tf * bg0;
  rgb[hw] = acc[1] + Tf * bg1;
  rgb[2 * hw] = acc[2] + Tf * bg2;
  out_depth[pix] = acc[3];
  out_alpha[pix] = 1.f - Tf;
  out_T[pix] = Tf;
  out_n[pix] = nlast;
}

// Lane exchanges of gfx950 that trade halves of two registers:
// permlane32_swap gives x the lower 32 lanes of y in place of its upper 32,
// permlane16_swap gives x the even 16-lane rows of y in place of its odd rows
// (and y what x gave up).  Adding the two results sums each value over lane
// pairs 32 (or 16) apart while packing two values into one register.
__device__ __forceinline__ float swap32_sum(float x, float y) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float swap16_sum(float x, float y) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Swap-add of two registers between the two halves of each group of 2m
// lanes (m = 8: row_ror:8 pairs lane i with i +- 8 of its row; m = 4:
// row_half_mirror pairs lane i with 7 - i of its 8-lane half): lanes of the
// lower m keep a's value summed with a's partner, lanes of the upper m keep
// b's.  With a == b this is a plain add of the partner (one instruction).
template <int kCtrl, int kM>
__device__ __forceinline__ float pair_sum(float a, float b, int lane) {
  const bool lo = (lane & kM) == 0;
  const float s = lo ? a : b, t = lo ? b : a;
  return s + __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(t), kCtrl, 0xF, 0xF, true));
}

// Sums of 12 values over the 64 lanes of the wave, by a transposing reduction that
// halves the lanes holding each value at every level while packing more values per
// register:
//  - 32-lane swaps and adds: value 2k in the lower half of register h[k],
//    2k + 1 in the upper half;
//  - 16-lane swaps and adds: four values per register q[i], one per row
//    (value 4 i + slot(r) in row r, slot = 0, 2, 1, 3);
//  - within rows, swap-adds 8 lanes apart (q[0] with q[1], q[2] with itself), then
//    4 apart, leave one value per 4-lane group of one register, and two DPP adds
//    sum each group.
// The result: the lane that wave_value() names holds the total of that value; the
// duplicates of q[2] are not named.  It costs 6 + 3 swaps and 18 VALU adds or
// selects; a plain row sum after the 16-lane level would take 21 adds.  The whole
// wave must be active.
__device__ __forceinline__ float wave_sums(const float (&g)[12], int lane) {
  float h[6], q[3];
#pragma unroll
  for (int k = 0; k < 6; ++k) h[k] = swap32_sum(g[2 * k], g[2 * k + 1]);
#pragma unroll
  for (int i = 0; i < 3; ++i) q[i] = swap16_sum(h[2 * i], h[2 * i + 1]);
  constexpr int kRor8 = 0x128, kHalfMirror = 0x141, kQuad1032 = 0xB1, kQuad2301 = 0x4E;
  const float z0 = pair_sum<kRor8, 8>(q[0], q[1], lane), z1 = pair_sum<kRor8, 8>(q[2], q[2], lane);
  float y = pair_sum<kHalfMirror, 4>(z0, z1, lane);
  y += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(y), kQuad1032, 0xF, 0xF, true));
  y += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(y), kQuad2301, 0xF, 0xF, true));
  // Keep the last add in every lane: callers store the sum from a few lanes,
  // and sinking the add into that branch splits the fused DPP add into a DPP
  // move plus an add (an empty asm that reads and writes y, no code).
  asm volatile("" : "+v"(y));
  return y;
}

// The value whose total lane `lane` holds after wave_sums, or -1 for the lanes that
// hold a duplicate or one of the same group (exactly one lane per value is named).
__device__ __forceinline__ int wave_value(int lane) {
  const int r = lane >> 4, grp = (lane >> 2) & 3;
  // 8 apart: lanes 0-7 of a row keep q[0], 8-15 q[1], and both q[2]; 4 apart:
  // groups 0 and 2 keep the first register's, 1 and 3 the second's
  if ((lane & 3) || grp == 3) return -1;
  const int qi = grp == 1 ? 2 : grp >> 1;
  return 4 * qi + (((r & 1) << 1) | (r >> 1));
}

// Backward.  Per pixel, walking the list from n_last - 1 down to 0 with the
// transmittance recovered as T_i = T_{i+1} / (1 - alpha_i) and the running
// "behind" value acc = sum_{j>i} alpha_j prod_{i<k<j}(1 - alpha_k) v_j +
// prod_{k>i}(1 - alpha_k)(bg . gC - gA), where v_j = c_j . gC + z_j gD:
//   dL/dalpha_i = T_i (v_i - acc_i).
// One such step at a pixel (a, b staged, b.w the list position), branch-free:
// where the entry was composited (visited, sigma >= 0 and alpha >= 1/255), T
// is recovered, acc updated, and wgt = alpha T and ds = dL/dsigma = -alpha
// dL/dalpha are formed.  Elsewhere the step runs with alpha = 0, which leaves
// T (times 1 / 1) and acc (plus 0) unchanged and gives wgt = ds = 0.
// dL/d(opacity) = -ds / opacity (both carry the factor exp(-sigma)), so it
// needs no sum of its own.  No gradient flows through an active 0.99 clamp
// (alpha = 0.99): those ds are cleared.
__device__ __forceinline__ float step_alpha(const float4& a, const float4& b, int nl, float fx, float fy) {
  const float dx = fx - a.x, dy = fy - a.y;
  const float sl = falloff_log2(a.z, a.w, b.x, dx, dy);
  const float G = b.y * __builtin_amdgcn_exp2f(-sl);
  // & and not &&: no branch
  return (__float_as_int(b.w) < nl) & composited(sl, b.z) ? fminf(LS_ALPHA_MAX, G) : 0.f;
}

// The band of a wave: unit = 4 tile + band, lane l its pixel (l & 7, l >> 3), or
// (l >> 3, l & 7) with kColumns.
struct BandCtx {
  int r, tile, band;
  int x, y;    // pixel of this lane
  int x0, y0;  // the band's first pixel
  bool inside;
  int64_t pix;  // pixel index in the image arrays (if inside)
};

template <bool kColumns>
__device__ __forceinline__ BandCtx band_ctx(const JobDev* jobs, const int32_t* tile_off, int R, int unit, int lane) {
  BandCtx c;
  c.tile = unit >> 2;
  c.band = unit & 3;
  c.r = find_segment<int32_t>(tile_off, R, c.tile);
  const JobDev& J = jobs[c.r];
  const int lt = c.tile - J.tile_off;
  const int ty = lt / J.TX, tx = lt - ty * J.TX;
  c.x0 = tx * kTile + 8 * (c.band & 1);
  c.y0 = ty * kTile + 8 * (c.band >> 1);
  c.x = c.x0 + (kColumns ? lane >> 3 : lane & 7);
  c.y = c.y0 + (kColumns ? lane & 7 : lane >> 3);
  c.inside = c.x < J.W && c.y < J.H;
  c.pix = J.pix_off + (int64_t)c.y * J.W + c.x;
  return c;
}

// Per-pixel state shared by both backward kernels: upstream gradients (scaled),
// final transmittance, entries visited, and the initial "behind" value.
struct BwdPixel {
  float T, gR, gG, gB, gD, acc;
  int nl;
  float lsum, lcnt;  // the pixel's L1 terms and 1 when it lies in Omega (L1 targets only), else 0
};

__device__ __forceinline__ float l1_sign(float d) { return d > 0.f ? 1.f : (d < 0.f ? -1.f : 0.f); }

__device__ __forceinline__ BwdPixel bwd_pixel(const BandCtx& c, const JobDev& J, float bg0, float bg1, float bg2,
                                              const float* fwd_T, const int32_t* fwd_n, const float* up_rgb,
                                              const float* up_depth, const float* up_alpha, const float* up_scale,
                                              const L1Targets& l1) {
  BwdPixel p{1.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0, 0.f, 0.f};
  if (c.inside) {
    const int64_t hw = (int64_t)J.W * J.H;
    const int64_t ci = 3 * J.pix_off + (int64_t)c.y * J.W + c.x;
    const float sc = up_scale ? up_scale[c.r] : 1.f;
    if (l1.pred_rgb) {
      // the loss gradient of this pixel, as the L1 loss kernel forms it
      const int64_t q = (int64_t)c.y * J.W + c.x;
      const float* trgb = l1.tgt_rgb ? l1.tgt_rgb + ci : J.tgt_rgb + q;
      const float td = l1.tgt_depth ? l1.tgt_depth[c.pix] : J.tgt_depth[q];
      const bool valid = td > 0.f;
      const float d0 = l1.pred_rgb[ci] - trgb[0], d1 = l1.pred_rgb[ci + hw] - trgb[hw];
      const float d2 = l1.pred_rgb[ci + 2 * hw] - trgb[2 * hw], dd = l1.pred_depth[c.pix] - td;
      p.gR = sc * (valid ? l1_sign(d0) : 0.f);
      p.gG = sc * (valid ? l1_sign(d1) : 0.f);
      p.gB = sc * (valid ? l1_sign(d2) : 0.f);
      p.gD = sc * (valid ? l1_sign(dd) : 0.f);
      if (valid) {  // summed as the loss kernel sums a pixel: depth, then the channels in order
        p.lsum = ((fabsf(dd) + fabsf(d0)) + fabsf(d1)) + fabsf(d2);
        p.lcnt = 1.f;
      }
    }
    if (up_rgb) { p.gR = sc * up_rgb[ci]; p.gG = sc * up_rgb[ci + hw]; p.gB = sc * up_rgb[ci + 2 * hw]; }
    if (up_depth) p.gD = sc * up_depth[c.pix];
    const float gA = up_alpha ? sc * up_alpha[c.pix] : 0.f;
    p.T = fwd_T[c.pix];
    p.nl = fwd_n[c.pix];
    p.acc = bg0 * p.gR + bg1 * p.gG + bg2 * p.gB - gA;
  }
  return p;
}

// What the gradients need of an entry is sums over the band's pixels of ds
// times 1, dx, dy, dx^2, dx dy, dy^2 and of wgt times the upstream gradients.
// They are taken eight entries at a time: the walk (lane = pixel) leaves ds
// and wgt of each entry in two rows of the wave's LDS, and then lane (e, y) =
// (lane >> 3, lane & 7) sums pixel row y of entry e on its own (moments about
// the band's centre, shifted to the splat's) before the eight rows of an entry
// are added across lanes.  So the products are formed once per lane for eight
// pixels and one cross-lane reduction serves eight entries.  An entry costs
// about 22 VALU instructions in the walk and 13 in the sums; with ten products a
// pixel and a reduction of as many values an entry it was 67.  VALU bound: 200k
// Gaussians at 1200x680, full, 218 -> 120 us (with the atomics below; 115 us
// since the XCDs take turns, see xcd_turns).  (The pose-only sums go by pixel
// columns, with every product rounded: see column_sums.)
// (FP32 matrix products that contract the same rows with the pixel factors
// cost more: twice the vector rate, but 10 of 32 result columns are of use,
// and they do not overlap with the SIMD's vector instructions.)
// The colour term v = c . (gR, gG, gB) + z gD of four entries at all 64
// pixels is four 4x4x1 matrix products, bit for bit the FMA chain.
constexpr int kBatch = 32;        // entries staged per round
constexpr int kRowStride = 68;    // floats per LDS row of 64 pixels: 16-byte aligned, rows 4 banks apart
constexpr int kRing = 128;        // positions waiting to be staged: < kBatch left over + 64 new
constexpr int kPoseRow = 6;       // pose only: sums of ds dx, ds dy, ds dx^2, ds dx dy, ds dy^2, wgt gD
using f32x4 = __attribute__((ext_vector_type(4))) float;

struct BandLds {
  float4 s0[kBatch], s1[kBatch], s2[kBatch];  // (u, v, hA, B), (hC, opacity, bound, list position), (r, g, b, z)
  float rows[16 * kRowStride];  // of eight entries: ds, then wgt
  int32_t ring[kRing];
};
struct FullBandLds : BandLds {
  int32_t item[kBatch];
};
constexpr int kPoseRound = 256;  // most list positions per round
struct PoseBandLds : BandLds {
  float late[kBatch];         // red of the entries that take green first (s2 holds 0 there)
  uint8_t place[kPoseRound];  // of the round's positions among the round's sums, or kNoPlace
};
constexpr uint8_t kNoPlace = 255;

// The upstream gradients of pixel row y = lane & 7 of the band, by way of the
// wave's LDS.
template <int kN>
__device__ __forceinline__ void row_factors(float* rows, int lane, const float (&g)[kN], float (&f)[kN][8]) {
#pragma unroll
  for (int q = 0; q < kN; ++q) rows[q * kRowStride + lane] = g[q];
  wave_sync();
#pragma unroll
  for (int q = 0; q < kN; ++q) {
    const float4* r = reinterpret_cast<const float4*>(rows + q * kRowStride + 8 * (lane & 7));
    const float4 a = r[0], b = r[1];
    f[q][0] = a.x; f[q][1] = a.y; f[q][2] = a.z; f[q][3] = a.w;
    f[q][4] = b.x; f[q][5] = b.y; f[q][6] = b.z; f[q][7] = b.w;
  }
  wave_sync();
}

// The band's entries in walk order (list positions descending): the forward's
// "used" bits (64 entries per word, word 0 the list's first 64; every word
// below the band's largest visited count was written) are expanded word by
// word into a ring of list positions.  take() stages the next kBatch of them
// (padded with entries that composite nowhere) and returns how many there are.
struct BandList {
  const uint64_t* used;
  int visited;      // entries the band's pixels visited: none from there on is listed
  int left;         // words of the list not yet loaded
  uint64_t mine;    // this lane's word of the current 64
  uint64_t busy;    // which of the current 64 words have bits left to expand
  int base;         // word index of lane 0's word
  int head, have;
  bool clamp;       // some staged entry's opacity reaches the 0.99 clamp
  uint32_t odd;     // kPose: whether the last entry taken was its chunk's 2nd, 4th, ...

  __device__ __forceinline__ BandList(BandLds& L, const uint64_t* u, int n)
      : used(u), visited(n), left((n + 63) >> 6), mine(0ull), busy(0ull), base(0), head(0), have(0), clamp(false),
        odd(0u) {
    if ((threadIdx.x & 63) == 0) L.ring[kRing - 1] = 1 << 30;  // before the first: of no chunk
  }

  // kPose: of the entries from position `lo` on, which get the places from
  // `place` on.  Chunks of 64 positions end at `top` (the lowest one at 0), and a
  // chunk's 2nd, 4th, ... entry keeps its red apart.
  template <bool kPose, class Lds>
  __device__ __forceinline__ int take(Lds& L, int lane, int start, const int32_t* items, const float4* rec,
                                      int lo = 0, int top = 0, int place = 0) {
    while (have < kBatch && (busy != 0ull || left > 0)) {
      if (busy == 0ull) {  // the next 64 words, the last one in lane 0
        base = left - 1;
        const int i = base - lane;
        mine = i >= 0 ? used[i] : 0ull;
        if (64 * i + 64 > visited) mine &= ~0ull >> (64 * i + 64 - visited);  // (i < ceil(visited / 64): by 63 at most)
        busy = __ballot(mine != 0ull);
        left = max(left - 64, 0);
        continue;
      }
      const int at = (int)__builtin_ctzll(busy);
      busy &= busy - 1ull;
      const uint32_t w0 = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)mine, at);
      const uint32_t w1 = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(mine >> 32), at);
      const uint64_t wd = ((uint64_t)w1 << 32) | w0;
      have += (int)__popcll(wd);
      // the word's highest bit comes first
      const uint32_t below = __builtin_amdgcn_mbcnt_hi(w1, __builtin_amdgcn_mbcnt_lo(w0, 0u));
      if (__builtin_amdgcn_inverse_ballot_w64(wd))
        L.ring[(head + have - 1 - (int)below) & (kRing - 1)] = 64 * (base - at) + lane;
    }
    wave_sync();
    const int pos = lane < min(have, kBatch) ? L.ring[(head + lane) & (kRing - 1)] : -1;
    const int n = (int)__popcll(__ballot(pos >= lo));  // (descending: the first n)
    const int chunk = (top - 1 - pos) >> 6;
    uint32_t late = 0u;
    if constexpr (kPose) {
      // (the ring still holds the entry before the first)
      const int before = L.ring[(head + lane - 1) & (kRing - 1)];
      const uint32_t first = (uint32_t)__ballot(lane < kBatch && chunk != ((top - 1 - before) >> 6));
      const uint32_t upto = first & (uint32_t)((2ull << lane) - 1ull);
      const int since = upto != 0u ? lane - (31 - __builtin_clz(upto)) : lane + 1 + (int)odd;
      late = (uint32_t)since & 1u;
      odd = n > 0 ? (uint32_t)__builtin_amdgcn_readlane((int)late, n - 1) : odd;
    }
    bool sat = false;
    if (lane < kBatch) {
      float4 a = make_float4(0.f, 0.f, 0.f, 0.f), b = a, c = a;
      if (lane < n) {
        const int it = items[start + pos];
        a = rec[(int64_t)it * 3];
        b = rec[(int64_t)it * 3 + 1];
        c = rec[(int64_t)it * 3 + 2];
        c.w = b.z;
        stage_conic(a, b);
        b.w = __int_as_float(pos);
        if constexpr (kPose)
          L.place[64 * chunk + pos - max(top - 64 * (chunk + 1), 0)] = (uint8_t)(place + lane);
        else
          L.item[lane] = it;
      }
      if constexpr (kPose) {
        L.late[lane] = late ? c.x : 0.f;
        c.x = late ? 0.f : c.x;
      }
      L.s0[lane] = a;
      L.s1[lane] = b;
      L.s2[lane] = c;
      sat = b.y >= LS_ALPHA_MAX;
    }
    clamp = __ballot(sat) != 0ull;
    wave_sync();
    head = (head + n) & (kRing - 1);
    have -= n;
    return n;
  }
};

// Eight steps of the walk, staged entries e0 .. e0 + 7, or the first four if no more
// are listed (e0 + 4 >= n): ds and wgt (kPose: wgt gD) of entry e0 + i at every
// pixel go to rows i and 8 + i.  Branch-free within four (padding entries composite
// nowhere; short lists are mostly padding: 64 renders of 4k items at 640x480, 10
// entries a tile, pose-only 660 -> 642 us and full 394 -> 381 us).  clamp: some staged entry's opacity reaches 0.99 (an
// opacity below it bounds alpha, and the clamp can not act).  kPose rounds ds as
// (T (v - acc)) alpha, and late[e] is the red that entry e adds after its green.
template <bool kPose>
__device__ __forceinline__ void walk_eight(BandLds& L, int lane, int e0, int n, bool clamp, float fx, float fy,
                                           BwdPixel& px, const float* late) {
#pragma unroll
  for (int h = 0; h < 8; h += 4) {
    if (h == 4 && e0 + 4 >= n) break;  // uniform
    const float4 c = L.s2[e0 + h + (lane & 3)];
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    v = __builtin_amdgcn_mfma_f32_4x4x1f32(c.x, px.gR, v, 0, 0, 0);
    v = __builtin_amdgcn_mfma_f32_4x4x1f32(c.y, px.gG, v, 0, 0, 0);
    if (kPose) v = __builtin_amdgcn_mfma_f32_4x4x1f32(late[e0 + h + (lane & 3)], px.gR, v, 0, 0, 0);
    v = __builtin_amdgcn_mfma_f32_4x4x1f32(c.z, px.gB, v, 0, 0, 0);
    v = __builtin_amdgcn_mfma_f32_4x4x1f32(c.w, px.gD, v, 0, 0, 0);
    // what does not depend on the earlier steps first, then the chain
    // through T and acc
    float al[4], rc[4];
#pragma unroll
    for (int i = 0; i < 4; i += 2) {
      const float4 a0 = L.s0[e0 + h + i], b0 = L.s1[e0 + h + i];
      const float4 a1 = L.s0[e0 + h + i + 1], b1 = L.s1[e0 + h + i + 1];
      al[i] = step_alpha(a0, b0, px.nl, fx, fy);
      al[i + 1] = step_alpha(a1, b1, px.nl, fx, fy);
      rc[i] = __builtin_amdgcn_rcpf(1.f - al[i]);
      rc[i + 1] = __builtin_amdgcn_rcpf(1.f - al[i + 1]);
      if (i == 0) __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      px.T *= rc[i];
      const float wgt = al[i] * px.T, d = v[i] - px.acc;
      px.acc = fmaf(al[i], d, px.acc);
      L.rows[(h + i) * kRowStride + lane] = kPose ? (px.T * -d) * al[i] : -wgt * d;
      L.rows[(8 + h + i) * kRowStride + lane] = kPose ? wgt * px.gD : wgt;
    }
    if (clamp) {  // uniform
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (al[i] >= LS_ALPHA_MAX) L.rows[(h + i) * kRowStride + lane] = 0.f;
    }
  }
  wave_sync();
}

// Lane (e, y)'s sums over pixel row y of entry e0 + e: S = ds dx, ds dy,
// ds dx^2, ds dx dy, ds dy^2, ds, then wgt times each of the kN factors.
// bx = the band's centre x, ry = row y's pixel centre.
template <int kN>
__device__ __forceinline__ void row_sums(const BandLds& L, int lane, int e0, float bx, float ry,
                                         const float (&f)[kN][8], float (&S)[6 + kN]) {
  const int e = lane >> 3;
  const float4* d4 = reinterpret_cast<const float4*>(L.rows + e * kRowStride + 8 * (lane & 7));
  const float4* w4 = reinterpret_cast<const float4*>(L.rows + (8 + e) * kRowStride + 8 * (lane & 7));
  const float4 x = d4[0], y = d4[1], p = w4[0], q = w4[1];
  const float2 uv = *reinterpret_cast<const float2*>(&L.s0[e0 + e]);
  const float s0 = x.x + y.w, s1 = x.y + y.z, s2 = x.z + y.y, s3 = x.w + y.x;
  const float d0 = y.w - x.x, d1 = y.z - x.y, d2 = y.y - x.z, d3 = y.x - x.w;
  const float r0 = (s0 + s1) + (s2 + s3);
  const float r1 = 3.5f * d0 + 2.5f * d1 + 1.5f * d2 + 0.5f * d3;
  const float r2 = 12.25f * s0 + 6.25f * s1 + 2.25f * s2 + 0.25f * s3;
  const float U = uv.x - bx, dy = ry - uv.y;
  S[0] = r1 - U * r0;
  S[1] = dy * r0;
  S[2] = r2 - U * (r1 + S[0]);
  S[3] = dy * S[0];
  S[4] = dy * S[1];
  S[5] = r0;
#pragma unroll
  for (int k = 0; k < kN; ++k)
    S[6 + k] = fmaf(q.w, f[k][7], fmaf(q.z, f[k][6], fmaf(q.y, f[k][5], fmaf(q.x, f[k][4],
               fmaf(p.w, f[k][3], fmaf(p.z, f[k][2], fmaf(p.y, f[k][1], p.x * f[k][0])))))));
}

// Within groups of eight lanes: the value of lane 7 - y, y ^ 2 or y ^ 1.
constexpr int kMirror8 = 0x141, kXor2 = 0x4E, kXor1 = 0xB1;
template <int kCtrl>
__device__ __forceinline__ float partner(float x) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), kCtrl, 0xF, 0xF, true));
}
__device__ __forceinline__ float sum8(float x) {
  x += partner<kMirror8>(x);
  x += partner<kXor2>(x);
  return x + partner<kXor1>(x);
}

// Largest of the 64 lanes' values (>= 0), as a scalar: DPP shifts within
// 16-lane rows, then the row ends broadcast to the later rows.
__device__ __forceinline__ int wave_max_i(int v) {
  v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false));  // row_shr:1
  v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false));  // row_shr:2
  v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false));  // row_shr:4
  v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false));  // row_shr:8
  v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false));  // row_bcast:15 -> rows 1, 3
  v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false));  // row_bcast:31 -> rows 2, 3
  return __builtin_amdgcn_readlane(v, 63);
}

// The band's L1 loss partial {sum, count} (L1 targets with loss_part).
__device__ __forceinline__ void band_loss(const L1Targets& l1, const BwdPixel& px, int unit, int lane) {
  if (!l1.loss_part) return;
  const float s = wave_sum(px.lsum), n = wave_sum(px.lcnt);
  if (lane == 0) reinterpret_cast<float2*>(l1.loss_part)[unit] = make_float2(s, n);
}

// Full mode: the ten sums of each (entry, band) are added to the item's
// accumulator by one atomic instruction, ten neighbouring lanes to one
// 64-byte line.  The atomics are limited by the requests (instruction x line)
// they make, not by their values (200k Gaussians at 1200x680, 1.4 M (entry,
// band) pairs: two requests per pair 183-216 us, one per pair 148 us at 40
// bytes per item and 124 us at 64, none 116 us, before the XCDs took turns).  The
// projection backward applies the factors that are the same for all pixels
// (conic, halves, 1 / opacity) once per item.  Few items over very many tiles make
// their lines wait: such a batch has copies of the accumulators (grad_copies), a
// tile's bands adding to different ones, and the projection backward adds them up.
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(5))) void k_composite_bwd(
    const JobDev* __restrict__ jobs, const int32_t* __restrict__ tile_off, int R, int T_total,
    const float4* __restrict__ rec, const int32_t* __restrict__ items, const int32_t* __restrict__ range,
    const uint64_t* __restrict__ used, int64_t ustride, float bg0, float bg1, float bg2,
    const float* __restrict__ fwd_T, const int32_t* __restrict__ fwd_n, const float* __restrict__ up_rgb,
    const float* __restrict__ up_depth, const float* __restrict__ up_alpha, const float* __restrict__ up_scale,
    float* __restrict__ g2d, GradCopies copies, L1Targets l1) {
  __shared__ __attribute__((aligned(16))) FullBandLds L;
  const int unit = xcd_turns<64>(blockIdx.x, 4 * T_total);
  if (unit >= 4 * T_total) return;
  g2d += (unit & (copies.n - 1)) * copies.stride;
  const int lane = threadIdx.x;
  const BandCtx c = band_ctx<false>(jobs, tile_off, R, unit, lane);
  const JobDev& J = jobs[c.r];
  const int start = range[2 * c.tile], end = range[2 * c.tile + 1];
  if (start == end && !l1.loss_part) return;  // uniform
  BwdPixel px = bwd_pixel(c, J, bg0, bg1, bg2, fwd_T, fwd_n, up_rgb, up_depth, up_alpha, up_scale, l1);
  band_loss(l1, px, unit, lane);
  BandList list(L, used + c.band * ustride + (start >> 6) + c.tile, min(wave_max_i(px.nl), end - start));
  if (list.left == 0) return;
  const float fx = (float)c.x + 0.5f, fy = (float)c.y + 0.5f;
  const int y = lane & 7;
  const float bx = (float)(c.x0 + 4), ry = (float)(c.y0 + y) + 0.5f;
  const float g[4] = {px.gD, px.gR, px.gG, px.gB};
  float f[4][8];
  row_factors(L.rows, lane, g, f);
  const bool hi = y & 4, b2 = y & 2, b1 = y & 1;
  const int k0 = 4 * (y & 1) + (y & 2) + (y >> 2);  // the value that this lane ends with
  for (int n = kBatch; n == kBatch;) {  // (a short batch is the last)
    n = list.take<false>(L, lane, start, items, rec);
    for (int e0 = 0; e0 < n; e0 += 8) {
      walk_eight<false>(L, lane, e0, n, list.clamp, fx, fy, px, nullptr);
      float S[kGrad2D];
      row_sums(L, lane, e0, bx, ry, f, S);
      // sums over the entry's eight lanes, halving the lanes that hold a
      // value at every level: ten values end in two registers
      float h[5];
#pragma unroll
      for (int k = 0; k < 5; ++k)
        h[k] = (hi ? S[2 * k + 1] : S[2 * k]) + partner<kMirror8>(hi ? S[2 * k] : S[2 * k + 1]);
      const float q0 = (b2 ? h[1] : h[0]) + partner<kXor2>(b2 ? h[0] : h[1]);
      const float q1 = (b2 ? h[3] : h[2]) + partner<kXor2>(b2 ? h[2] : h[3]);
      float z1 = h[4] + partner<kXor2>(h[4]);
      // by way of LDS to sixteen lanes per entry
      float* out = L.rows + (lane >> 3) * kGradStride;
      out[k0] = (b1 ? q1 : q0) + partner<kXor1>(b1 ? q0 : q1);
      z1 += partner<kXor1>(z1);
      if ((y & 3) == 0) out[8 + (y >> 2)] = z1;
      wave_sync();
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        const int e = e0 + 4 * p + (lane >> 4), k = lane & 15;
        const float v = L.rows[64 * p + lane];
        if (e < n && k < kGrad2D && v != 0.f) atomic_add_f32(g2d + (int64_t)L.item[e] * kGradStride + k, v);
      }
      wave_sync();
    }
  }
}

// Pose-only mode (registration, tracking): only the gradients a pose
// correction acts through (u, v, conic, depth) are formed, one block per tile, a
// wave per band.  The waves walk their bands over a round of list positions
// (from the tile's last visited one down) and leave each entry's six sums in LDS;
// then lane j of wave c adds up the bands of the round's position j of chunk c (64
// positions), turns the sums into the image-space gradients and applies the pose
// Jacobian of its Gaussian, and the chunks' sums are added, in a fixed order, to
// the tile's running sum, written once as the tile's 12-value partial: no atomics,
// so the pose gradient is deterministic and independent of the other renders.
//
// Every rounding is fixed: a registration follows its pose gradients for a
// hundred Adam steps, whose quotient turns a changed last bit of a component that
// cancels into another pose, and a view's residual moves by up to 1e-4 of itself.
// Products are therefore rounded per pixel, and an entry's pixels summed as a
// tree: rows y and y + 4, y + 2, y + 1, then columns x and 7 - x, x ^ 1, x ^ 2;
// then its bands in order, the chunk's entries by wave_sums, and four chunks as
// (0 + 1) + (2 + 3).  The colour term v is the FMA chain red, green, blue, depth
// for a band's 1st, 3rd, ... composited entry of a chunk, and green, red, blue,
// depth for its 2nd, 4th, ...
//
// An entry costs about 23 VALU instructions in the walk and 14 in the sums (53
// with the products in the walk and a reduction of six values an entry).  Bound
// by their issue and by the waves that wait for the tile's slowest at a round's
// end: 16 views of 640x480 of 150k/120k 472 -> 358 us, 97k at 640x480 92 -> 68 us.
// What a round costs besides its entries is the larger part of the wait, so rounds
// are long: 256 positions where each band's entries fit kPosePlaces places (39 KB
// of LDS, four blocks on a CU), else 128, which always fit.  (One place per
// position: rounds of 128 392 us, of 64 473, of 256 in 51 KB and three blocks 445, to
// 374 then; one wave per tile, its bands in turn, 476 us, and 97k 146 us.  Sums by pixel
// rows, a wave per band and no common round, with the Jacobian per (entry, band):
// 290 and 56 us, but other roundings.)  Of short lists the fixed part counts: waves
// without a chunk of 64 positions skip its sums, and no batch is taken after a
// short one (64 renders of 4k items at 640x480, 10 entries a tile, 642 -> 610 us,
// 128 of 2k at 160x120 96 -> 91; with a reduction of every entry in its band
// 505 and 94, where dense ones took 472 us).  Less LDS for more waves spills: 892 us
// with five on a SIMD.
__device__ __forceinline__ float uniform(float x) {
  return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(x)));
}

constexpr int kPosePlaces = 128;  // a band's entries with sums per round
static_assert(kPosePlaces < kNoPlace && kPosePlaces >= kPoseRound / 2, "a half round always fits");

// Lane (e, x)'s sums over pixel column x of entry e0 + e.  fx = the column's
// pixel centre, fy = the eight rows'.  (Products and sums are rounded apart.)
__device__ __forceinline__ void column_sums(const BandLds& L, int lane, int e0, float fx, const float (&fy)[8],
                                            float (&S)[kPoseRow]) {
#pragma clang fp contract(off)
  const int e = lane >> 3;
  const float4* d4 = reinterpret_cast<const float4*>(L.rows + e * kRowStride + 8 * (lane & 7));
  const float4* w4 = reinterpret_cast<const float4*>(L.rows + (8 + e) * kRowStride + 8 * (lane & 7));
  const float4 d0 = d4[0], d1 = d4[1], w0 = w4[0], w1 = w4[1];
  const float2 uv = *reinterpret_cast<const float2*>(&L.s0[e0 + e]);
  const float ds[8] = {d0.x, d0.y, d0.z, d0.w, d1.x, d1.y, d1.z, d1.w};
  const float dx = fx - uv.x;
  float g[5][8];
#pragma unroll
  for (int y = 0; y < 8; ++y) {
    const float dy = fy[y] - uv.y;
    g[0][y] = ds[y] * dx;
    g[1][y] = ds[y] * dy;
    g[2][y] = g[0][y] * dx;
    g[3][y] = g[0][y] * dy;
    g[4][y] = g[1][y] * dy;
  }
#pragma unroll
  for (int q = 0; q < 5; ++q)
    S[q] = ((g[q][0] + g[q][4]) + (g[q][2] + g[q][6])) + ((g[q][1] + g[q][5]) + (g[q][3] + g[q][7]));
  S[5] = ((w0.x + w1.x) + (w0.z + w1.z)) + ((w0.y + w1.y) + (w0.w + w1.w));
}

// One band's walk over the list positions [lo, top): the sums of its i-th entry go
// to part[i][kPoseRow].  x0, y0: the band's first pixel.
__device__ __forceinline__ void pose_walk(PoseBandLds& L, int lane, BandList& list, int start, int top, int lo,
                                          const int32_t* __restrict__ items, const float4* __restrict__ rec, int x0,
                                          int y0, BwdPixel& px, float* part) {
  const int x = lane & 7;
  const float fx = (float)(x0 + (lane >> 3)) + 0.5f, fy = (float)(y0 + x) + 0.5f;
  const float colx = (float)(x0 + x) + 0.5f;
  float rowy[8];
#pragma unroll
  for (int y = 0; y < 8; ++y) rowy[y] = (float)(y0 + y) + 0.5f;
  const bool hi = x & 4, b1 = x & 2, b0 = x & 1;
  const int k0 = b1 ? 4 + (x >> 2) : 2 * (x & 1) + (x >> 2);  // the value that this lane ends with
  const bool puts = !(b1 && b0);
  part += (lane >> 3) * kPoseRow + k0;
  for (int place = 0, n = kBatch; n == kBatch; place += n) {  // (a short batch is the last)
    n = list.take<true>(L, lane, start, items, rec, lo, top, place);
    for (int e0 = 0; e0 < n; e0 += 8) {
      walk_eight<true>(L, lane, e0, n, list.clamp, fx, fy, px, L.late);
      float S[kPoseRow];
      column_sums(L, lane, e0, colx, rowy, S);
      // sums over the entry's eight lanes, halving the lanes that hold a value at
      // every level: six values end in one register
      float h[3];
#pragma unroll
      for (int k = 0; k < 3; ++k)
        h[k] = (hi ? S[2 * k + 1] : S[2 * k]) + partner<kMirror8>(hi ? S[2 * k] : S[2 * k + 1]);
      const float q0 = (b0 ? h[1] : h[0]) + partner<kXor1>(b0 ? h[0] : h[1]);
      const float q1 = h[2] + partner<kXor1>(h[2]);
      const float v = (b1 ? q1 : q0) + partner<kXor2>(b1 ? q0 : q1);
      if (puts && e0 + (lane >> 3) < n) part[(place + e0) * kPoseRow] = v;
      wave_sync();
    }
  }
}

// Whether the used entries of every band among the kPoseRound positions below
// `top` have places.  words: band 0's row; lanes 8 b .. 8 b + 4 take band b's words.
__device__ __forceinline__ bool round_fits(const uint64_t* __restrict__ words, int64_t ustride, const int* visited,
                                           int top, int lane) {
  const int b = (lane >> 3) & 3, lo = max(top - kPoseRound, 0), i = (lo >> 6) + (lane & 7), end = min(top, visited[b]);
  uint64_t m = 64 * i < end ? words[b * ustride + i] : 0ull;
  if (64 * i < lo) m &= ~0ull << (lo & 63);
  if (64 * i < end && 64 * i + 64 > end) m &= ~0ull >> (64 * i + 64 - end);
  int n = (int)__popcll(m);
  n += __builtin_amdgcn_mov_dpp(n, kMirror8, 0xF, 0xF, true);
  n += __builtin_amdgcn_mov_dpp(n, kXor2, 0xF, 0xF, true);
  n += __builtin_amdgcn_mov_dpp(n, kXor1, 0xF, 0xF, true);
  return __ballot(n > kPosePlaces) == 0ull;
}

// A Gaussian's record and camera-space state, as the pose gradient reads them.
struct PoseItem {
  float4 r0, r1, a0, a1, a2;
};
__device__ __forceinline__ PoseItem pose_item(const float4* __restrict__ rec, const float4* __restrict__ aux,
                                              int64_t it) {
  return PoseItem{rec[it * 3], rec[it * 3 + 1], aux[it * 3], aux[it * 3 + 1], aux[it * 3 + 2]};
}

// a . b of three, as fma(a2, b2, fma(a0, b0, a1 b1)).
__device__ __forceinline__ float dot3(float a0, float b0, float a1, float b1, float a2, float b2) {
#pragma clang fp contract(off)
  return __builtin_fmaf(a2, b2, __builtin_fmaf(a0, b0, a1 * b1));
}

// The rotation of q / |q| (row-major).
__device__ __forceinline__ void pose_rot(float w, float x, float y, float z, float (&R)[9]) {
#pragma clang fp contract(off)
  const float inv = rsqrtf(__builtin_fmaf(z, z, __builtin_fmaf(y, y, __builtin_fmaf(w, w, x * x))));
  w *= inv;
  x *= inv;
  y *= inv;
  z *= inv;
  const float wx = w * x, wy = w * y, wz = w * z;
  R[0] = __builtin_fmaf(__builtin_fmaf(y, y, z * z), -2.f, 1.f);
  R[1] = 2.f * __builtin_fmaf(x, y, -wz);
  R[2] = 2.f * __builtin_fmaf(x, z, wy);
  R[3] = 2.f * __builtin_fmaf(x, y, wz);
  R[4] = __builtin_fmaf(__builtin_fmaf(x, x, z * z), -2.f, 1.f);
  R[5] = 2.f * __builtin_fmaf(y, z, -wx);
  R[6] = 2.f * __builtin_fmaf(x, z, -wy);
  R[7] = 2.f * __builtin_fmaf(y, z, wx);
  R[8] = __builtin_fmaf(__builtin_fmaf(x, x, y * y), -2.f, 1.f);
}

// The pose-gradient terms pc of a Gaussian from its list entry's sums: the chain
// of camera_space_grads and, with p = R_d p0 + t_d and Sc = R_d Sc0 R_d^T, dL/dR_d
// = dp p0^T + 2 G Sc R_d (pc[0..8]) and dL/dt_d = dp (pc[9..11]).  Contracted by
// hand: what a compiler would contract changes with the code around it.
__device__ __forceinline__ void pose_terms(float fx, float fy, const PoseItem& g, const float (&sum)[kPoseRow],
                                           const float (&Rd)[9], const float (&td)[3], float (&pc)[kPoseAcc]) {
#pragma clang fp contract(off)
#define FMA __builtin_fmaf
  // the conic as the staged one gives it
  const float cA = kTwoLn2 * (g.r0.z * kHalfLog2e), cB = kLn2 * (g.r0.w * kLog2e);
  const float cC = kTwoLn2 * (g.r1.x * kHalfLog2e);
  const float du = -FMA(sum[0], cA, sum[1] * cB), dv = -FMA(sum[0], cB, sum[1] * cC);
  const float dA = 0.5f * sum[2], dB = sum[3], dC = 0.5f * sum[4], dz = sum[5];
  const float px = g.a0.x, py = g.a0.y, pz = g.a0.z;
  const float S[9] = {g.a0.w, g.a1.x, g.a1.y, g.a1.x, g.a1.z, g.a1.w, g.a1.y, g.a1.w, g.a2.x};
  const float iz = 1.0f / pz, iz2 = iz * iz, iz3 = iz * iz2;
  // J0 = (j00, 0, j02), J1 = (0, j11, j12); their products with S
  const float j00 = fx * iz, j02 = px * -fx * iz * iz, j11 = fy * iz, j12 = py * -fy * iz * iz;
  float s0[3], s1[3];
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    s0[i] = FMA(S[3 * i + 2], j02, S[3 * i] * j00);
    s1[i] = FMA(S[3 * i + 2], j12, S[3 * i + 1] * j11);
  }
  const float a = FMA(j02, s0[2], j00 * s0[0]) + LS_EPS_2D;
  const float b = FMA(j02, s1[2], j00 * s1[0]);
  const float c = FMA(j12, s1[2], j11 * s1[1]) + LS_EPS_2D;
  const float bb = b * b, det = FMA(a, c, -bb);
  const float id2 = 1.0f / (det * det);
  const float ga = FMA(-dC, bb, FMA(dB, b * c, -(dA * (c * c)))) * id2;
  const float gb = FMA(dC, b * (a + a), FMA(dA, (b + b) * c, -(dB * FMA(b, b + b, det)))) * id2;
  const float gc = FMA(-dC, a * a, FMA(dB, b * a, -(dA * bb))) * id2;
  const float hb = 0.5f * gb, ga2 = ga + ga, gc2 = gc + gc, j22 = j02 * j12;
  const float G01 = j00 * j11 * hb, m02 = j00 * j12 * hb, m12 = j11 * j02 * hb;
  const float G[9] = {j00 * (j00 * ga), G01, FMA(j02, j00 * ga, m02),
                      G01, j11 * (j11 * gc), FMA(j12, j11 * gc, m12),
                      FMA(j00, j02 * ga, m02), FMA(j11, j12 * gc, m12),
                      FMA(j12, j12 * gc, FMA(j02, j02 * ga, (j22 + j22) * hb))};
  const float gJ00 = FMA(s0[0], ga2, s1[0] * gb), gJ02 = FMA(s0[2], ga2, s1[2] * gb);
  const float gJ11 = FMA(s1[1], gc2, s0[1] * gb), gJ12 = FMA(s1[2], gc2, s0[2] * gb);
  float dp[3];
  dp[0] = FMA(iz, fx * du, -(iz2 * (fx * gJ02)));
  dp[1] = FMA(iz, fy * dv, -(iz2 * (fy * gJ12)));
  dp[2] = dz + FMA(iz2, px * (fx * -du), -(iz2 * (py * (fy * dv))));
  dp[2] = FMA(-iz2, fx * gJ00, dp[2]);
  dp[2] = FMA(iz3, px * (fx * (gJ02 + gJ02)), dp[2]);
  dp[2] = FMA(-iz2, fy * gJ11, dp[2]);
  dp[2] = FMA(iz3, py * (fy * (gJ12 + gJ12)), dp[2]);
  const float d[3] = {px - td[0], py - td[1], pz - td[2]};
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    float gs[3];  // row i of G Sc
#pragma unroll
    for (int k = 0; k < 3; ++k)
      gs[k] = dot3(S[k], G[3 * i], S[3 + k], G[3 * i + 1], S[6 + k], G[3 * i + 2]);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const float q0 = dot3(Rd[k], d[0], Rd[3 + k], d[1], Rd[6 + k], d[2]);
      pc[3 * i + k] = FMA(q0, dp[i], 2.f * dot3(Rd[k], gs[0], Rd[3 + k], gs[1], Rd[6 + k], gs[2]));
    }
    pc[9 + i] = dp[i];
  }
#undef FMA
}

__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(4))) void k_composite_bwd_pose(
    const JobDev* __restrict__ jobs, const int32_t* __restrict__ tile_off, int R, int T_total,
    const float4* __restrict__ rec, const float4* __restrict__ aux, const float* __restrict__ pose,
    const int32_t* __restrict__ items, const int32_t* __restrict__ range, const uint64_t* __restrict__ used,
    int64_t ustride, float bg0, float bg1, float bg2, const float* __restrict__ fwd_T,
    const int32_t* __restrict__ fwd_n, const float* __restrict__ up_rgb, const float* __restrict__ up_depth,
    const float* __restrict__ up_alpha, const float* __restrict__ up_scale, float* __restrict__ tile_part,
    L1Targets l1) {
  __shared__ __attribute__((aligned(16))) PoseBandLds band[4];
  __shared__ __attribute__((aligned(16))) float part[4][kPosePlaces * kPoseRow];
  __shared__ float wred[4][kPoseAcc];
  __shared__ int visited[4];
  const int tile = xcd_turns<16>(blockIdx.x, T_total);
  if (tile >= T_total) return;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  PoseBandLds& L = band[w];
  const BandCtx c = band_ctx<true>(jobs, tile_off, R, 4 * tile + w, lane);
  const JobDev& J = jobs[c.r];
  const int start = range[2 * tile], end = range[2 * tile + 1];
  const uint64_t* const words = used + (start >> 6) + tile;
  if (start == end && !l1.loss_part) {  // uniform for the block
    if ((int)threadIdx.x < kPoseAcc) tile_part[(int64_t)tile * kPoseAcc + threadIdx.x] = 0.f;
    return;
  }
  BwdPixel px = bwd_pixel(c, J, bg0, bg1, bg2, fwd_T, fwd_n, up_rgb, up_depth, up_alpha, up_scale, l1);
  band_loss(l1, px, 4 * tile + w, lane);
  const int mine = min(wave_max_i(px.nl), end - start);
  if (lane == 0) visited[w] = mine;
  reinterpret_cast<uint32_t*>(L.place)[lane] = 0x01010101u * kNoPlace;
  static_assert(kPoseRound == 4 * 64, "a word of places per lane");
  __syncthreads();
  const int last = max(max(visited[0], visited[1]), max(visited[2], visited[3]));
  float total = 0.f;  // of pose value threadIdx.x
  if (last > 0) {     // uniform for the block
    // the render's correction, kept in scalar registers
    float Rd[9] = {1.f, 0.f, 0.f, 0.f, 1.f, 0.f, 0.f, 0.f, 1.f}, td[3] = {0.f, 0.f, 0.f};
    if (pose && 64 * w < last) {  // (the wave has a chunk)
      const float* pr = pose + 7 * c.r;
      pose_rot(pr[0], pr[1], pr[2], pr[3], Rd);
#pragma unroll
      for (int k = 0; k < 9; ++k) Rd[k] = uniform(Rd[k]);
      td[0] = pr[4];
      td[1] = pr[5];
      td[2] = pr[6];
    }
    BandList list(L, words + w * ustride, mine);
    int chunk0 = 0;  // of the four that are added up, the round's first
    for (int top = last, lo; top > 0; top = lo) {
      const bool whole = chunk0 == 0 && (top <= kPosePlaces || round_fits(words, ustride, visited, top, lane));
      const int chunks = whole ? kPoseRound / 64 : kPosePlaces / 64;
      lo = max(top - 64 * chunks, 0);
      pose_walk(L, lane, list, start, top, lo, items, rec, c.x0, c.y0, px, part[w]);
      const int chunk = w - chunk0;  // this wave's, if the round has it
      const bool turn = chunk >= 0 && chunk < chunks && 64 * chunk < top;
      const int end = top - 64 * chunk, base = max(end - 64, 0);
      const bool has = turn && lane < end;
      PoseItem g;  // (loaded while the other waves walk)
      if (has) g = pose_item(rec, aux, items[start + base + lane]);
      __syncthreads();
      if (turn) {
        float pc[kPoseAcc];
#pragma unroll
        for (int q = 0; q < kPoseAcc; ++q) pc[q] = 0.f;
        float sum[kPoseRow] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        bool any = false;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          const int place = band[b].place[64 * chunk + lane];
          if (place != kNoPlace) {
            any = true;
            band[b].place[64 * chunk + lane] = kNoPlace;
#pragma unroll
            for (int q = 0; q < kPoseRow; ++q) sum[q] += part[b][place * kPoseRow + q];
          }
        }
        if (any) pose_terms(J.fx, J.fy, g, sum, Rd, td, pc);
        const float out = wave_sums(pc, lane);
        const int v = wave_value(lane);
        if (v >= 0) wred[w][v] = out;
      }
      __syncthreads();
      chunk0 += lo > 0 ? chunks : (top + 63) >> 6;
      if (chunk0 == 4 || lo == 0) {
        if ((int)threadIdx.x < kPoseAcc) {
          float s[4];
#pragma unroll
          for (int q = 0; q < 4; ++q) s[q] = q < chunk0 ? wred[q][threadIdx.x] : 0.f;
          total += (s[0] + s[1]) + (s[2] + s[3]);
        }
        chunk0 = 0;
      }
    }
  }
  if ((int)threadIdx.x < kPoseAcc) tile_part[(int64_t)tile * kPoseAcc + threadIdx.x] = total;
}

// Work statistics of a forward pass: entries evaluated and composited.
__global__ __launch_bounds__(kBlock) void k_render_stats(const JobDev* __restrict__ jobs,
                                                         const int32_t* __restrict__ tile_off, int R, int T_total,
                                                         const float4* __restrict__ rec,
                                                         const int32_t* __restrict__ items,
                                                         const int32_t* __restrict__ range,
                                                         const int32_t* __restrict__ fwd_n,
                                                         unsigned long long* __restrict__ stats) {
  __shared__ float4 s0[kBlock], s1[kBlock];
  const int tile = xcd_remap(blockIdx.x, T_total);
  if (tile >= T_total) return;
  const TileCtx c = tile_ctx(jobs, tile_off, R, tile);
  const int start = range[2 * tile], end = range[2 * tile + 1];
  const float fx = (float)c.x + 0.5f, fy = (float)c.y + 0.5f;
  const int nl = c.inside ? fwd_n[c.pix] : 0;
  unsigned long long visited = c.inside ? (unsigned long long)min(nl + 1, end - start) : 0ull;
  unsigned long long comp = 0;
  for (int chunk = start; chunk < end; chunk += kBlock) {
    const int e = chunk + threadIdx.x;
    if (e < end) {
      const int64_t it = items[e];
      float4 a = rec[it * 3 + 0], b = rec[it * 3 + 1];
      stage_conic(a, b);
      s0[threadIdx.x] = a;
      s1[threadIdx.x] = b;
    }
    __syncthreads();
    const int cnt = min(kBlock, end - chunk);
    for (int j = 0; j < cnt; ++j) {
      if (chunk + j - start >= nl) break;
      const float4 a = s0[j];
      const float4 b = s1[j];
      const float dx = fx - a.x, dy = fy - a.y;
      const float sl = falloff_log2(a.z, a.w, b.x, dx, dy);
      if (composited(sl, b.z)) ++comp;
    }
    __syncthreads();
  }
  for (int off = 32; off > 0; off >>= 1) {
    visited += __shfl_xor(visited, off, 64);
    comp += __shfl_xor(comp, off, 64);
  }
  if ((threadIdx.x & 63) == 0) {
    atomicAdd(stats, visited);
    atomicAdd(stats + 1, comp);
  }
}

}  // namespace ls

namespace ls {
void launch_render_stats(const JobDev* jobs, const int32_t* tile_off, int R, int T, const float* rec,
                         const int32_t* items, const int32_t* range, const int32_t* nl, int64_t* stats,
                         hipStream_t s) {
  launch_fill_i32(reinterpret_cast<int32_t*>(stats), 4, 0, s);
  if (T <= 0) return;
  hipLaunchKernelGGL(k_render_stats, dim3(8 * ((T + 7) / 8)), dim3(kBlock), 0, s, jobs, tile_off, R, T,
                     reinterpret_cast<const float4*>(rec), items, range, nl,
                     reinterpret_cast<unsigned long long*>(stats));
}

static inline int xcd_grid(int total) { return 8 * ((total + 7) / 8); }

void launch_composite_fwd(const JobDev* jobs, const int32_t* tile_off, int R, int T, const float* rec,
                          const int32_t* items, const int32_t* range, const float* bg, float* rgb, float* depth,
                          float* alpha, float* Tf, int32_t* nl, uint64_t* used, int64_t ustride,
                          hipStream_t s) {
  if (T <= 0) return;
  // LS_COVER=0 (read at every launch; for tests and measurements): stage by
  // the band rectangle test alone, whatever pixels have stopped
  const char* cv = std::getenv("LS_COVER");
  const int cover = (cv && cv[0] == '0' && cv[1] == '\0') ? 0 : 1;
  hipLaunchKernelGGL(k_composite_fwd_band, dim3(xcd_grid(4 * T)), dim3(64), 0, s, jobs, tile_off, R, T,
                     reinterpret_cast<const float4*>(rec), items, range, bg[0], bg[1], bg[2], rgb, depth, alpha, Tf,
                     nl, used, ustride, cover);
}

void launch_composite_bwd(const JobDev* jobs, const int32_t* tile_off, int R, int T, const float* rec,
                          const float* aux, const float* pose, const int32_t* items, const int32_t* range,
                          const uint64_t* used, int64_t ustride, const float* bg, const float* Tf,
                          const int32_t* nl,
                          const float* up_rgb, const float* up_depth, const float* up_alpha, const float* up_scale,
                          float* g2d, GradCopies copies, float* tile_part, int pose_only, hipStream_t s,
                          const L1Targets* l1) {
  if (T <= 0) return;
  const L1Targets l1v = l1 ? *l1 : L1Targets{nullptr, nullptr, nullptr, nullptr, nullptr};
  const float4* rec4 = reinterpret_cast<const float4*>(rec);
  const float4* aux4 = reinterpret_cast<const float4*>(aux);
  if (pose_only) {
    hipLaunchKernelGGL(k_composite_bwd_pose, dim3(xcd_grid(T)), dim3(kBlock), 0, s, jobs, tile_off, R, T, rec4, aux4,
                       pose, items, range, used, ustride, bg[0], bg[1], bg[2], Tf, nl, up_rgb, up_depth, up_alpha,
                       up_scale, tile_part, l1v);
    return;
  }
  hipLaunchKernelGGL(k_composite_bwd, dim3(xcd_grid(4 * T)), dim3(64), 0, s, jobs, tile_off, R, T, rec4, items, range,
                     used, ustride, bg[0], bg[1], bg[2], Tf, nl, up_rgb, up_depth, up_alpha, up_scale, g2d, copies,
                     l1v);
}
}  // namespace ls
