// Tile binning of large images and of sparse batches on gfx950: the depth-sorted
// items' (tile, item) pairs, emitted in depth order and sorted by tile.
//
// Distributing every sorted item over all of its render's tiles (binning.hip) costs
// in proportion to items x tiles, this to the instances; batch_host draws the line by
// the lists' capacity.
// Bound by the passes over the pairs, 20 bytes each and in runs of a few dozen keys:
// 110 M pairs of 20-bit keys 2.8 ms (emission 0.33, a pass 0.7), 16 M of 0.56 M tiles
// 0.46 ms; below a few million by the launches, 12 after the depth order (300k items,
// 0.9 M instances at 2560 x 1440: 111 us).
#include "common.h"

#include <algorithm>

#include "kernels.h"

namespace ls {

constexpr int kPairThreads = 256;
constexpr int kPairRounds = 8;  // rounds of kPairThreads sorted items per block
constexpr int kEmitWaves = 8;
int64_t pair_item_blocks(int64_t M) { return (M + kPairThreads * kPairRounds - 1) / (kPairThreads * kPairRounds); }
// Instances that an emission wave writes: 64 to 512, so that up to 2 M of them
// still make 1,024 blocks.
constexpr int kSpanMin = 64, kSpanMax = 512, kSpanWaves = 1024 * kEmitWaves;
static int64_t spans_of(int64_t cap, int64_t span) { return (cap + span - 1) / span; }
static int64_t emit_span(int64_t cap) {
  return std::min<int64_t>(std::max<int64_t>(32 * spans_of(cap, 32 * kSpanWaves), kSpanMin), kSpanMax);
}
int64_t pair_spans_room(int64_t cap) {
  return std::max(spans_of(cap, kSpanMax), std::min<int64_t>(spans_of(cap, kSpanMin), kSpanWaves));
}

// The renders' first places in the sequence of all sorted items, kept_off[R] = K of
// them, and the pairs as one segment of a sort of `blocks` blocks.  One block.
__global__ __launch_bounds__(1024) void k_pair_renders(const JobDev* __restrict__ jobs, int R,
                                                       const int32_t* __restrict__ kept,
                                                       int32_t* __restrict__ kept_off, PairSegs seg, int blocks) {
  __shared__ int32_t wsum[16];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  int32_t base = 0;
  for (int r0 = 0; r0 < R; r0 += 1024) {
    const int r = r0 + threadIdx.x;
    const int32_t mine = r < R && jobs[r].n > 0 ? kept[r] : 0;
    const int32_t x = (int32_t)wave_incl_sum((uint32_t)mine);
    if (lane == 63) wsum[w] = x;
    __syncthreads();
    int32_t run = base + x - mine;
    for (int k = 0; k < 16; ++k) {
      run += k < w ? wsum[k] : 0;
      base += wsum[k];
    }
    if (r < R) kept_off[r] = run;
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    kept_off[R] = base;
    seg.blk_off[0] = 0;
    seg.blk_off[1] = blocks;
    seg.base[0] = 0;
  }
}

// The sorted items of all renders, one after another.
struct PairItems {
  const uint32_t* order;
  const int64_t* item_off;
  const int32_t* kept_off;
  int R;
  __device__ __forceinline__ uint32_t at(int64_t k, int& r) const {
    r = R > 1 ? find_segment<int32_t>(kept_off, R, (int32_t)k) : 0;
    return order[item_off[r] + (k - kept_off[r])];
  }
};

// Instances of each block of kPairThreads x kPairRounds items.
__global__ __launch_bounds__(kPairThreads) void k_pair_count(PairItems items, const int32_t* __restrict__ tiles,
                                                             uint64_t* __restrict__ bsum) {
  __shared__ uint64_t ws[kPairThreads / 64];
  const int64_t base = (int64_t)blockIdx.x * kPairRounds * kPairThreads, n = items.kept_off[items.R];
  uint64_t s = 0;
  int r;
#pragma unroll
  for (int i = 0; i < kPairRounds; ++i) {
    const int64_t k = base + i * kPairThreads + threadIdx.x;
    s += k < n ? (uint32_t)tiles[items.at(k, r)] : 0u;
  }
  for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
  if ((threadIdx.x & 63) == 0) ws[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) bsum[blockIdx.x] = (ws[0] + ws[1]) + (ws[2] + ws[3]);
}

// First instance of every item (clamped to the capacity): the sum of the earlier
// blocks, formed by each block for itself, plus the prefix in the block.  The item
// that holds instance m * span (m < nspan) is recorded in first[m].  Block 0 also
// writes count = {min(I, cap), I > cap, min(I, INT32_MAX), 0}.
__global__ __launch_bounds__(kPairThreads) void k_pair_offsets(PairItems items, const int32_t* __restrict__ tiles,
                                                               const uint64_t* __restrict__ bsum, int nblk,
                                                               uint32_t* __restrict__ offs, int64_t cap, int64_t span,
                                                               int64_t nspan, uint32_t* __restrict__ first,
                                                               int32_t* __restrict__ count) {
  constexpr int kWaves = kPairThreads / 64;
  __shared__ uint64_t wbefore[kWaves], wall[kWaves], wt[kPairRounds][kWaves];
  const int64_t base = (int64_t)blockIdx.x * kPairRounds * kPairThreads, n = items.kept_off[items.R];
  if (blockIdx.x != 0 && base >= n) return;  // no item here (block 0 writes the counts)
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  uint64_t before = 0, all = 0;
  for (int b = threadIdx.x; b < (blockIdx.x == 0 ? nblk : (int)blockIdx.x); b += kPairThreads) {
    const uint64_t v = bsum[b];
    all += v;
    before += b < (int)blockIdx.x ? v : 0u;
  }
  for (int off = 32; off > 0; off >>= 1) {
    before += __shfl_xor(before, off, 64);
    all += __shfl_xor(all, off, 64);
  }
  if (lane == 0) {
    wbefore[w] = before;
    wall[w] = all;
  }
  uint32_t c[kPairRounds];
  uint64_t x[kPairRounds];
  int r;
#pragma unroll
  for (int i = 0; i < kPairRounds; ++i) {
    const int64_t k = base + i * kPairThreads + threadIdx.x;
    c[i] = k < n ? (uint32_t)tiles[items.at(k, r)] : 0u;
  }
#pragma unroll
  for (int i = 0; i < kPairRounds; ++i) {
    // (64 items' tiles may pass 2^32: low and high halves)
    const uint64_t incl = (uint64_t)wave_incl_sum(c[i] & 0xFFFFu) + ((uint64_t)wave_incl_sum(c[i] >> 16) << 16);
    x[i] = incl - c[i];
    if (lane == 63) wt[i][w] = incl;
  }
  __syncthreads();
  uint64_t run = (wbefore[0] + wbefore[1]) + (wbefore[2] + wbefore[3]);
#pragma unroll
  for (int i = 0; i < kPairRounds; ++i) {
    uint64_t pre = run;
#pragma unroll
    for (int u = 0; u < kWaves; ++u) {
      pre += u < w ? wt[i][u] : 0u;
      run += wt[i][u];
    }
    const int64_t k = base + i * kPairThreads + threadIdx.x;
    if (k < n) {
      const int64_t o = (int64_t)(pre + x[i]);
      offs[k] = (uint32_t)min(o, cap);
      for (int64_t m = (o + span - 1) / span; m < nspan && m * span < o + c[i]; ++m) first[m] = (uint32_t)k;
    }
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    const int64_t I = (int64_t)((wall[0] + wall[1]) + (wall[2] + wall[3]));
    count[0] = (int32_t)min(I, cap);
    count[1] = I > cap ? 1 : 0;
    count[2] = (int32_t)min(I, (int64_t)INT32_MAX);
    count[3] = 0;
  }
}

// Inclusive prefix maximum over the 64 lanes (DPP, as wave_incl_sum); -1 is the
// identity.
__device__ __forceinline__ int wave_incl_max(int v) {
  v = max(v, __builtin_amdgcn_update_dpp(-1, v, 0x111, 0xF, 0xF, false));  // row_shr:1
  v = max(v, __builtin_amdgcn_update_dpp(-1, v, 0x112, 0xF, 0xF, false));  // row_shr:2
  v = max(v, __builtin_amdgcn_update_dpp(-1, v, 0x114, 0xF, 0xF, false));  // row_shr:4
  v = max(v, __builtin_amdgcn_update_dpp(-1, v, 0x118, 0xF, 0xF, false));  // row_shr:8
  v = max(v, __builtin_amdgcn_update_dpp(-1, v, 0x142, 0xA, 0xF, false));  // row_bcast:15 -> rows 1, 3
  v = max(v, __builtin_amdgcn_update_dpp(-1, v, 0x143, 0xC, 0xF, false));  // row_bcast:31 -> rows 2, 3
  return v;
}

// Emission of the pairs in depth order, one wave per span of consecutive
// instances (so every wave has the same work, however many tiles its items
// cover).  The wave takes the items from the span's first one on, 64 at a time,
// lane l item kb + l: its first instance, its tile rectangle and the key of the
// rectangle's first tile.  It fills the span 64 instances at a time, lane l
// writing instance W0 + l, so every store is one contiguous run; windows stop at
// the end of the loaded items, and the next 64 items start there.  The owner of an
// instance is the last item that starts at or before it: items starting inside
// the window mark their start (LDS), a prefix maximum over the lanes carries each
// mark forward, and places before the first start keep the previous owner (at
// first, lane 0: the item that holds the span's first instance).  Within its
// owner's rectangle, instance q lies in row q / width.  Instances at or beyond the
// capacity are not written.
__global__ __launch_bounds__(64 * kEmitWaves) void k_pair_emit(const JobDev* __restrict__ jobs, PairItems items,
                                                               const float4* __restrict__ rec,
                                                               const int32_t* __restrict__ radius,
                                                               const int32_t* __restrict__ tiles,
                                                               const uint32_t* __restrict__ offs,
                                                               const int32_t* __restrict__ count,
                                                               const uint32_t* __restrict__ first, int64_t span_len,
                                                               int64_t nspan, uint32_t* __restrict__ kout,
                                                               uint32_t* __restrict__ vout) {
  __shared__ int marks[kEmitWaves][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t I = count[0];  // already clamped to the capacity
  const int64_t span = (int64_t)blockIdx.x * kEmitWaves + w;
  if (span >= nspan || span * span_len >= I) return;  // uniform for the wave; no barrier follows
  const int64_t n = items.kept_off[items.R];
  const int64_t iend = min((span + 1) * span_len, I);
  int64_t kb = first[span], W0 = span * span_len;
  while (W0 < iend && kb < n) {
    const int64_t k = kb + lane;
    const int last = (int)min((int64_t)63, n - 1 - kb);  // last lane with an item
    uint32_t off = 0xFFFFFFFFu, it = 0;
    int nt = 0, base_key = 0, stride = 0, wdt = 1;
    if (k < n) {
      int r;
      off = offs[k];
      it = items.at(k, r);
      nt = tiles[it];
      const JobDev& J = jobs[r];
      const float2 uv = *reinterpret_cast<const float2*>(rec + (int64_t)it * 3);
      const Rect rc = tile_rect(uv.x, uv.y, radius[it], J.TX, J.TY);
      wdt = max(rc.x1 - rc.x0, 1);
      base_key = J.tile_off + rc.y0 * J.TX + rc.x0;
      stride = J.TX - wdt;
    }
    const float inv = 1.0f / (float)wdt;
    const int64_t past = (int64_t)off + nt;  // (of the last lane: past the loaded items' instances)
    const int64_t cend = min(((int64_t)__builtin_amdgcn_readlane((int)(past >> 32), last) << 32) |
                                 (uint32_t)__builtin_amdgcn_readlane((int)past, last),
                             iend);
    int carry = 0;
    while (W0 < cend) {
      marks[w][lane] = -1;
      const int64_t rel = (int64_t)off - W0;
      if (nt > 0 && rel >= 0 && rel < 64) marks[w][(int)rel] = lane;
      wave_sync();
      int o = wave_incl_max(marks[w][lane]);
      o = o < 0 ? carry : o;
      carry = __builtin_amdgcn_readlane(o, 63);
      const int64_t i = W0 + lane;
      const int o_key = __shfl(base_key, o, 64), o_stride = __shfl(stride, o, 64), o_wdt = __shfl(wdt, o, 64);
      const float o_inv = __shfl(inv, o, 64);
      const uint32_t o_off = (uint32_t)__shfl((int)off, o, 64), o_it = (uint32_t)__shfl((int)it, o, 64);
      if (i < cend) {
        const int q = (int)(i - (int64_t)o_off);
        int dy = (int)((float)q * o_inv);
        if ((dy + 1) * o_wdt <= q)
          ++dy;
        else if (dy * o_wdt > q)
          --dy;
        kout[i] = (uint32_t)(o_key + dy * o_stride + q);
        vout[i] = o_it;
      }
      wave_sync();
      W0 = min(W0 + 64, cend);
    }
    kb += 64;
  }
}

// [start, end) of each tile's run in the sorted keys (the others' are cleared
// before).  A thread takes 4 consecutive keys (one 16-byte load, and its
// neighbours' edge keys; keys that are not 16-byte aligned are read one by one).
__global__ __launch_bounds__(256) void k_pair_ranges(const uint32_t* __restrict__ keys,
                                                     const int32_t* __restrict__ count, int32_t* __restrict__ range) {
  const int64_t k0 = 4 * ((int64_t)blockIdx.x * blockDim.x + threadIdx.x);
  const int64_t n = count[0];
  if (k0 >= n) return;
  uint32_t kk[6];  // keys k0 - 1 .. k0 + 4 (valid where 0 <= index < n)
  kk[0] = k0 > 0 ? keys[k0 - 1] : 0u;
  if (k0 + 4 <= n && (reinterpret_cast<uintptr_t>(keys) & 15) == 0) {
    const uint4 q = *reinterpret_cast<const uint4*>(keys + k0);
    kk[1] = q.x;
    kk[2] = q.y;
    kk[3] = q.z;
    kk[4] = q.w;
  } else {
    for (int j = 0; j < 4; ++j) kk[1 + j] = k0 + j < n ? keys[k0 + j] : 0u;
  }
  kk[5] = k0 + 4 < n ? keys[k0 + 4] : 0u;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int64_t k = k0 + j;
    if (k >= n) break;
    const int64_t t = kk[1 + j];
    if (k == 0 || kk[j] != (uint32_t)t) range[2 * t] = (int32_t)k;
    if (k == n - 1 || kk[2 + j] != (uint32_t)t) range[2 * t + 1] = (int32_t)(k + 1);
  }
}

void launch_bin_pairs(const BinLaunch& b, hipStream_t s) {
  const PairLaunch& p = b.pairs;
  const int R = b.tab.R, nblk = (int)pair_item_blocks(b.M);
  const int per = sort_per(b.cap, [&](int per) { return sort_blocks_of(b.cap, per); });
  const int blocks = sort_blocks_of(b.cap, per);
  hipLaunchKernelGGL(k_pair_renders, dim3(1), dim3(1024), 0, s, b.jobs, R, (const int32_t*)b.kept, p.kept_off, p.seg,
                     blocks);
  const PairItems items{b.v0, b.item_off, p.kept_off, R};
  uint32_t* offs = b.k0;  // (free after the depth sort)
  hipLaunchKernelGGL(k_pair_count, dim3(nblk), dim3(kPairThreads), 0, s, items, b.tiles, p.bsum);
  const int64_t span = emit_span(b.cap), nspan = spans_of(b.cap, span);
  hipLaunchKernelGGL(k_pair_offsets, dim3(nblk), dim3(kPairThreads), 0, s, items, b.tiles, (const uint64_t*)p.bsum,
                     nblk, offs, b.cap, span, nspan, p.first, b.count);
  launch_fill_i32(b.range, 2 * (int64_t)b.T, 0, s);
  if (b.cap == 0) return;
  // as few passes as 8-bit digits take, with the bits split evenly: fewer digits
  // leave longer runs to write (137 M pairs of 18-bit keys: 4.8 ms with 8, 8 and 2
  // bits, 4.0 with 6 each)
  int bits = 1;
  while (bits < 31 && (int64_t)b.T > (int64_t)1 << bits) ++bits;
  const int passes = (bits + 7) / 8, width = (bits + passes - 1) / passes;
  uint32_t* item = reinterpret_cast<uint32_t*>(b.item);
  uint32_t *ka = passes & 1 ? p.tk : b.tile_of, *va = passes & 1 ? p.tv : item;
  uint32_t *kb = passes & 1 ? b.tile_of : p.tk, *vb = passes & 1 ? item : p.tv;
  hipLaunchKernelGGL(k_pair_emit, dim3((unsigned)((nspan + kEmitWaves - 1) / kEmitWaves)), dim3(64 * kEmitWaves), 0,
                     s, b.jobs, items, reinterpret_cast<const float4*>(b.rec), b.radius, b.tiles,
                     (const uint32_t*)offs, (const int32_t*)b.count, (const uint32_t*)p.first, span, nspan, ka, va);
  const SegTable seg{p.seg.blk_off, p.seg.base, 1, b.count};
  for (int k = 0; k < passes; ++k) {
    launch_seg_pass(ka, va, kb, vb, seg, blocks, blocks, per, width * k, width, p.hist, false, s);
    std::swap(ka, kb);
    std::swap(va, vb);
  }
  hipLaunchKernelGGL(k_pair_ranges, dim3((unsigned)((b.cap + 1023) / 1024)), dim3(256), 0, s,
                     (const uint32_t*)b.tile_of, (const int32_t*)b.count, b.range);
}

}  // namespace ls
