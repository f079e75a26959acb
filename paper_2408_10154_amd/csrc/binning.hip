// Tile binning on gfx950: a depth sort of each render's items and a stable
// distribution of the sorted items over the render's tiles.
//
// Order of the final list: (tile, FP32 depth bits, item).
//
//  1. The items with tiles are sorted by depth bits, render by render (LSD
//     radix sort, stable: ties keep ascending item order).  A render of up to
//     16,384 items has them ranked by comparison, in a batch of such renders a
//     block each sorts them in LDS, in one launch; larger ones take a histogram
//     and a scatter per digit, and the scatter forms its digit bases from the
//     block histograms itself (or, of many blocks, a scan does).
//  2. The sorted items are cut into chunks.  One block per chunk counts the
//     items of every tile of its render, a scan over the chunks turns the
//     counts into each chunk's first place in each tile's list, and one block
//     per chunk then writes the instances straight to their final places.
//     Large images and sparse batches go by binning_pairs.hip instead.
//
// Every instance is written once, and no (tile, item) pairs are sorted: the
// pair sort it replaces moved each instance three times in 8 launches (all of
// binning: 200k items, 1200 x 680, 143 -> 91 us and 22 launches -> 11; eight
// renders of 150k items, 640 x 480, 157 -> 109 us; 23k items, 317 x 211, 90 ->
// 52 us and 10 launches; 4,096 items, 160 x 120, 81 -> 29 us and 3 launches).
// What is left is bound by latency: launches of 3 to 10 us on tens to hundreds
// of blocks, each a chain of dependent loads.
#include "common.h"

#include <algorithm>

#include "kernels.h"

namespace ls {

__global__ void k_fill_i32(int32_t* __restrict__ p, int64_t n, int32_t v) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t k = i; k < n; k += stride) p[k] = v;
}

// ---------------------------------------------------------------------------
// Segmented stable radix sort: segment s holds its (key, value) pairs at
// base[s] .. base[s] + len[s] (len on the device) and owns the sort blocks
// blk_off[s] .. blk_off[s + 1), kPer x kSortThreads keys each (sort_per), of
// which those with keys work.
//
// Four passes of 8-bit digits.  (Three of 11, 11 and 10 bits, in two launches
// less: 17k items' binning 62.3 us against 61.1, 40k 75 against 67, 65k 85
// against 70; 30 renders of 20k 127 against 129.)

constexpr int kSortWaves = kSortThreads / 64;
constexpr int kSortBits = 8;
// Words between two blocks' histograms: 256 counts, and some more so that one
// digit's counts spread over the memory channels (109 M pairs, 26,700 blocks: 3,254
// us at 256 words, 3,069 at 272, 3,081 at 320; 42 M, 10,300: 1,388, 1,419 and 1,265).
constexpr int kHistRow = 320;
template <int kBits>
struct Digit {
  static constexpr int kBins = 1 << kBits;
  static constexpr int kPer = kBins > kSortThreads ? kBins / kSortThreads : 1;  // bins per thread (1 or 2)
  static constexpr int kThreads = kBins / kPer;                                 // threads with bins
  __device__ __forceinline__ static uint32_t of(uint32_t key, int shift, uint32_t mask = kBins - 1) {
    return (key >> shift) & mask;
  }
};

// Exclusive prefix of one value per thread over the first kThreads threads (the
// others' values are ignored); every thread of the block calls it.
template <int kThreads>
__device__ __forceinline__ uint32_t digit_excl(uint32_t v, uint32_t* wsum) {
  const int w = threadIdx.x >> 6;
  const uint32_t x = wave_incl_sum(v);
  if ((threadIdx.x & 63) == 63 && w < kThreads / 64) wsum[w] = x;
  __syncthreads();
  uint32_t before = 0;
#pragma unroll
  for (int k = 0; k < kThreads / 64; ++k) before += k < w ? wsum[k] : 0u;
  return before + x - v;
}

// Ranks of the wave's keys among its earlier keys of the same digit: 64 at a
// time in order, a ballot match per 64 keys, and the wave's running digit
// counts in its own LDS row (cleared here).
template <int kBits, int kPer>
__device__ __forceinline__ void wave_ranks(const uint32_t (&key)[kPer], const bool (&ok)[kPer], int shift,
                                           uint32_t mask, uint16_t* row, int lane, uint32_t (&rk)[kPer]) {
  const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
#pragma unroll
  for (int d = 0; d < Digit<kBits>::kBins / 128; ++d) reinterpret_cast<uint32_t*>(row)[64 * d + lane] = 0u;
  wave_sync();
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const uint32_t d = Digit<kBits>::of(key[j], shift, mask);
    const uint64_t valid = __ballot(ok[j]);
    rk[j] = 0u;
    if (valid != 0ull) {  // uniform
      uint32_t plo = (uint32_t)valid, phi = (uint32_t)(valid >> 32);
#pragma unroll
      for (int b = 0; b < kBits; ++b) {
        const uint32_t sign = (uint32_t)((int32_t)(d << (31 - b)) >> 31);  // all ones where the bit is set
        const uint64_t m = __ballot(sign != 0u);
        plo &= ~((uint32_t)m ^ sign);
        phi &= ~((uint32_t)(m >> 32) ^ sign);
      }
      const uint64_t peers = ((uint64_t)phi << 32) | plo;
      const uint32_t rank = (uint32_t)__popcll(peers & lt);
      const uint32_t before = ok[j] ? row[d] : 0u;
      rk[j] = before + rank;
      if (ok[j] && rank == 0) row[d] = (uint16_t)(before + (uint32_t)__popcll(peers));
      wave_sync();
    }
  }
}

// The block's digit starts, after every wave has ranked (and a barrier): each
// wave's row turns into its first place for each digit in the block's digit
// order (at most 8,192 keys: 16 bits); lstart: the local starts of
// the thread's digits (threads below kThreads); returns the number of keys up
// to and with them.
template <int kBits>
__device__ __forceinline__ uint32_t digit_starts(uint16_t (*wcnt)[Digit<kBits>::kBins], uint32_t* wsum,
                                                 uint32_t (&lstart)[Digit<kBits>::kPer]) {
  using D = Digit<kBits>;
  const bool mine = (int)threadIdx.x < D::kThreads;
  uint32_t c[kSortWaves], cnt = 0;  // two 16-bit counts, or one
  if (mine) {
#pragma unroll
    for (int k = 0; k < kSortWaves; ++k) {
      c[k] = D::kPer == 2 ? reinterpret_cast<const uint32_t*>(wcnt[k])[threadIdx.x] : wcnt[k][threadIdx.x];
      cnt += c[k];  // (sums stay below 2^16)
    }
  }
  const uint32_t first = cnt & 0xFFFFu, both = first + (cnt >> 16);
  lstart[0] = digit_excl<D::kThreads>(both, wsum);
  if (D::kPer == 2) lstart[D::kPer - 1] = lstart[0] + first;
  if (mine) {
    uint32_t run = D::kPer == 2 ? lstart[0] | (lstart[D::kPer - 1] << 16) : lstart[0];
#pragma unroll
    for (int k = 0; k < kSortWaves; ++k) {
      if (D::kPer == 2)
        reinterpret_cast<uint32_t*>(wcnt[k])[threadIdx.x] = run;
      else
        wcnt[k][threadIdx.x] = (uint16_t)run;
      run += c[k];
    }
  }
  return lstart[0] + both;
}

// Digit counts of every block's keys: hist[block][digit].
template <int kPer>
__global__ __launch_bounds__(kSortThreads) void k_seg_hist(const uint32_t* __restrict__ keys, SegTable seg, int shift,
                                                           uint32_t mask, uint32_t* __restrict__ hist) {
  using D = Digit<kSortBits>;
  constexpr int kKeys = kPer * kSortThreads;
  __shared__ uint32_t h[D::kBins];
  const int s = find_segment<int32_t>(seg.blk_off, seg.S, (int32_t)blockIdx.x);
  const int c = blockIdx.x - seg.blk_off[s];
  const int m = min(seg.len[s] - c * kKeys, kKeys);
  if (m <= 0) return;  // uniform for the block
  for (int d = threadIdx.x; d < D::kBins; d += kSortThreads) h[d] = 0u;
  const uint32_t* __restrict__ k0 = keys + seg.base[s] + (int64_t)c * kKeys;
  uint32_t key[kPer];
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const int i = j * kSortThreads + threadIdx.x;
    key[j] = i < m ? k0[i] : 0u;
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kPer; ++j)
    if (j * kSortThreads + (int)threadIdx.x < m) atomicAdd(&h[D::of(key[j], shift, mask)], 1u);
  __syncthreads();
  for (int d = threadIdx.x; d < D::kBins; d += kSortThreads) hist[(int64_t)blockIdx.x * kHistRow + d] = h[d];
}

// Sums of digit d's counts over the segment's blocks and over those before this
// one, kParts threads per digit; the results in threads d below kThreads.
// The rows are few (98 for 200k keys; at most kScanRows), so every block can add
// them up and no scan launch is needed.
__device__ __forceinline__ void digit_bases(const uint32_t* __restrict__ rows, int nrows, int c, uint32_t* ta,
                                            uint32_t* tb, uint32_t& total, uint32_t& before) {
  using D = Digit<kSortBits>;
  constexpr int kParts = kSortThreads / D::kThreads, kAhead = 16;
  const int d = threadIdx.x & (D::kThreads - 1), p = threadIdx.x / D::kThreads;
  total = before = 0u;
  for (int r0 = p; r0 < nrows; r0 += kAhead * kParts) {
    uint32_t v[kAhead];
#pragma unroll
    for (int k = 0; k < kAhead; ++k)
      v[k] = r0 + k * kParts < nrows ? rows[(int64_t)(r0 + k * kParts) * kHistRow + d] : 0u;
#pragma unroll
    for (int k = 0; k < kAhead; ++k) {
      total += v[k];
      before += r0 + k * kParts < c ? v[k] : 0u;
    }
  }
  ta[threadIdx.x] = total;
  tb[threadIdx.x] = before;
  __syncthreads();
  total = before = 0u;
  if ((int)threadIdx.x < D::kThreads)
#pragma unroll
    for (int k = 0; k < kParts; ++k) {
      total += ta[k * D::kThreads + d];
      before += tb[k * D::kThreads + d];
    }
}

// Stable scatter of one digit: ranks in the waves, the block's keys placed in
// LDS by digit, then written out in that order, so that stores are contiguous
// along each digit's run.  kFirst: the block's own keys, blk_cnt of them, as
// k_depth_prep left them (len[s] is written); else kKeys of the segment's
// len[s].  kLast: only the values are written.  sums: k_seg_scan has turned the
// counts into each block's bases, and these are the segments' digit totals; or
// NULL, and every block adds the counts up for itself.
template <int kPer, bool kFirst, bool kLast>
__global__ __launch_bounds__(kSortThreads) void k_seg_scatter(const uint32_t* __restrict__ kin,
                                                              const uint32_t* __restrict__ vin,
                                                              uint32_t* __restrict__ kout,
                                                              uint32_t* __restrict__ vout, SegTable seg, int shift,
                                                              uint32_t mask, const uint32_t* __restrict__ hist,
                                                              const int32_t* __restrict__ blk_cnt,
                                                              const uint32_t* __restrict__ sums) {
  using D = Digit<kSortBits>;
  constexpr int kKeys = kPer * kSortThreads;
  __shared__ __attribute__((aligned(4))) uint16_t wcnt[kSortWaves][D::kBins];
  __shared__ uint32_t sk[kKeys], sv[kKeys];
  __shared__ uint32_t delta[D::kBins];  // global minus local start of each digit's run (mod 2^32)
  __shared__ uint32_t wsum[2][kSortWaves];
  const int s = find_segment<int32_t>(seg.blk_off, seg.S, (int32_t)blockIdx.x);
  const int b0 = seg.blk_off[s], c = blockIdx.x - b0;
  const int n = kFirst ? 0 : seg.len[s];
  const int m = kFirst ? blk_cnt[blockIdx.x] : min(n - c * kKeys, kKeys);
  const int nrows = kFirst ? seg.blk_off[s + 1] - b0 : (n + kKeys - 1) / kKeys;
  if (m <= 0 && !(kFirst && c == 0)) return;  // uniform for the block
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t in0 = seg.base[s] + (int64_t)c * kKeys;
  uint32_t key[kPer], val[kPer], rk[kPer];
  bool ok[kPer];
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const int i = w * 64 * kPer + j * 64 + lane;
    ok[j] = i < m;
    key[j] = ok[j] ? kin[in0 + i] : 0u;
    val[j] = ok[j] ? vin[in0 + i] : 0u;
  }
  uint32_t total = 0u, before = 0u, lstart[1];
  if (sums == nullptr) {
    digit_bases(hist + (int64_t)b0 * kHistRow, nrows, c, sk, sv, total, before);
  } else if ((int)threadIdx.x < D::kThreads) {
    total = sums[s * D::kBins + threadIdx.x];
    before = hist[(int64_t)blockIdx.x * kHistRow + threadIdx.x];
  }
  const uint32_t first = digit_excl<D::kThreads>(total, wsum[0]);  // of the thread's digit, in the segment
  if (kFirst && c == 0 && threadIdx.x == D::kThreads - 1) seg.len[s] = (int32_t)(first + total);
  wave_ranks<kSortBits, kPer>(key, ok, shift, mask, wcnt[w], lane, rk);
  __syncthreads();
  digit_starts<kSortBits>(wcnt, wsum[1], lstart);
  if ((int)threadIdx.x < D::kThreads) delta[threadIdx.x] = first + before - lstart[0];
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kPer; ++j)
    if (ok[j]) {
      const uint32_t pos = wcnt[w][D::of(key[j], shift, mask)] + rk[j];
      sk[pos] = key[j];
      sv[pos] = val[j];
    }
  __syncthreads();
  const int64_t out0 = seg.base[s];
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const int i = j * kSortThreads + threadIdx.x;
    if (i < m) {
      const uint32_t k = sk[i];
      const int64_t pos = out0 + (uint32_t)(delta[D::of(k, shift, mask)] + (uint32_t)i);
      if (!kLast) kout[pos] = k;
      vout[pos] = sv[i];
    }
  }
}

// Segments of many blocks: the digits' counts turned into each block's bases, in
// place, and the segments' digit totals into sums.  kScanDigits digits of a
// segment to a block, kParts threads to a digit, each a run of blocks.  kFirst as
// above.
//
// A scatter block that adds up its segment's counts for itself reads 1 KB per
// block, so a pass reads the square of the blocks: past kScanRows of them the
// launch costs less (binning without and with it at 1200 x 680: 500k items, 245
// blocks, 96 and 100 us; 1M, 489, 157 and 151 us; 10M, 2,442, 1,161 and 743 us).
constexpr int kScanRows = 256, kScanDigits = 16;
template <int kPer, bool kFirst>
__global__ __launch_bounds__(1024) void k_seg_scan(SegTable seg, uint32_t* __restrict__ hist,
                                                   uint32_t* __restrict__ sums) {
  using D = Digit<kSortBits>;
  constexpr int kKeys = kPer * kSortThreads, kParts = 1024 / kScanDigits, kAhead = 16;
  __shared__ uint32_t part[kParts][kScanDigits];
  const int s = blockIdx.x / (D::kBins / kScanDigits), d0 = blockIdx.x % (D::kBins / kScanDigits) * kScanDigits;
  const int d = threadIdx.x % kScanDigits, p = threadIdx.x / kScanDigits;
  const int b0 = seg.blk_off[s], all = seg.blk_off[s + 1] - b0;
  const int rows = kFirst ? all : (seg.len[s] + kKeys - 1) / kKeys;
  const int per = (rows + kParts - 1) / kParts, lo = min(p * per, rows), hi = min(lo + per, rows);
  uint32_t* __restrict__ col = hist + (int64_t)b0 * kHistRow + d0 + d;
  uint32_t sum = 0;
  for (int r = lo; r < hi; r += kAhead) {
    uint32_t v[kAhead];
#pragma unroll
    for (int k = 0; k < kAhead; ++k) v[k] = r + k < hi ? col[(int64_t)(r + k) * kHistRow] : 0u;
#pragma unroll
    for (int k = 0; k < kAhead; ++k) sum += v[k];
  }
  part[p][d] = sum;
  __syncthreads();
  uint32_t run = 0, total = 0;
#pragma unroll 16
  for (int k = 0; k < kParts; ++k) {
    run += k < p ? part[k][d] : 0u;
    total += part[k][d];
  }
  for (int r = lo; r < hi; r += kAhead) {
    uint32_t v[kAhead];
#pragma unroll
    for (int k = 0; k < kAhead; ++k) v[k] = r + k < hi ? col[(int64_t)(r + k) * kHistRow] : 0u;
#pragma unroll
    for (int k = 0; k < kAhead; ++k)
      if (r + k < hi) {
        col[(int64_t)(r + k) * kHistRow] = run;
        run += v[k];
      }
  }
  if (p == 0) sums[s * D::kBins + d0 + d] = total;
}

int64_t seg_hist_words(int64_t nblk, int nseg) {
  return kHistRow * std::max<int64_t>(nblk, 1) + (int64_t)Digit<kSortBits>::kBins * nseg;
}

// ---------------------------------------------------------------------------
// Depth order of each render's items.

// Larger renders: each block compacts its items with tiles (in item order) and
// counts the first digit of their depth bits.
template <int kPer>
__global__ __launch_bounds__(kSortThreads) void k_depth_prep(const JobDev* __restrict__ jobs, SegTable seg,
                                                             const float4* __restrict__ rec,
                                                             const int32_t* __restrict__ tiles,
                                                             uint32_t* __restrict__ keys, uint32_t* __restrict__ vals,
                                                             uint32_t* __restrict__ hist,
                                                             int32_t* __restrict__ blk_cnt) {
  using D = Digit<kSortBits>;
  constexpr int kKeys = kPer * kSortThreads;
  __shared__ uint32_t h[D::kBins];
  __shared__ uint32_t cnt[kPer][kSortWaves];
  const int s = find_segment<int32_t>(seg.blk_off, seg.S, (int32_t)blockIdx.x);
  const int c = blockIdx.x - seg.blk_off[s];
  const int n = jobs[s].n, lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t base = seg.base[s] + (int64_t)c * kKeys;
  for (int d = threadIdx.x; d < D::kBins; d += kSortThreads) h[d] = 0u;
  uint64_t keep[kPer];
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const int i = j * kSortThreads + threadIdx.x;
    keep[j] = __ballot(c * kKeys + i < n && tiles[base + i] > 0);
    if (lane == 0) cnt[j][w] = (uint32_t)__popcll(keep[j]);
  }
  uint32_t key[kPer];
#pragma unroll
  for (int j = 0; j < kPer; ++j)
    key[j] = __builtin_amdgcn_inverse_ballot_w64(keep[j])
                 ? __float_as_uint(rec[(base + j * kSortThreads + threadIdx.x) * 3 + 1].z)
                 : 0u;
  __syncthreads();
  uint32_t run = 0;
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    uint32_t at = run;
#pragma unroll
    for (int k = 0; k < kSortWaves; ++k) {
      at += k < w ? cnt[j][k] : 0u;
      run += cnt[j][k];
    }
    if (__builtin_amdgcn_inverse_ballot_w64(keep[j])) {
      const int64_t pos = base + at + __builtin_amdgcn_mbcnt_hi((uint32_t)(keep[j] >> 32),
                                                                __builtin_amdgcn_mbcnt_lo((uint32_t)keep[j], 0u));
      keys[pos] = key[j];
      vals[pos] = (uint32_t)(base + j * kSortThreads + threadIdx.x);
      atomicAdd(&h[D::of(key[j], 0)], 1u);
    }
  }
  __syncthreads();
  for (int d = threadIdx.x; d < D::kBins; d += kSortThreads) hist[(int64_t)blockIdx.x * kHistRow + d] = h[d];
  if (threadIdx.x == 0) blk_cnt[blockIdx.x] = (int32_t)run;
}

// Small renders, of up to kItems items: each item's place is the number of
// items before it, by comparison with all of them.  A block holds the render's
// depth bits in LDS (all ones: no tiles) and takes 64 of its items, one per
// lane; a wave counts over a sixteenth of the keys.  off256: the renders' first
// blocks of 256 items.
//
// A key costs a wave a compare and an add with carry, and the keys of 4,096 items
// 2,000 cycles; the rest is the launch and two dependent loads.  All of binning
// in a graph, with this and with one block sorting each render in LDS: 1,500
// items 28 and 32 us, 4,096 33 and 38 us, 8,192 43 and 53 us; with this and with
// the radix passes: 7,000 35 and 51 us, 12,000 47 and 56 us, 16,384 55.5 and 56.5
// us, where the line lies.  Batches do better with the LDS sort from kRankPairs pairs on: 4 renders
// of 3,000 items 30 and 34 us, 4 of 8,000 54 and 53 us, 8 of 5,000 53 and 49 us
// (and the radix passes 4 of 8,000 59 us, 16 of 8,192 82 against 72 us).
constexpr int kRankWaves = 16;

// n += the number of k's components that are below key (kEqual: or equal).
// (The masks of four compares at once: used straight after its compare, a mask
// takes wait states.)
template <bool kEqual>
__device__ __forceinline__ void count4(uint32_t& n, uint32_t key, const uint4& k) {
  uint64_t a, b, c, d;
  if (kEqual)
    asm("v_cmp_ge_u32_e64 %1, %5, %6\n\tv_cmp_ge_u32_e64 %2, %5, %7\n\t"
        "v_cmp_ge_u32_e64 %3, %5, %8\n\tv_cmp_ge_u32_e64 %4, %5, %9\n\t"
        "v_addc_co_u32_e64 %0, %1, %0, 0, %1\n\tv_addc_co_u32_e64 %0, %2, %0, 0, %2\n\t"
        "v_addc_co_u32_e64 %0, %3, %0, 0, %3\n\tv_addc_co_u32_e64 %0, %4, %0, 0, %4"
        : "+v"(n), "=&s"(a), "=&s"(b), "=&s"(c), "=&s"(d)
        : "v"(key), "v"(k.x), "v"(k.y), "v"(k.z), "v"(k.w));
  else
    asm("v_cmp_gt_u32_e64 %1, %5, %6\n\tv_cmp_gt_u32_e64 %2, %5, %7\n\t"
        "v_cmp_gt_u32_e64 %3, %5, %8\n\tv_cmp_gt_u32_e64 %4, %5, %9\n\t"
        "v_addc_co_u32_e64 %0, %1, %0, 0, %1\n\tv_addc_co_u32_e64 %0, %2, %0, 0, %2\n\t"
        "v_addc_co_u32_e64 %0, %3, %0, 0, %3\n\tv_addc_co_u32_e64 %0, %4, %0, 0, %4"
        : "+v"(n), "=&s"(a), "=&s"(b), "=&s"(c), "=&s"(d)
        : "v"(key), "v"(k.x), "v"(k.y), "v"(k.z), "v"(k.w));
}

// Those of keys[lo] .. keys[hi), a multiple of 64 of them, 64 in flight.
template <bool kEqual>
__device__ __forceinline__ void count_keys(uint32_t& n, uint32_t key, const uint32_t* keys, int lo, int hi) {
  for (int i = lo; i < hi; i += 64) {
    uint4 k[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) k[j] = reinterpret_cast<const uint4*>(keys + i)[j];
#pragma unroll
    for (int j = 0; j < 16; ++j) count4<kEqual>(n, key, k[j]);
  }
}

template <int kItems>
__global__ __launch_bounds__(64 * kRankWaves) void k_depth_rank(const JobDev* __restrict__ jobs, SegTable seg,
                                                                const int32_t* __restrict__ off256,
                                                                const float4* __restrict__ rec,
                                                                const int32_t* __restrict__ tiles,
                                                                uint32_t* __restrict__ order) {
  constexpr int kThreads = 64 * kRankWaves;
  constexpr uint32_t kNone = 0xFFFFFFFFu;
  __shared__ __attribute__((aligned(16))) uint32_t keys[kItems];
  __shared__ uint32_t part[kRankWaves][64];
  __shared__ int kept[kRankWaves];
  const int blk = blockIdx.x >> 2, s = find_segment<int32_t>(off256, seg.S, blk);
  const int q0 = (blk - off256[s]) * 256 + (blockIdx.x & 3) * 64, n = jobs[s].n;
  if (q0 >= n) return;  // uniform for the block
  const int64_t base = seg.base[s];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int padded = (n + kThreads - 1) / kThreads * kThreads;
  int valid = 0;
  for (int i0 = 0; i0 < padded; i0 += 4 * kThreads) {
    bool ok[4];
    uint32_t z[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int i = i0 + j * kThreads + threadIdx.x;
      ok[j] = i < n && tiles[base + i] > 0;
      valid += (int)__popcll(__ballot(ok[j]));
    }
#pragma unroll
    for (int j = 0; j < 4; ++j)
      z[j] = ok[j] ? min(__float_as_uint(rec[(base + i0 + j * kThreads + threadIdx.x) * 3 + 1].z), kNone - 1u) : kNone;
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (i0 + j * kThreads < padded) keys[i0 + j * kThreads + threadIdx.x] = z[j];
  }
  if (lane == 0) kept[w] = valid;
  __syncthreads();
  if (q0 == 0 && threadIdx.x == 0) {
    int all = 0;
    for (int k = 0; k < kRankWaves; ++k) all += kept[k];
    seg.len[s] = all;
  }
  const uint32_t key = keys[q0 + lane];
  if (__syncthreads_or(key != kNone) == 0) return;
  // this wave's share, in fours; equal keys keep their order, so those of an
  // earlier place count as smaller, and the block's own 64 are compared by place
  const int per = padded / kRankWaves, lo = w * per, hi = lo + per;
  const int a = min(max(q0, lo), hi), b = max(min(q0 + 64, hi), a);
  uint32_t below = 0;
  count_keys<true>(below, key, keys, lo, a);
  for (int i = a; i < b; i += 4) {
    const uint4 k = *reinterpret_cast<const uint4*>(keys + i);
    const int at = q0 + lane - i;
    below += k.x < key + (at > 0 ? 1u : 0u) ? 1u : 0u;
    below += k.y < key + (at > 1 ? 1u : 0u) ? 1u : 0u;
    below += k.z < key + (at > 2 ? 1u : 0u) ? 1u : 0u;
    below += k.w < key + (at > 3 ? 1u : 0u) ? 1u : 0u;
  }
  count_keys<false>(below, key, keys, b, hi);
  part[w][lane] = below;
  __syncthreads();
  if (w == 0 && key != kNone) {
    uint32_t rank = 0;
#pragma unroll
    for (int k = 0; k < kRankWaves; ++k) rank += part[k][lane];
    order[base + rank] = (uint32_t)(base + q0 + lane);
  }
}

// Batches of small renders, where comparing all pairs would take longer: one
// block sorts a whole render of up to kPer * 1,024 items in LDS, three passes of
// ranks, digit starts and LDS moves, each a chain of barriers (4,096 items 16
// us, eight renders of 5,000 20 us, and 24 us by comparison).
template <int kBits, int kPer>
__global__ __launch_bounds__(kSortThreads) void k_depth_sort_small(const JobDev* __restrict__ jobs, SegTable seg,
                                                                   const float4* __restrict__ rec,
                                                                   const int32_t* __restrict__ tiles,
                                                                   uint32_t* __restrict__ order) {
  using D = Digit<kBits>;
  __shared__ __attribute__((aligned(4))) uint16_t wcnt[kSortWaves][D::kBins];
  __shared__ uint32_t sk[kPer * kSortThreads], sv[kPer * kSortThreads];
  __shared__ uint32_t wsum[kSortWaves];
  __shared__ uint32_t kept;
  const int s = blockIdx.x;
  const int n = jobs[s].n, lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t base = jobs[s].item_off;
  uint32_t key[kPer], val[kPer], rk[kPer];
  bool ok[kPer];
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const int i = w * 64 * kPer + j * 64 + lane;
    ok[j] = i < n && tiles[base + i] > 0;
    val[j] = (uint32_t)(base + i);
  }
#pragma unroll
  for (int j = 0; j < kPer; ++j) key[j] = ok[j] ? __float_as_uint(rec[(int64_t)val[j] * 3 + 1].z) : 0u;
  int m = 0;
#pragma unroll 1
  for (int shift = 0; shift < 32; shift += kBits) {
    wave_ranks<kBits, kPer>(key, ok, shift, D::kBins - 1, wcnt[w], lane, rk);
    __syncthreads();
    uint32_t lstart[D::kPer];
    const uint32_t upto = digit_starts<kBits>(wcnt, wsum, lstart);
    if (threadIdx.x == D::kThreads - 1) kept = upto;
    __syncthreads();
    m = (int)kept;
#pragma unroll
    for (int j = 0; j < kPer; ++j)
      if (ok[j]) {
        const uint32_t pos = wcnt[w][D::of(key[j], shift)] + rk[j];
        sk[pos] = key[j];
        sv[pos] = val[j];
      }
    __syncthreads();
    if (shift + kBits < 32)
#pragma unroll
      for (int j = 0; j < kPer; ++j) {
        const int i = w * 64 * kPer + j * 64 + lane;
        ok[j] = i < m;
        key[j] = ok[j] ? sk[i] : 0u;
        val[j] = ok[j] ? sv[i] : 0u;
      }
  }
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const int i = j * kSortThreads + threadIdx.x;
    if (i < m) order[base + i] = sv[i];
  }
  if (threadIdx.x == 0) seg.len[s] = m;
}

// ---------------------------------------------------------------------------
// Distribution over the tiles.  A block works on one chunk of a render's
// sorted items and one window of its tiles (at most kWindowTiles; the whole
// image up to 1,024 x 1,024 or 1200 x 680 pixels), kPlaceItems items at a
// time, and a thread on a few tiles of the window.  For 64 items (a wave) the
// items that reach a tile are a 64-bit word: those that reach its row and its
// column, and the words of the window's rows and columns are transposed line
// masks.  So a tile counts its items with a population count and lists them in
// depth order by walking its words, with no atomics and no matter how large
// the items' rectangles are.  Measured for 1.6 M instances of 200k items:
// counts 13 us and lists 27 us (LDS atomics per (item, tile), balanced over
// items: 81 and 249 us; words by a ballot per line: 20 and 29 us).  Windows of
// 1,024 tiles instead repeat the words: 21 and 33 us.

constexpr int kWindowSide = 256;    // most tiles of a window's row
constexpr int kPlaceThreads = 1024;
constexpr int kPlaceItems = 512;
constexpr int kPlaceGroups = kPlaceItems / 64;
constexpr int kPlaceTiles = kWindowTiles / kPlaceThreads;  // tiles per thread
static_assert(2 * kPlaceGroups * 64 == kPlaceThreads, "a wave per group for the rows and one for the columns");

struct Window {
  int w, h, nx, ny;  // a window's tiles, windows per row and column
};
__host__ __device__ inline Window window_of(int TX, int TY) {
  Window o;
  o.w = TX < kWindowSide ? TX : kWindowSide;
  o.h = kWindowTiles / o.w < TY ? kWindowTiles / o.w : TY;
  o.h = o.h < kWindowSide ? o.h : kWindowSide;
  o.nx = (TX + o.w - 1) / o.w;
  o.ny = (TY + o.h - 1) / o.h;
  return o;
}
int windows_of(int TX, int TY) {
  const Window w = window_of(TX, TY);
  return w.nx * w.ny;
}

// Chunks hold `chunk` items.  The nearest items cover the most tiles; with
// `ramp` a render's first chunks are therefore cut finer, 64 items (16 chunks),
// then 128 and 256 (16 chunks each), so that no block writes many times the
// others' instances (k_place: 200k items 92 -> 29 us, 4 renders of 21k and 17k
// items 17 -> 14 us).  A batch of more than 560 chunks fills the CUs as it is,
// and finer chunks only add counts to scan (16 renders of 150k and 120k items:
// counts and lists 104 us without, 121 us with; 8 of 150k 53 and 66 us).
constexpr int kRamp = 16 * (64 + 128 + 256);
__host__ __device__ inline int chunk_first(int c, int chunk, bool ramp) {
  if (!ramp) return chunk * c;
  return c < 16 ? 64 * c : c < 32 ? 1024 + 128 * (c - 16) : c < 48 ? 3072 + 256 * (c - 32) : kRamp + chunk * (c - 48);
}
__host__ __device__ inline int chunks_of(int n, int chunk, bool ramp) {
  if (!ramp) return (n + chunk - 1) / chunk;
  return n <= 1024 ? (n + 63) / 64
         : n <= 3072 ? 16 + (n - 1024 + 127) / 128
         : n <= kRamp ? 32 + (n - 3072 + 255) / 256 : 48 + (n - kRamp + chunk - 1) / chunk;
}
int bin_chunks(int n, int chunk, bool ramp) { return chunks_of(n, chunk, ramp); }

struct PlaceCtx {
  int r, chunk, x0, y0, w, h;  // render, chunk, window in tiles
  int first, n;                // the chunk's items
};

// Block -> work unit: neighbouring chunks, whose instances are neighbours in
// the lists, on one XCD.  A single render's units are mapped over those that
// have items, so that all XCDs work.
__device__ __forceinline__ int place_unit(const BinTables& t, const JobDev* jobs, const int32_t* kept, int units) {
  if (t.R > 1) return (int)blockIdx.x < 8 * ((units + 7) / 8) ? xcd_remap(blockIdx.x, units) : units;
  const int busy = units > 0 ? chunks_of(kept[0], t.chunk, true) * (units / chunks_of(jobs[0].n, t.chunk, true)) : 0;
  const int u = xcd_remap(blockIdx.x, busy);
  return u < busy && (int)blockIdx.x < 8 * ((busy + 7) / 8) ? u : units;
}

__device__ __forceinline__ bool place_ctx(const JobDev* jobs, const BinTables& t, const int32_t* kept, int unit,
                                          PlaceCtx& c) {
  c.r = find_segment<int32_t>(t.work_off, t.R, unit);
  const JobDev& J = jobs[c.r];
  const Window win = window_of(J.TX, J.TY);
  const int nw = win.nx * win.ny, local = unit - t.work_off[c.r];
  c.chunk = local / nw;
  const int k = local - c.chunk * nw, wy = k / win.nx;
  c.x0 = (k - wy * win.nx) * win.w;
  c.y0 = wy * win.h;
  c.w = min(win.w, J.TX - c.x0);
  c.h = min(win.h, J.TY - c.y0);
  c.first = chunk_first(c.chunk, t.chunk, t.ramp);
  c.n = min(kept[c.r], chunk_first(c.chunk + 1, t.chunk, t.ramp)) - c.first;
  return c.n > 0;
}

struct PlaceLds {
  uint64_t row[kPlaceGroups][kWindowSide];  // per 64 items and window row: the items that reach it
  uint64_t col[kPlaceGroups][kWindowSide];
  uint32_t id[kPlaceItems];
};

// The lowest k bits (none for k <= 0, all for k >= 64).
__device__ __forceinline__ uint64_t bits_below(int k) {
  return k <= 0 ? 0ull : k >= 64 ? ~0ull : (1ull << k) - 1ull;
}

// One step of the bit transpose: blocks of kStep x kStep bits change places
// with the lane kStep away.
template <int kStep>
__device__ __forceinline__ uint32_t transpose_step(uint32_t v, uint32_t low) {
  const bool up = (threadIdx.x & kStep) != 0;
  const uint32_t o = (uint32_t)__builtin_amdgcn_ds_swizzle((int)v, (kStep << 10) | 0x1F);
  return up ? (v & ~low) | ((o >> kStep) & low) : (v & low) | ((o & low) << kStep);
}

// Bit k of lane l's word becomes bit l of lane k's: the items' line masks
// turned into the lines' item masks, 70 instructions against 8 per line with a
// ballot each.
__device__ __forceinline__ uint64_t transpose64(uint64_t v) {
  const auto r = __builtin_amdgcn_permlane32_swap((uint32_t)v, (uint32_t)(v >> 32), false, false);
  uint32_t w[2] = {r[0], r[1]};
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    w[i] = transpose_step<16>(w[i], 0x0000FFFFu);
    w[i] = transpose_step<8>(w[i], 0x00FF00FFu);
    w[i] = transpose_step<4>(w[i], 0x0F0F0F0Fu);
    w[i] = transpose_step<2>(w[i], 0x33333333u);
    w[i] = transpose_step<1>(w[i], 0x55555555u);
  }
  return ((uint64_t)w[1] << 32) | w[0];
}

// The row and column words (and item ids) of n <= kPlaceItems sorted items.
// Wave g < kPlaceGroups takes the rows of items 64 g .., wave kPlaceGroups + g
// their columns.  Ends with a barrier.
__device__ __forceinline__ void window_words(PlaceLds& L, const JobDev& J, const PlaceCtx& c,
                                             const uint32_t* __restrict__ ord, int n,
                                             const float4* __restrict__ rec, const int32_t* __restrict__ radius) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, g = w & (kPlaceGroups - 1), i = 64 * g + lane;
  if (64 * g < n) {
    int lo = 0, hi = 0;  // this item's first and past-the-last row (column) in the window
    if (i < n) {
      const uint32_t it = ord[i];
      const float2 uv = *reinterpret_cast<const float2*>(rec + (int64_t)it * 3);
      const Rect rc = tile_rect(uv.x, uv.y, radius[it], J.TX, J.TY);
      const bool any = rc.x1 > rc.x0 && rc.y1 > rc.y0;
      if (w < kPlaceGroups) {
        L.id[i] = it;
        lo = rc.y0 - c.y0;
        hi = any ? rc.y1 - c.y0 : lo;
      } else {
        lo = rc.x0 - c.x0;
        hi = any ? rc.x1 - c.x0 : lo;
      }
    }
    uint64_t* out = w < kPlaceGroups ? L.row[g] : L.col[g];
    const int len = w < kPlaceGroups ? c.h : c.w;
    for (int k0 = 0; k0 < len; k0 += 64) {
      const uint64_t word = transpose64(bits_below(hi - k0) & ~bits_below(lo - k0));
      if (k0 + lane < len) out[k0 + lane] = word;
    }
  }
  __syncthreads();
}

// Items of the chunk per tile: cnt[chunk][tile of the render].
__global__ __launch_bounds__(kPlaceThreads) void k_chunk_count(const JobDev* __restrict__ jobs, BinTables t,
                                                               int units, const int32_t* __restrict__ kept,
                                                               const uint32_t* __restrict__ order,
                                                               const float4* __restrict__ rec,
                                                               const int32_t* __restrict__ radius,
                                                               uint32_t* __restrict__ cnt) {
  __shared__ PlaceLds L;
  const int unit = place_unit(t, jobs, kept, units);
  if (unit >= units) return;
  PlaceCtx c;
  if (!place_ctx(jobs, t, kept, unit, c)) return;  // uniform
  const JobDev& J = jobs[c.r];
  const int nt = c.w * c.h;
  const uint32_t* __restrict__ ord = order + J.item_off + c.first;
  uint32_t v[kPlaceTiles];
#pragma unroll
  for (int j = 0; j < kPlaceTiles; ++j) v[j] = 0u;
  for (int i0 = 0; i0 < c.n; i0 += kPlaceItems) {
    const int n = min(c.n - i0, kPlaceItems);
    if (i0 > 0) __syncthreads();
    window_words(L, J, c, ord + i0, n, rec, radius);
#pragma unroll
    for (int j = 0; j < kPlaceTiles; ++j) {
      const int k = j * kPlaceThreads + threadIdx.x;
      if (k < nt) {
        const int y = k / c.w, x = k - y * c.w;
        for (int g = 0; 64 * g < n; ++g) v[j] += (uint32_t)__popcll(L.row[g][y] & L.col[g][x]);
      }
    }
  }
  uint32_t* __restrict__ row = cnt + t.cnt_off[c.r] + (int64_t)c.chunk * (J.TX * J.TY);
#pragma unroll
  for (int j = 0; j < kPlaceTiles; ++j) {
    const int k = j * kPlaceThreads + threadIdx.x, y = k / c.w;
    if (k < nt) row[(c.y0 + y) * J.TX + c.x0 + (k - y * c.w)] = v[j];
  }
}

// Per tile: the chunks' counts turned into exclusive prefixes, the total, and
// the totals of the tiles before it in its group of 64 (at most 2^32 - 1); per
// group the sum of the totals.  16 threads per tile, each a run of chunks.
__global__ __launch_bounds__(1024) void k_chunk_scan(const JobDev* __restrict__ jobs, BinTables t,
                                                     const int32_t* __restrict__ tile_off, int T,
                                                     const int32_t* __restrict__ kept, uint32_t* __restrict__ cnt,
                                                     uint32_t* __restrict__ total, uint32_t* __restrict__ before,
                                                     uint64_t* __restrict__ blk_total) {
  constexpr int kParts = 16, kRun = 32;
  __shared__ uint32_t sums[kParts][64];
  const int tile = blockIdx.x * 64 + (threadIdx.x & 63), p = threadIdx.x >> 6;
  const bool in = tile < T;
  const int r = find_segment<int32_t>(tile_off, t.R, in ? tile : T - 1);
  const JobDev& J = jobs[r];
  const int nt = J.TX * J.TY;
  const int rows = J.n > 0 ? chunks_of(kept[r], t.chunk, t.ramp) : 0;
  const int per = (rows + kParts - 1) / kParts;
  const int lo = min(p * per, rows), hi = in ? min(lo + per, rows) : lo;
  uint32_t* __restrict__ col = cnt + t.cnt_off[r] + (in ? tile - J.tile_off : 0);
  uint32_t v[kRun], s = 0;
#pragma unroll
  for (int k = 0; k < kRun; ++k) {
    v[k] = lo + k < hi ? col[(int64_t)(lo + k) * nt] : 0u;
    s += v[k];
  }
  for (int k = lo + kRun; k < hi; ++k) s += col[(int64_t)k * nt];
  sums[p][threadIdx.x & 63] = s;
  __syncthreads();
  uint32_t run = 0, all = 0;
#pragma unroll
  for (int k = 0; k < kParts; ++k) {
    const uint32_t x = sums[k][threadIdx.x & 63];
    run += k < p ? x : 0u;
    all += x;
  }
#pragma unroll
  for (int k = 0; k < kRun; ++k)
    if (lo + k < hi) {
      col[(int64_t)(lo + k) * nt] = run;
      run += v[k];
    }
  for (int k = lo + kRun; k < hi; ++k) {
    const uint32_t x = col[(int64_t)k * nt];
    col[(int64_t)k * nt] = run;
    run += x;
  }
  if (p == 0) {
    const uint64_t mine = in ? all : 0u;
    uint64_t sum = mine;  // inclusive over the lanes
    for (int off = 1; off < 64; off <<= 1) {
      const uint64_t y = __shfl_up(sum, off, 64);
      if ((int)threadIdx.x >= off) sum += y;
    }
    if (in) {
      total[tile] = all;
      before[tile] = (uint32_t)min(sum - mine, (uint64_t)UINT32_MAX);
    }
    if (threadIdx.x == 63) blk_total[blockIdx.x] = sum;
  }
}

// Where each group of 64 tiles starts in the lists: the groups' sums turned
// into exclusive prefixes; the whole sum into all[0].  One block.
__global__ __launch_bounds__(1024) void k_group_starts(uint64_t* __restrict__ group, int n,
                                                       uint64_t* __restrict__ all) {
  __shared__ uint64_t wsum[16];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  uint64_t base = 0;
  for (int i0 = 0; i0 < n; i0 += 1024) {
    const int i = i0 + threadIdx.x;
    const uint64_t mine = i < n ? group[i] : 0ull;
    uint64_t x = mine;
    for (int off = 1; off < 64; off <<= 1) {
      const uint64_t y = __shfl_up(x, off, 64);
      if (lane >= off) x += y;
    }
    if (lane == 63) wsum[w] = x;
    __syncthreads();
    uint64_t run = base + x - mine;
    for (int k = 0; k < 16; ++k) {
      run += k < w ? wsum[k] : 0ull;
      base += wsum[k];
    }
    if (i < n) group[i] = run;
    __syncthreads();
  }
  if (threadIdx.x == 0) all[0] = base;
}

// The lists' table, a share of the tiles per block: every tile's [start, end)
// (clamped to the capacity; empty tiles 0, 0) and tile_of, eight tiles to a
// wave, in whole lines; and count = {min(I, cap), I > cap, min(I, INT32_MAX),
// 0}.  start, total: where a tile's list starts and its length.
template <class Start, class Total>
__device__ __forceinline__ void list_table(const Start& start, const Total& total, uint64_t all, int T, uint64_t cap,
                                           uint32_t* __restrict__ tile_of, int32_t* __restrict__ range,
                                           int32_t* __restrict__ count) {
  const int lane = threadIdx.x & 63;
  for (int k = blockIdx.x + (threadIdx.x >> 6) * gridDim.x; 8 * k < T; k += gridDim.x * (kPlaceThreads / 64)) {
    const int tile = 8 * k + lane;
    uint64_t a = 0, e = 0;
    if (lane < 8 && tile < T) {
      a = start(tile);
      e = min(a + total(tile), cap);
      a = min(a, cap);
      range[2 * tile] = a < e ? (int32_t)a : 0;
      range[2 * tile + 1] = a < e ? (int32_t)e : 0;
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)a, j);
      const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)e, j);
      for (uint32_t i = lo + lane; i < hi; i += 64) tile_of[i] = (uint32_t)(8 * k + j);
    }
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    count[0] = (int32_t)min(all, cap);
    count[1] = all > cap ? 1 : 0;
    count[2] = (int32_t)min(all, (uint64_t)INT32_MAX);
    count[3] = 0;
  }
}

// Exclusive prefixes of the n <= kFewGroups group sums in LDS, by one block of
// 1,024 threads; returns the whole sum.
__device__ __forceinline__ uint64_t group_starts(const uint64_t* __restrict__ group, int n, uint64_t* out) {
  __shared__ uint64_t wsum[16];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const uint64_t mine = (int)threadIdx.x < n ? group[threadIdx.x] : 0ull;
  uint64_t x = mine;
  for (int off = 1; off < 64; off <<= 1) {
    const uint64_t y = __shfl_up(x, off, 64);
    if (lane >= off) x += y;
  }
  if (lane == 63) wsum[w] = x;
  __syncthreads();
  uint64_t run = x - mine, all = 0;
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    run += k < w ? wsum[k] : 0ull;
    all += wsum[k];
  }
  out[threadIdx.x] = run;
  __syncthreads();
  return all;
}

// The instances of a chunk, written to their places: every tile lists the
// chunk's items that reach it, from the tile's start plus the earlier chunks'
// count on.  A thread walks all words of its tile as one sequence, so a wave
// takes as many steps as its fullest tile has items.  A scattered store costs a
// CU about a clock per lane, so tile_of is left to list_table.
//
// kFew: up to kFewGroups groups of 64 tiles, whose starts every block works out
// for itself from the groups' sums; a launch for it and for the table took 3 to
// 5 us.  More come from k_group_starts (kMany).  kOwn: a single render of up to
// kPlaceThreads tiles whose counts, up to kOwnCounts, every block scans for
// itself in one to four rounds of loads (4,096 items at 160 x 120, 2,800 counts:
// 4.2 us for k_chunk_scan against 1.1 us here; 23k items at 317 x 211, 22k
// counts: 5.0 against 2.1 us).
constexpr int kFewGroups = kPlaceThreads;
constexpr int kOwnCounts = 32768;
enum PlaceStarts { kMany, kFew, kOwn };

// kOwn: the tiles' totals over all chunks and over those before `chunk`, and
// the tiles' starts, by the whole block; returns the sum of the totals.
struct OwnScan {
  uint32_t total[kPlaceThreads], before[kPlaceThreads], start[kPlaceThreads];
};
__device__ __forceinline__ uint32_t own_scan(OwnScan& o, const uint32_t* __restrict__ cnt, int T, int rows, int chunk) {
  __shared__ uint32_t wsum[kPlaceThreads / 64];
  const int parts = kPlaceThreads / T, part = threadIdx.x / T, tile = threadIdx.x - part * T;
  uint32_t all = 0, pre = 0;
  if (part < parts)
    for (int r0 = part; r0 < rows; r0 += 16 * parts) {
      uint32_t v[16];
#pragma unroll
      for (int k = 0; k < 16; ++k) v[k] = r0 + k * parts < rows ? cnt[(r0 + k * parts) * T + tile] : 0u;
#pragma unroll
      for (int k = 0; k < 16; ++k) {
        all += v[k];
        pre += r0 + k * parts < chunk ? v[k] : 0u;
      }
    }
  o.total[threadIdx.x] = all;
  o.before[threadIdx.x] = pre;
  __syncthreads();
  all = pre = 0u;
  if ((int)threadIdx.x < T)
    for (int k = 0; k < parts; ++k) {
      all += o.total[k * T + threadIdx.x];
      pre += o.before[k * T + threadIdx.x];
    }
  const int w = threadIdx.x >> 6;
  const uint32_t x = wave_incl_sum(all);
  if ((threadIdx.x & 63) == 63) wsum[w] = x;
  __syncthreads();
  uint32_t run = x - all, sum = 0;
#pragma unroll
  for (int k = 0; k < kPlaceThreads / 64; ++k) {
    run += k < w ? wsum[k] : 0u;
    sum += wsum[k];
  }
  o.total[threadIdx.x] = all;
  o.before[threadIdx.x] = pre;
  o.start[threadIdx.x] = run;
  __syncthreads();
  return sum;
}

template <PlaceStarts kStarts>
__global__ __launch_bounds__(kPlaceThreads) void k_place(const JobDev* __restrict__ jobs, BinTables t, int units,
                                                         const int32_t* __restrict__ kept,
                                                         const uint32_t* __restrict__ order,
                                                         const float4* __restrict__ rec,
                                                         const int32_t* __restrict__ radius,
                                                         const uint32_t* __restrict__ cnt,
                                                         const uint32_t* __restrict__ total,
                                                         const uint32_t* __restrict__ before,
                                                         const uint64_t* __restrict__ group, int T, uint32_t cap,
                                                         uint32_t* __restrict__ tile_of, int32_t* __restrict__ item,
                                                         int32_t* __restrict__ range, int32_t* __restrict__ count) {
  __shared__ PlaceLds L;
  __shared__ uint64_t starts[kStarts == kFew ? kFewGroups : 1];
  __shared__ OwnScan own[1];
  const int ngroup = (T + 63) / 64;
  PlaceCtx c;
  bool work;  // uniform
  auto find_work = [&] {
    const int unit = place_unit(t, jobs, kept, units);
    work = unit < units && place_ctx(jobs, t, kept, unit, c);
  };
  uint64_t all;
  if (kStarts == kOwn) {
    find_work();
    all = own_scan(own[0], cnt, T, chunks_of(kept[0], t.chunk, t.ramp), work ? c.chunk : 0);
  } else {
    all = kStarts == kFew ? group_starts(group, ngroup, starts) : group[ngroup];
  }
  auto start_of = [&](int tile) {
    return kStarts == kOwn ? (uint64_t)own[0].start[tile]
                           : (kStarts == kFew ? starts[tile >> 6] : group[tile >> 6]) + before[tile];
  };
  auto total_of = [&](int tile) { return kStarts == kOwn ? own[0].total[tile] : total[tile]; };
  // (first: at the end it is every block's tail, 29 -> 36 us at 200k items)
  list_table(start_of, total_of, all, T, cap, tile_of, range, count);
  if (kStarts != kOwn) find_work();
  if (!work) return;
  const JobDev& J = jobs[c.r];
  const int nt = c.w * c.h;
  const uint32_t* __restrict__ ord = order + J.item_off + c.first;
  const uint32_t* __restrict__ row = cnt + t.cnt_off[c.r] + (int64_t)c.chunk * (J.TX * J.TY);
  uint32_t place[kPlaceTiles];
#pragma unroll
  for (int j = 0; j < kPlaceTiles; ++j) {
    const int k = j * kPlaceThreads + threadIdx.x, y = k / c.w, rt = (c.y0 + y) * J.TX + c.x0 + (k - y * c.w);
    const int tile = J.tile_off + rt;
    const uint32_t earlier = k >= nt ? 0u : kStarts == kOwn ? own[0].before[tile] : row[rt];
    place[j] = k < nt ? (uint32_t)min(start_of(tile), (uint64_t)cap) + earlier : 0u;
  }
  for (int i0 = 0; i0 < c.n; i0 += kPlaceItems) {
    const int n = min(c.n - i0, kPlaceItems);
    if (i0 > 0) __syncthreads();
    window_words(L, J, c, ord + i0, n, rec, radius);
#pragma unroll
    for (int j = 0; j < kPlaceTiles; ++j) {
      const int k = j * kPlaceThreads + threadIdx.x;
      if (k < nt) {
        const int y = k / c.w, x = k - y * c.w;
        uint32_t any = 0u;  // groups with items here
#pragma unroll
        for (int g = 0; g < kPlaceGroups; ++g)
          if (64 * g < n) any |= (L.row[g][y] & L.col[g][x]) != 0ull ? 1u << g : 0u;
        uint32_t at = place[j];
        int g = 0;
        uint64_t bits = 0ull;
        while (bits != 0ull || any != 0u) {
          if (bits == 0ull) {
            g = (int)__builtin_ctz(any);
            any &= any - 1u;
            bits = L.row[g][y] & L.col[g][x];
          }
          const int e = (int)__builtin_ctzll(bits);
          bits &= bits - 1ull;
          if (at < cap) item[at] = (int32_t)L.id[64 * g + e];
          ++at;
        }
        place[j] = at;
      }
    }
  }
}

}  // namespace ls

namespace ls {
void launch_fill_i32(int32_t* p, int64_t n, int32_t v, hipStream_t s) {
  if (n <= 0) return;
  const int64_t blocks = std::min<int64_t>((n + 255) / 256, 4096);
  hipLaunchKernelGGL(k_fill_i32, dim3((unsigned)blocks), dim3(256), 0, s, p, n, v);
}

// The scan of a pass whose largest segment has `rows` blocks, if that is worth it;
// returns the digit totals for the scatter, or NULL.
template <int kPer, bool kFirst>
static const uint32_t* seg_scan(const SegTable& seg, int blocks, int rows, uint32_t* hist, hipStream_t s) {
  if (rows <= kScanRows) return nullptr;
  uint32_t* sums = hist + (int64_t)kHistRow * blocks;
  hipLaunchKernelGGL((k_seg_scan<kPer, kFirst>), dim3(Digit<kSortBits>::kBins / kScanDigits * seg.S), dim3(1024), 0, s,
                     seg, hist, sums);
  return sums;
}

template <int kPer>
static void seg_pass(const uint32_t* kin, const uint32_t* vin, uint32_t* kout, uint32_t* vout, const SegTable& seg,
                     int blocks, int rows, int shift, int bits, uint32_t* hist, bool last, hipStream_t s) {
  const dim3 grid(blocks), block(kSortThreads);
  const uint32_t mask = (1u << bits) - 1u;
  hipLaunchKernelGGL(k_seg_hist<kPer>, grid, block, 0, s, kin, seg, shift, mask, hist);
  const uint32_t* sums = seg_scan<kPer, false>(seg, blocks, rows, hist, s);
  const int32_t* none = nullptr;
  auto scatter = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, block, 0, s, kin, vin, kout, vout, seg, shift, mask, (const uint32_t*)hist, none,
                       sums);
  };
  if (last)
    scatter(k_seg_scatter<kPer, false, true>);
  else
    scatter(k_seg_scatter<kPer, false, false>);
}

// The depth sort of larger renders; the order ends in v0.
template <int kPer>
static void depth_passes(const BinLaunch& b, const SegTable& seg, hipStream_t s) {
  const dim3 grid(b.sort_blocks), block(kSortThreads);
  const int rows = sort_blocks_of(b.max_items, kPer);
  hipLaunchKernelGGL(k_depth_prep<kPer>, grid, block, 0, s, b.jobs, seg, reinterpret_cast<const float4*>(b.rec),
                     b.tiles, b.k0, b.v0, b.hist, b.blk_cnt);
  const uint32_t* sums = seg_scan<kPer, true>(seg, b.sort_blocks, rows, b.hist, s);
  hipLaunchKernelGGL((k_seg_scatter<kPer, true, false>), grid, block, 0, s, (const uint32_t*)b.k0,
                     (const uint32_t*)b.v0, b.k1, b.v1, seg, 0, 255u, (const uint32_t*)b.hist,
                     (const int32_t*)b.blk_cnt, sums);
  seg_pass<kPer>(b.k1, b.v1, b.k0, b.v0, seg, b.sort_blocks, rows, 8, 8, b.hist, false, s);
  seg_pass<kPer>(b.k0, b.v0, b.k1, b.v1, seg, b.sort_blocks, rows, 16, 8, b.hist, false, s);
  seg_pass<kPer>(b.k1, b.v1, b.k0, b.v0, seg, b.sort_blocks, rows, 24, 8, b.hist, true, s);
}

void launch_bin_sort(const BinLaunch& b, hipStream_t s) {
  const float4* rec4 = reinterpret_cast<const float4*>(b.rec);
  const SegTable seg{b.tab.blk_off, b.item_off, b.tab.R, b.kept};
  const uint32_t* order = b.v0;
  const dim3 block(kSortThreads);
  if (b.max_items <= kRankItems && (b.tab.R == 1 || b.rank_pairs <= kRankPairs)) {
    auto rank = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, dim3(4 * b.blocks256), dim3(64 * kRankWaves), 0, s, b.jobs, seg, b.off256, rec4,
                         b.tiles, b.v0);
    };
    if (b.max_items <= 4096)
      rank(k_depth_rank<4096>);
    else
      rank(k_depth_rank<kRankItems>);
  } else if (b.max_items <= 8 * kSortThreads) {
    auto small = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, dim3(b.tab.R), block, 0, s, b.jobs, seg, rec4, b.tiles, b.v0);
    };
    if (b.max_items <= 4 * kSortThreads)
      small(k_depth_sort_small<11, 4>);
    else
      small(k_depth_sort_small<11, 8>);
  } else {
    const auto passes = b.sort_per == 1   ? depth_passes<1>
                        : b.sort_per == 2 ? depth_passes<2>
                        : b.sort_per == 3 ? depth_passes<3>
                                          : depth_passes<4>;
    passes(b, seg, s);
  }
  if (b.pairs.tk) {
    launch_bin_pairs(b, s);
    return;
  }
  const dim3 work(8 * ((b.units + 7) / 8));
  if (b.units > 0)
    hipLaunchKernelGGL(k_chunk_count, work, dim3(kPlaceThreads), 0, s, b.jobs, b.tab, b.units,
                       (const int32_t*)b.kept, order, rec4, b.radius, b.cnt);
  const int ngroup = (b.T + 63) / 64;
  const bool own = b.tab.R == 1 && b.T <= kPlaceThreads && b.counts <= kOwnCounts;
  if (!own)
    hipLaunchKernelGGL(k_chunk_scan, dim3(ngroup), dim3(1024), 0, s, b.jobs, b.tab, b.tile_off, b.T,
                       (const int32_t*)b.kept, b.cnt, b.tile_total, b.tile_before, b.groups);
  // at least a block per 1,024 tiles for the table
  const dim3 place(std::max(work.x, 8u * ((unsigned)b.T / 8192u + 1u)));
  auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, place, dim3(kPlaceThreads), 0, s, b.jobs, b.tab, b.units, (const int32_t*)b.kept,
                       order, rec4, b.radius, (const uint32_t*)b.cnt, (const uint32_t*)b.tile_total,
                       (const uint32_t*)b.tile_before, (const uint64_t*)b.groups, b.T, (uint32_t)b.cap, b.tile_of,
                       b.item, b.range, b.count);
  };
  if (own) {
    launch(k_place<kOwn>);
  } else if (ngroup <= kFewGroups) {
    launch(k_place<kFew>);
  } else {
    hipLaunchKernelGGL(k_group_starts, dim3(1), dim3(1024), 0, s, b.groups, ngroup, b.groups + ngroup);
    launch(k_place<kMany>);
  }
}

void launch_seg_pass(const uint32_t* kin, const uint32_t* vin, uint32_t* kout, uint32_t* vout, const SegTable& seg,
                     int blocks, int rows, int per, int shift, int bits, uint32_t* hist, bool last, hipStream_t s) {
  const auto pass = per == 1 ? seg_pass<1> : per == 2 ? seg_pass<2> : per == 3 ? seg_pass<3> : seg_pass<4>;
  pass(kin, vin, kout, vout, seg, blocks, rows, shift, bits, hist, last, s);
}
}  // namespace ls
