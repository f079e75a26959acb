// Opacity pruning of a submap after mapping (supplement, Implementation
// Details, submap update): every Gaussian whose opacity is below o_thre is
// removed and the others are compacted, in order, into new arrays.
//
// The keep test is taken on the stored FP32 logit against the FP32 rounding
// of logit(o_thre) (sigmoid is increasing), so it needs no transcendental and
// its decisions are reproducible: keep <=> logit >= tau (NaN is pruned).
//
// Per-tile keep counts, one block scanning the counts into tile offsets (and
// the total), then the scatter, which re-derives each item's rank within its
// tile from ballots and copies every component of the kept items; sets of up
// to 262,144 items leave the scan to the scatter.  Rows of the outputs are
// `count` floats apart, so they come out in the ls_gaussians layout for the new
// Gaussian count.  Bound by launches below 100k items and by the rows' bytes
// above (15 arrays, 42 rows, half kept: 200k 51 MB, 10.6 us at the rate of a
// large copy, 16.8 in all; 1M 254 MB, 53 and 75 us).
#include <algorithm>

#include "kernels.h"

namespace ls {

constexpr int kPruneThreads = 256;
// Items per thread: 4 for large sets; 1 below kPruneSmall items, so that a
// submap-sized set still spreads over more blocks than the GPU has CUs.
constexpr int kPruneSmall = 1 << 20;
__host__ __device__ constexpr int prune_tile(int rounds) { return kPruneThreads * rounds; }
// Up to kPruneOwn tiles every scatter block adds up the tile counts for itself
// and the scan is left out (15 arrays, 42 rows: 20k items 13.1 -> 11.2 us,
// 200k 23.2 -> 22.0; at 2,700 tiles the blocks read 30 MB of counts: 44 -> 47,
// so larger sets keep it).  The arrays are then dealt to as many blocks per
// tile as the chip holds at once (8 blocks on each of 256 CUs), two to five:
// a wave's rows are a chain of loads and stores.  2k items 11.1 -> 6.5 us, 20k
// 11.2 -> 6.7, 100k 15.0 -> 10.4 (five parts), 200k 22.0 -> 16.8 (two; three
// 20.3, five 18.6), 262k 22.5 -> 18.2 (two; five 22.5).
constexpr int kPruneOwn = 1024;
static int prune_parts(int tiles, int narrays) {
  return std::max(1, std::min(narrays, std::min(5, std::max(2, 2048 / tiles))));
}

__device__ __forceinline__ bool prune_keep(float w, float tau) { return w >= tau; }

template <int kPruneRounds>
__global__ __launch_bounds__(kPruneThreads) void k_prune_count(const float* __restrict__ logit, int n, float tau,
                                                               int32_t* __restrict__ tile_count) {
  const int64_t base = (int64_t)blockIdx.x * prune_tile(kPruneRounds);
  int c = 0;
#pragma unroll
  for (int r = 0; r < kPruneRounds; ++r) {
    const int64_t i = base + r * kPruneThreads + threadIdx.x;
    c += (i < n && prune_keep(logit[i], tau)) ? 1 : 0;
  }
  __shared__ int ws[kPruneThreads / 64];
  for (int off = 32; off > 0; off >>= 1) c += __shfl_xor(c, off, 64);
  if ((threadIdx.x & 63) == 0) ws[threadIdx.x >> 6] = c;
  __syncthreads();
  if (threadIdx.x == 0) tile_count[blockIdx.x] = (ws[0] + ws[1]) + (ws[2] + ws[3]);
}

// One block: exclusive scan of the tile counts into offsets, total to *count
// (sets of more than kPruneOwn tiles).
__global__ __launch_bounds__(1024) void k_prune_scan(const int32_t* __restrict__ tile_count, int ntiles,
                                                     int32_t* __restrict__ tile_off, int32_t* __restrict__ count) {
  __shared__ int32_t wsum[16];
  const int per = (ntiles + 1023) / 1024;
  const int b = threadIdx.x * per, e = min(b + per, ntiles);
  int32_t s = 0;
  for (int i = b; i < e; ++i) s += tile_count[i];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  int32_t x = s;
  for (int off = 1; off < 64; off <<= 1) {
    const int32_t y = __shfl_up(x, off, 64);
    if (lane >= off) x += y;
  }
  if (lane == 63) wsum[w] = x;
  __syncthreads();
  int32_t run = x - s;
  for (int k = 0; k < w; ++k) run += wsum[k];
  for (int i = b; i < e; ++i) {
    tile_off[i] = run;
    run += tile_count[i];
  }
  if (threadIdx.x == 1023) *count = run;
}

// kOwn: tile_off holds the tiles' counts, *count is written here, and the
// arrays are dealt to gridDim.y blocks.
template <int kPruneRounds, bool kOwn>
__global__ __launch_bounds__(kPruneThreads) void k_prune_scatter(const float* __restrict__ logit, int n, float tau,
                                                                 const int32_t* __restrict__ tile_off,
                                                                 int32_t* __restrict__ count, PruneArrays arr,
                                                                 int32_t* __restrict__ kept) {
  __shared__ int32_t wcnt[kPruneRounds][kPruneThreads / 64];
  __shared__ int2 wown[kPruneThreads / 64];
  const int64_t base = (int64_t)blockIdx.x * prune_tile(kPruneRounds);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const uint64_t below = lane == 0 ? 0ull : (~0ull >> (64 - lane));
  bool keep[kPruneRounds];
  int rank[kPruneRounds];
#pragma unroll
  for (int r = 0; r < kPruneRounds; ++r) {
    const int64_t i = base + r * kPruneThreads + threadIdx.x;
    keep[r] = i < n && prune_keep(logit[i], tau);
    const uint64_t m = __ballot(keep[r]);
    rank[r] = __popcll(m & below);
    if (lane == 0) wcnt[r][w] = __popcll(m);
  }
  if (kOwn) {
    int2 s = make_int2(0, 0);  // kept in the tiles before this one, and in all
    for (int i = threadIdx.x; i < (int)gridDim.x; i += kPruneThreads) {
      const int c = tile_off[i];
      s.x += i < (int)blockIdx.x ? c : 0;
      s.y += c;
    }
    for (int off = 32; off > 0; off >>= 1) {
      s.x += __shfl_xor(s.x, off, 64);
      s.y += __shfl_xor(s.y, off, 64);
    }
    if (lane == 0) wown[w] = s;
  }
  __syncthreads();
  const int total = kOwn ? (wown[0].y + wown[1].y) + (wown[2].y + wown[3].y) : count[0];
  if (kOwn && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *count = total;
  const int64_t stride = total;
  int64_t pos[kPruneRounds];
  int run = kOwn ? (wown[0].x + wown[1].x) + (wown[2].x + wown[3].x) : tile_off[blockIdx.x];
#pragma unroll
  for (int r = 0; r < kPruneRounds; ++r) {
    int before = run;
    for (int k = 0; k < w; ++k) before += wcnt[r][k];
    pos[r] = before + rank[r];
    if (keep[r] && blockIdx.y == 0) kept[pos[r]] = (int32_t)(base + r * kPruneThreads + threadIdx.x);
    run += (wcnt[r][0] + wcnt[r][1]) + (wcnt[r][2] + wcnt[r][3]);
  }
  // one row at a time: the four rounds' loads are issued before their stores
  for (int a = blockIdx.y; a < kPruneArrays; a += gridDim.y) {
    if (a >= arr.count) break;  // uniform
    const float* __restrict__ src = arr.src[a];
    float* __restrict__ dst = arr.dst[a];
    for (int c = 0; c < arr.comp[a]; ++c) {
      float v[kPruneRounds];
#pragma unroll
      for (int r = 0; r < kPruneRounds; ++r)
        v[r] = keep[r] ? src[(int64_t)c * n + base + r * kPruneThreads + threadIdx.x] : 0.f;
#pragma unroll
      for (int r = 0; r < kPruneRounds; ++r)
        if (keep[r]) dst[c * stride + pos[r]] = v[r];
    }
  }
}

static int prune_rounds(int n) { return n < kPruneSmall ? 1 : 4; }

size_t prune_workspace_bytes(int n) {
  const size_t tiles = (size_t)std::max((n + prune_tile(prune_rounds(n)) - 1) / prune_tile(prune_rounds(n)), 1);
  return 2 * ((4 * tiles + 255) & ~(size_t)255);
}

template <int kRounds>
static void launch_prune_rounds(const float* logit, int n, float tau, const PruneArrays& arr, int32_t* kept,
                                int32_t* count, void* work, hipStream_t s) {
  const int tiles = std::max((n + prune_tile(kRounds) - 1) / prune_tile(kRounds), 1);
  int32_t* tile_count = static_cast<int32_t*>(work);
  int32_t* tile_off = tile_count + (((4 * (size_t)tiles + 255) & ~(size_t)255) / 4);
  hipLaunchKernelGGL(k_prune_count<kRounds>, dim3(tiles), dim3(kPruneThreads), 0, s, logit, n, tau, tile_count);
  if (kRounds == 1 && tiles <= kPruneOwn) {
    hipLaunchKernelGGL((k_prune_scatter<kRounds, true>), dim3(tiles, prune_parts(tiles, arr.count)), dim3(kPruneThreads), 0, s, logit, n, tau,
                       (const int32_t*)tile_count, count, arr, kept);
    return;
  }
  hipLaunchKernelGGL(k_prune_scan, dim3(1), dim3(1024), 0, s, (const int32_t*)tile_count, tiles, tile_off, count);
  if (n > 0)
    hipLaunchKernelGGL((k_prune_scatter<kRounds, false>), dim3(tiles), dim3(kPruneThreads), 0, s, logit, n, tau,
                       (const int32_t*)tile_off, count, arr, kept);
}

void launch_prune(const float* logit, int n, float tau, const PruneArrays& arr, int32_t* kept, int32_t* count,
                  void* work, hipStream_t s) {
  if (prune_rounds(n) == 1)
    launch_prune_rounds<1>(logit, n, tau, arr, kept, count, work, s);
  else
    launch_prune_rounds<4>(logit, n, tau, arr, kept, count, work, s);
}

}  // namespace ls
