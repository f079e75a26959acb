// Geometric overlap ratio of two submaps (supplement, loop detection,
// Eq. 9): the fraction of reciprocal nearest-neighbour pairs between the
// Gaussian means of P, moved by an estimate of T_{P->Q}, and those of Q whose
// distance is below tau_1.
//
// Every nearest neighbour is exact: both point sets are sorted along a
// 30-bit Hilbert curve and cut into leaves of 16 points and superblocks of 64
// leaves, each with its bounding box.  A wave of 32 query points visits the
// candidate superblocks and leaves nearest box first and skips any box that is
// farther from every one of its points than that point's current best (with a
// margin over FP32 rounding), so no skipped point can win or tie.  Distances and the
// transform follow one fixed FP32 rounding sequence (no fused multiply-add)
// so that matches and ties are reproducible: d^2 = (dx^2 + dy^2) + dz^2,
// ties to the lower index.
#include <algorithm>
#include <cmath>
#include <mutex>
#include <vector>

#include "kernels.h"

namespace ls {

constexpr int kOvLeaf = 16;       // points per leaf
constexpr int kOvSuper = 64;      // leaves per superblock (one per lane of a wave)
constexpr int kOvQuery = 32;      // query points per wave, two lanes each
constexpr int kOvMany = 16;       // of 64 leaves: more are first tested against every query point
constexpr int kOvBoxBlocks = 256; // blocks of the bounding-box reduction
constexpr float kOvPrune = 1.f - 1e-5f;  // a box is skipped only if lb^2 * kOvPrune > bound

__device__ __forceinline__ float sq_dist_rn(float ax, float ay, float az, float bx, float by, float bz) {
#pragma clang fp contract(off)
  const float dx = ax - bx, dy = ay - by, dz = az - bz;
  return (dx * dx + dy * dy) + dz * dz;
}

__device__ __forceinline__ float wave_max_f(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}
__device__ __forceinline__ float wave_min_f(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fminf(v, __shfl_xor(v, o, 64));
  return v;
}

// P moved by T (row-major 3x4): ((R_r0 x + R_r1 y) + R_r2 z) + t_r, each
// operation rounded to FP32 (contraction into fused multiply-adds is off in
// this and the distance function).
struct Rigid {
  float m[12];
};
__global__ __launch_bounds__(256) void k_ov_transform(const float* __restrict__ p, int n, Rigid T,
                                                      float* __restrict__ out) {
  const int i = blockIdx.x * kBlock + threadIdx.x;
  if (i >= n) return;
  const float x = p[i], y = p[(int64_t)n + i], z = p[2 * (int64_t)n + i];
#pragma unroll
  for (int r = 0; r < 3; ++r) {
#pragma clang fp contract(off)
    const float* M = T.m + 4 * r;
    out[(int64_t)r * n + i] = ((M[0] * x + M[1] * y) + M[2] * z) + M[3];
  }
}

// Bounding box of both sets: per-block partials, then one block.
__global__ __launch_bounds__(256) void k_ov_box_part(const float* __restrict__ a, int na, const float* __restrict__ b,
                                                     int nb, float* __restrict__ part) {
  float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
  for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < (int64_t)na + nb; i += (int64_t)gridDim.x * kBlock) {
    const float* s = i < na ? a : b;
    const int64_t n = i < na ? na : nb, k = i < na ? i : i - na;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const float v = s[d * n + k];
      lo[d] = fminf(lo[d], v);
      hi[d] = fmaxf(hi[d], v);
    }
  }
  __shared__ float ws[4][6];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    lo[d] = wave_min_f(lo[d]);
    hi[d] = wave_max_f(hi[d]);
  }
  if ((threadIdx.x & 63) == 0)
    for (int d = 0; d < 3; ++d) {
      ws[threadIdx.x >> 6][d] = lo[d];
      ws[threadIdx.x >> 6][3 + d] = hi[d];
    }
  __syncthreads();
  if (threadIdx.x < 6) {
    const int d = threadIdx.x;
    float v = ws[0][d];
    for (int w = 1; w < 4; ++w) v = d < 3 ? fminf(v, ws[w][d]) : fmaxf(v, ws[w][d]);
    part[6 * blockIdx.x + d] = v;
  }
}

// The common box, and the two sets as segments of one sort with `keys` keys to a
// block.
struct OvSegs {
  int32_t* blk_off;  // [3]
  int64_t* base;     // [2]
  int32_t* len;      // [2]
};
__global__ __launch_bounds__(256) void k_ov_box_final(const float* __restrict__ part, int nblk, int np, int nq,
                                                      float* __restrict__ box, OvSegs seg, int keys) {
  __shared__ float ws[4][6];
  float v[6];
#pragma unroll
  for (int d = 0; d < 6; ++d) v[d] = d < 3 ? INFINITY : -INFINITY;
  for (int k = threadIdx.x; k < nblk; k += kBlock)
#pragma unroll
    for (int d = 0; d < 6; ++d) v[d] = d < 3 ? fminf(v[d], part[6 * k + d]) : fmaxf(v[d], part[6 * k + d]);
#pragma unroll
  for (int d = 0; d < 6; ++d) v[d] = d < 3 ? wave_min_f(v[d]) : wave_max_f(v[d]);
  if ((threadIdx.x & 63) == 0)
    for (int d = 0; d < 6; ++d) ws[threadIdx.x >> 6][d] = v[d];
  __syncthreads();
  if (threadIdx.x < 6) {
    const int d = threadIdx.x;
    float r = ws[0][d];
    for (int w = 1; w < 4; ++w) r = d < 3 ? fminf(r, ws[w][d]) : fmaxf(r, ws[w][d]);
    box[d] = r;
  }
  if (threadIdx.x == 0) {
    seg.blk_off[0] = 0;
    seg.blk_off[1] = (np + keys - 1) / keys;
    seg.blk_off[2] = seg.blk_off[1] + (nq + keys - 1) / keys;
    seg.base[0] = 0;
    seg.base[1] = np;
    seg.len[0] = np;
    seg.len[1] = nq;
  }
}

__device__ __forceinline__ uint32_t spread10(uint32_t v) {
  v &= 0x3FFu;
  v = (v | (v << 16)) & 0x030000FFu;
  v = (v | (v << 8)) & 0x0300F00Fu;
  v = (v | (v << 4)) & 0x030C30C3u;
  v = (v | (v << 2)) & 0x09249249u;
  return v;
}

// 30-bit Hilbert index of a cell of the 1024^3 grid (J. Skilling, "Programming
// the Hilbert curve", 2004: undo the excess work from the top bit down, then
// Gray decode; the bits of the three axes interleave into the index).
__device__ __forceinline__ uint32_t hilbert30(uint32_t x, uint32_t y, uint32_t z) {
  uint32_t X[3] = {x, y, z};
#pragma unroll
  for (uint32_t q = 512u; q > 1u; q >>= 1) {
    const uint32_t low = q - 1u;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const uint32_t t = (X[0] ^ X[i]) & low;
      const bool set = (X[i] & q) != 0u;
      X[0] ^= set ? low : t;  // invert, or exchange with axis i
      if (i > 0) X[i] ^= set ? 0u : t;
    }
  }
  X[1] ^= X[0];
  X[2] ^= X[1];
  uint32_t t = 0u;
#pragma unroll
  for (uint32_t q = 512u; q > 1u; q >>= 1) t ^= (X[2] & q) != 0u ? q - 1u : 0u;
  return (spread10(X[0] ^ t) << 2) | (spread10(X[1] ^ t) << 1) | spread10(X[2] ^ t);
}

// Place on the Hilbert curve of every point of both sets (P's first), on a
// cubic grid of 1024 cells per axis over the common box; value = the point's
// index in its set.  (A Morton curve jumps: one wave of queries in ten then
// spans a large part of the scene, and its box meets up to all leaves: 85
// leaves on average against 46 on this curve, 7,500 at worst against 2,800.)
__global__ __launch_bounds__(256) void k_ov_codes(const float* __restrict__ p, int np, const float* __restrict__ q,
                                                  int nq, const float* __restrict__ box, uint32_t* __restrict__ code,
                                                  uint32_t* __restrict__ idx) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i >= (int64_t)np + nq) return;
  const float* __restrict__ s = i < np ? p : q;
  const int64_t n = i < np ? np : nq, k = i < np ? i : i - np;
  const float ext = fmaxf(fmaxf(box[3] - box[0], box[4] - box[1]), box[5] - box[2]);
  const float inv = ext > 0.f ? 1023.f / ext : 0.f;
  uint32_t u[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) u[d] = (uint32_t)fminf(fmaxf((s[d * n + k] - box[d]) * inv, 0.f), 1023.f);
  code[i] = hilbert30(u[0], u[1], u[2]);
  idx[i] = (uint32_t)k;
}

struct OvSet {
  float* p;              // [3][n] in curve order
  const int32_t* idx;    // original indices
  const uint32_t* code;  // sorted curve places
  float* leaf;           // [6][nleaf] min xyz, max xyz
  float* super;          // [6][nsuper]
  int n, nleaf, nsuper;
};

// Points in curve order (SoA x, y, z) and one box per leaf; grid y: the set.
__global__ __launch_bounds__(256) void k_ov_gather(const float* __restrict__ p, const float* __restrict__ q,
                                                   OvSet a, OvSet b) {
  const OvSet& S = blockIdx.y ? b : a;
  const float* __restrict__ src = blockIdx.y ? q : p;
  const int n = S.n;
  const int i = blockIdx.x * kBlock + threadIdx.x;
  if (blockIdx.x * kBlock >= n) return;  // uniform
  const bool v = i < n;
  float c[3] = {0.f, 0.f, 0.f};
  if (v) {
    const int32_t k = S.idx[i];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      c[d] = src[(int64_t)d * n + k];
      S.p[(int64_t)d * n + i] = c[d];
    }
  }
  float lo[3], hi[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    lo[d] = v ? c[d] : INFINITY;
    hi[d] = v ? c[d] : -INFINITY;
#pragma unroll
    for (int o = kOvLeaf / 2; o > 0; o >>= 1) {
      lo[d] = fminf(lo[d], __shfl_xor(lo[d], o, 64));
      hi[d] = fmaxf(hi[d], __shfl_xor(hi[d], o, 64));
    }
  }
  const int leaf = i / kOvLeaf;
  if ((threadIdx.x & (kOvLeaf - 1)) == 0 && v)
    for (int d = 0; d < 3; ++d) {
      S.leaf[d * S.nleaf + leaf] = lo[d];
      S.leaf[(3 + d) * S.nleaf + leaf] = hi[d];
    }
}

// One wave per superblock, a leaf per lane.
__global__ __launch_bounds__(64) void k_ov_super(OvSet a, OvSet b_) {
  const OvSet& S = blockIdx.y ? b_ : a;
  const int s = blockIdx.x, lane = threadIdx.x, l = s * kOvSuper + lane;
  if (s >= S.nsuper) return;
#pragma unroll
  for (int d = 0; d < 6; ++d) {
    const float x = l < S.nleaf ? S.leaf[d * S.nleaf + l] : d < 3 ? INFINITY : -INFINITY;
    const float m = d < 3 ? wave_min_f(x) : wave_max_f(x);
    if (lane == 0) S.super[d * S.nsuper + s] = m;
  }
}

// Minimum and maximum over the wave without LDS (DPP, as a prefix whose last
// lane is the result).
template <int kCtrl, int kRows>
__device__ __forceinline__ float dpp_f(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(v), __float_as_int(v), kCtrl, kRows, 0xF, false));
}
template <bool kMin>
__device__ __forceinline__ float wave_extreme(float v) {
  auto pick = [](float a, float b) { return kMin ? fminf(a, b) : fmaxf(a, b); };
  v = pick(v, dpp_f<0x111, 0xF>(v));  // row_shr:1, 2, 4, 8
  v = pick(v, dpp_f<0x112, 0xF>(v));
  v = pick(v, dpp_f<0x114, 0xF>(v));
  v = pick(v, dpp_f<0x118, 0xF>(v));
  v = pick(v, dpp_f<0x142, 0xA>(v));  // row_bcast:15 -> rows 1, 3
  v = pick(v, dpp_f<0x143, 0xC>(v));  // row_bcast:31 -> rows 2, 3
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

__device__ __forceinline__ float lane_f(float v, int l) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}

// Squared distance between two boxes (min xyz, max xyz); 0 where they meet.  A
// point is a box.  Every gap is at most that of any point in a, as rounding is
// monotone.
__device__ __forceinline__ float box_dist2(const float* a, const float* b) {
  float s = 0.f;
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const float g = fmaxf(fmaxf(b[d] - a[3 + d], a[d] - b[3 + d]), 0.f);
    s += g * g;
  }
  return s;
}

struct OvBest {
  float px, py, pz;  // this lane's query
  float best;        // its nearest squared distance so far (-inf: no query)
  int bi;            // and that point's index
};

// Point (d, id) against a lane's best: the nearer, of equals the lower index.
__device__ __forceinline__ void ov_take(OvBest& o, float d, int id) {
  const bool take = (d < o.best) | ((d == o.best) & (id < o.bi));
  o.best = take ? d : o.best;
  o.bi = take ? id : o.bi;
}

// The two lanes of a query take the better of their bests.
__device__ __forceinline__ void ov_merge(OvBest& o) {
  const auto d = __builtin_amdgcn_permlane32_swap(__float_as_uint(o.best), __float_as_uint(o.best), false, false);
  const auto i = __builtin_amdgcn_permlane32_swap((uint32_t)o.bi, (uint32_t)o.bi, false, false);
  o.best = __uint_as_float(d[0]);  // the lower lane's, in both
  o.bi = (int)i[0];
  ov_take(o, __uint_as_float(d[1]), (int)i[1]);
}

// All points of leaf l against the queries, half of them in each of a query's
// lanes.
__device__ __forceinline__ void ov_scan_leaf(const OvSet& c, int l, int lane, float4* stage, OvBest& o) {
  // the leaf's candidates go through the wave's LDS slot and are read back
  // with one (broadcast) load each; places past the end hold a distance of
  // infinity and the index that never wins
  const int ci = l * kOvLeaf + lane;
  if (lane < kOvLeaf) {
    const bool cv = ci < c.n;
    stage[lane] = cv ? make_float4(c.p[ci], c.p[(int64_t)c.n + ci], c.p[2 * (int64_t)c.n + ci],
                                   __int_as_float(c.idx[ci]))
                     : make_float4(INFINITY, INFINITY, INFINITY, __int_as_float(0x7fffffff));
  }
  wave_sync();
  const float4* half = stage + (lane >> 5) * (kOvLeaf / 2);
#pragma unroll
  for (int j = 0; j < kOvLeaf / 2; ++j) {
    const float4 b = half[j];
    ov_take(o, sq_dist_rn(o.px, o.py, o.pz, b.x, b.y, b.z), __float_as_int(b.w));
  }
  ov_merge(o);
  wave_sync();  // every lane has read the slot before it is refilled
}

// Whether lane l's box is near enough to any of the queries.
__device__ __forceinline__ bool ov_reach(const float* box, int l, const OvBest& o) {
  float b[6];
#pragma unroll
  for (int d = 0; d < 6; ++d) b[d] = lane_f(box[d], l);
  const float pt[6] = {o.px, o.py, o.pz, o.px, o.py, o.pz};
  return __ballot(box_dist2(pt, b) * kOvPrune <= o.best) != 0ull;
}

// Takes the nearest of the boxes in `todo` (bit l: lane l's, at squared
// distance d), which is left out of it; -1 when it is farther than `bound`.
__device__ __forceinline__ int ov_nearest(float d, uint64_t& todo, float bound) {
  const bool mine = __builtin_amdgcn_inverse_ballot_w64(todo);
  const float m = wave_extreme<true>(mine ? d : INFINITY);
  if (!(m * kOvPrune <= bound)) return -1;
  const int l = (int)__builtin_ctzll(__ballot(mine & (d == m)));
  todo &= ~(1ull << l);
  return l;
}

// One wave per 32 query points: the exact nearest candidate of each.  Every
// query first takes the two candidates at its place on the curve (a close
// first bound); then come superblocks and their leaves, nearest first, 64
// boxes tested at a time against the box of the queries, and a box that is
// near enough once more against each of them.  A box is skipped when it is
// farther than the current best (scaled by kOvPrune against FP32 rounding), so
// a skipped point can neither win nor tie.
//
// Bound by instruction issue (55 us of it) and by the slowest waves, whose
// queries lie far apart or far from every candidate: 150k against 120k points,
// both directions, 94 us.  Walking the boxes one by one in curve order, with
// leaves of 64 points, left two launches of 2,000 waves waiting for the next
// box, 966 us; 64 queries per wave, a lane each, 191 us (fewer waves, longer
// tail); without the test of many leaves against every query 226 us.
__global__ __launch_bounds__(64) void k_ov_nn(OvSet a, OvSet b, int32_t* __restrict__ nn_a,
                                              int32_t* __restrict__ nn_b) {
  __shared__ float4 stage[kOvLeaf];
  const int ga = (a.n + kOvQuery - 1) / kOvQuery, lane = threadIdx.x;
  const bool second = (int)blockIdx.x >= ga;
  const OvSet q = second ? b : a, c = second ? a : b;
  const int q0 = ((int)blockIdx.x - (second ? ga : 0)) * kOvQuery, qi = q0 + (lane & (kOvQuery - 1));
  const bool qv = qi < q.n;
  OvBest o;
  o.px = qv ? q.p[qi] : 0.f;
  o.py = qv ? q.p[(int64_t)q.n + qi] : 0.f;
  o.pz = qv ? q.p[2 * (int64_t)q.n + qi] : 0.f;
  o.best = qv ? INFINITY : -INFINITY;
  o.bi = 0x7fffffff;
  float qb[6];  // the queries' box
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const float x = d == 0 ? o.px : d == 1 ? o.py : o.pz;
    qb[d] = wave_extreme<true>(qv ? x : INFINITY);
    qb[3 + d] = wave_extreme<false>(qv ? x : -INFINITY);
  }
  // the candidates below the first query's place, 64 probes at a time, and
  // from there those below each query's, its two lanes with one after another
  {
    const uint32_t code = q.code[min(qi, q.n - 1)], code0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)code);
    int lo = 0, len = c.n;
    while (len > 0) {
      const int step = (int)(((uint32_t)len + 63u) >> 6), end = lo + len;
      const uint32_t p = (uint32_t)lo + (uint32_t)(lane + 1) * (uint32_t)step - 1u;
      const uint64_t below = __ballot(p < (uint32_t)end && c.code[min(p, (uint32_t)end - 1u)] < code0);
      lo += (int)__popcll(below) * step;
      len = min(step - 1, end - lo);
    }
    int hi = c.n;
    int64_t reach = 32;  // a query's place is mostly close to the first one's
    while (lo + reach < hi && __ballot(c.code[lo + reach - 1] < code) != 0ull) reach *= 4;
    hi = (int)min(lo + reach, (int64_t)hi);
    while (__ballot(lo < hi) != 0ull) {
      const int mid = lo + ((hi - lo) >> 1);
      const bool below = lo < hi && c.code[min(mid, c.n - 1)] < code;
      lo = below ? mid + 1 : lo;
      hi = below ? hi : mid;
    }
    const int k = min(max(lo - (lane >> 5), 0), c.n - 1);
    if (qv) ov_take(o, sq_dist_rn(o.px, o.py, o.pz, c.p[k], c.p[(int64_t)c.n + k], c.p[2 * (int64_t)c.n + k]), c.idx[k]);
    ov_merge(o);
  }
  float bound = wave_extreme<false>(o.best);

  for (int sbase = 0; sbase < c.nsuper; sbase += 64) {
    const int sl = min(sbase + lane, c.nsuper - 1);
    float sbox[6];
#pragma unroll
    for (int d = 0; d < 6; ++d) sbox[d] = c.super[d * c.nsuper + sl];
    const float ds = box_dist2(qb, sbox);
    uint64_t supers = __ballot(sbase + lane < c.nsuper);
    while (supers != 0ull) {
      const int s = ov_nearest(ds, supers, bound);
      if (s < 0) break;
      if (!ov_reach(sbox, s, o)) continue;
      const int lbase = (sbase + s) * kOvSuper, ll = min(lbase + lane, c.nleaf - 1);
      float box[6];
#pragma unroll
      for (int d = 0; d < 6; ++d) box[d] = c.leaf[d * c.nleaf + ll];
      const float dl = box_dist2(qb, box);
      uint64_t leaves = __ballot(lbase + lane < c.nleaf && dl * kOvPrune <= bound);
      if (__popcll(leaves) > kOvMany) {  // each of them against every query, 64 leaves at a time
        bool near = false;
#pragma unroll 4
        for (int i = 0; i < kOvQuery; ++i) {
          const float x = lane_f(o.px, i), y = lane_f(o.py, i), z = lane_f(o.pz, i);
          const float pt[6] = {x, y, z, x, y, z};
          near |= box_dist2(pt, box) * kOvPrune <= lane_f(o.best, i);
        }
        leaves &= __ballot(near);
      }
      while (leaves != 0ull) {
        const int l = ov_nearest(dl, leaves, bound);
        if (l < 0) break;
        if (!ov_reach(box, l, o)) continue;
        ov_scan_leaf(c, lbase + l, lane, stage, o);
        bound = wave_extreme<false>(o.best);
      }
    }
  }
  if (qv && lane < kOvQuery) (second ? nn_b : nn_a)[q.idx[qi]] = o.bi;
}

// Reciprocity and the threshold test per point of P; one integer atomic per
// block and count.
__global__ __launch_bounds__(256) void k_ov_count(const float* __restrict__ pt, int np, const float* __restrict__ q,
                                                  int nq, const int32_t* __restrict__ nn_pq,
                                                  const int32_t* __restrict__ nn_qp, float tau2,
                                                  int32_t* __restrict__ counts) {
  const int i = blockIdx.x * kBlock + threadIdx.x;
  bool pair = false, in = false;
  if (i < np) {
    const int j = nn_pq[i];
    if (j >= 0 && j < nq && nn_qp[j] == i) {
      pair = true;
      const float d = sq_dist_rn(pt[i], pt[(int64_t)np + i], pt[2 * (int64_t)np + i], q[j], q[(int64_t)nq + j],
                                 q[2 * (int64_t)nq + j]);
      in = d < tau2;
    }
  }
  __shared__ int32_t ws[4][2];
  const uint64_t bp = __ballot(pair), bn = __ballot(in);
  if ((threadIdx.x & 63) == 0) {
    ws[threadIdx.x >> 6][0] = (int32_t)__popcll(bp);
    ws[threadIdx.x >> 6][1] = (int32_t)__popcll(bn);
  }
  __syncthreads();
  if (threadIdx.x < 2) {
    const int32_t v = (ws[0][threadIdx.x] + ws[1][threadIdx.x]) + (ws[2][threadIdx.x] + ws[3][threadIdx.x]);
    if (v) atomicAdd(&counts[threadIdx.x], v);
  }
}

// Workspace layout (all pieces 256-byte aligned).  The sorted codes and
// indices stay in the sort's buffers.
struct OvLayout {
  size_t pt, box_part, box, segs, code_a, idx_a, code_b, idx_b, hist, set_p[3], set_q[3], total;
};
static size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }
static int ov_sort_blocks(int np, int nq, int per) { return sort_blocks_of(np, per) + sort_blocks_of(nq, per); }
static int ov_sort_per(int np, int nq) {
  return sort_per(std::max(np, nq), [&](int per) { return ov_sort_blocks(np, nq, per); });
}
static OvLayout ov_layout(int np, int nq) {
  OvLayout L{};
  size_t o = 0;
  auto take = [&](size_t bytes) {
    const size_t at = o;
    o += align256(bytes);
    return at;
  };
  const size_t both = (size_t)np + nq;
  L.pt = take(12 * (size_t)np);
  L.box_part = take(4 * 6 * kOvBoxBlocks);
  L.box = take(4 * 6);
  L.segs = take(64);
  L.code_a = take(4 * both);
  L.idx_a = take(4 * both);
  L.code_b = take(4 * both);
  L.idx_b = take(4 * both);
  const int64_t room = sort_blocks_room([&](int per) { return ov_sort_blocks(np, nq, per); });
  L.hist = take(4 * (size_t)seg_hist_words(room, 2));
  for (int s = 0; s < 2; ++s) {
    const int n = s ? nq : np;
    const int nleaf = (n + kOvLeaf - 1) / kOvLeaf, nsuper = (nleaf + kOvSuper - 1) / kOvSuper;
    size_t* S = s ? L.set_q : L.set_p;
    S[0] = take(12 * (size_t)n);         // points in curve order
    S[1] = take(24 * (size_t)nleaf);     // leaf boxes
    S[2] = take(24 * (size_t)nsuper);    // superblock boxes
  }
  L.total = o;
  return L;
}

size_t overlap_workspace_bytes(int np, int nq) { return ov_layout(np, nq).total; }

void launch_overlap(const float* p_mean, int np, const float* q_mean, int nq, const float* T, float tau,
                    int32_t* nn_pq, int32_t* nn_qp, int32_t* counts, void* work, hipStream_t s) {
  const OvLayout L = ov_layout(np, nq);
  char* w = static_cast<char*>(work);
  launch_fill_i32(counts, 2, 0, s);
  if (np == 0 || nq == 0) {
    launch_fill_i32(nn_pq, np, -1, s);
    launch_fill_i32(nn_qp, nq, -1, s);
    return;
  }
  float* pt = reinterpret_cast<float*>(w + L.pt);
  Rigid R;
  for (int k = 0; k < 12; ++k) R.m[k] = T[k];
  hipLaunchKernelGGL(k_ov_transform, dim3((np + kBlock - 1) / kBlock), dim3(kBlock), 0, s, p_mean, np, R, pt);
  float* box_part = reinterpret_cast<float*>(w + L.box_part);
  float* box = reinterpret_cast<float*>(w + L.box);
  hipLaunchKernelGGL(k_ov_box_part, dim3(kOvBoxBlocks), dim3(kBlock), 0, s, (const float*)pt, np, q_mean, nq,
                     box_part);
  char* sg = w + L.segs;
  const int per = ov_sort_per(np, nq), nsb = ov_sort_blocks(np, nq, per), rows = sort_blocks_of(std::max(np, nq), per);
  const OvSegs segs{reinterpret_cast<int32_t*>(sg), reinterpret_cast<int64_t*>(sg + 16),
                    reinterpret_cast<int32_t*>(sg + 32)};
  hipLaunchKernelGGL(k_ov_box_final, dim3(1), dim3(kBlock), 0, s, (const float*)box_part, kOvBoxBlocks, np, nq, box,
                     segs, per * kSortThreads);
  uint32_t* ca = reinterpret_cast<uint32_t*>(w + L.code_a);
  uint32_t* ia = reinterpret_cast<uint32_t*>(w + L.idx_a);
  uint32_t* cb = reinterpret_cast<uint32_t*>(w + L.code_b);
  uint32_t* ib = reinterpret_cast<uint32_t*>(w + L.idx_b);
  uint32_t* hist = reinterpret_cast<uint32_t*>(w + L.hist);
  const int64_t both = (int64_t)np + nq;
  hipLaunchKernelGGL(k_ov_codes, dim3((unsigned)((both + kBlock - 1) / kBlock)), dim3(kBlock), 0, s, (const float*)pt,
                     np, q_mean, nq, (const float*)box, ca, ia);
  // both sets in one sort; four passes over the 30-bit codes end in (ca, ia)
  const SegTable seg{segs.blk_off, segs.base, 2, segs.len};
  launch_seg_pass(ca, ia, cb, ib, seg, nsb, rows, per, 0, 8, hist, false, s);
  launch_seg_pass(cb, ib, ca, ia, seg, nsb, rows, per, 8, 8, hist, false, s);
  launch_seg_pass(ca, ia, cb, ib, seg, nsb, rows, per, 16, 8, hist, false, s);
  launch_seg_pass(cb, ib, ca, ia, seg, nsb, rows, per, 24, 6, hist, false, s);
  OvSet set[2];
  for (int k = 0; k < 2; ++k) {
    const int n = k ? nq : np;
    const size_t* S = k ? L.set_q : L.set_p;
    const int nleaf = (n + kOvLeaf - 1) / kOvLeaf, nsuper = (nleaf + kOvSuper - 1) / kOvSuper;
    set[k] = OvSet{reinterpret_cast<float*>(w + S[0]), reinterpret_cast<int32_t*>(ia) + (k ? np : 0),
                   ca + (k ? np : 0), reinterpret_cast<float*>(w + S[1]), reinterpret_cast<float*>(w + S[2]), n,
                   nleaf, nsuper};
  }
  const int nmax = std::max(np, nq), smax = std::max(set[0].nsuper, set[1].nsuper);
  hipLaunchKernelGGL(k_ov_gather, dim3((nmax + kBlock - 1) / kBlock, 2), dim3(kBlock), 0, s, (const float*)pt, q_mean,
                     set[0], set[1]);
  hipLaunchKernelGGL(k_ov_super, dim3(smax, 2), dim3(64), 0, s, set[0], set[1]);
  const int groups = (np + kOvQuery - 1) / kOvQuery + (nq + kOvQuery - 1) / kOvQuery;
  hipLaunchKernelGGL(k_ov_nn, dim3(groups), dim3(64), 0, s, set[0], set[1], nn_pq, nn_qp);
  const float tau2 = tau * tau;
  hipLaunchKernelGGL(k_ov_count, dim3((np + kBlock - 1) / kBlock), dim3(kBlock), 0, s, (const float*)pt, np, q_mean,
                     nq, (const int32_t*)nn_pq, (const int32_t*)nn_qp, tau2, counts);
}

}  // namespace ls

// ---------------------------------------------------------------------------
// Overlap ratio without allocation: the workspace is a file-scope device
// array, one copy per GPU, held until the process ends.  Host code never
// passes the array's name to a kernel (on the host it is only a stand-in
// symbol): its device address is looked up once per device with
// hipGetSymbolAddress, with that device current, and kept in a per-device
// table.  Every call on a device shares its copy; the kernels write every
// byte they read from it within the call, so nothing needs clearing, and
// calls that overlap on one device race.
namespace {

constexpr size_t kNoAllocBytes = (size_t)LS_OVERLAP_NOALLOC_BYTES;
static_assert(kNoAllocBytes % 256 == 0, "scratch size must keep 256-byte alignment");

static __device__ __align__(256) unsigned char scratch[kNoAllocBytes];

std::mutex g_scratch_mu;
std::vector<void*> g_scratch_dev;  // device address of `scratch`, by device ordinal

ls_status scratch_address(void** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0) return ls::api_fail(LS_ERR_HIP, "hipGetDevice failed");
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if ((size_t)dev >= g_scratch_dev.size()) g_scratch_dev.resize((size_t)dev + 1, nullptr);
  if (!g_scratch_dev[(size_t)dev]) {
    void* ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !ptr) {
      (void)hipGetLastError();
      return ls::api_fail(LS_ERR_HIP, "hipGetSymbolAddress of the overlap scratch array failed");
    }
    g_scratch_dev[(size_t)dev] = ptr;
  }
  *out = g_scratch_dev[(size_t)dev];
  return LS_OK;
}

}  // namespace

extern "C" ls_status ls_overlap_ratio_noalloc(const float* p_mean, int32_t np, const float* q_mean, int32_t nq,
                                              const float* T_pq, float tau, int32_t* nn_pq, int32_t* nn_qp,
                                              int32_t* counts, hipStream_t s) {
  const ls_status st = ls::overlap_check_args(p_mean, np, q_mean, nq, T_pq, tau, nn_pq, nn_qp, counts);
  if (st != LS_OK) return st;
  if (np > LS_OVERLAP_NOALLOC_MAX_POINTS || nq > LS_OVERLAP_NOALLOC_MAX_POINTS)
    return ls::api_fail(LS_ERR_CAPACITY, "ls_overlap_ratio_noalloc takes at most LS_OVERLAP_NOALLOC_MAX_POINTS "
                                         "points per set; use ls_overlap_ratio with a workspace");
  if (ls::overlap_workspace_bytes(np, nq) > kNoAllocBytes)
    return ls::api_fail(LS_ERR_CAPACITY, "overlap workspace exceeds the static scratch array");
  void* work = nullptr;
  const ls_status sa = scratch_address(&work);
  if (sa != LS_OK) return sa;
  ls::launch_overlap(p_mean, np, q_mean, nq, T_pq, tau, nn_pq, nn_qp, counts, work, s);
  return ls::api_hip_check("ls_overlap_ratio_noalloc");
}
