// Submap-update (mapping) loss of Sec. 3.1, Eq. 3-5: the colour term mixing
// L1 and SSIM (Eq. 4), the L1 depth term, and the isotropic regulariser on
// the Gaussian scales (Eq. 5), each with its gradient.
//
// SSIM is the windowed index with an 11 x 11 Gaussian window (sigma 1.5,
// weights summing to 1), zero padding outside the image, C1 = 0.01^2 and
// C2 = 0.03^2, per colour channel, averaged over channels and pixels.  Its
// gradient follows from the three partial derivatives of the per-pixel index
// with respect to the x-side windowed moments (mu_x, E[x^2], E[xy]):
//   dS/dx(q) = sum_p w(p - q) (A_p + 2 x_q B_p + y_q C_p)
// i.e. the same window applied to the maps A, B, C (the window is symmetric).
#include <algorithm>
#include <cmath>

#include "kernels.h"

namespace ls {

constexpr int kSsimR = 5;                    // window radius: 11 taps
constexpr int kSsimTaps = 2 * kSsimR + 1;
constexpr int kSsimT = 32;                   // output tile side
constexpr int kSsimM = kSsimT + 2 * kSsimR;  // 42: side of the region whose SSIM terms reach the tile
constexpr int kSsimI = kSsimT + 4 * kSsimR;  // 52: side of the input region those terms read
// Each filter pass gives a thread a strip of consecutive outputs along the
// filter direction, so an input is read once per strip rather than once per
// tap.  LDS rows have odd lengths and the lanes of a pass run across its
// strips, so that no pass has bank conflicts.
constexpr int kInRow = kSsimI + 1;                   // inputs: 52 rows of 52
constexpr int kInMap = kSsimI * kInRow;
constexpr int kInLoads = (kSsimI * kSsimI + kBlock - 1) / kBlock;  // 11 per thread and image
constexpr int kMomRow = kSsimM + 1;                  // row-filtered moments: 52 rows of 42
constexpr int kMomMap = kSsimI * kMomRow;
constexpr int kDerMap = kSsimM * kMomRow;            // derivative maps: 42 rows of 42
constexpr int kOutRow = kSsimT + 1;                  // row-filtered derivatives: 42 rows of 32
constexpr int kOutMap = kSsimM * kOutRow;
constexpr int kInStrip = 11;                         // moment row pass: 52 rows x 4 strips
constexpr int kInStrips = (kSsimM + kInStrip - 1) / kInStrip;
constexpr int kMomStrip = 7;                         // moment column pass: 42 columns x 6 strips
constexpr int kMomStrips = kSsimM / kMomStrip;
constexpr int kDerStrip = 8;                         // derivative row pass: 42 rows x 4 strips
constexpr int kDerStrips = kSsimT / kDerStrip;
constexpr int kOutStrip = kSsimT * kSsimT / kBlock;  // derivative column pass: 32 columns x 8 strips of 4
static_assert(kSsimM % kMomStrip == 0 && kSsimT % kDerStrip == 0, "whole strips");
static_assert(kSsimI * kInStrips <= kBlock && kSsimM * kMomStrips <= kBlock && kSsimM * kDerStrips <= kBlock,
              "one strip per thread");
static_assert(kSsimT * (kSsimT / kOutStrip) == kBlock, "one output strip per thread");
constexpr int kSsimLds = 3 * (kDerMap + kOutMap);  // 38 KB: four blocks per CU
static_assert(2 * kInMap + kInStrip <= kSsimLds && 3 * kMomMap <= kSsimLds,
              "inputs, three of the moments and derivatives take turns");
constexpr float kSsimC1 = 0.01f * 0.01f;
constexpr float kSsimC2 = 0.03f * 0.03f;

struct SsimWindow {
  float w[kSsimTaps];
};

// Pixels with a target depth, per 1024-pixel block (blocks never straddle
// renders).
__global__ __launch_bounds__(256) void k_valid_count(const JobDev* __restrict__ jobs,
                                                     const int32_t* __restrict__ pblk_off, int R,
                                                     const float* __restrict__ tgt_depth, float* __restrict__ part) {
  const int r = find_segment<int32_t>(pblk_off, R, (int32_t)blockIdx.x);
  const JobDev& J = jobs[r];
  const int64_t hw = (int64_t)J.W * J.H;
  const int64_t b0 = (int64_t)(blockIdx.x - pblk_off[r]) * 1024;
  float cnt = 0.f;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int64_t p = b0 + (int64_t)k * 256 + threadIdx.x;
    if (p < hw) {
      const float td = tgt_depth ? tgt_depth[J.pix_off + p] : J.tgt_depth[p];
      cnt += td > 0.f ? 1.f : 0.f;
    }
  }
  cnt = wave_sum(cnt);
  __shared__ float ws[4];
  if ((threadIdx.x & 63) == 0) ws[threadIdx.x >> 6] = cnt;
  __syncthreads();
  if (threadIdx.x == 0) part[blockIdx.x] = (ws[0] + ws[1]) + (ws[2] + ws[3]);
}

// Block-wide sum of one value per thread (256 threads), fixed order; the
// total is returned to thread 0.
__device__ __forceinline__ float block_sum(float v, float* ws) {
  v = wave_sum(v);
  if ((threadIdx.x & 63) == 0) ws[threadIdx.x >> 6] = v;
  __syncthreads();
  return (ws[0] + ws[1]) + (ws[2] + ws[3]);
}

// One block per render: 1 / |Omega| (0 when no pixel has a target depth).
__global__ __launch_bounds__(256) void k_valid_inv(const int32_t* __restrict__ pblk_off, int R,
                                                   const float* __restrict__ part, float* __restrict__ inv) {
  __shared__ float ws[4];
  const int r = blockIdx.x;
  float c = 0.f;
  for (int b = pblk_off[r] + threadIdx.x; b < pblk_off[r + 1]; b += kBlock) c += part[b];
  c = block_sum(c, ws);
  if (threadIdx.x == 0) inv[r] = c > 0.f ? 1.f / c : 0.f;
}

// The same in kValidParts parts per render, for a kernel whose waves add them up for
// themselves (valid_inv); a launch for that took 2 to 5 us.  `blocks` of a render
// write a part each, and zeros to the parts that are no block's; where they are more
// than the parts, k_valid_fold adds them up.
constexpr int kValidThreads = 1024;
__global__ __launch_bounds__(kValidThreads) void k_valid_parts(const JobDev* __restrict__ jobs,
                                                               const float* __restrict__ tgt_depth, int blocks,
                                                               float* __restrict__ part) {
  constexpr int kAhead = 8;
  const int r = blockIdx.x / blocks, b = blockIdx.x - r * blocks;
  const JobDev& J = jobs[r];
  const int64_t hw = (int64_t)J.W * J.H, step = (int64_t)blocks * kValidThreads;
  const float* __restrict__ td = tgt_depth ? tgt_depth + J.pix_off : J.tgt_depth;
  int cnt = 0;
  for (int64_t p0 = (int64_t)b * kValidThreads + threadIdx.x; p0 < hw; p0 += kAhead * step) {
    float v[kAhead];
#pragma unroll
    for (int k = 0; k < kAhead; ++k) v[k] = p0 + k * step < hw ? td[p0 + k * step] : 0.f;
#pragma unroll
    for (int k = 0; k < kAhead; ++k) cnt += v[k] > 0.f ? 1 : 0;
  }
  const float sum = wave_sum((float)cnt);
  __shared__ float ws[kValidThreads / 64];
  if ((threadIdx.x & 63) == 0) ws[threadIdx.x >> 6] = sum;
  __syncthreads();
  if (threadIdx.x == 0) {
    float all = 0.f;
#pragma unroll
    for (int k = 0; k < kValidThreads / 64; ++k) all += ws[k];
    part[(int64_t)r * max(blocks, kValidParts) + b] = all;
  }
  const int k = b + blocks * (1 + threadIdx.x);
  if (k < kValidParts) part[(int64_t)r * kValidParts + k] = 0.f;
}

__global__ __launch_bounds__(kValidParts) void k_valid_fold(const float* __restrict__ many, float* __restrict__ part) {
  float c = 0.f;  // (whole numbers: any order)
#pragma unroll
  for (int k = 0; k < kValidPartsMany / kValidParts; ++k)
    c += many[(int64_t)blockIdx.x * kValidPartsMany + k * kValidParts + threadIdx.x];
  part[(int64_t)blockIdx.x * kValidParts + threadIdx.x] = c;
}

// 1 / |Omega| of render r (0 when no pixel has a target depth), in every lane.
__device__ __forceinline__ float valid_inv(const float* __restrict__ part, int r) {
  static_assert(kValidParts == 64, "a part per lane");
  const float c = wave_sum(part[r * kValidParts + (threadIdx.x & 63)]);
  return c > 0.f ? 1.f / c : 0.f;
}

// One block per (render, colour channel, 32 x 32 output tile).  The block
// stages the 52 x 52 input region of both images in LDS, filters the five
// windowed moments separably (rows, then columns) over the 42 x 42 region
// whose SSIM terms reach the tile, forms the index and its derivative maps
// A, B, C there (zero outside the image), filters those back onto the tile
// and writes the weighted colour gradient; channel-0 blocks also handle the
// depth term.  Partials per block: (sum of SSIM over the tile, L1 colour
// sum and L1 depth sum over its pixels with a target depth).
//
// Bound by vector instruction issue (1,800 instructions per wave and block).
// All stages share one piece of LDS, for four blocks on a CU: the row pass
// keeps a strip's 55 moments in registers until every thread is done with the
// inputs, and then hands over three of them, and the other two after those.
// 1200 x 680: 49 us; with inputs and five moments apart in 65 KB (two blocks)
// and strips whose lanes met in the same banks 62 us; all five moments at once
// in 44 KB (three blocks) 53 us.  (Filtering x^2 + y^2 as one map takes 43 us,
// but its rounding moves gradients by 2e-5 where a window is nearly flat.)
__global__ __launch_bounds__(256) void k_loss_ssim(const JobDev* __restrict__ jobs,
                                                   const int32_t* __restrict__ sblk_off, int R, int nblk,
                                                   const float* __restrict__ pred_rgb,
                                                   const float* __restrict__ pred_depth,
                                                   const float* __restrict__ tgt_rgb,
                                                   const float* __restrict__ tgt_depth,
                                                   const float* __restrict__ valid, SsimWindow win,
                                                   float lambda_ssim, float lambda_color, float lambda_depth,
                                                   float* __restrict__ g_rgb, float* __restrict__ g_depth,
                                                   float* __restrict__ part) {
  __shared__ float lds[kSsimLds];
  const int blk = xcd_remap(blockIdx.x, nblk);
  if (blk >= nblk) return;
  const int r = find_segment<int32_t>(sblk_off, R, (int32_t)blk);
  const JobDev& J = jobs[r];
  const int W = J.W, H = J.H;
  const int tx = (W + kSsimT - 1) / kSsimT, ty = (H + kSsimT - 1) / kSsimT;
  const int local = blk - sblk_off[r];
  const int ch = local / (tx * ty);
  const int t = local - ch * tx * ty;
  const int x0 = (t % tx) * kSsimT, y0 = (t / tx) * kSsimT;
  const float inv = valid_inv(valid, r);
  const int64_t hw = (int64_t)W * H;
  const float* __restrict__ X = pred_rgb + 3 * J.pix_off + ch * hw;
  const float* __restrict__ Y = (tgt_rgb ? tgt_rgb + 3 * J.pix_off : J.tgt_rgb) + ch * hw;

  {
    // every load of the input region is issued before the first is used
    float xv[kInLoads], yv[kInLoads];
#pragma unroll
    for (int j = 0; j < kInLoads; ++j) {
      const int i = threadIdx.x + kBlock * j;
      const int rr = i / kSsimI, cc = i - rr * kSsimI;
      const int gy = y0 - 2 * kSsimR + rr, gx = x0 - 2 * kSsimR + cc;
      xv[j] = 0.f;
      yv[j] = 0.f;
      if (rr < kSsimI && gx >= 0 && gx < W && gy >= 0 && gy < H) {
        const int64_t p = (int64_t)gy * W + gx;
        xv[j] = X[p];
        yv[j] = Y[p];
      }
    }
#pragma unroll
    for (int j = 0; j < kInLoads; ++j) {
      const int i = threadIdx.x + kBlock * j;
      const int rr = i / kSsimI, cc = i - rr * kSsimI;
      if (rr < kSsimI) {
        lds[rr * kInRow + cc] = xv[j];
        lds[kInMap + rr * kInRow + cc] = yv[j];
      }
    }
  }
  __syncthreads();

  // row pass: the five moments of each input row at the 42 moment columns
  // (the last strip's columns past them are not stored)
  const int rs = threadIdx.x / kSsimI, rr = threadIdx.x - rs * kSsimI, rc0 = rs * kInStrip;
  const bool row_item = rs < kInStrips;
  float a[kInStrip], b[kInStrip], c[kInStrip], d[kInStrip], e[kInStrip];
#pragma unroll
  for (int o = 0; o < kInStrip; ++o) a[o] = b[o] = c[o] = d[o] = e[o] = 0.f;
  if (row_item) {
    const float* xr = lds + rr * kInRow + rc0;
    const float* yr = xr + kInMap;
#pragma unroll
    for (int k = 0; k < kInStrip + 2 * kSsimR; ++k) {
      const float xv = xr[k], yv = yr[k];
      const float xx = xv * xv, yy = yv * yv, xy = xv * yv;
#pragma unroll
      for (int o = 0; o < kInStrip; ++o) {
        const int tap = k - o;
        if (tap >= 0 && tap < kSsimTaps) {
          const float w = win.w[tap];
          a[o] += w * xv;
          b[o] += w * yv;
          c[o] += w * xx;
          d[o] += w * yy;
          e[o] += w * xy;
        }
      }
    }
  }
  float* row_out = lds + rr * kMomRow + rc0;
  __syncthreads();  // every thread is done with the inputs
  if (row_item) {
#pragma unroll
    for (int o = 0; o < kInStrip; ++o)
      if (rc0 + o < kSsimM) {
        row_out[o] = a[o];
        row_out[kMomMap + o] = b[o];
        row_out[2 * kMomMap + o] = c[o];
      }
  }
  __syncthreads();

  // column pass, SSIM index and its derivative maps on the 42 x 42 region:
  // one strip of kMomStrip rows of one moment column per thread, three of the
  // moments first and then the other two in their place
  float dA[kMomStrip], dB[kMomStrip], dC[kMomStrip];
  float ssum = 0.f;
  const int mc = threadIdx.x % kSsimM, r0 = (threadIdx.x / kSsimM) * kMomStrip;
  const bool col_item = threadIdx.x < kSsimM * kMomStrips;
  float mx[kMomStrip], my[kMomStrip], exx[kMomStrip], eyy[kMomStrip], exy[kMomStrip];
#pragma unroll
  for (int q = 0; q < kMomStrip; ++q) mx[q] = my[q] = exx[q] = eyy[q] = exy[q] = dA[q] = dB[q] = dC[q] = 0.f;
  const float* col_in = lds + (col_item ? r0 * kMomRow + mc : 0);
#pragma unroll
  for (int k = 0; k < kMomStrip + 2 * kSsimR; ++k) {
    const float* in = col_in + k * kMomRow;
    const float v0 = in[0], v1 = in[kMomMap], v2 = in[2 * kMomMap];
#pragma unroll
    for (int q = 0; q < kMomStrip; ++q) {
      const int tap = k - q;
      if (tap >= 0 && tap < kSsimTaps) {
        const float w = win.w[tap];
        mx[q] += w * v0;
        my[q] += w * v1;
        exx[q] += w * v2;
      }
    }
  }
  __syncthreads();
  if (row_item) {
#pragma unroll
    for (int o = 0; o < kInStrip; ++o)
      if (rc0 + o < kSsimM) {
        row_out[o] = d[o];
        row_out[kMomMap + o] = e[o];
      }
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kMomStrip + 2 * kSsimR; ++k) {
    const float* in = col_in + k * kMomRow;
    const float v3 = in[0], v4 = in[kMomMap];
#pragma unroll
    for (int q = 0; q < kMomStrip; ++q) {
      const int tap = k - q;
      if (tap >= 0 && tap < kSsimTaps) {
        const float w = win.w[tap];
        eyy[q] += w * v3;
        exy[q] += w * v4;
      }
    }
  }
  if (col_item) {
    const int gx = x0 - kSsimR + mc;
#pragma unroll
    for (int q = 0; q < kMomStrip; ++q) {
      const int mr = r0 + q;
      const int gy = y0 - kSsimR + mr;
      if (gx >= 0 && gx < W && gy >= 0 && gy < H) {
        const float vx = exx[q] - mx[q] * mx[q], vy = eyy[q] - my[q] * my[q], cxy = exy[q] - mx[q] * my[q];
        const float n1 = 2.f * mx[q] * my[q] + kSsimC1, n2 = 2.f * cxy + kSsimC2;
        const float i1 = 1.f / (mx[q] * mx[q] + my[q] * my[q] + kSsimC1), i2 = 1.f / (vx + vy + kSsimC2);
        const float sv = n1 * n2 * i1 * i2;
        dA[q] = 2.f * my[q] * (n2 - n1) * i1 * i2 - 2.f * mx[q] * sv * (i1 - i2);
        dB[q] = -sv * i2;
        dC[q] = 2.f * n1 * i1 * i2;
        if (mr >= kSsimR && mr < kSsimR + kSsimT && mc >= kSsimR && mc < kSsimR + kSsimT) ssum += sv;
      }
    }
  }
  __syncthreads();  // every thread is done with the moments
  if (col_item) {
#pragma unroll
    for (int q = 0; q < kMomStrip; ++q) {
      const int i = (r0 + q) * kMomRow + mc;
      lds[i] = dA[q];
      lds[kDerMap + i] = dB[q];
      lds[2 * kDerMap + i] = dC[q];
    }
  }
  // this thread's output strip (column ocol, rows o0 .. o0 + kOutStrip - 1):
  // its pixels are issued now and used at the end
  const int ocol = threadIdx.x % kSsimT, o0 = (threadIdx.x / kSsimT) * kOutStrip;
  float xq[kOutStrip], yq[kOutStrip], tq[kOutStrip], dq[kOutStrip];
#pragma unroll
  for (int q = 0; q < kOutStrip; ++q) {
    const int gy = y0 + o0 + q, gx = x0 + ocol;
    xq[q] = yq[q] = tq[q] = dq[q] = 0.f;
    if (gx < W && gy < H) {
      const int64_t p = (int64_t)gy * W + gx;
      xq[q] = X[p];
      yq[q] = Y[p];
      tq[q] = tgt_depth ? tgt_depth[J.pix_off + p] : J.tgt_depth[p];
      if (ch == 0) dq[q] = pred_depth[J.pix_off + p];
    }
  }
  __syncthreads();

  // row pass over the derivative maps: 42 rows x 32 output columns
  float* rowed = lds + 3 * kDerMap;
  if (threadIdx.x < kSsimM * kDerStrips) {
    const int row = threadIdx.x % kSsimM, s0 = (threadIdx.x / kSsimM) * kDerStrip;
    const float* in = lds + row * kMomRow + s0;
    float a[kDerStrip], b[kDerStrip], c[kDerStrip];
#pragma unroll
    for (int o = 0; o < kDerStrip; ++o) a[o] = b[o] = c[o] = 0.f;
#pragma unroll
    for (int k = 0; k < kDerStrip + 2 * kSsimR; ++k) {
      const float va = in[k], vb = in[kDerMap + k], vc = in[2 * kDerMap + k];
#pragma unroll
      for (int o = 0; o < kDerStrip; ++o) {
        const int tap = k - o;
        if (tap >= 0 && tap < kSsimTaps) {
          const float w = win.w[tap];
          a[o] += w * va;
          b[o] += w * vb;
          c[o] += w * vc;
        }
      }
    }
    float* out = rowed + row * kOutRow + s0;
#pragma unroll
    for (int o = 0; o < kDerStrip; ++o) {
      out[o] = a[o];
      out[kOutMap + o] = b[o];
      out[2 * kOutMap + o] = c[o];
    }
  }
  __syncthreads();

  // column pass onto the tile (a strip of kOutStrip rows of one column per
  // thread) and the weighted gradients
  const float k_l1 = lambda_color * (1.f - lambda_ssim) * inv;
  const float k_ss = -lambda_color * lambda_ssim / (3.f * (float)hw);
  const float k_d = lambda_depth * inv;
  float l1 = 0.f, l1d = 0.f;
  {
    float fa[kOutStrip], fb[kOutStrip], fc[kOutStrip];
#pragma unroll
    for (int q = 0; q < kOutStrip; ++q) fa[q] = fb[q] = fc[q] = 0.f;
#pragma unroll
    for (int k = 0; k < kOutStrip + 2 * kSsimR; ++k) {
      const int li = (o0 + k) * kOutRow + ocol;
      const float va = rowed[li], vb = rowed[kOutMap + li], vc = rowed[2 * kOutMap + li];
#pragma unroll
      for (int q = 0; q < kOutStrip; ++q) {
        const int tap = k - q;
        if (tap >= 0 && tap < kSsimTaps) {
          const float w = win.w[tap];
          fa[q] += w * va;
          fb[q] += w * vb;
          fc[q] += w * vc;
        }
      }
    }
    const int gx = x0 + ocol;
#pragma unroll
    for (int q = 0; q < kOutStrip; ++q) {
      const int gy = y0 + o0 + q;
      if (gx < W && gy < H) {
        const int64_t p = (int64_t)gy * W + gx;
        const float xv = xq[q], yv = yq[q];
        const float td = tq[q];
        const bool valid = td > 0.f;
        const float dc = xv - yv;
        float g = k_ss * (fa[q] + 2.f * xv * fb[q] + yv * fc[q]);
        if (valid) {
          l1 += fabsf(dc);
          g += dc > 0.f ? k_l1 : (dc < 0.f ? -k_l1 : 0.f);
        }
        if (g_rgb) g_rgb[3 * J.pix_off + ch * hw + p] = g;
        if (ch == 0) {
          const float dd = dq[q] - td;
          if (valid) l1d += fabsf(dd);
          if (g_depth) g_depth[J.pix_off + p] = valid ? (dd > 0.f ? k_d : (dd < 0.f ? -k_d : 0.f)) : 0.f;
        }
      }
    }
  }
  ssum = wave_sum(ssum);
  l1 = wave_sum(l1);
  l1d = wave_sum(l1d);
  __shared__ float ws[4][3];
  if ((threadIdx.x & 63) == 0) {
    ws[threadIdx.x >> 6][0] = ssum;
    ws[threadIdx.x >> 6][1] = l1;
    ws[threadIdx.x >> 6][2] = l1d;
  }
  __syncthreads();
  if (threadIdx.x < 3) {
    const int q = threadIdx.x;
    part[3 * (int64_t)blk + q] = (ws[0][q] + ws[1][q]) + (ws[2][q] + ws[3][q]);
  }
}

// One block per render: ordered sums of the block partials and the loss
//   lc ((1 - ls) L1_rgb + ls (1 - mean SSIM)) + ld L1_depth.
constexpr int kMapReduceThreads = 1024;
__global__ __launch_bounds__(kMapReduceThreads) void k_map_reduce(const JobDev* __restrict__ jobs,
                                                                  const int32_t* __restrict__ sblk_off, int R,
                                                                  const float* __restrict__ part,
                                                                  const float* __restrict__ valid, float lambda_ssim,
                                                                  float lambda_color, float lambda_depth,
                                                                  float* __restrict__ loss,
                                                                  float* __restrict__ scale) {
  constexpr int kWaves = kMapReduceThreads / 64, kAhead = 4;
  __shared__ float ws[3][kWaves];
  const int r = blockIdx.x, end = sblk_off[r + 1];
  const float inv = valid_inv(valid, r);
  float s = 0.f, c = 0.f, d = 0.f;
  for (int b = sblk_off[r] + threadIdx.x; b < end; b += kAhead * kMapReduceThreads) {
    float v[kAhead][3];
#pragma unroll
    for (int k = 0; k < kAhead; ++k)
#pragma unroll
      for (int q = 0; q < 3; ++q)
        v[k][q] = b + k * kMapReduceThreads < end ? part[3 * (int64_t)(b + k * kMapReduceThreads) + q] : 0.f;
#pragma unroll
    for (int k = 0; k < kAhead; ++k) {
      s += v[k][0];
      c += v[k][1];
      d += v[k][2];
    }
  }
  s = wave_sum(s);
  c = wave_sum(c);
  d = wave_sum(d);
  if ((threadIdx.x & 63) == 0) {
    ws[0][threadIdx.x >> 6] = s;
    ws[1][threadIdx.x >> 6] = c;
    ws[2][threadIdx.x >> 6] = d;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    s = c = d = 0.f;
#pragma unroll
    for (int k = 0; k < kWaves; ++k) {
      s += ws[0][k];
      c += ws[1][k];
      d += ws[2][k];
    }
    const float n = 3.f * (float)jobs[r].W * (float)jobs[r].H;
    if (loss)
      loss[r] = lambda_color * ((1.f - lambda_ssim) * c * inv + lambda_ssim * (1.f - s / n)) + lambda_depth * d * inv;
    if (scale) scale[r] = 1.f;
  }
}

// Isotropic regulariser (Eq. 5): per Gaussian sum_j |s_j - mean(s)| with
// s = exp(log_scale); its gradient coef * s_j (sign(d_j) - mean_i sign(d_i))
// is added to grad; one partial sum per block.
template <int kThreads>
__global__ __launch_bounds__(kThreads) void k_isotropic(const float* __restrict__ log_scale, int64_t n, float coef,
                                                   float* __restrict__ grad, float* __restrict__ part) {
  float acc = 0.f;
  for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n; i += (int64_t)gridDim.x * kThreads) {
    const float s0 = expf(log_scale[i]), s1 = expf(log_scale[n + i]), s2 = expf(log_scale[2 * n + i]);
    const float m = (s0 + s1 + s2) * (1.f / 3.f);
    const float d0 = s0 - m, d1 = s1 - m, d2 = s2 - m;
    acc += (fabsf(d0) + fabsf(d1)) + fabsf(d2);
    if (grad) {
      const float g0 = d0 > 0.f ? 1.f : (d0 < 0.f ? -1.f : 0.f);
      const float g1 = d1 > 0.f ? 1.f : (d1 < 0.f ? -1.f : 0.f);
      const float g2 = d2 > 0.f ? 1.f : (d2 < 0.f ? -1.f : 0.f);
      const float gm = (g0 + g1 + g2) * (1.f / 3.f);
      grad[i] += coef * s0 * (g0 - gm);
      grad[n + i] += coef * s1 * (g1 - gm);
      grad[2 * n + i] += coef * s2 * (g2 - gm);
    }
  }
  acc = wave_sum(acc);
  __shared__ float ws[kThreads / 64];
  if ((threadIdx.x & 63) == 0) ws[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    float sum = 0.f;
#pragma unroll
    for (int k = 0; k < kThreads / 64; ++k) sum += ws[k];
    part[blockIdx.x] = sum;
  }
}

__global__ __launch_bounds__(256) void k_isotropic_reduce(const float* __restrict__ part, int nblk, float coef,
                                                          float* __restrict__ loss) {
  float v = 0.f;
  for (int b = threadIdx.x; b < nblk; b += kBlock) v += part[b];
  v = wave_sum(v);
  __shared__ float ws[4];
  if ((threadIdx.x & 63) == 0) ws[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0) loss[0] = coef * ((ws[0] + ws[1]) + (ws[2] + ws[3]));
}

static SsimWindow ssim_window() {
  SsimWindow w;
  double g[kSsimTaps], tot = 0.0;
  for (int k = 0; k < kSsimTaps; ++k) {
    const double d = k - kSsimR;
    g[k] = std::exp(-d * d / (2.0 * 1.5 * 1.5));
    tot += g[k];
  }
  for (int k = 0; k < kSsimTaps; ++k) w.w[k] = (float)(g[k] / tot);
  return w;
}

void launch_valid_inv(const JobDev* jobs, const int32_t* pblk_off_d, int npblk, int R, const float* tgt_depth,
                      float* cnt_part, float* inv, hipStream_t s) {
  if (npblk > 0)
    hipLaunchKernelGGL(k_valid_count, dim3(npblk), dim3(256), 0, s, jobs, pblk_off_d, R, tgt_depth, cnt_part);
  if (R > 0) hipLaunchKernelGGL(k_valid_inv, dim3(R), dim3(kBlock), 0, s, pblk_off_d, R, (const float*)cnt_part, inv);
}

int ssim_blocks(int W, int H) { return 3 * ((W + kSsimT - 1) / kSsimT) * ((H + kSsimT - 1) / kSsimT); }

void launch_loss_mapping(const JobDev* jobs, int npblk, int max_pblk, const int32_t* sblk_off_d, int nsblk, int R,
                         const float* pred_rgb,
                         const float* pred_depth, const float* tgt_rgb, const float* tgt_depth, float lambda_ssim,
                         float lambda_color, float lambda_depth, float* g_rgb, float* g_depth, float* map_part,
                         float* loss, float* scale, hipStream_t s) {
  float* valid = map_part + 3 * (int64_t)nsblk;
  // A block per 1,024 pixels of a render, up to 64, and 256 of large images (with 64
  // whatever the size 512 renders of 33 x 17 took 57 us, 4 with one, and 4096 x 4096
  // 108 us, 37 with 256), but no more than that on average over the renders.
  const bool many = max_pblk > 2048 && npblk / R >= kValidPartsMany;
  const int blocks = many ? kValidPartsMany : std::max(1, std::min({max_pblk, npblk / R, kValidParts}));
  float* count = many ? valid + (int64_t)kValidParts * R : valid;
  hipLaunchKernelGGL(k_valid_parts, dim3(blocks * R), dim3(kValidThreads), 0, s, jobs, tgt_depth, blocks, count);
  if (many) hipLaunchKernelGGL(k_valid_fold, dim3(R), dim3(kValidParts), 0, s, (const float*)count, valid);
  if (nsblk > 0) {
    const int grid = 8 * ((nsblk + 7) / 8);
    hipLaunchKernelGGL(k_loss_ssim, dim3(grid), dim3(kBlock), 0, s, jobs, sblk_off_d, R, nsblk, pred_rgb, pred_depth,
                       tgt_rgb, tgt_depth, (const float*)valid, ssim_window(), lambda_ssim, lambda_color,
                       lambda_depth, g_rgb, g_depth, map_part);
  }
  hipLaunchKernelGGL(k_map_reduce, dim3(R), dim3(kMapReduceThreads), 0, s, jobs, sblk_off_d, R, (const float*)map_part,
                     (const float*)valid, lambda_ssim, lambda_color, lambda_depth, loss, scale);
}

void launch_loss_isotropic(const float* log_scale, int64_t n, float lambda_reg, float* loss, float* grad, float* part,
                           hipStream_t s) {
  const float coef = n > 0 ? lambda_reg / (float)n : 0.f;
  // the work array holds 256 partials: past a block of 256 items each, larger
  // blocks (200k items: 7.1 us with four rounds of 256, 4.9 us with one of 1,024)
  const int per = n <= (int64_t)kIsotropicBlocks * kBlock ? kBlock : 1024;
  const int nblk = (int)std::min<int64_t>(std::max<int64_t>((n + per - 1) / per, 1), kIsotropicBlocks);
  if (per == kBlock)
    hipLaunchKernelGGL(k_isotropic<kBlock>, dim3(nblk), dim3(kBlock), 0, s, log_scale, n, coef, grad, part);
  else
    hipLaunchKernelGGL(k_isotropic<1024>, dim3(nblk), dim3(1024), 0, s, log_scale, n, coef, grad, part);
  hipLaunchKernelGGL(k_isotropic_reduce, dim3(1), dim3(kBlock), 0, s, (const float*)part, nblk, coef, loss);
}

}  // namespace ls
