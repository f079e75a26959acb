// L1 registration/tracking loss with its image gradients, and fused Adam.
#include "common.h"
#include "kernels.h"

#include <algorithm>

namespace ls {

constexpr int kLossPix = 4;  // pixels per thread
constexpr int kLossBlockPix = 256 * kLossPix;
constexpr int kSelBins = kSelHistBins;  // bins of a median selection pass

// Per-render exposure coefficients (a, b) of the rendered colour, C' =
// exp(a) C + b (registration with exposure compensation); identity without.
struct Exposure {
  float gain, offset;
  bool on;
};
__device__ __forceinline__ Exposure exposure_of(const float* expo, int r) {
  Exposure e{1.f, 0.f, expo != nullptr};
  if (e.on) {
    e.gain = expf(expo[2 * r]);
    e.offset = expo[2 * r + 1];
  }
  return e;
}

// Block sums of the exposure-gradient terms (sum g' e^a C and sum g' over
// the block's pixels and channels, g' = dL/dC' before the 1/|Omega| scale).
__device__ __forceinline__ void exposure_partials(float sa, float sb, float* epart) {
  sa = wave_sum(sa);
  sb = wave_sum(sb);
  __shared__ float we[4][2];
  if ((threadIdx.x & 63) == 0) { we[threadIdx.x >> 6][0] = sa; we[threadIdx.x >> 6][1] = sb; }
  __syncthreads();
  if (threadIdx.x < 2) {
    const int q = threadIdx.x;
    epart[2 * (int64_t)blockIdx.x + q] = (we[0][q] + we[1][q]) + (we[2][q] + we[3][q]);
  }
}

// One pixel's inputs to the loss kernels.
struct PixIn {
  float td, pd, al, pc[3], tc[3];
};

// Loads every pixel of the thread (kLossPix, 256 apart) before any is used,
// so the thread waits for memory once; pixels past the image read as zero.
// Targets come batch-laid-out (tgt_* non-null) or per render from the job.
__device__ __forceinline__ void load_pixels(const JobDev& J, int64_t hw, int64_t b0, const float* __restrict__ pred_rgb,
                                            const float* __restrict__ pred_depth,
                                            const float* __restrict__ pred_alpha,
                                            const float* __restrict__ tgt_rgb,
                                            const float* __restrict__ tgt_depth, PixIn (&in)[kLossPix]) {
#pragma unroll
  for (int k = 0; k < kLossPix; ++k) {
    const int64_t p = b0 + (int64_t)k * 256 + threadIdx.x;
    PixIn v{0.f, 0.f, 0.f, {0.f, 0.f, 0.f}, {0.f, 0.f, 0.f}};
    if (p < hw) {
      const int64_t pi = J.pix_off + p;
      const int64_t ci = 3 * J.pix_off + p;
      const float* trgb = tgt_rgb ? tgt_rgb + ci : J.tgt_rgb + p;
      v.td = tgt_depth ? tgt_depth[pi] : J.tgt_depth[p];
      v.pd = pred_depth[pi];
      if (pred_alpha) v.al = pred_alpha[pi];
#pragma unroll
      for (int ch = 0; ch < 3; ++ch) {
        v.pc[ch] = pred_rgb[ci + ch * hw];
        v.tc[ch] = trgb[ch * hw];
      }
    }
    in[k] = v;
  }
}

// Per block of 1024 pixels (blocks never straddle renders): writes sign
// gradients on valid pixels and the block's (sum |residual|, valid count);
// with exposure coefficients the colour residual is taken on exp(a) C + b,
// the colour gradient carries the factor exp(a) and epart receives the
// block's exposure-gradient terms.
__global__ __launch_bounds__(256) void k_loss_l1(const JobDev* __restrict__ jobs, const int32_t* __restrict__ pblk_off,
                                                 int R, const float* __restrict__ pred_rgb,
                                                 const float* __restrict__ pred_depth,
                                                 const float* __restrict__ tgt_rgb,
                                                 const float* __restrict__ tgt_depth, float* __restrict__ g_rgb,
                                                 float* __restrict__ g_depth, float* __restrict__ part,
                                                 const float* __restrict__ expo, float* __restrict__ epart) {
  const int r = find_segment<int32_t>(pblk_off, R, (int32_t)blockIdx.x);
  const JobDev& J = jobs[r];
  const int64_t hw = (int64_t)J.W * J.H;
  const int64_t b0 = (int64_t)(blockIdx.x - pblk_off[r]) * kLossBlockPix;
  const Exposure ex = exposure_of(expo, r);
  float s = 0.f, cnt = 0.f, sa = 0.f, sb = 0.f;
  PixIn in[kLossPix];
  load_pixels(J, hw, b0, pred_rgb, pred_depth, nullptr, tgt_rgb, tgt_depth, in);
#pragma unroll
  for (int k = 0; k < kLossPix; ++k) {
    const int64_t p = b0 + (int64_t)k * 256 + threadIdx.x;
    if (p >= hw) continue;
    const int64_t pi = J.pix_off + p;
    const int64_t ci = 3 * J.pix_off + p;
    const float td = in[k].td;
    const bool valid = td > 0.f;
    float l = 0.f;
    const float dd = in[k].pd - td;
    l += fabsf(dd);
    if (g_depth) g_depth[pi] = valid ? (dd > 0.f ? 1.f : (dd < 0.f ? -1.f : 0.f)) : 0.f;
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) {
      const float pc = in[k].pc[ch];
      const float dc = (ex.on ? ex.gain * pc + ex.offset : pc) - in[k].tc[ch];
      l += fabsf(dc);
      const float sg = dc > 0.f ? 1.f : (dc < 0.f ? -1.f : 0.f);
      if (g_rgb) g_rgb[ci + ch * hw] = valid ? (ex.on ? ex.gain * sg : sg) : 0.f;
      if (valid && ex.on) {
        sa += sg * ex.gain * pc;
        sb += sg;
      }
    }
    if (valid) { s += l; cnt += 1.f; }
  }
  if (epart) exposure_partials(sa, sb, epart);
  s = wave_sum(s);
  cnt = wave_sum(cnt);
  __shared__ float ws[4][2];
  if ((threadIdx.x & 63) == 0) { ws[threadIdx.x >> 6][0] = s; ws[threadIdx.x >> 6][1] = cnt; }
  __syncthreads();
  if (threadIdx.x < 2) {
    const int q = threadIdx.x;
    part[2 * (int64_t)blockIdx.x + q] = (ws[0][q] + ws[1][q]) + (ws[2][q] + ws[3][q]);
  }
}

// One wave per render: ordered sum of the block partials; with exposure
// partials, also dL/d(a, b) = (1/|Omega|) (sum g' e^a C, sum g').  clear: the
// last histograms of the median selection, zeroed for the next call.
__global__ void k_loss_reduce(const int32_t* __restrict__ pblk_off, int R, const float* __restrict__ part,
                              float* __restrict__ loss, float* __restrict__ scale, const float* __restrict__ epart,
                              float* __restrict__ egrad, uint32_t* __restrict__ clear) {
  const int r = blockIdx.x;
  if (r >= R) return;
  if (clear)
#pragma unroll
    for (int i = 0; i < kSelBins / 256; ++i)
      reinterpret_cast<uint4*>(clear + (int64_t)r * kSelBins)[i * 64 + threadIdx.x] = make_uint4(0u, 0u, 0u, 0u);
  float s = 0.f, c = 0.f, sa = 0.f, sb = 0.f;
  for (int b = pblk_off[r] + threadIdx.x; b < pblk_off[r + 1]; b += 64) {
    s += part[2 * (int64_t)b];
    c += part[2 * (int64_t)b + 1];
    if (epart) {
      sa += epart[2 * (int64_t)b];
      sb += epart[2 * (int64_t)b + 1];
    }
  }
  s = wave_sum(s);
  c = wave_sum(c);
  if (epart) {
    sa = wave_sum(sa);
    sb = wave_sum(sb);
  }
  if (threadIdx.x == 0) {
    const float inv = c > 0.f ? 1.f / c : 0.f;
    if (loss) loss[r] = c > 0.f ? s / c : 0.f;
    if (scale) scale[r] = inv;
    if (egrad) {
      egrad[2 * r] = sa * inv;
      egrad[2 * r + 1] = sb * inv;
    }
  }
}

// Per-render L1 loss from the partials {sum, count} per 8x8 band that the
// compositing backward wrote with L1 targets: one block per render, strided
// per-thread sums, wave sums, then the waves in order.  Bound by its loads'
// latency: 1,024 threads with eight loads in flight each (1200 x 680, 12,900
// partials: 4.7 us, against 6.7 us with 256 threads and four).
constexpr int kTileLossThreads = 1024;
__global__ __launch_bounds__(kTileLossThreads) void k_tile_loss_reduce(const JobDev* __restrict__ jobs, int R,
                                                                       const float* __restrict__ part,
                                                                       float* __restrict__ loss) {
  constexpr int kWaves = kTileLossThreads / 64;
  __shared__ float ws[2][kWaves];
  const int r = blockIdx.x;
  if (r >= R) return;
  const JobDev& J = jobs[r];
  const int nt = 4 * J.TX * J.TY;
  const float2* p2 = reinterpret_cast<const float2*>(part) + 4 * (int64_t)J.tile_off;
  float s = 0.f, c = 0.f;
  for (int t0 = threadIdx.x; t0 < nt; t0 += 8 * kTileLossThreads) {
    float2 v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int t = t0 + k * kTileLossThreads;
      v[k] = t < nt ? p2[t] : make_float2(0.f, 0.f);
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      s += v[k].x;
      c += v[k].y;
    }
  }
  s = wave_sum(s);
  c = wave_sum(c);
  if ((threadIdx.x & 63) == 0) {
    ws[0][threadIdx.x >> 6] = s;
    ws[1][threadIdx.x >> 6] = c;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    float ts = 0.f, tc = 0.f;
#pragma unroll
    for (int k = 0; k < kWaves; ++k) {
      ts += ws[0][k];
      tc += ws[1][k];
    }
    loss[r] = tc > 0.f ? ts / tc : 0.f;
  }
}

// ---------------------------------------------------------------------------
// Tracking loss with masks (Eq. 2 and the supplement's tracking-loss
// details).  The inlier mask needs, per render, the median of the depth
// error e = |D - D*| over pixels with D* > 0.  It is found exactly by radix
// selection on the bit patterns of the non-negative FP32 errors (their
// unsigned order is their numeric order): three passes over 11, 11 and 10
// bits, each a histogram of the errors that match the digits fixed so far.
// The digit that holds the element of rank floor((n-1)/2) is found by every
// block of the next kernel for itself, from the finished histogram (8 KB, 0.7
// us): a launch of its own took 3.4 us, three times per loss (tracking step of
// 4,096 items at 160 x 120: 105 -> 98 us, of 97k at 640 x 480: 214 -> 206 us).
// A histogram
// is zeroed again by a kernel after its last reader (no memset, so the
// sequence can be captured in a graph).

struct SelState {
  uint32_t prefix, mask, k, n;
};

// The selection workspace of R renders: the state after the first and after
// the second digit, then three histograms per render.
struct SelWork {
  SelState* state;  // [2][R]
  uint32_t* hist;   // [3][R][kSelBins]
  int R;
  __device__ __forceinline__ uint32_t* bins(int pass, int r) const {
    return hist + ((int64_t)pass * R + r) * kSelBins;
  }
};

__device__ __forceinline__ int sel_shift(int pass) { return pass == 0 ? 21 : (pass == 1 ? 10 : 0); }
__device__ __forceinline__ int sel_bins(int pass) { return pass == 2 ? 1024 : 2048; }

__device__ __forceinline__ float depth_error(float d, float t) { return fabsf(d - t); }

// State after digit `pass` of render r, from that digit's histogram and the
// state before; every thread of the block (256) calls it and gets the result.
__device__ __forceinline__ SelState sel_next(const SelWork& w, int r, int pass) {
  __shared__ uint32_t wsum[4];
  __shared__ SelState found;
  const int shift = sel_shift(pass), nb = sel_bins(pass);
  const int per = nb / 256;  // 8 or 4 bins per thread
  const uint4* g = reinterpret_cast<const uint4*>(w.bins(pass, r) + threadIdx.x * per);
  const uint4 a = g[0], b = per > 4 ? g[1] : make_uint4(0u, 0u, 0u, 0u);
  SelState st{0u, 0u, 0u, 0u};
  if (pass > 0) st = w.state[(pass - 1) * w.R + r];
  const uint32_t c[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
  uint32_t mine = 0;
#pragma unroll
  for (int j = 0; j < 8; ++j) mine += c[j];
  // block-wide exclusive scan of the per-thread sums
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  uint32_t incl = mine;
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(incl, o, 64);
    if (lane >= o) incl += y;
  }
  if (lane == 63) wsum[wv] = incl;
  __syncthreads();
  uint32_t before = incl - mine;
  for (int k = 0; k < wv; ++k) before += wsum[k];
  if (pass == 0) {
    st.n = wsum[0] + wsum[1] + wsum[2] + wsum[3];
    st.k = st.n ? (st.n - 1u) / 2u : 0u;
  }
  if (st.n == 0u) return st;  // the same for every thread
  if (st.k >= before && st.k < before + mine) {  // in one thread
    uint32_t cum = before;
    int d = 0;
#pragma unroll
    for (int j = 0; j < 7; ++j) {
      const bool past = d == j && st.k >= cum + c[j];
      cum += past ? c[j] : 0u;
      d += past ? 1 : 0;
    }
    found = SelState{st.prefix | ((uint32_t)(threadIdx.x * per + d) << shift), st.mask | ((uint32_t)(nb - 1) << shift),
                     st.k - cum, st.n};
  }
  __syncthreads();
  return found;
}

__device__ __forceinline__ void clear_bins(uint32_t* bins, bool first) {
  if (!first) return;
  for (int i = threadIdx.x; i < kSelBins; i += 256) bins[i] = 0u;
}

// Histogram of the depth errors' digit of this pass.  kMany: `per` pieces of
// kLossBlockPix pixels to a block and `share` blocks to a render (some past a smaller
// render's end); else one piece, without the loop.
template <bool kMany>
__global__ __launch_bounds__(256) void k_err_hist(const JobDev* __restrict__ jobs, const int32_t* __restrict__ pblk_off,
                                                  int R, const float* __restrict__ pred_depth,
                                                  const float* __restrict__ tgt_depth, SelWork sel, int pass, int per,
                                                  int share) {
  __shared__ uint32_t h[kSelBins];
  const int r = kMany ? (int)blockIdx.x / share : find_segment<int32_t>(pblk_off, R, (int32_t)blockIdx.x);
  const JobDev& J = jobs[r];
  const int64_t hw = (int64_t)J.W * J.H;
  const int64_t piece = kMany ? (int64_t)(blockIdx.x - r * share) * per : (int64_t)blockIdx.x - pblk_off[r];
  const int64_t b0 = piece * kLossBlockPix;
  if (kMany && b0 >= hw) return;
  const bool first = piece == 0;  // the render's first block
  const int shift = sel_shift(pass), nb = sel_bins(pass);
  // every pixel of the thread is loaded before any is counted (one wait for
  // memory, overlapping the histogram clear)
  float td[kLossPix], pd[kLossPix];
#pragma unroll
  for (int k = 0; k < kLossPix; ++k) {
    const int64_t p = b0 + (int64_t)k * 256 + threadIdx.x;
    const bool in = p < hw;
    td[k] = in ? (tgt_depth ? tgt_depth[J.pix_off + p] : J.tgt_depth[p]) : 0.f;
    pd[k] = in ? pred_depth[J.pix_off + p] : 0.f;
  }
  for (int i = threadIdx.x; i < nb; i += 256) h[i] = 0u;
  SelState st{0u, 0u, 0u, 0u};
  if (pass > 0) {
    st = sel_next(sel, r, pass - 1);
    if (first && threadIdx.x == 0) sel.state[(pass - 1) * R + r] = st;
    if (pass == 2) clear_bins(sel.bins(0, r), first);
  }
  __syncthreads();
  for (int i = 0;;) {
    float td1[kLossPix], pd1[kLossPix];
    const bool more = kMany && ++i < per && b0 + (int64_t)i * kLossBlockPix < hw;
    if (more) {
#pragma unroll
      for (int k = 0; k < kLossPix; ++k) {  // the next piece, while this one is counted
        const int64_t p = b0 + (int64_t)i * kLossBlockPix + (int64_t)k * 256 + threadIdx.x;
        const bool in = p < hw;
        td1[k] = in ? (tgt_depth ? tgt_depth[J.pix_off + p] : J.tgt_depth[p]) : 0.f;
        pd1[k] = in ? pred_depth[J.pix_off + p] : 0.f;
      }
    }
#pragma unroll
    for (int k = 0; k < kLossPix; ++k) {
      if (!(td[k] > 0.f)) continue;  // out-of-image pixels carry td = 0
      const uint32_t bits = __float_as_uint(depth_error(pd[k], td[k]));
      if ((bits & st.mask) == st.prefix) atomicAdd(&h[(bits >> shift) & (uint32_t)(nb - 1)], 1u);
    }
    if (!more) break;
#pragma unroll
    for (int k = 0; k < kLossPix; ++k) {
      td[k] = td1[k];
      pd[k] = pd1[k];
    }
  }
  __syncthreads();
  uint32_t* __restrict__ g = sel.bins(pass, r);
  for (int i = threadIdx.x; i < nb; i += 256)
    if (h[i]) atomicAdd(&g[i], h[i]);
}

// Per block of 1024 pixels: the masked, weighted L1 of Eq. 2 with its
// gradient w.r.t. the rendered colour and depth (the alpha weight is a
// constant), and the block's (sum, valid count) partials.
__global__ __launch_bounds__(256) void k_loss_track(const JobDev* __restrict__ jobs,
                                                    const int32_t* __restrict__ pblk_off, int R,
                                                    const float* __restrict__ pred_rgb,
                                                    const float* __restrict__ pred_depth,
                                                    const float* __restrict__ pred_alpha,
                                                    const float* __restrict__ tgt_rgb,
                                                    const float* __restrict__ tgt_depth,
                                                    SelWork sel, float* __restrict__ median, float lambda_c,
                                                    float inlier_k, int alpha_power, float* __restrict__ g_rgb,
                                                    float* __restrict__ g_depth, float* __restrict__ part,
                                                    const float* __restrict__ expo, float* __restrict__ epart) {
  const int r = find_segment<int32_t>(pblk_off, R, (int32_t)blockIdx.x);
  const JobDev& J = jobs[r];
  const int64_t hw = (int64_t)J.W * J.H;
  const int64_t b0 = (int64_t)(blockIdx.x - pblk_off[r]) * kLossBlockPix;
  const Exposure ex = exposure_of(expo, r);
  float s = 0.f, cnt = 0.f, sa = 0.f, sb = 0.f;
  PixIn in[kLossPix];
  load_pixels(J, hw, b0, pred_rgb, pred_depth, alpha_power > 0 ? pred_alpha : nullptr, tgt_rgb, tgt_depth, in);
  float thr = 0.f;
  if (inlier_k > 0.f) {
    const SelState st = sel_next(sel, r, 2);
    const float med = st.n ? __uint_as_float(st.prefix) : 0.f;
    const bool first = (int)blockIdx.x == pblk_off[r];
    if (first && threadIdx.x == 0) median[r] = med;
    clear_bins(sel.bins(1, r), first);
    thr = inlier_k * med;
  }
#pragma unroll
  for (int k = 0; k < kLossPix; ++k) {
    const int64_t p = b0 + (int64_t)k * 256 + threadIdx.x;
    if (p >= hw) continue;
    const int64_t pi = J.pix_off + p;
    const int64_t ci = 3 * J.pix_off + p;
    const float td = in[k].td;
    const bool valid = td > 0.f;
    const float dd = in[k].pd - td;
    float w = 0.f;
    if (valid && (inlier_k <= 0.f || depth_error(in[k].pd, td) <= thr)) {
      w = 1.f;
      if (alpha_power > 0) {
        const float a = in[k].al;
        for (int e = 0; e < alpha_power; ++e) w *= a;
      }
    }
    const float wc = w * lambda_c, wd = w * (1.f - lambda_c);
    float lc = 0.f;
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) {
      const float pc = in[k].pc[ch];
      const float dc = (ex.on ? ex.gain * pc + ex.offset : pc) - in[k].tc[ch];
      lc += fabsf(dc);
      const float gc = dc > 0.f ? wc : (dc < 0.f ? -wc : 0.f);
      if (g_rgb) g_rgb[ci + ch * hw] = ex.on ? ex.gain * gc : gc;
      if (ex.on) {
        sa += gc * ex.gain * pc;
        sb += gc;
      }
    }
    if (g_depth) g_depth[pi] = dd > 0.f ? wd : (dd < 0.f ? -wd : 0.f);
    if (valid) {
      s += wc * lc + wd * fabsf(dd);
      cnt += 1.f;
    }
  }
  if (epart) exposure_partials(sa, sb, epart);
  s = wave_sum(s);
  cnt = wave_sum(cnt);
  __shared__ float ws[4][2];
  if ((threadIdx.x & 63) == 0) { ws[threadIdx.x >> 6][0] = s; ws[threadIdx.x >> 6][1] = cnt; }
  __syncthreads();
  if (threadIdx.x < 2) {
    const int q = threadIdx.x;
    part[2 * (int64_t)blockIdx.x + q] = (ws[0][q] + ws[1][q]) + (ws[2][q] + ws[3][q]);
  }
}

struct AdamArgs {
  float* param[16];
  float* grad[16];
  float* m[16];
  float* v[16];
  int64_t n[16];
  float lr[16];
};

__global__ __launch_bounds__(256) void k_adam(AdamArgs a, float beta1, float beta2, float eps, float bc1, float bc2,
                                              int zero_grad) {
  const int gidx = blockIdx.y;
  const int64_t n = a.n[gidx];
  float* __restrict__ p = a.param[gidx];
  float* __restrict__ g = a.grad[gidx];
  float* __restrict__ m = a.m[gidx];
  float* __restrict__ v = a.v[gidx];
  const float lr = a.lr[gidx];
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    float pi = p[i], mi = m[i], vi = v[i];
    adam_update(pi, mi, vi, g[i], lr, beta1, beta2, eps, bc1, bc2);
    p[i] = pi;
    m[i] = mi;
    v[i] = vi;
    if (zero_grad) g[i] = 0.f;
  }
}

}  // namespace ls

namespace ls {
void launch_loss_l1(const JobDev* jobs, const int32_t* pblk_off_d, int R, int npblk, const float* pred_rgb,
                    const float* pred_depth, const float* tgt_rgb, const float* tgt_depth, float* g_rgb,
                    float* g_depth, float* part, float* loss, float* scale, hipStream_t s, const float* expo,
                    float* epart, float* egrad) {
  if (npblk > 0)
    hipLaunchKernelGGL(k_loss_l1, dim3(npblk), dim3(256), 0, s, jobs, pblk_off_d, R, pred_rgb, pred_depth, tgt_rgb,
                       tgt_depth, g_rgb, g_depth, part, expo, epart);
  hipLaunchKernelGGL(k_loss_reduce, dim3(R), dim3(64), 0, s, pblk_off_d, R, (const float*)part, loss, scale,
                     (const float*)epart, egrad, (uint32_t*)nullptr);
}

constexpr int kHistBlocks = 1024;
void launch_loss_track(const JobDev* jobs, const int32_t* pblk_off_d, int R, int npblk, int max_pblk,
                       const float* pred_rgb,
                       const float* pred_depth, const float* pred_alpha, const float* tgt_rgb, const float* tgt_depth,
                       float lambda_c, float inlier_k, int alpha_power, uint32_t* sel, float* median, float* g_rgb,
                       float* g_depth, float* part, float* loss, float* scale, hipStream_t s, const float* expo,
                       float* epart, float* egrad) {
  const SelWork w{reinterpret_cast<SelState*>(sel), sel + 8 * (int64_t)R, R};
  const bool select = inlier_k > 0.f;
  if (npblk > 0) {
    // Each block of the histograms reads the last pass's bins and adds its own to the
    // render's, which takes as long as a piece of its pixels.  So past kHistBlocks
    // pieces a block has several (loss without and with, us: 4096 x 4096 974 and 352,
    // 2048 x 1536 183 and 102, 16 x 1920 x 1080 661 and 481; at 512 blocks the last
    // 547, at 2,048 the second 116), unless renders of very different sizes would
    // leave most blocks without one.
    const int per = (npblk + kHistBlocks - 1) / kHistBlocks, share = (max_pblk + per - 1) / per;
    const bool many = per > 1 && (int64_t)share * R <= npblk;
    if (select)
      for (int pass = 0; pass < 3; ++pass)
        hipLaunchKernelGGL(many ? k_err_hist<true> : k_err_hist<false>, dim3(many ? share * R : npblk), dim3(256), 0, s,
                           jobs, pblk_off_d, R, pred_depth, tgt_depth, w, pass, per, share);
    hipLaunchKernelGGL(k_loss_track, dim3(npblk), dim3(256), 0, s, jobs, pblk_off_d, R, pred_rgb, pred_depth,
                       pred_alpha, tgt_rgb, tgt_depth, w, median, lambda_c, inlier_k, alpha_power, g_rgb, g_depth,
                       part, expo, epart);
  }
  hipLaunchKernelGGL(k_loss_reduce, dim3(R), dim3(64), 0, s, pblk_off_d, R, (const float*)part, loss, scale,
                     (const float*)epart, egrad, select ? w.hist + 2 * (int64_t)R * kSelBins : nullptr);
}

void launch_tile_loss_reduce(const JobDev* jobs, int R, const float* loss_part, float* loss, hipStream_t s) {
  if (R > 0) hipLaunchKernelGGL(k_tile_loss_reduce, dim3(R), dim3(kTileLossThreads), 0, s, jobs, R, loss_part, loss);
}

void launch_adam(const ls_adam_group* g, int ng, float beta1, float beta2, float eps, float bc1, float bc2,
                 int zero_grad, hipStream_t s) {
  AdamArgs a{};
  int64_t maxn = 0;
  for (int i = 0; i < ng; ++i) {
    a.param[i] = g[i].param;
    a.grad[i] = g[i].grad;
    a.m[i] = g[i].m;
    a.v[i] = g[i].v;
    a.n[i] = g[i].n;
    a.lr[i] = g[i].lr;
    maxn = std::max(maxn, g[i].n);
  }
  if (maxn == 0) return;
  const int64_t bx = std::min<int64_t>((maxn + 255) / 256, 2048);
  hipLaunchKernelGGL(k_adam, dim3((unsigned)bx, ng), dim3(256), 0, s, a, beta1, beta2, eps, bc1, bc2, zero_grad);
}
}  // namespace ls
