// Host-side launchers of the gfx950 kernels (defined next to each kernel).
#pragma once

#include <algorithm>

#include "common.h"

namespace ls {

// Error reporting of the C ABI (api.cpp): set the thread's ls_last_error()
// text and return `st`; turn a pending HIP error into LS_ERR_HIP.
ls_status api_fail(ls_status st, const char* msg);
ls_status api_hip_check(const char* what);

void launch_fill_i32(int32_t* p, int64_t n, int32_t v, hipStream_t s);

// Copies of the image-space gradient accumulators, `stride` floats apart (a power
// of two of them; 1: the accumulators alone).
struct GradCopies {
  int n;
  int64_t stride;
};

struct ViewOpt;
// live (or NULL: every render) gates each render on its active flag: the
// items of a frozen render project to radius 0, so it has no tile instances.
void launch_project(const JobDev* jobs, const int32_t* blk_off, int R, int nblk, const float* pose, float* rec,
                    int32_t* radius, int32_t* tiles, float* aux, const ViewOpt* live, hipStream_t s);

// One Adam update of a parameter from its gradient, with explicit FMAs so
// that every kernel applying it (k_adam, the fused backward) gives the same
// bits.
__device__ __forceinline__ void adam_update(float& p, float& m, float& v, float g, float lr, float beta1, float beta2,
                                            float eps, float bc1, float bc2) {
  m = __builtin_fmaf(beta1, m, (1.f - beta1) * g);
  v = __builtin_fmaf(beta2, v, (1.f - beta2) * g * g);
  p -= lr * (m * bc1) / (sqrtf(v * bc2) + eps);
}

// Adam state of the fused projection backward: per render (at most
// kAdamRenders) and per parameter array (mean, log_scale, quat, opacity,
// rgb) the moments and the learning rate; bias corrections of the step.
constexpr int kAdamRenders = 16;
struct GaussAdamArgs {
  float* m[kAdamRenders][5];
  float* v[kAdamRenders][5];
  float lr[kAdamRenders][5];
  float beta1, beta2, eps, bc1, bc2;
  // optional pose step in the pose reduction: [R][7] pose and moments (NULL: none)
  float* pose;
  float* pose_m;
  float* pose_v;
  float lr_rot, lr_trans;
};

// adam (or NULL): instead of accumulating the Gaussian gradients into grads,
// apply one Adam step to each Gaussian's parameters (the arrays its render
// job points to) from its gradient; culled items step with zero gradients.
void launch_project_bwd(const JobDev* jobs, const int32_t* blk_off, int R, int nblk, const float* pose,
                        const int32_t* radius, const float* aux, float* g2d, GradCopies copies,
                        const GradDev* grads, int want_gauss,
                        float* pose_part, int want_pose, float* pose_grad, hipStream_t s,
                        const GaussAdamArgs* adam = nullptr);
void launch_pose_reduce_tiles(const JobDev* jobs, int R, const float* pose, const float* tile_part, float* pose_grad,
                              hipStream_t s);

// Segments of a radix sort: segment s holds its keys at base[s] ..
// base[s] + len[s] and owns the sort blocks blk_off[s] .. blk_off[s + 1), one
// per `per` x kSortThreads keys of the most it may hold.  All arrays on the
// device.
struct SegTable {
  const int32_t* blk_off;  // [S + 1]
  const int64_t* base;     // [S]
  int S;
  int32_t* len;            // [S]
};
inline int sort_blocks_of(int64_t n, int per) { return (int)((n + per * kSortThreads - 1) / (per * kSortThreads)); }
// Keys per thread of a sort block, 1 to 4, for segments of up to max_n keys in
// `blocks(per)` blocks in all.  Short blocks use more CUs, but every block adds
// up its segment's counts, 64 blocks' in one round of loads, and a second round
// of blocks costs a whole block's time.  So: one key if the largest segment has
// up to 64 such blocks and each has a CU to itself, else the fewest from two with
// which all blocks are on the chip at once (two on each of 256 CUs).  Binning of
// renders with 1 and 2 keys: 17k items 56.7 and 61.2 us, 65k 68.1 and 70.6, 97k
// 77.3 and 76.7, 200k 109 and 103, 10 x 17k (170 blocks) 81.4 and 83.6, 16 x 20k
// (320) 98.8 and 92.4, 3 x 80k 90.1 and 88.1; with 2, 3 and 4: 97k 77.5, 80.5
// and 84.2, 200k 102, 105 and 107, 3 x 80k 90, 92 and 96, 8 x 150k 210 (586
// blocks), 192 (391) and 200, 16 x 135k 172, 154 (704) and 148.
constexpr int kSortResident = 512;
template <class Blocks>
inline int sort_per(int64_t max_n, const Blocks& blocks) {
  constexpr int kRound = 64, kCus = kSortResident / 2;
  if (sort_blocks_of(max_n, 1) <= kRound && blocks(1) <= kCus) return 1;
  int per = 2;
  while (per < kSortPerMax && blocks(per) > kSortResident) ++per;
  return per;
}
// Room for the sort blocks of these sizes and of all smaller ones (blocks fall
// where sort_per rises): a workspace for some size serves the smaller ones.
template <class Blocks>
inline int64_t sort_blocks_room(const Blocks& blocks) {
  return std::max<int64_t>(blocks(kSortPerMax), std::min<int64_t>(blocks(1), kSortResident));
}
// Words of the digit histograms of `blocks` sort blocks and of the `segments`'
// digit totals.
int64_t seg_hist_words(int64_t blocks, int segments);
// One stable pass over the digit of `bits` <= 8 bits at `shift` (binning.hip), from
// (kin, vin) to (kout, vout); last: kout is not written.  rows: the largest
// segment's sort blocks.
void launch_seg_pass(const uint32_t* kin, const uint32_t* vin, uint32_t* kout, uint32_t* vout, const SegTable& seg,
                     int blocks, int rows, int per, int shift, int bits, uint32_t* hist, bool last, hipStream_t s);

// Device tables of a batch's binning: per render the sort blocks, the chunk x
// window work units and the count matrices (chunks x tiles words) before it.
struct BinTables {
  const int32_t* blk_off;   // [R + 1]
  const int32_t* work_off;  // [R + 1]
  const int64_t* cnt_off;   // [R + 1]
  int R;
  int chunk;                // sorted items per chunk
  bool ramp;                // the first chunks are smaller
};
// Tile windows of a render and chunks of n sorted items (host tables).
int windows_of(int TX, int TY);
int bin_chunks(int n, int chunk, bool ramp);

// Workspace of the pair sort (binning_pairs.hip); all NULL where the lists are not
// made by it.
struct PairSegs {
  int32_t* blk_off;  // [2]
  int64_t* base;     // [1]
};
struct PairLaunch {
  int32_t* kept_off;  // [R + 1]
  uint64_t* bsum;     // [pair_item_blocks(M)]
  uint32_t* first;    // [pair_spans_room(cap)]
  uint32_t *tk, *tv;  // [cap]
  uint32_t* hist;     // seg_hist_words(pair_sort_blocks_room(cap), 1)
  PairSegs seg;
};
int64_t pair_item_blocks(int64_t M);
// Room for the spans of every capacity up to `cap`, as of the sort blocks.
int64_t pair_spans_room(int64_t cap);
inline int64_t pair_sort_blocks_room(int64_t cap) {
  return sort_blocks_room([&](int per) { return sort_blocks_of(cap, per); });
}

struct BinLaunch {
  const JobDev* jobs;
  const int64_t* item_off;
  const int32_t* tile_off;
  BinTables tab;
  int T, max_items, sort_blocks, sort_per, units, blocks256;
  const int32_t* off256;        // [R + 1]: first block of 256 items of each render; blocks256 of them
  int64_t rank_pairs;           // sum over the renders of the squared item count
  int64_t counts;               // words of the count matrices
  int64_t M;                    // items
  PairLaunch pairs;
  const float* rec;
  const int32_t* radius;
  const int32_t* tiles;
  int64_t cap;
  uint32_t *k0, *v0, *k1, *v1;  // sort buffers [M]
  uint32_t* hist;               // seg_hist_words(sort_blocks, R)
  int32_t* blk_cnt;             // [sort_blocks]
  int32_t* kept;                // [R]: items with tiles
  uint32_t* cnt;                // count matrices
  uint32_t* tile_total;         // [T]
  uint32_t* tile_before;        // [T]: totals of the tiles before it in its group of 64
  uint64_t* groups;             // [ceil(T / 64) + 1]: totals of the groups, and room for their sum
  uint32_t* tile_of;
  int32_t* item;
  int32_t* range;
  int32_t* count;
};
void launch_bin_sort(const BinLaunch& b, hipStream_t s);
// The lists from the depth order (v0, kept) by a sort of pairs.
void launch_bin_pairs(const BinLaunch& b, hipStream_t s);

// used: 4 rows (one per band) of ustride = used_slots(capacity, T) 64-bit
// words; the forward sets bit l of slot (start / 64) + tile + k of row q when
// some pixel of band q composited list entry start + 64 k + l of the tile
// (chunks a band never walked keep old bits: the backward reads only
// positions below the band's largest n_last).
inline int64_t used_slots(int64_t cap, int T) { return cap / 64 + T + 2; }
void launch_composite_fwd(const JobDev* jobs, const int32_t* tile_off, int R, int T, const float* rec,
                          const int32_t* items, const int32_t* range, const float* bg, float* rgb, float* depth,
                          float* alpha, float* Tf, int32_t* nl, uint64_t* used, int64_t ustride, hipStream_t s);

// The plain colour + depth L1 of registration (Sec. 3.2), formed per pixel
// by the pose-only backward itself from the forward's images and the targets
// instead of read from a loss kernel's gradient images: on pixels with a
// target depth, sign(rendered - target) per colour channel and for depth,
// times the render's 1 / |Omega| (up_scale); 0 elsewhere.  Targets in the
// batch's image layout, or NULL: each render's own (JobDev.tgt_*).  With
// loss_part, each 8x8 band also writes {sum over its pixels in Omega of the L1
// terms (|D - D*| + sum_c |C_c - C*_c|), number of those pixels}.
struct L1Targets {
  const float* pred_rgb;    // forward colour [3][P]; NULL: off
  const float* pred_depth;  // forward depth [P]
  const float* tgt_rgb;
  const float* tgt_depth;
  float* loss_part;         // [4 T][2], one row per 8x8 band (4 tile + band), or NULL
};

// Per-render L1 loss from the band partials: loss[r] = sum / count over the
// render's bands in a fixed order (0 when the render has no pixel in Omega).
void launch_tile_loss_reduce(const JobDev* jobs, int R, const float* loss_part, float* loss, hipStream_t s);

// used, ustride: the flags the forward wrote for the same bins: the backward
// walks only the entries some pixel of the band composited.
void launch_composite_bwd(const JobDev* jobs, const int32_t* tile_off, int R, int T, const float* rec,
                          const float* aux, const float* pose, const int32_t* items, const int32_t* range,
                          const uint64_t* used, int64_t ustride, const float* bg, const float* Tf, const int32_t* nl,
                          const float* up_rgb,
                          const float* up_depth, const float* up_alpha, const float* up_scale,
                          float* g2d, GradCopies copies,
                          float* tile_part, int pose_only, hipStream_t s,
                          const L1Targets* l1 = nullptr);

// Registration helpers (reg_kernels.hip).
struct ViewOpt {
  float lr_rot, lr_trans;
  int32_t step;    // Adam steps taken so far
  int32_t active;  // 0: frozen (no update)
  float best;      // lowest loss seen (early exit)
  int32_t stall;   // iterations since the loss last improved on best by more than the tolerance
  float resid;     // loss at the pose the view froze at
  int32_t pad;
};
// Adam on one render's 7 pose values (lr_rot for q, lr_trans for t) from its
// gradient g, and on its 2 exposure coefficients when given (lr_expo), bias
// correction from the render's own step count; the gradients are consumed
// (zeroed).  Early exit (exit_patience > 0) freezes a view at its current
// pose (whose loss is the one just computed) instead of stepping once, for
// exit_patience iterations in a row,
//   exit_mode 0: its loss has not improved on its best by more than exit_tol
//                (relative);
//   exit_mode 1: its Adam step would have been small: the largest
//                |m_hat| / (sqrt(v_hat) + eps) over its 7 pose values (the
//                step in units of the learning rate) is below exit_tol.
// Frozen views keep their pose.
struct PoseAdamArgs {
  float* pose;
  float* grad;  // [R][7], zeroed here
  float* m;
  float* v;
  ViewOpt* opt;
  const float* loss;
  float beta1, beta2, eps, exit_tol;
  int exit_patience, exit_mode;
  float* expo;  // exposure coefficients (a, b) per render, or NULL
  float* egrad;
  float* em;
  float* ev;
  float lr_expo;
};

// One render's pose, gradient so far and moments.  A reduction loads them before
// its sums: read where they are used, seven loads wait for each other's stores
// (pose reduction with its step, 16 views of 1,200 rows: 7.8 -> 6.8 us, one of
// 782 rows: 6.0 -> 5.2 us).
struct PoseState {
  float p[7], g[7], m[7], v[7];
};
__device__ __forceinline__ PoseState load_pose_state(const float* pose, const float* grad, const float* m,
                                                     const float* v, int r) {
  PoseState s;
#pragma unroll
  for (int k = 0; k < 7; ++k) {
    s.p[k] = pose[7 * r + k];
    s.g[k] = grad[7 * r + k];
    s.m[k] = m ? m[7 * r + k] : 0.f;
    s.v[k] = m ? v[7 * r + k] : 0.f;
  }
  return s;
}

__device__ inline void pose_adam_view(const PoseAdamArgs& a, int r, const PoseState& st, ViewOpt o,
                                      const float (&g)[7]) {
  if (o.active) {
    const int step = o.step + 1;
    const float bc1 = 1.f / (1.f - __powf(a.beta1, (float)step));
    const float bc2 = 1.f / (1.f - __powf(a.beta2, (float)step));
    float mn[7], vn[7], ratio = 0.f;
#pragma unroll
    for (int k = 0; k < 7; ++k) {
      mn[k] = a.beta1 * st.m[k] + (1.f - a.beta1) * g[k];
      vn[k] = a.beta2 * st.v[k] + (1.f - a.beta2) * g[k] * g[k];
      ratio = fmaxf(ratio, fabsf(mn[k] * bc1) / (sqrtf(vn[k] * bc2) + a.eps));
    }
    bool step_now = true;
    if (a.exit_patience > 0) {
      const float l = a.loss[r];
      if (a.exit_mode == 1) {
        o.stall = ratio < a.exit_tol ? o.stall + 1 : 0;
        o.best = o.step == 0 ? l : fminf(o.best, l);
      } else if (o.step == 0 || l < o.best * (1.f - a.exit_tol)) {
        o.best = o.step == 0 ? l : fminf(o.best, l);
        o.stall = 0;
      } else {
        o.best = fminf(o.best, l);
        ++o.stall;
      }
      if (o.stall >= a.exit_patience) {
        o.active = 0;
        o.resid = l;
        step_now = false;
      }
    }
    if (step_now) {
#pragma unroll
      for (int k = 0; k < 7; ++k) {
        const int i = 7 * r + k;
        a.m[i] = mn[k];
        a.v[i] = vn[k];
        const float lr = k < 4 ? o.lr_rot : o.lr_trans;
        a.pose[i] = st.p[k] - lr * (mn[k] * bc1) / (sqrtf(vn[k] * bc2) + a.eps);
      }
      if (a.expo) {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          const int i = 2 * r + k;
          const float eg = a.egrad[i];
          const float mi = a.beta1 * a.em[i] + (1.f - a.beta1) * eg;
          const float vi = a.beta2 * a.ev[i] + (1.f - a.beta2) * eg * eg;
          a.em[i] = mi;
          a.ev[i] = vi;
          a.expo[i] -= a.lr_expo * (mi * bc1) / (sqrtf(vi * bc2) + a.eps);
        }
      }
      o.step = step;
    }
    a.opt[r] = o;
  }
#pragma unroll
  for (int k = 0; k < 7; ++k) a.grad[7 * r + k] = 0.f;
  if (a.expo) {
    a.egrad[2 * r] = 0.f;
    a.egrad[2 * r + 1] = 0.f;
  }
}

// sticky[0] |= overflow; sticky[1] keeps the instance count required at the
// first overflow (the pose before any step taken on truncated lists).
__device__ inline void or_flag(const int32_t* count, int32_t* sticky) {
  if (count[1] != 0) {
    if (sticky[0] == 0) sticky[1] = count[2];
    sticky[0] = 1;
  }
}

// Joint registration on the device (one T = T_{P->Q} per pair shared by its
// views, optimised by Adam in double precision).  Per view: its keyframe's
// rotation, translation and unit quaternion, the pair and whether it is a
// keyframe of Q; per pair: T (unnormalised quaternion, translation), its
// moments and its views [first, first + count).
struct JointView {
  double Rc[9], tc[3], qc[4];
  int32_t pair, reverse;
};
struct JointPair {
  double T[7], m[7], v[7];
  int32_t first, count;
};
struct JointAdam {
  double lr_rot, lr_trans, beta1, beta2, eps, bc1, bc2;  // bc = 1 / (1 - beta^step)
};
// pose[r] = the camera-frame correction Delta of view r under its pair's T:
// C^-1 T^-1 C for a keyframe of P, C^-1 T C for one of Q.
void launch_joint_poses(const JointView* views, int R, const JointPair* pairs, float* pose, hipStream_t s);
// One Adam step of every pair's T from its views' pose gradients (chained
// through the Jacobian of T -> Delta by central differences of that smooth
// map in double precision), then the views' new corrections; the pose
// gradients are cleared.
void launch_joint_step(const JointView* views, JointPair* pairs, int npairs, float* pose_grad, float* pose,
                       const JointAdam& a, hipStream_t s);

// One iteration's end in pose-only registration: per render, the tile
// partials reduced to its pose gradient (as launch_pose_reduce_tiles) and
// its Adam step (pose_adam_view) in one launch; render 0 also updates the
// sticky overflow flag from count (as launch_or_flag).
void launch_pose_reduce_adam(const JobDev* jobs, int R, const float* tile_part, const PoseAdamArgs& a,
                             const int32_t* count, int32_t* sticky, hipStream_t s);
void launch_pose_init(float* pose, float* m, float* v, ViewOpt* opt, int R, hipStream_t s);
void launch_or_flag(const int32_t* count, int32_t* sticky, hipStream_t s);
// Per render: fraction of the pixels with a target depth > 0 whose rendered
// alpha is >= 0.5 (part: 2 floats per 1024-pixel block).
void launch_view_coverage(const JobDev* jobs, const int32_t* pblk_off, int R, int npblk, const float* alpha,
                          const float* tgt_depth, float* part, float* coverage, hipStream_t s);
// Per-view exposure coefficients (a, b) [R][2] with their Adam moments and
// gradient, or all null.
struct ExpoState {
  float *expo, *m, *v, *grad;
};
void launch_state_remap(const float* opose, const float* om, const float* ov, const ViewOpt* oopt, float* npose,
                        float* nm, float* nv, float* ngrad, ViewOpt* nopt, const int32_t* map, const ViewOpt* init_opt,
                        int R, hipStream_t s, ExpoState oe = {}, ExpoState ne = {});
void launch_all_finite(const float* a, int64_t n, int32_t* bad, hipStream_t s);

void launch_render_stats(const JobDev* jobs, const int32_t* tile_off, int R, int T, const float* rec,
                         const int32_t* items, const int32_t* range, const int32_t* nl, int64_t* stats, hipStream_t s);

// The loss launchers take optional exposure coefficients (expo [R][2], the
// colour residual then taken on exp(a) C + b) with their block partials
// (epart, 2 floats per 1024-pixel block) and gradients (egrad [R][2]).
void launch_loss_l1(const JobDev* jobs, const int32_t* pblk_off_d, int R, int npblk, const float* pred_rgb,
                    const float* pred_depth, const float* tgt_rgb, const float* tgt_depth, float* g_rgb,
                    float* g_depth, float* part, float* loss, float* scale, hipStream_t s,
                    const float* expo = nullptr, float* epart = nullptr, float* egrad = nullptr);
// Tracking loss with masks; sel = per-render selection workspace
// (sel_words(R) uint32, zero on first use, histograms left zeroed after each
// call).
void launch_loss_track(const JobDev* jobs, const int32_t* pblk_off_d, int R, int npblk, int max_pblk,
                       const float* pred_rgb,
                       const float* pred_depth, const float* pred_alpha, const float* tgt_rgb, const float* tgt_depth,
                       float lambda_c, float inlier_k, int alpha_power, uint32_t* sel, float* median, float* g_rgb,
                       float* g_depth, float* part, float* loss, float* scale, hipStream_t s,
                       const float* expo = nullptr, float* epart = nullptr, float* egrad = nullptr);
constexpr int kSelHistBins = 2048;
inline int64_t sel_words(int R) { return (int64_t)R * (8 + 3 * kSelHistBins); }

// Mapping loss (mapping_loss.hip).  SSIM blocks of a W x H render (3 colour
// channels x 32 x 32 tiles); map_part: 3 floats per SSIM block + kValidParts + kValidPartsMany per render.
int ssim_blocks(int W, int H);
constexpr int kValidParts = 64, kValidPartsMany = 256;
void launch_loss_mapping(const JobDev* jobs, int npblk, int max_pblk, const int32_t* sblk_off_d, int nsblk, int R,
                         const float* pred_rgb,
                         const float* pred_depth, const float* tgt_rgb, const float* tgt_depth, float lambda_ssim,
                         float lambda_color, float lambda_depth, float* g_rgb, float* g_depth, float* map_part,
                         float* loss, float* scale, hipStream_t s);
// Per render 1 / |Omega| (pixels with a target depth; 0 when none) into inv
// [R]; cnt_part = npblk floats.  Targets as for L1Targets.
void launch_valid_inv(const JobDev* jobs, const int32_t* pblk_off_d, int npblk, int R, const float* tgt_depth,
                      float* cnt_part, float* inv, hipStream_t s);
// Isotropic regulariser; part = kIsotropicBlocks floats.
constexpr int kIsotropicBlocks = LS_ISOTROPIC_WORK_FLOATS;
void launch_loss_isotropic(const float* log_scale, int64_t n, float lambda_reg, float* loss, float* grad, float* part,
                           hipStream_t s);

// Map adjustment (adjust.hip): validated descriptors, any count.
int launch_adjust_submaps(const ls_submap_adjust* subs, int count, hipStream_t s);

// Opacity pruning (prune.hip): up to kPruneArrays SoA arrays [comp][n]
// compacted to [comp][count] by the keep test logit >= tau.
constexpr int kPruneArrays = 16;
struct PruneArrays {
  const float* src[kPruneArrays];
  float* dst[kPruneArrays];
  int comp[kPruneArrays];
  int count;
};
size_t prune_workspace_bytes(int n);
void launch_prune(const float* logit, int n, float tau, const PruneArrays& arr, int32_t* kept, int32_t* count,
                  void* work, hipStream_t s);

// Overlap ratio (overlap.hip).
ls_status overlap_check_args(const float* p_mean, int32_t np, const float* q_mean, int32_t nq, const float* T_pq,
                             float tau, const int32_t* nn_pq, const int32_t* nn_qp, const int32_t* counts);
size_t overlap_workspace_bytes(int np, int nq);
void launch_overlap(const float* p_mean, int np, const float* q_mean, int nq, const float* T, float tau,
                    int32_t* nn_pq, int32_t* nn_qp, int32_t* counts, void* work, hipStream_t s);

void launch_adam(const ls_adam_group* g, int ng, float beta1, float beta2, float eps, float bc1, float bc2,
                 int zero_grad, hipStream_t s);

}  // namespace ls
