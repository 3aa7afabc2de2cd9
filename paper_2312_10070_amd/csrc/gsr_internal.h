// Internal declarations of libgsr: launch-constant structs, device helpers
// shared by the forward and backward kernels, and the host-side launchers.
// gfx950 (CDNA4) only: wave64, 256-thread workgroups for the tile kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gsr.h"

namespace gsr {

constexpr float kLog2e = 1.4426950408889634f;
constexpr int kTileThreads = 256;  // one pixel per lane, 4 waves per tile
constexpr int kWave = 64;
constexpr int kRec = 4;  // float4s per projected record
// The support box is taken at level (1 + kBoxSlack) ln(o / alpha_min) + kBoxSlack
// of sigma instead of ln(o / alpha_min).
constexpr float kBoxSlack = 1e-3f;


// Launch constants of one render (by value into every kernel).
struct Raster {
  int W, H;
  int tw, th;         // tile shape (tw * th == 256)
  int tw_log2;        // log2(tw)
  int ntx, nty;       // tiles per row / column
  int n_tiles;        // ntx * nty (per view)
  float fx, fy, cx, cy, near_z;
  float lowpass, amin, amax, tmin;
  float log2_amin;    // log2(amin)
  float limx, limy;   // guard band on x/z and y/z inside the Jacobian
  float bg0, bg1, bg2;
};

// Per-Gaussian record written by the projection kernel. The quadratic form of
// Eq. 4 is stored pre-scaled so that one pair costs three FMAs:
//   p = pa dx^2 + pb dx dy + pc dy^2 = -sigma * log2(e),   alpha = o * 2^p.
//   rec_uvab = (u, v, pa, pb), rec_cob = (pc, o, bx, by), rec_rgbz = (r, g, b, z_cam)
// The three float4s of a record are interleaved in one 64-byte slot (kRec
// float4s, the fourth unused): a record gathered by its index touches one
// cache line instead of three. rec_uvab[kRec i], rec_cob[kRec i], ... address
// record i.
// where bx / by carry the pixel support box as bit patterns px0 | px1 << 16 and
// py0 | py1 << 16 (a wave skips records whose box misses its pixels).
struct PairEval {
  float alpha;   // min(alpha_max, o 2^p)
  float e;       // 2^p = exp(-sigma)
  bool use;      // alpha >= alpha_min
  bool clamped;  // o 2^p > alpha_max (alpha does not depend on o, sigma)
};

// The single definition of every per-pair discrete decision. The forward and
// the backward both call it, so skip / clamp decisions agree bit for bit. FP
// contraction is pinned: only the explicit fmaf calls fuse.
__device__ __forceinline__ PairEval eval_pair(float dx, float dy, float pa, float pb, float pc, float o,
                                              float amin, float amax) {
#pragma clang fp contract(off)
  const float t = pc * dy;
  const float p = fmaf(pa * dx, dx, fmaf(pb * dx, dy, t * dy));
  PairEval r;
  r.e = __builtin_amdgcn_exp2f(p);
  const float raw = o * r.e;
  r.clamped = raw > amax;
  r.alpha = fminf(raw, amax);  // = clamped ? amax : raw (raw is finite: p is)
  r.use = r.alpha >= amin;
  return r;
}

// Work index of a workgroup. Workgroups are dealt round-robin to the 8 XCDs
// (each with its own L2); this gives each XCD a contiguous run of row-major
// tiles so neighbouring tiles, which share most Gaussians, hit the same L2
// (the forward of few or short lists: 320x240 with 92K Gaussians 75.4 -> 73.4 us).
__device__ __forceinline__ int xcd_tile(int b, int nb) {
  const int q = nb >> 3, r = nb & 7;
  const int x = b & 7, i = b >> 3;
  return x * q + (x < r ? x : r) + i;
}

// The same with chunks of kXcdChunk consecutive indices dealt to the XCDs in
// turn: every XCD gets a share of each part of the work, so one whose part is
// dense does not end last (the backward of few or short lists, whose waves do
// not share their fetches, and the seeding queries).
constexpr int kXcdChunk = 16;
__device__ __forceinline__ int xcd_chunk(int b, int nb) {
  const int full = nb / (8 * kXcdChunk) * (8 * kXcdChunk);
  const int x = b & 7, i = b >> 3;
  return b < full ? ((i / kXcdChunk) * 8 + x) * kXcdChunk + i % kXcdChunk : b;
}

// The sum of `a` over a lane pair that differs in bit 5 (bit 4) in the lane
// whose bit is 0, and of `b` in the other one.
__device__ __forceinline__ float perm_add32(float a, float b) {
  auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(p[0]) + __uint_as_float(p[1]);
}
__device__ __forceinline__ float perm_add16(float a, float b) {
  auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(p[0]) + __uint_as_float(p[1]);
}
template <int CTRL>
__device__ __forceinline__ float dpp_f(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, false));
}
__device__ __forceinline__ int wave_max_int(int v) {
  for (int o = 32; o > 0; o >>= 1) v = max(v, __shfl_xor(v, o, 64));
  return v;
}

__device__ __forceinline__ float wave_sum_all(float v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// Rotation matrix of a unit quaternion (w, x, y, z), row-major.
__device__ __forceinline__ void quat_rot(float w, float x, float y, float z, float R[9]) {
  const float xx = x * x, yy = y * y, zz = z * z;
  const float xy = x * y, xz = x * z, yz = y * z, wx = w * x, wy = w * y, wz = w * z;
  R[0] = 1.f - 2.f * (yy + zz);
  R[1] = 2.f * (xy - wz);
  R[2] = 2.f * (xz + wy);
  R[3] = 2.f * (xy + wz);
  R[4] = 1.f - 2.f * (xx + zz);
  R[5] = 2.f * (yz - wx);
  R[6] = 2.f * (xz - wy);
  R[7] = 2.f * (yz + wx);
  R[8] = 1.f - 2.f * (xx + yy);
}

// Gradient of <G, R(q)> w.r.t. a unit quaternion, then through q / |q|.
__device__ __forceinline__ void quat_rot_vjp(const float qh[4], float inv_norm, const float G[9], float gq[4]) {
  const float w = qh[0], x = qh[1], y = qh[2], z = qh[3];
  float gw = 2.f * (x * (G[7] - G[5]) + y * (G[2] - G[6]) + z * (G[3] - G[1]));
  float gx = 2.f * (y * (G[1] + G[3]) + z * (G[2] + G[6]) + w * (G[7] - G[5])) - 4.f * x * (G[4] + G[8]);
  float gy = 2.f * (x * (G[1] + G[3]) + w * (G[2] - G[6]) + z * (G[5] + G[7])) - 4.f * y * (G[0] + G[8]);
  float gz = 2.f * (w * (G[3] - G[1]) + x * (G[2] + G[6]) + y * (G[5] + G[7])) - 4.f * z * (G[0] + G[4]);
  const float d = w * gw + x * gx + y * gy + z * gz;
  gq[0] = (gw - w * d) * inv_norm;
  gq[1] = (gx - x * d) * inv_norm;
  gq[2] = (gy - y * d) * inv_norm;
  gq[3] = (gz - z * d) * inv_norm;
}

// ---------------------------------------------------------------------------
// Host-side launchers (defined in the .hip files, called by gsr_api.cpp).
// ---------------------------------------------------------------------------

struct ProjectArgs {
  int64_t n;
  const float *means, *scales, *quats, *opacities, *colors;
  const float* pose7;  // device
  float4* rec_uvab;
  float4* rec_cob;
  float4* rec_rgbz;
  int4* rect;          // (tx0 | tx1 << 16, ty0 | ty1 << 16, depth bits, tiles); see BinArgs
  uint32_t* counts;    // tiles per Gaussian (0 = culled)
  int n_views;         // outputs are [n_views * n]; view v uses pose7 + 7 v
};
void launch_project(const Raster& R, const ProjectArgs& a, hipStream_t s);

// Exclusive scan of n uint32 values; writes the total to *total (device) and,
// if total_host is not NULL, to that device-visible pinned host word.
// temp must hold scan_temp_words(n) uint32.
int64_t scan_temp_words(int64_t n);
void launch_exclusive_scan(const uint32_t* in, uint32_t* out, int64_t n, uint32_t* total, uint32_t* temp,
                           hipStream_t s, uint32_t* total_host = nullptr);

// Seeding candidates (k_seed.hip): chosen pixels back-projected to world
// points [m,3] with their colours [m,3], in pixel order; the count goes to
// count_host (pinned, device-visible). temp: seed_sample_temp_words(W H) uint32.
struct SeedSample {
  const float *color, *depth, *alpha, *u, *pose7;  // alpha NULL: a sub-map's first keyframe
  int W, H;
  float fx, fy, cx, cy;
  float p_uniform, p_grad, g2thre, alpha_n;
};
int64_t seed_sample_temp_words(int64_t P);
void launch_seed_sample(const SeedSample& a, float* points, float* colors, uint32_t* temp, uint32_t* count_host,
                        hipStream_t s);

// New Gaussians from the kept seeding points (k_seed.hip): rows 0..n_new-1 of
// the outputs, in point order; count_host (pinned, device-visible) receives
// n_new. temp: seed_init_temp_words(m) uint32.
struct SeedInit {
  int64_t m;
  const float* points;   // [m,3]
  const float* pcolors;  // [m,3]
  const float* nn_d2;    // [m]
  const int32_t* keep;   // [m]
  float *means, *scales, *quats, *opacities, *colors;
};
int64_t seed_init_temp_words(int64_t m);
void launch_seed_init(const SeedInit& a, uint32_t* temp, uint32_t* count_host, hipStream_t s);
// Seeding neighbour queries (k_seed.hip): nn_d2[j] = min(r_max^2, min_i |q_j - p_i|^2),
// keep[j] = nn_d2[j] >= rho^2 (either output may be NULL); rho <= r_max.
// temp: seed_temp_words(n) uint32, 16-byte aligned; launch_seed_grid fills it
// with the hash grid of the means, launch_seed_query then answers the queries.
uint32_t seed_buckets(int64_t n);
int64_t seed_temp_words(int64_t n);
void launch_seed_grid(const float* means, int64_t n, float r_max, uint32_t* temp, hipStream_t s);
void launch_seed_query(int64_t n, const float* points, int64_t m, float rho, float r_max, float* nn_d2,
                       int32_t* keep, const uint32_t* temp, hipStream_t s);

// Opacity pruning / compaction: in[0..4] = means, scales, quats, opacities,
// colors (widths 3, 3, 4, 1, 3), in[5..9] / in[10..14] their Adam moments
// (NULL = absent; out[t] NULL exactly where in[t] is). Keeps the Gaussians
// with mask[i] != 0 (mask given) or opacity >= thre (mask NULL), in their
// order, at the front of out; the count goes to kept_host (pinned,
// device-visible). temp: prune_temp_words(n) uint32.
struct PruneArgs {
  const float* in[15];
  float* out[15];
};
int64_t prune_temp_words(int64_t n);
void launch_prune(const PruneArgs& a, int64_t n, float thre, const int32_t* mask, uint32_t* temp, uint32_t* kept_host,
                  hipStream_t s);

// Tile binning (see k_sort.hip). Workgroup w of view v handles the Gaussians
// [w c, (w + 1) c) with c = ceil(n / n_wg); M[v][w][tile] is the offset of
// its pairs inside the range of the (view, tile) item, R[item] that range (a
// workgroup's offsets lie side by side: written and read in runs, 1200x680 of
// 1M 24 -> 20 us counting and 24 -> 21 placing against [item][w]).
// rect[o] = (tx0 | tx1 << 16, ty0 | ty1 << 16, float bits of the camera
// depth, number of tiles; 0 = not binned): everything binning reads, 16 bytes.
struct BinArgs {
  int64_t n;
  int n_views;
  int n_wg;                // workgroups per view
  const int4* rect;
  uint32_t* M;             // [n_views][n_wg][n_tiles]
  uint32_t* T;             // [n_items] pair totals; zero between launches
  int2* R;                 // [n_items] unclipped ranges
  int* order;              // [n_items] items from the longest list to the shortest, if that pays
  bool order_always;       // or in any case
  uint32_t* ticket;        // zero between launches
  uint32_t* K;             // overlap count
  uint32_t* K_host;        // NULL or a device-visible host word that also receives K
  int64_t cap;             // positions >= cap are dropped and flagged
  uint64_t* keys;          // [cap] (depth bits << 32 | record index)
  int* overflow;
  int2* ranges;            // [n_items] written by the placement pass (NULL while counting)
};
// Do the passes over n items with K list entries go by length? With less work
// than that the order costs more than it gives: forward alone against forward
// and backward, 320x240 with 31K Gaussians (K about 65,000) 41.8 -> 45.9 us and
// 84.2 -> 85.7, 560x360 with 81K (170,000) 53.4 -> 55.1 and 112 -> 111, with
// 242K (390,000) 93.2 -> 92.0 and 207 -> 195, 800x500 with 480K 138 -> 121 and
// 329 -> 301. Nor where there are many items and most have a short list, as one
// workgroup makes the order; binning to backward, even scenes and ones with half
// of the entries in a sixteenth of the image: 262,144 items with 2 entries each
// 2551 -> 2911 us and 2437 -> 2744, with 22 3530 -> 3976 and 3901 -> 4010;
// 65,536 with 9 722 -> 794 and 776 -> 781, with 29 953 -> 1043 and 1169 -> 1029,
// with 88 1640 -> 1723 and 2296 -> 1721; 14,400 with 40 243 -> 251 and 314 ->
// 262. n is asked where the launch is made, K on the device, where it
// is known: what a state's workspace has room for says nothing about this call.
// A persistent grid's workgroups take the longest first whatever n and K are: a
// long list that one of them takes last is what the launch ends with (forward,
// 499 lists of 1500 and one of 3000 in the last tile on 256 workgroups: 261 us
// by position, 185 by length).
constexpr int kOrderItems = 512;
constexpr uint32_t kOrderEntries = 1 << 18;
__host__ __device__ __forceinline__ uint32_t order_least(int64_t n) {  // K from which on n items go by length
  const int64_t k = 24 * n > kOrderEntries ? 24 * n : kOrderEntries;
  return k < 0xffffffffll ? (uint32_t)k : 0xffffffffu;
}
struct ItemOrder {
  const int* items;   // NULL = by position
  const uint32_t* K;  // by length if *K >= least
  uint32_t least;
};
// The item that is taken i-th, where item `at` stands in for it.
__device__ __forceinline__ int item_at(const ItemOrder& o, int i, int at) {
  if (!o.items) return at;
  const int it = o.items[i];  // (read beside K, not after it)
  return *o.K >= o.least ? it : at;
}
// Compute units of the chip. (A partition of it has fewer: what follows from
// this number there is no longer the best split or order, but a right one.)
constexpr int kUnits = 256;
// Workgroups of the compositing passes that a compute unit holds (forward: 26
// of its 160 KB of LDS each; backward: 20 waves of at most 96 registers). A
// persistent grid of as many or more per compute unit bounds nothing, and one
// workgroup per item is faster, as no workgroup waits for its slowest wave
// between items: 8 views of 1200x680, 1M Gaussians, 474 -> 358 us forward
// and 986 -> 880 us backward. A smaller grid is run as asked for.
constexpr int kFwdHeld = 6, kBwdHeld = 5;

// Workgroups per view: 1,024 Gaussians each, at most 128, and over all views at
// most one per compute unit, but four per view. Every workgroup reserves room
// on every tile it meets, with an atomic on a word that all of the view's
// workgroups share: 8 views of 1M, 128 per view 120 us counting and 98 placing,
// 64 109 and 98, 32 98 and 92; one view, 256 instead of 128 24 us instead of 20
// and 21 each. 17 views of 640x480 of 200K, counting and placing with the sort,
// 15 per view 66 and 110 us, 16 (one in the last round) 72 and 122; 64 views,
// four 253 and 412, eight 262 and 411, 16 272 and 409, 32 276 and 375.
int bin_workgroups(int64_t n, int64_t views);
// M, R and K from the tile rectangles (LDS histograms, one reservation atomic
// per (tile, workgroup), the last workgroup scans the tile totals).
void launch_bin_count(const Raster& R, const BinArgs& a, hipStream_t s);
// ranges from R, slot placement (LDS counters seeded from R and M), then one
// LDS sort per tile writing ids[cap] (record indices in depth order).
// scratch: [cap] keys, used by ranges longer than LDS holds.
void launch_tile_bins(const Raster& R, const BinArgs& a, int64_t n_items, int2* ranges, uint64_t* scratch,
                      uint32_t* ids, const ItemOrder& order, hipStream_t s);

struct FwdArgs {
  const int2* ranges;
  const uint32_t* ids;
  const float4* rec_uvab;
  const float4* rec_cob;
  const float4* rec_rgbz;
  float *color, *depth, *alpha, *Tfin;  // [V,3,H,W] / [V,H,W]
  int* last;
  unsigned long long* stats;  // non-NULL: count work only, write no outputs
  int n_items;                // views * tiles; item = view * n_tiles + tile
  int* queue;                 // persistent launch: work counter (zeroed first)
  ItemOrder order;            // the order in which the items are taken
  int blocks;                 // persistent launch: workgroups (0 = one per item)
};
void launch_render_fwd(const Raster& R, const FwdArgs& a, hipStream_t s);

// The compositing backward adds a Gaussian's sums with atomics, in an order
// that varies from run to run. Up to this many (Gaussian, view) pairs the sums
// are doubles, and eight runs gave the same gradients to the bit; as floats, up
// to 1e-6 of a group's largest lay between them, and 1e-8 to 4e-7 in the norm,
// at 8,000 as at 500,000 Gaussians. What that costs, backward and projection
// backward with floats and with doubles: 8,000 Gaussians at 160x120 26.4 us and
// 26.5, 32,000 at 320x240 33.5 and 34.4, 64,000 at 480x320 43.8 and 45.1, 128,000
// at 640x480 65.2 and 67.1, 300,000 110 and 116, 500,000 at 1200x680 188 and 202:
// the line lies where it reaches about a microsecond.
constexpr int64_t kWideSums = 32768;

struct BwdArgs {
  const int2* ranges;
  const uint32_t* ids;
  const float4* rec_uvab;
  const float4* rec_cob;
  const float4* rec_rgbz;
  const float* Tfin;
  const int* last;
  const float *gC, *gD, *gA;
  float* g2d;  // [V*n, 10] floats, or doubles if `wide`: sums of q (dx, dy, dx^2, dx dy, dy^2, 1), q = dL/do; r, g, b, z
  bool wide;       // see kWideSums
  bool geom_only;  // only fields 0-4 and 9 are needed (no opacity or colour gradient wanted)
  int n_items;
  int* queue;
  ItemOrder order;
  int blocks;
  // deterministic backward (both NULL otherwise): per (list position,
  // 8x8 block of the tile) sums [K, 4, 10 or 6] and per list position the
  // mask of the blocks that stored one (zero before the launch)
  float* part;
  uint32_t* mask;
};
void launch_render_bwd(const Raster& R, const BwdArgs& a, hipStream_t s);
// Deterministic backward: list positions of each record's tiles (before the
// compositing pass), and the fixed-order sums into g2d (after it).
void launch_det_rev(const Raster& R, const int2* ranges, const uint32_t* ids, const int4* rect, const uint32_t* goff,
                    uint32_t* rev, int n_items, hipStream_t s);
void launch_det_reduce(const int4* rect, const uint32_t* goff, const uint32_t* rev, const uint32_t* mask,
                       const float* part, int64_t n_rec, bool geom_only, float* g2d, hipStream_t s);

// Adam applied by the projection backward to each Gaussian's gradient as soon
// as it is complete (groups: means, scales, quats, opacities, colors); p[i]
// are the parameters the forward read, updated in place.
struct AdamFused {
  float *p[5], *m[5], *v[5];
  float lr[5];
  float b1, b2, eps, bc1, bc2;
  float reg_w;  // Eq. 11 weight lambda_reg / N added to the scale gradient before the step; 0 = none
  bool on;
};

// Isotropic scale regulariser (Eq. 11) of one Gaussian: returns
// sum_i |s_i - sbar| with sbar = (s0 + s1 + s2) / 3, and writes
// d[j] = w (sign(r_j) - mean_i sign(r_i)), r = s - sbar, sign(0) = 0.
// Contraction is pinned so every kernel that applies it rounds alike.
__device__ __forceinline__ float reg_term(float s0, float s1, float s2, float w, float d[3]) {
#pragma clang fp contract(off)
  const float sbar = (s0 + s1 + s2) / 3.f;
  const float r0 = s0 - sbar, r1 = s1 - sbar, r2 = s2 - sbar;
  const float g0 = (float)((r0 > 0.f) - (r0 < 0.f)), g1 = (float)((r1 > 0.f) - (r1 < 0.f)),
              g2 = (float)((r2 > 0.f) - (r2 < 0.f));
  const float gm = (g0 + g1 + g2) / 3.f;
  d[0] = w * (g0 - gm);
  d[1] = w * (g1 - gm);
  d[2] = w * (g2 - gm);
  return fabsf(r0) + fabsf(r1) + fabsf(r2);
}

struct ProjectBwdArgs {
  int64_t n;
  const float *means, *scales, *quats, *opacities, *colors;
  const float* pose7;
  const uint32_t* counts;
  bool wide;    // g2d holds doubles
  float* g2d;  // read, then cleared (zero again for the next backward)
  float *g_means, *g_scales, *g_quats, *g_opacities, *g_colors;  // may be NULL; summed over views
  float* pose_acc;  // [n_views][blocks][12] per-workgroup dL/dR_p (9, row-major), dL/dt (3); NULL = skip
  int n_views;
  AdamFused adam;  // adam.on: apply Adam instead of (or as well as) writing the gradients
};
// workgroups of the projection backward (one per 256 Gaussians)
int64_t project_bwd_blocks(int64_t n);
void launch_project_bwd(const Raster& R, const ProjectBwdArgs& a, hipStream_t s);
// Sums the per-workgroup pose partials in a fixed order and converts them.
// Adam on the 7 pose parameters (q: lr_q, t: lr_t), bias-corrected with the
// step count kept in state = [m(8), v(8), step(1)]; element i of a step.
__device__ __forceinline__ void pose_adam_elem(float* pose, float* state, int i, float gi, float t, float lr_q,
                                               float lr_t, float b1, float b2, float eps) {
  const float mi = b1 * state[i] + (1.f - b1) * gi;
  const float vi = b2 * state[8 + i] + (1.f - b2) * gi * gi;
  state[i] = mi;
  state[8 + i] = vi;
  const float bc1 = 1.f - powf(b1, t), bc2 = 1.f - powf(b2, t);
  const float lr = i < 4 ? lr_q : lr_t;
  pose[i] -= lr * (mi / bc1) / (sqrtf(vi / bc2) + eps);
}

struct PoseAdam {
  float* state;  // NULL: no step
  float lr_q, lr_t, b1, b2, eps;
};

// With adam.state non-NULL (one view), also applies the pose Adam step to
// pose7 (in place) with the gradient just formed.
void launch_pose_finalize(const float* pose7, const float* pose_acc, int64_t blocks, float* dL_dpose7,
                          float* dL_dtwist6, int n_views, hipStream_t s, const PoseAdam* adam = nullptr);

void launch_fill_u32(uint32_t* p, uint32_t v, int64_t n, hipStream_t s);
void launch_fill_f32(float* p, float v, int64_t n, hipStream_t s);

// red: reduce_temp_words() uint32, zero before its first use (the loss kernels
// leave it zero again).
int64_t reduce_temp_words();
void launch_loss_l1(const float* C, const float* D, const float* Ct, const float* Dt, int64_t P, float wc, float wd,
                    float* loss, float* gC, float* gD, uint32_t* red, hipStream_t s);
// Adds weight * L_reg (Eq. 11) of scales [n,3] to *loss and, if g != NULL, its
// gradient to g [n,3].
void launch_loss_reg(const float* scales, int64_t n, float weight, float* loss, float* g, uint32_t* red,
                     hipStream_t s);
// Adds weight (1 - SSIM(X, Y)) to *loss and its gradient to gX ([3,H,W]).
void launch_loss_ssim(const float* X, const float* Y, int H, int W, float weight, float* loss, float* gX,
                      uint32_t* red, hipStream_t s);
// temp: track_temp_words() uint32, zero before the first call (every call leaves it zero)
int64_t track_temp_words();
void launch_loss_track(const float* C, const float* D, const float* A, const float* Ct, const float* Dt, int64_t P,
                       float lambda_c, float inlier_mult, float* loss, float* gC, float* gD, float* median,
                       uint32_t* temp, hipStream_t s);
void launch_adam(float* p, float* m, float* v, const float* g, int64_t n, float lr, float b1, float b2, float eps,
                 float bc1, float bc2, hipStream_t s);

void launch_pose_adam(float* pose, float* state, const float* g, float lr_q, float lr_t, float b1, float b2, float eps,
                      hipStream_t s);
// One bias-corrected Adam step (Kingma & Ba) on one value; bc1 = 1 - b1^t,
// bc2 = 1 - b2^t. Contraction is pinned so every kernel that applies it (the
// group step, the single-tensor step and the step fused into the projection
// backward) rounds identically.
__device__ __forceinline__ void adam_one(float& p, float& m, float& v, float g, float lr, float b1, float b2,
                                         float eps, float bc1, float bc2) {
#pragma clang fp contract(off)
  m = b1 * m + (1.f - b1) * g;
  v = b2 * v + (1.f - b2) * g * g;
  p -= lr * (m / bc1) / (sqrtf(v / bc2) + eps);
}

constexpr int kAdamGroups = 8;
struct AdamGroups {
  float* p[kAdamGroups];
  float* m[kAdamGroups];
  float* v[kAdamGroups];
  const float* g[kAdamGroups];
  float lr[kAdamGroups];
  int64_t off[kAdamGroups + 1];
  int n;
};
void launch_adam_multi(const AdamGroups& a, float b1, float b2, float eps, float bc1, float bc2, hipStream_t s);

// Tracking-initialisation CNN (k_initnet.hip). BF16 values travel as uint16_t bits.
int conv_kp(int C);
void launch_conv_fwd(int B, int H, int W, int C, const uint16_t* in, const uint16_t* wk, const float* bias,
                     uint16_t* out, hipStream_t st);
void launch_conv_bwd_data(int B, int H, int W, const uint16_t* dout, const uint16_t* wt, const uint16_t* in,
                          uint16_t* din, hipStream_t st);
void launch_conv_bwd_weight(int B, int H, int W, int C, const uint16_t* dy, const uint16_t* in, float* dw, float* db,
                            hipStream_t st);
void launch_head_fwd(int B, int OH, int OW, const uint16_t* act, const float* wfc, const float* bfc, float* pool,
                     float* out, hipStream_t st);
void launch_head_bwd(int B, int OH, int OW, const float* out, const float* label, const float* scale,
                     const float* pool, const float* wfc, const uint16_t* act, const float* dout, float* dwfc,
                     float* dbfc, uint16_t* dact, float* loss, hipStream_t st);
struct CastWeights {
  int n;  // layers
  int C[4];
  const float* w[4];
  uint16_t *wk[4], *wt[4];
};
void launch_cast_weights(const CastWeights& a, hipStream_t st);
void launch_pack_input(const float* rc, const float* rd, const float* oc, const float* od, int H, int W, int f,
                       float depth_scale, uint16_t* out, hipStream_t st);
void launch_pose_const_velocity(const float* p0, const float* p1, float* out, hipStream_t s);
void launch_pose_apply_twist(const float* pose, const float* xi, float* out, hipStream_t s);

}  // namespace gsr
