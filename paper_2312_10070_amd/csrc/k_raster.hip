// Per-tile compositing. One 256-thread workgroup per (view, tile) item, one
// pixel per lane: each wave covers an 8x8 pixel block of the tile and each
// 16-lane row of a wave (one DPP row) a 4x4 quadrant of that block. Gaussian
// records of the item's depth-sorted list are staged through LDS in batches
// (one coalesced fetch per record per workgroup). Skipping a record for a
// block or quadrant cannot change the result: outside its support box (taken
// with a small slack) a Gaussian's alpha stays below alpha_min by more than
// FP32 rounding, and the ellipse test keeps a margin too.
//
// Forward: front to back (Eq. 3 colour, Eq. 4 alpha, Eq. 6 depth), batches of
// 448 records (the largest that keeps six workgroups per CU in LDS). Each
// wave tests, 64 records at a time, which records can reach alpha >=
// alpha_min in its block (support box, then an exact ellipse-versus-rectangle
// test) and in which of its quadrants (support box), and appends their LDS
// offsets to one visit list per quadrant. The four rows
// of the wave then walk their own lists side by side, each lane reading its
// row's record from LDS, so a record is visited only by the quadrants it can
// reach; a row whose list has ended reads an all-zero record (alpha = 0). A
// lane stops before the Gaussian that would take its transmittance below
// T_min; a quadrant whose lanes have all stopped gets no further entries, a
// wave leaves the batch as soon as all its lanes have stopped, and the
// workgroup stops fetching batches once all four waves have.
//
// Backward: back to front from each pixel's last composited Gaussian. The
// transmittance in front of Gaussian j is recomputed as T_j = T_{j+1} /
// (1 - alpha_j) instead of being stored; suffix sums of c alpha T and z alpha
// T give the second terms of dC/dalpha and Eq. 8. Per pair, ten partials
// (sums of q (dx, dy, dx^2, dx dy, dy^2, 1) with q = dL/do = dL/dp / (o ln 2)
// for alpha = o 2^p, then colour and direct depth; six of them for a pose-only
// backward) are summed over the pixels of a wave's 8x8 block, four records at
// a time, on the matrix cores (see bwd_item), and a record's sums go out with
// one atomic per field. Each wave fetches, tests and walks its records by
// itself: the waves of a workgroup never wait for one another.
// A deterministic variant stores the wave's sums per (list position, block)
// instead and a second pass adds them per Gaussian in a fixed order.
//
// Launch shapes, both from the longest list to the shortest where that pays
// (see ItemOrder): one workgroup per item, or a persistent grid whose
// workgroups pull items from a counter until the queue is empty
// (multi-keyframe mapping).
#include <type_traits>

#include "gsr_internal.h"

namespace gsr {

namespace {

// Records the forward stages in LDS per batch, capacity of a quadrant's visit
// list, and the LDS slot of an all-zero record (u = v = 0, zero conic, o = 0:
// alpha = 0 at every pixel), which a row reads once its list has ended.
constexpr int kFwdBatch = 448;
constexpr int kListCap = 128;
constexpr int kWavesPerTile = kTileThreads / kWave;
static_assert(kFwdBatch % kWave == 0 && kListCap % 4 == 0 && kListCap >= kWave,
              "batch / list shape");

struct Block {
  int x0, x1, y0, y1;  // inclusive pixel rectangle of a wave (8x8)
};

struct Pixel {
  int tile, view;
  int px, py;
  int quad;     // 4x4 quadrant of the block (row-major) = DPP row of the lane
  bool inside;
  float fpx, fpy;
  int64_t p;    // pixel index inside the view
  int64_t off;  // view * W * H
  Block blk;
};

// Each wave covers one 8x8 pixel block of the tile (a square block meets fewer
// support boxes than a 16x4 or 32x2 strip), the four blocks row-major in the
// tile; lane row r = lane / 16 covers quadrant r of the block (row-major),
// lanes row-major in the quadrant.
__device__ __forceinline__ Pixel item_pixel(const Raster& Rr, int item) {
  Pixel q;
  q.view = item / Rr.n_tiles;
  q.tile = item - q.view * Rr.n_tiles;
  const int tyi = q.tile / Rr.ntx, txi = q.tile - tyi * Rr.ntx;
  const int tid = threadIdx.x, w = tid >> 6, l = tid & 63;
  const int bpr_log2 = Rr.tw_log2 - 3;  // 8x8 blocks per tile row: 1, 2 or 4
  const int bx = w & ((1 << bpr_log2) - 1), by = w >> bpr_log2;
  q.blk.x0 = txi * Rr.tw + 8 * bx;
  q.blk.x1 = q.blk.x0 + 7;
  q.blk.y0 = tyi * Rr.th + 8 * by;
  q.blk.y1 = q.blk.y0 + 7;
  q.quad = l >> 4;
  q.px = q.blk.x0 + 4 * (q.quad & 1) + (l & 3);
  q.py = q.blk.y0 + 4 * (q.quad >> 1) + ((l >> 2) & 3);
  q.inside = q.px < Rr.W && q.py < Rr.H;
  q.fpx = (float)q.px;
  q.fpy = (float)q.py;
  q.p = (int64_t)q.py * Rr.W + q.px;
  q.off = (int64_t)q.view * Rr.W * Rr.H;
  return q;
}

// Can the record reach alpha >= alpha_min anywhere in the block? alpha = o 2^p
// with p = pa dx^2 + pb dx dy + pc dy^2 <= 0 (pa, pc < 0), so it needs
// max over the block of p >= log2(alpha_min / o). If the centre lies in the
// block the maximum is 0; otherwise it lies on the block edge(s) facing the
// centre, where p restricted to the edge is a 1D concave quadratic whose
// maximiser is clamped to the edge. The continuous block contains every pixel
// centre, and the threshold carries a margin of 1e-3 (FP32 rounding of p is
// ~1e-6), so a skipped record has alpha < alpha_min at every pixel: the
// result cannot change, only the work.
__device__ __forceinline__ bool ellipse_meets(const float4& g, const float4& cb, const Block& s, float log2_amin) {
  const float u = g.x, v = g.y, pa = g.z, pb = g.w, pc = cb.x;
  const float thr = log2_amin - __builtin_amdgcn_logf(cb.y) - 1e-3f;  // log2(alpha_min / o)
  const float X0 = (float)s.x0, X1 = (float)s.x1, Y0 = (float)s.y0, Y1 = (float)s.y1;
  const float cx = fminf(fmaxf(u, X0), X1), cy = fminf(fmaxf(v, Y0), Y1);
  float best = (cx == u && cy == v) ? 0.f : -INFINITY;
  if (cx != u) {  // edge x = cx: maximise over y
    const float dX = cx - u;
    const float y = fminf(fmaxf(v - pb * dX * __builtin_amdgcn_rcpf(2.f * pc), Y0), Y1);
    const float dy = y - v;
    best = fmaxf(best, fmaf(pa * dX, dX, fmaf(pb * dX, dy, pc * dy * dy)));
  }
  if (cy != v) {  // edge y = cy: maximise over x
    const float dY = cy - v;
    const float x = fminf(fmaxf(u - pb * dY * __builtin_amdgcn_rcpf(2.f * pa), X0), X1);
    const float dx = x - u;
    best = fmaxf(best, fmaf(pa * dx, dx, fmaf(pb * dx, dY, pc * dY * dY)));
  }
  return best >= thr;
}

// Quadrants of the block (bit k = quadrant k, row-major) the record may reach:
// the packed support box (x0 | x1 << 16, y0 | y1 << 16) must meet the block
// and, if EXACT, the record must pass the ellipse test on the block; a
// quadrant must also meet the support box.
template <bool EXACT>
__device__ __forceinline__ uint32_t quad_mask(const float4& g, const float4& cb, const Block& s, float log2_amin) {
  const uint32_t bx = __float_as_uint(cb.z), by = __float_as_uint(cb.w);
  const int x0 = (int)(bx & 0xffffu), x1 = (int)(bx >> 16), y0 = (int)(by & 0xffffu), y1 = (int)(by >> 16);
  bool meets = (x0 <= s.x1) & (x1 >= s.x0) & (y0 <= s.y1) & (y1 >= s.y0);  // no short-circuit branches
  if (EXACT) meets = meets && ellipse_meets(g, cb, s, log2_amin);
  const uint32_t L = x0 <= s.x0 + 3, R = x1 >= s.x0 + 4, T = y0 <= s.y0 + 3, B = y1 >= s.y0 + 4;
  const uint32_t m = (L & T) | ((R & T) << 1) | ((L & B) << 2) | ((R & B) << 3);
  return meets ? m : 0u;
}

// Can the record reach alpha >= alpha_min anywhere in the block (support box,
// then the ellipse test)?
__device__ __forceinline__ bool block_meets(const float4& g, const float4& cb, const Block& s, float log2_amin) {
  const uint32_t bx = __float_as_uint(cb.z), by = __float_as_uint(cb.w);
  const int x0 = (int)(bx & 0xffffu), x1 = (int)(bx >> 16), y0 = (int)(by & 0xffffu), y1 = (int)(by >> 16);
  return ((x0 <= s.x1) & (x1 >= s.x0) & (y0 <= s.y1) & (y1 >= s.y0)) && ellipse_meets(g, cb, s, log2_amin);
}

__device__ __forceinline__ bool box_holds(float fbx, float fby, int px, int py) {
  const uint32_t bx = __float_as_uint(fbx), by = __float_as_uint(fby);
  return (px >= (int)(bx & 0xffffu)) & (px <= (int)(bx >> 16)) & (py >= (int)(by & 0xffffu)) & (py <= (int)(by >> 16));
}

// Lanes whose bit is set in the wave-uniform mask m append `val` to `list`
// after its first `len` entries, in lane order.
__device__ __forceinline__ void list_append(uint16_t* list, int len, uint64_t m, int lane, int val) {
  if ((m >> lane) & 1ull) {
    const int below = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
    list[len + below] = (uint16_t)val;
  }
}

// The float4 at byte offset `boff` of an LDS array.
__device__ __forceinline__ float4 lds_at(const float4* arr, int boff) {
  return *reinterpret_cast<const float4*>(reinterpret_cast<const char*>(arr) + boff);
}

struct FwdSmem {
  static constexpr int kBatch = kFwdBatch, kDummy = kFwdBatch;
  float4 uvab[kBatch + 1];
  float4 cob[kBatch + 1];
  float4 rgbz[kBatch + 1];
  uint16_t list[kWavesPerTile][4][kListCap + 4];
};

// Where the backward's sums go: float or double atomics (see kWideSums), or
// stored per (list position, block) for the deterministic option.
enum BwdSums { kFloat, kWide, kStored };

// Backward: a wave's ring of records still to be walked (u, v, pa, pb | pc, o,
// list position, Gaussian id | r, g, b, z). Up to three are left when the next
// chunk of 64 is appended.
constexpr int kRing = 128;
struct BwdWave {
  float4 uvab[kRing];
  float4 copg[kRing];
  float4 rgbz[kRing];
};

// The all-zero record; written once per workgroup before its first barrier.
__device__ __forceinline__ void init_smem(FwdSmem& sm) {
  if (threadIdx.x == 0) {
    sm.uvab[FwdSmem::kDummy] = make_float4(0.f, 0.f, 0.f, 0.f);
    sm.cob[FwdSmem::kDummy] = make_float4(0.f, 0.f, 0.f, 0.f);
    sm.rgbz[FwdSmem::kDummy] = make_float4(0.f, 0.f, 0.f, 0.f);
  }
}

// STATS = true: instead of writing outputs, count the algorithmic work (for the
// benchmark's roofline): pairs whose pixel lies in the Gaussian's support box
// before the pixel stops, and pairs composited. The lists then come from the
// support boxes alone, so every such pair is visited.
template <bool STATS>
__device__ __forceinline__ void fwd_item(const Raster& Rr, const FwdArgs& a, int item, FwdSmem& sm) {
  constexpr int kBatch = FwdSmem::kBatch, kDummy = FwdSmem::kDummy;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const Pixel q = item_pixel(Rr, item);
  const int2 rg = a.ranges[item];
  const int start = rg.x, end = rg.y;
  // T > 0: the lane is compositing; T < 0: it has stopped and -T is its final
  // transmittance (T >= T_min > 0 while compositing, so the sign is free).
  float T = q.inside ? 1.f : -1.f, C0 = 0.f, C1 = 0.f, C2 = 0.f, D = 0.f;
  int last16 = 0;  // 16 x (list position of the last composited Gaussian + 1)
  uint32_t n_eval = 0, n_comp = 0;
  const uint16_t* mylist = sm.list[w][q.quad];

  for (int base = start; base < end; base += kBatch) {
    if (__syncthreads_count(T > 0.f) == 0) break;
#pragma unroll
    for (int h = 0; h < (kBatch + kTileThreads - 1) / kTileThreads; ++h) {
      const int sl = h * kTileThreads + tid, i = base + sl;
      if (sl < kBatch && i < end) {
        const uint32_t gid = a.ids[i];
        sm.uvab[sl] = a.rec_uvab[kRec * gid];
        sm.cob[sl] = a.rec_cob[kRec * gid];
        sm.rgbz[sl] = a.rec_rgbz[kRec * gid];
      }
    }
    __syncthreads();
    const int cnt = min(kBatch, end - base);
    const int nch = (cnt + kWave - 1) / kWave;
    int k = 0;
    while (k < nch) {
      // one segment: append chunks to the quadrant lists until one would overflow
      const uint64_t alive = __ballot(T > 0.f);
      if (alive == 0) break;
      int len0 = 0, len1 = 0, len2 = 0, len3 = 0;
      for (; k < nch; ++k) {
        const int r = k * kWave + lane;
        const uint32_t qm = r < cnt ? quad_mask<!STATS>(sm.uvab[r], sm.cob[r], q.blk, Rr.log2_amin) : 0u;
        // a quadrant whose lanes have all stopped takes no entries
        const uint64_t m0 = (alive & 0xffffull) ? __ballot(qm & 1u) : 0ull;
        const uint64_t m1 = (alive & 0xffff0000ull) ? __ballot(qm & 2u) : 0ull;
        const uint64_t m2 = (alive & 0xffff00000000ull) ? __ballot(qm & 4u) : 0ull;
        const uint64_t m3 = (alive & 0xffff000000000000ull) ? __ballot(qm & 8u) : 0ull;
        const int c0 = __popcll(m0), c1 = __popcll(m1), c2 = __popcll(m2), c3 = __popcll(m3);
        if (len0 + c0 > kListCap || len1 + c1 > kListCap || len2 + c2 > kListCap || len3 + c3 > kListCap) break;
        // entries are LDS byte offsets of the slot inside each record array
        list_append(sm.list[w][0], len0, m0, lane, 16 * r);
        list_append(sm.list[w][1], len1, m1, lane, 16 * r);
        list_append(sm.list[w][2], len2, m2, lane, 16 * r);
        list_append(sm.list[w][3], len3, m3, lane, 16 * r);
        len0 += c0;
        len1 += c1;
        len2 += c2;
        len3 += c3;
      }
      const int myl = q.quad == 0 ? len0 : (q.quad == 1 ? len1 : (q.quad == 2 ? len2 : len3));
      const int maxl = __builtin_amdgcn_readfirstlane(max(max(len0, len1), max(len2, len3)));
      // (list position + 1) * 16 of slot 0: last16 = code + byte offset
      const int code = 16 * (base - start + 1);
      __builtin_amdgcn_wave_barrier();
      // One step per record of the row's list. Every lane runs the same
      // instructions: a skipped pair (alpha < alpha_min, or the all-zero
      // record) acts as alpha = 0; a stopped lane has T < 0, so its Tn <
      // T_min and it adds w = 0 and keeps T.
      auto step = [&](const float4& g, const float4& cb, const float4& cz, int jb) {
        const PairEval pe = eval_pair(q.fpx - g.x, q.fpy - g.y, g.z, g.w, cb.x, cb.y, Rr.amin, Rr.amax);
        if (STATS && T > 0.f && jb != 16 * kDummy && box_holds(cb.z, cb.w, q.px, q.py)) ++n_eval;
        const float al = pe.use ? pe.alpha : 0.f;
        const float Tn = T * (1.f - al);
        const bool comp = Tn >= Rr.tmin;  // false for a stopped lane and at the stop
        const float wt = comp ? al * T : 0.f;
        C0 = fmaf(cz.x, wt, C0);
        C1 = fmaf(cz.y, wt, C1);
        C2 = fmaf(cz.z, wt, C2);
        D = fmaf(cz.w, wt, D);
        last16 = (comp && pe.use) ? code + jb : last16;
        if (STATS && comp && pe.use) ++n_comp;
        T = comp ? Tn : -fabsf(T);
      };
      // walk while some lane is compositing and its row's list has not ended
      auto going = [&](int t) { return (t < maxl) & ((__ballot(T > 0.f) & __ballot(t < myl)) != 0); };
      // Software pipeline, unrolled by two so that no record is copied
      // between registers: while step t runs on one record set, the other
      // set receives the record of step t + 1 from LDS, and the list entry of
      // step t + 2 is read (entries past the row's list end are not used).
      // The walk condition is checked before every second step only: a step
      // after it turned false is a no-op (every lane has stopped, or every
      // row reads the all-zero record), and entries up to kListCap + 2 exist
      // for its reads. The loop is tested at its end (one exit) and the test
      // itself has no branch, so the body is one basic block and the carried
      // sums stay in the same registers around it.
      int jA = 0 < myl ? mylist[0] : 16 * kDummy;
      int jn = mylist[1];
      float4 gA = lds_at(sm.uvab, jA), cbA = lds_at(sm.cob, jA), czA = lds_at(sm.rgbz, jA);
      if (going(0)) {
        int t = 0;
        do {
          const int jB = t + 1 < myl ? jn : 16 * kDummy;
          jn = mylist[t + 2];
          const float4 gB = lds_at(sm.uvab, jB), cbB = lds_at(sm.cob, jB), czB = lds_at(sm.rgbz, jB);
          step(gA, cbA, czA, jA);
          ++t;
          jA = t + 1 < myl ? jn : 16 * kDummy;
          jn = mylist[t + 2];
          gA = lds_at(sm.uvab, jA);
          cbA = lds_at(sm.cob, jA);
          czA = lds_at(sm.rgbz, jA);
          step(gB, cbB, czB, jB);
          ++t;
        } while (going(t));
      }
      __builtin_amdgcn_wave_barrier();
    }
  }
  if (STATS) {
    unsigned long long e = n_eval, cm = n_comp;
    for (int o = 32; o > 0; o >>= 1) {
      e += __shfl_xor(e, o, 64);
      cm += __shfl_xor(cm, o, 64);
    }
    if (lane == 0) {
      atomicAdd(&a.stats[0], e);
      atomicAdd(&a.stats[1], cm);
    }
    return;
  }
  if (q.inside) {
    T = fabsf(T);
    const int64_t P = (int64_t)Rr.W * Rr.H;
    const int64_t p = q.off + q.p;
    float* col = a.color + 3 * q.off;
    col[q.p] = fmaf(T, Rr.bg0, C0);
    col[P + q.p] = fmaf(T, Rr.bg1, C1);
    col[2 * P + q.p] = fmaf(T, Rr.bg2, C2);
    a.depth[p] = D;
    a.alpha[p] = 1.f - T;
    a.Tfin[p] = T;
    a.last[p] = last16 >> 4;
  }
}

// The values of lane ^ 4 and lane ^ 8 (inside a 16-lane row).
template <int CTRL>
__device__ __forceinline__ float dpp_all(float v) {  // every lane has a source lane
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
__device__ __forceinline__ float row_xor4(float v) { return dpp_all<0x1b>(dpp_all<0x141>(v)); }  // half_mirror, quad_perm [3,2,1,0]
__device__ __forceinline__ float row_xor8(float v) { return dpp_all<0x128>(v); }                 // row_ror:8

typedef float f32x4 __attribute__((ext_vector_type(4)));

// D_b[i][j] += A_b[i] B_b[j] for the wave's 16 blocks b of four lanes: A's row
// i and B's column j lie in lane 4 b + i and 4 b + j, D's element (i, j) in
// register i of lane 4 b + j. Each element is one fused multiply-add.
__device__ __forceinline__ f32x4 outer4(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c, 0, 0, 0);
}

// In every group of four lanes, the transpose of the 4x4 matrices a and b
// (register s of lane i becomes register i of lane s): two exchanges of lane
// pairs, each element one select whose one side comes from the partner lane.
// A lane's values reach only their own places, whatever they hold (NaN and
// infinities too). Written as one block because the select takes a partner
// lane's value only with its mask in VCC; the waits are those that a DPP read
// of a freshly written register needs (two) at the start and between the
// exchanges, and that a matrix instruction's read needs at the end.
__device__ __forceinline__ void transpose4(float a[4], float b[4], uint64_t even, uint64_t low) {
  const uint64_t odd = ~even, high = ~low;
  float p0, p1, p2, p3, q0, q1, q2, q3;
#define GSR_SEL(d, x, y, perm) "v_cndmask_b32_dpp " d ", " x ", " y ", vcc quad_perm:" perm " row_mask:0xf bank_mask:0xf\n"
  asm("s_mov_b64 vcc, %[ev]\n"
      "s_nop 1\n"
      GSR_SEL("%[p0]", "%[a1]", "%[a0]", "[1,0,3,2]")
      GSR_SEL("%[p2]", "%[a3]", "%[a2]", "[1,0,3,2]")
      GSR_SEL("%[q0]", "%[b1]", "%[b0]", "[1,0,3,2]")
      GSR_SEL("%[q2]", "%[b3]", "%[b2]", "[1,0,3,2]")
      "s_mov_b64 vcc, %[od]\n"
      GSR_SEL("%[p1]", "%[a0]", "%[a1]", "[1,0,3,2]")
      GSR_SEL("%[p3]", "%[a2]", "%[a3]", "[1,0,3,2]")
      GSR_SEL("%[q1]", "%[b0]", "%[b1]", "[1,0,3,2]")
      GSR_SEL("%[q3]", "%[b2]", "%[b3]", "[1,0,3,2]")
      "s_mov_b64 vcc, %[lo]\n"
      "s_nop 1\n"
      GSR_SEL("%[a0]", "%[p2]", "%[p0]", "[2,3,0,1]")
      GSR_SEL("%[a1]", "%[p3]", "%[p1]", "[2,3,0,1]")
      GSR_SEL("%[b0]", "%[q2]", "%[q0]", "[2,3,0,1]")
      GSR_SEL("%[b1]", "%[q3]", "%[q1]", "[2,3,0,1]")
      "s_mov_b64 vcc, %[hi]\n"
      GSR_SEL("%[a2]", "%[p0]", "%[p2]", "[2,3,0,1]")
      GSR_SEL("%[a3]", "%[p1]", "%[p3]", "[2,3,0,1]")
      GSR_SEL("%[b2]", "%[q0]", "%[q2]", "[2,3,0,1]")
      GSR_SEL("%[b3]", "%[q1]", "%[q3]", "[2,3,0,1]")
      "s_nop 1"
      : [a0] "+v"(a[0]), [a1] "+v"(a[1]), [a2] "+v"(a[2]), [a3] "+v"(a[3]), [b0] "+v"(b[0]), [b1] "+v"(b[1]),
        [b2] "+v"(b[2]), [b3] "+v"(b[3]), [p0] "=&v"(p0), [p1] "=&v"(p1), [p2] "=&v"(p2), [p3] "=&v"(p3),
        [q0] "=&v"(q0), [q1] "=&v"(q1), [q2] "=&v"(q2), [q3] "=&v"(q3)
      : [ev] "s"(even), [od] "s"(odd), [lo] "s"(low), [hi] "s"(high)
      : "vcc");
#undef GSR_SEL
}

// Column of the [n, 10] gradient sums that field f of the six-field
// reduction adds to.
__device__ __forceinline__ int g2d_field6(int f) { return f < 5 ? f : 9; }

// Per-pixel state of the backward: the forward's final transmittance and last
// composited position, the upstream gradients, and the running suffix term.
struct BwdPix {
  float T, g0, g1, g2, gd, gS, gA;
  int last;
};

// dL/dalpha_j = T_j (g . c_j) - (g . S_j + ga T_fin) / (1 - alpha_j) with the
// suffix sums S_j = sum_{u > j} c_u alpha_u T_u + T_fin bg (colour) and
// sum_{u > j} z_u alpha_u T_u (depth), g = (gC, gD). Only the dot product
// gS = g . S_j is needed; the background enters it through T_fin bg.
__device__ __forceinline__ BwdPix bwd_pixel(const Raster& Rr, const BwdArgs& a, const Pixel& q) {
  BwdPix b{1.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0};
  float ga = 0.f;
  if (q.inside) {
    const int64_t P = (int64_t)Rr.W * Rr.H;
    const int64_t p = q.off + q.p;
    const float* gC = a.gC + 3 * q.off;
    b.T = a.Tfin[p];
    b.last = a.last[p];
    b.g0 = gC[q.p];
    b.g1 = gC[P + q.p];
    b.g2 = gC[2 * P + q.p];
    b.gd = a.gD[p];
    ga = a.gA ? a.gA[p] : 0.f;
  }
  b.gS = b.T * (b.g0 * Rr.bg0 + b.g1 * Rr.bg1 + b.g2 * Rr.bg2);
  b.gA = ga * b.T;
  return b;
}

// The sums of wt (g_r, g_g, g_b, g_d) over a group's four pixels, for a block
// with an upstream gradient that is not finite: a pixel that did not composite
// the record (wt = 0) adds nothing to it, where an outer product would add 0
// times that gradient, a NaN.
template <int CTRL>
__device__ __forceinline__ void add_if_hit(const BwdPix& b, float wt, f32x4& r) {
  const f32x4 g = {dpp_all<CTRL>(b.g0), dpp_all<CTRL>(b.g1), dpp_all<CTRL>(b.g2), dpp_all<CTRL>(b.gd)};
#pragma unroll
  for (int i = 0; i < 4; ++i) r[i] = wt != 0.f ? fmaf(g[i], wt, r[i]) : r[i];
}
__device__ __forceinline__ f32x4 sums_of_hits(const BwdPix& b, const float (&wT)[4]) {
  f32x4 r = {0.f, 0.f, 0.f, 0.f};
  add_if_hit<0x00>(b, wT[0], r);
  add_if_hit<0x55>(b, wT[1], r);
  add_if_hit<0xaa>(b, wT[2], r);
  add_if_hit<0xff>(b, wT[3], r);
  return r;
}

// Backward of one wave's 8x8 block (block w of the item's tile), with NF = 10
// fields (mapping) or 6 (a pose-only backward). The wave reads the records of
// the tile's list in chunks of 64 from the largest `last` of its pixels
// downwards, appends those that can reach alpha >= alpha_min in its block
// (support box, then the ellipse test) to a ring in LDS, and walks the ring
// four records per step, each lane its own pixel.
//
// The sums over the block's pixels are contractions and run on the matrix
// cores, in FP32 (4x4x1 outer products, exact fused multiply-adds). With q =
// dL/do and wt = alpha T of the step's four records:
//  - g . c (upstream gradient dot colour and depth) of four records: four
//    outer products of the records' channels with the pixels' gradients;
//  - q and wt are transposed inside each group of four lanes, so that a lane
//    holds one record's values at the group's four pixels, which lie in one
//    pixel row;
//  - the group's sums of q (1, dx, dx^2) about the record's centre; as y is
//    constant in the group, the moments with dy follow with a few operations.
//    (Not as outer products with the pixels' x, moved to the centre afterwards:
//    no faster, and for a Gaussian smaller than the group the difference of
//    large terms: at a variance of 0.25 px^2 the sum of q dx^2 was off by
//    3.4e-7 rms, now by 6.4e-8.)
//  - the group's sums of wt (g_r, g_g, g_b, g_d): outer products with the
//    pixels' gradients.
// The 16 groups are then added by exchanges that split the fields over the
// lanes, and one 40-lane atomic adds the four records' fields to the [n, 10]
// gradient sums (the projection backward multiplies the moments by the opacity).
//
// Bound by VALU issue (about 0.9 while a CU is busy): some 200 issue slots per
// step of four records, where DPP sums of every pair's ten products and one
// 64-lane butterfly per record took about 80 per record. A matrix instruction
// takes two slots, so those are used where one replaces more than two
// operations; the transposes as outer products with unit vectors (180 us) and
// the pixel offsets as outer products (no change) are not.
// Measured at 1200x680 with 500K Gaussians / 640x480 with 500K, six fields:
// 267 / 146 us before (there a block walk, here one of per-quadrant lists with
// LDS accumulators, both with workgroup batches and barriers), 175 / 118 us
// then, 169 / 107 now that tiles go by length (188 / 114 traced). On the way: the same sums with workgroup batches of 512 records 198 /
// 149 us; visit lists per 4x4 quadrant (0.6 of the steps, but sums per
// quadrant) with LDS float atomics 330 / 158 us, as those take about two
// cycles per lane, with global atomics 1.1 ms / 344 us, as they need several
// times the cache lines of atomic traffic.
//
// kStored: the wave's sums of a record are stored to a.part at (list position of
// the record, block of the tile) and the block's bit set in a.mask instead; a
// later pass adds them per Gaussian in a fixed order, so the result does not
// depend on the order waves run in.
//
// ALPHA: with an upstream gradient of alpha. Its term gA = dL/dA T_fin is
// subtracted from the suffix sum per pair. Folded into the sum from the start,
// which takes no operation, it has every addition rounded to its size (an alpha
// gradient a thousand times the colour's, 200 layers: dL/do off by 2.2e-7 rms,
// so 5.4e-8). A kernel of its own, as the operation costs the others 3 %.
template <int NF, BwdSums SUMS, bool ALPHA>
__device__ __forceinline__ void bwd_item(const Raster& Rr, const BwdArgs& a, int item, BwdWave* smem) {
  constexpr int H = NF / 2;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const Pixel q = item_pixel(Rr, item);
  BwdPix b = bwd_pixel(Rr, a, q);
  // per-lane constants: lane 4 b + i holds, for pixel s of block b, row i of
  // the upstream gradients, and the pixel's x
  const int li = lane & 3;
  const bool b2 = (lane >> 2) & 1, b3 = (lane >> 3) & 1;
  // the field a lane's sum ends with (see the reduction below), or -1
  const int b54 = ((lane >> 5) & 1) + 2 * ((lane >> 4) & 1);
  const int fld0 = NF == 10 ? (b2 ? 8 + b54 : 4 * (int)b3 + b54) : 4 * (int)b3 + b54;
  const int fld = NF == 10 ? ((b2 && (b3 || b54 > 1)) ? -1 : fld0) : ((b2 || fld0 > 5) ? -1 : fld0);
  // some upstream gradient of the block is not finite (0 times it is NaN)
  const bool odd = __ballot(!(0.f * b.g0 + 0.f * b.g1 + 0.f * b.g2 + 0.f * b.gd == 0.f)) != 0;
  float xs[4], G[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) xs[s] = (float)(q.blk.x0 + 4 * (q.quad & 1) + s);
#define GSR_GRAD_ROW(s, ctrl)                                                                                    \
  {                                                                                                      \
    const float t0 = dpp_f<ctrl>(b.g0), t1 = dpp_f<ctrl>(b.g1), t2 = dpp_f<ctrl>(b.g2), t3 = dpp_f<ctrl>(b.gd); \
    G[s] = li == 0 ? t0 : (li == 1 ? t1 : (li == 2 ? t2 : t3));                                          \
  }
  GSR_GRAD_ROW(0, 0x00)
  GSR_GRAD_ROW(1, 0x55)
  GSR_GRAD_ROW(2, 0xaa)
  GSR_GRAD_ROW(3, 0xff)
#undef GSR_GRAD_ROW
  const int start = a.ranges[item].x;
  const int wmax = __builtin_amdgcn_readfirstlane(wave_max_int(b.last));
  BwdWave& sm = smem[w];

  // Records come in chunks of 64, the highest positions first: lane l reads
  // the record at position pos0 - l, tests it, and appends it to the ring if
  // it can reach the block. The next chunk's records are read while the
  // current ones are walked.
  uint32_t gid = 0;
  float4 uvab = make_float4(0.f, 0.f, 0.f, 0.f), cob = uvab, rgbz = uvab;
  auto fetch = [&](int pos0) {
    const int pos = pos0 - lane;
    if (pos >= 0) {
      gid = a.ids[start + pos];
      uvab = a.rec_uvab[kRec * gid];
      cob = a.rec_cob[kRec * gid];
      rgbz = a.rec_rgbz[kRec * gid];
    }
  };
  fetch(wmax - 1);
  int head = 0, tail = 0;
  for (int pos0 = wmax - 1; pos0 >= 0; pos0 -= kWave) {
    const bool meets = pos0 - lane >= 0 && block_meets(uvab, cob, q.blk, Rr.log2_amin);
    const uint64_t m = __ballot(meets);
    if (meets) {
      const int below = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
      const int sl = (tail + below) & (kRing - 1);
      sm.uvab[sl] = uvab;
      sm.copg[sl] = make_float4(cob.x, cob.y, __int_as_float(pos0 - lane), __uint_as_float(gid));
      sm.rgbz[sl] = rgbz;
    }
    tail += __popcll(m);
    if (pos0 < kWave) {
      // no more records: all-zero ones (alpha = 0) fill the last step
      if (lane < 3) {
        const int sl = (tail + lane) & (kRing - 1);
        sm.uvab[sl] = make_float4(0.f, 0.f, 0.f, 0.f);
        sm.copg[sl] = make_float4(0.f, 0.f, __int_as_float(-1), 0.f);
        sm.rgbz[sl] = make_float4(0.f, 0.f, 0.f, 0.f);
      }
      tail += 3;
    }
    fetch(pos0 - kWave);
    __builtin_amdgcn_wave_barrier();
    for (; tail - head >= 4; head += 4) {
      const int h = head & (kRing - 1);
      float4 g[4], co[4];
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        g[s] = sm.uvab[h + s];
        co[s] = sm.copg[h + s];
      }
      const float4 cz = sm.rgbz[h + li], mine = sm.copg[h + li];  // the record this lane sums
      const float2 uv = *reinterpret_cast<const float2*>(&sm.uvab[h + li]);  // its centre
      f32x4 gc = {0.f, 0.f, 0.f, 0.f}, Wm = gc;
      float qT[4], wT[4];
      gc = outer4(cz.w, b.gd, gc);
      gc = outer4(cz.z, b.g2, gc);
      gc = outer4(cz.y, b.g1, gc);
      gc = outer4(cz.x, b.g0, gc);
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const float dx = q.fpx - g[s].x, dy = q.fpy - g[s].y;
        const PairEval pe = eval_pair(dx, dy, g[s].z, g[s].w, co[s].x, co[s].y, Rr.amin, Rr.amax);
        const bool hit = (__float_as_int(co[s].z) < b.last) & pe.use;  // the all-zero record never passes `use`
        // A lane without a hit runs the same instructions with alpha = 0: its
        // transmittance and suffix term are unchanged, q and wt are 0.
        const float al = hit ? pe.alpha : 0.f;
        const float inv = __builtin_amdgcn_rcpf(1.f - al);  // 1 ulp; alpha <= alpha_max < 1
        const float Tj = b.T * inv;
        const float wt = al * Tj;
        const float dA = fmaf(Tj, gc[s], -inv * (ALPHA ? b.gS - b.gA : b.gS));
        b.gS = fmaf(gc[s], wt, b.gS);
        b.T = Tj;
        // a clamped alpha does not depend on o or sigma
        qT[s] = (hit & !pe.clamped) ? dA * pe.e : 0.f;
        wT[s] = wt;
      }
      transpose4(qT, wT, 0x5555555555555555ull, 0x3333333333333333ull);
#pragma unroll
      for (int s = 0; s < 4; ++s) Wm = outer4(G[s], wT[s], Wm);
      if (odd) Wm = sums_of_hits(b, wT);
      // moments about the record's centre (u, v)
      float dx[4], qx[4];
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        dx[s] = xs[s] - uv.x;
        qx[s] = qT[s] * dx[s];
      }
      const float dy = q.fpy - uv.y;
      const float m = (qT[0] + qT[1]) + (qT[2] + qT[3]), mx = (qx[0] + qx[1]) + (qx[2] + qx[3]);
      const float mxx = fmaf(qx[3], dx[3], fmaf(qx[2], dx[2], fmaf(qx[1], dx[1], qx[0] * dx[0])));
      const float my = dy * m, mxy = dy * mx, myy = dy * my;
      float v[NF];
      v[0] = mx;
      v[1] = my;
      v[2] = mxx;
      v[3] = mxy;
      v[4] = myy;
      if (NF == 10) {
        v[5] = m;
        v[NF - 4] = Wm[0];
        v[NF - 3] = Wm[1];
        v[NF - 2] = Wm[2];
      }
      v[NF - 1] = Wm[3];
      // The wave's sum over its 16 blocks, the fields split over the lanes'
      // bits 5 .. 2: one field (or none) per lane and record is left.
      float r5[H], r4[(H + 1) / 2];
#pragma unroll
      for (int f = 0; f < H; ++f) r5[f] = perm_add32(v[2 * f], v[2 * f + 1]);
#pragma unroll
      for (int f = 0; f < (H + 1) / 2; ++f) r4[f] = perm_add16(r5[2 * f], 2 * f + 1 < H ? r5[2 * f + 1] : 0.f);
      float o;
      if (NF == 10) {
        const float a0 = (b3 ? r4[1] : r4[0]) + row_xor8(b3 ? r4[0] : r4[1]);
        const float a1 = r4[2] + row_xor8(r4[2]);
        o = (b2 ? a1 : a0) + row_xor4(b2 ? a0 : a1);
      } else {
        const float a0 = (b3 ? r4[1] : r4[0]) + row_xor8(b3 ? r4[0] : r4[1]);
        o = a0 + row_xor4(a0);
      }
      const int pos = __float_as_int(mine.z);
      if (fld >= 0 && pos >= 0) {
        if (SUMS == kStored) {
          const int64_t slot = start + pos;  // position in the ids array
          a.part[(slot * 4 + w) * NF + fld] = o;
          if (fld == 0) atomicOr(a.mask + slot, 1u << w);
        } else {
          const int64_t at = 10 * (int64_t)__float_as_uint(mine.w) + (NF == 10 ? fld : g2d_field6(fld));
          if (SUMS == kWide) atomicAdd(reinterpret_cast<double*>(a.g2d) + at, (double)o);
          else atomicAdd(a.g2d + at, o);
        }
      }
    }
    __builtin_amdgcn_wave_barrier();
  }
}

template <bool STATS>
__global__ __launch_bounds__(kTileThreads) void k_render_fwd(Raster Rr, FwdArgs a) {
  __shared__ FwdSmem sm;
  init_smem(sm);
  const int b = (int)blockIdx.x;
  fwd_item<STATS>(Rr, a, item_at(a.order, b, xcd_tile(b, (int)gridDim.x)), sm);
}

template <int NF, BwdSums SUMS, bool ALPHA>
__global__ __launch_bounds__(kTileThreads, 5) void k_render_bwd(Raster Rr, BwdArgs a) {
  __shared__ BwdWave sm[kWavesPerTile];
  const int b = (int)blockIdx.x;
  bwd_item<NF, SUMS, ALPHA>(Rr, a, item_at(a.order, b, xcd_chunk(b, (int)gridDim.x)), sm);
}

// Persistent workgroups: take the next item from the queue until it is empty.
// Every workgroup reaches the exit once the counter passes n_items.
__device__ __forceinline__ int next_item(int* queue, const ItemOrder& order, int n_items, int* s_item) {
  __syncthreads();
  if (threadIdx.x == 0) *s_item = atomicAdd(queue, 1);
  __syncthreads();
  const int qi = *s_item;
  if (qi >= n_items) return -1;
  return item_at(order, qi, qi);
}

__global__ __launch_bounds__(kTileThreads) void k_render_fwd_persistent(Raster Rr, FwdArgs a) {
  __shared__ FwdSmem sm;
  __shared__ int s_item;
  init_smem(sm);
  for (;;) {
    const int item = next_item(a.queue, a.order, a.n_items, &s_item);
    if (item < 0) break;
    fwd_item<false>(Rr, a, item, sm);
  }
}

template <int NF, BwdSums SUMS, bool ALPHA>
__global__ __launch_bounds__(kTileThreads, 5) void k_render_bwd_persistent(Raster Rr, BwdArgs a) {
  __shared__ BwdWave sm[kWavesPerTile];
  __shared__ int s_item;
  for (;;) {
    const int item = next_item(a.queue, a.order, a.n_items, &s_item);
    if (item < 0) break;
    bwd_item<NF, SUMS, ALPHA>(Rr, a, item, sm);
  }
}

// Deterministic backward, before the compositing pass: rev[goff[o] + j] =
// list position of record o in the j-th tile of its tile rectangle (row-major),
// where goff is the exclusive scan of the records' tile counts.
__global__ __launch_bounds__(256) void k_det_rev(Raster Rr, const int2* __restrict__ ranges,
                                               const uint32_t* __restrict__ ids, const int4* __restrict__ rect,
                                               const uint32_t* __restrict__ goff, uint32_t* __restrict__ rev) {
  const int item = blockIdx.x;
  const int tile = item % Rr.n_tiles;
  const int ty = tile / Rr.ntx, tx = tile - ty * Rr.ntx;
  const int2 rg = ranges[item];
  for (int i = rg.x + (int)threadIdx.x; i < rg.y; i += blockDim.x) {
    const uint32_t o = ids[i];
    const int4 r = rect[o];
    const int tx0 = r.x & 0xffff, tx1 = (int)((uint32_t)r.x >> 16), ty0 = r.y & 0xffff;
    rev[goff[o] + (uint32_t)((ty - ty0) * (tx1 - tx0 + 1) + (tx - tx0))] = (uint32_t)i;
  }
}

// Deterministic backward, after the compositing pass: one thread per (record,
// field) adds the stored block sums of its tiles (tiles in row-major order
// of the record's rectangle, blocks in order) and stores the total into
// the [n, 10] gradient sums.
template <int NF>
__global__ __launch_bounds__(256) void k_det_reduce(const int4* __restrict__ rect, const uint32_t* __restrict__ goff,
                                                  const uint32_t* __restrict__ rev, const uint32_t* __restrict__ mask,
                                                  const float* __restrict__ part, int64_t n_rec,
                                                  float* __restrict__ g2d) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= n_rec * NF) return;
  const int64_t o = idx / NF;
  const int f = (int)(idx - o * NF);
  const int cnt = rect[o].w;
  if (cnt == 0) return;
  const uint32_t b = goff[o];
  float sum = 0.f;
  for (int j = 0; j < cnt; ++j) {
    const int64_t slot = rev[b + j];
    uint32_t m = mask[slot];
    while (m) {
      const int blk = __builtin_ctz(m);
      m &= m - 1u;
      sum += part[(slot * 4 + blk) * NF + f];
    }
  }
  g2d[10 * o + (NF == 10 ? f : g2d_field6(f))] = sum;
}

// Support-box pairs before each pixel's last composited Gaussian: the pairs
// the backward must evaluate (work counter; reads the forward's `last`).
__global__ __launch_bounds__(kTileThreads) void k_count_bwd_pairs(Raster Rr, FwdArgs a) {
  __shared__ float4 s_cob[kTileThreads];
  const int item = blockIdx.x;
  const Pixel q = item_pixel(Rr, item);
  const int last = q.inside ? a.last[q.off + q.p] : 0;
  const int2 rg = a.ranges[item];
  unsigned long long n = 0;
  for (int base = rg.x; base < rg.y; base += kTileThreads) {
    __syncthreads();
    if (base + (int)threadIdx.x < rg.y) s_cob[threadIdx.x] = a.rec_cob[kRec * a.ids[base + threadIdx.x]];
    __syncthreads();
    const int cnt = min(kTileThreads, rg.y - base);
    for (int j = 0; j < cnt; ++j)
      if (base - rg.x + j < last && box_holds(s_cob[j].z, s_cob[j].w, q.px, q.py)) ++n;
  }
  for (int o = 32; o > 0; o >>= 1) n += __shfl_xor(n, o, 64);
  if ((threadIdx.x & 63) == 0) atomicAdd(&a.stats[2], n);
}

}  // namespace

void launch_render_fwd(const Raster& R, const FwdArgs& a, hipStream_t s) {
  if (a.stats) {
    hipLaunchKernelGGL(k_render_fwd<true>, dim3((unsigned)a.n_items), dim3(kTileThreads), 0, s, R, a);
    hipLaunchKernelGGL(k_count_bwd_pairs, dim3((unsigned)a.n_items), dim3(kTileThreads), 0, s, R, a);
  } else if (a.blocks > 0) {
    launch_fill_u32(reinterpret_cast<uint32_t*>(a.queue), 0u, 1, s);
    hipLaunchKernelGGL(k_render_fwd_persistent, dim3((unsigned)a.blocks), dim3(kTileThreads), 0, s, R, a);
  } else {
    hipLaunchKernelGGL(k_render_fwd<false>, dim3((unsigned)a.n_items), dim3(kTileThreads), 0, s, R, a);
  }
}

void launch_render_bwd(const Raster& R, const BwdArgs& a, hipStream_t s) {
  const dim3 tb(kTileThreads);
  const bool det = a.part != nullptr;
  const bool queue = a.blocks > 0;
  const dim3 grid((unsigned)(queue ? a.blocks : a.n_items));
  if (queue) launch_fill_u32(reinterpret_cast<uint32_t*>(a.queue), 0u, 1, s);
  auto go = [&](auto one, auto many) {
    if (queue) hipLaunchKernelGGL(many, grid, tb, 0, s, R, a);
    else hipLaunchKernelGGL(one, grid, tb, 0, s, R, a);
  };
  auto with = [&](auto nf, auto sums) {
    constexpr int NF = decltype(nf)::value;
    constexpr BwdSums SUMS = decltype(sums)::value;
    if (a.gA) go(k_render_bwd<NF, SUMS, true>, k_render_bwd_persistent<NF, SUMS, true>);
    else go(k_render_bwd<NF, SUMS, false>, k_render_bwd_persistent<NF, SUMS, false>);
  };
  auto fields = [&](auto nf) {
    if (det) with(nf, std::integral_constant<BwdSums, kStored>());
    else if (a.wide) with(nf, std::integral_constant<BwdSums, kWide>());
    else with(nf, std::integral_constant<BwdSums, kFloat>());
  };
  // ten fields, or the six of a pose-only backward
  if (a.geom_only) fields(std::integral_constant<int, 6>());
  else fields(std::integral_constant<int, 10>());
}

void launch_det_rev(const Raster& R, const int2* ranges, const uint32_t* ids, const int4* rect, const uint32_t* goff,
                    uint32_t* rev, int n_items, hipStream_t s) {
  if (n_items <= 0) return;
  hipLaunchKernelGGL(k_det_rev, dim3((unsigned)n_items), dim3(256), 0, s, R, ranges, ids, rect, goff, rev);
}

void launch_det_reduce(const int4* rect, const uint32_t* goff, const uint32_t* rev, const uint32_t* mask,
                       const float* part, int64_t n_rec, bool geom_only, float* g2d, hipStream_t s) {
  if (n_rec <= 0) return;
  const int nf = geom_only ? 6 : 10;
  const unsigned g = (unsigned)((n_rec * nf + 255) / 256);
  if (geom_only)
    hipLaunchKernelGGL(k_det_reduce<6>, dim3(g), dim3(256), 0, s, rect, goff, rev, mask, part, n_rec, g2d);
  else
    hipLaunchKernelGGL(k_det_reduce<10>, dim3(g), dim3(256), 0, s, rect, goff, rev, mask, part, n_rec, g2d);
}

}  // namespace gsr
