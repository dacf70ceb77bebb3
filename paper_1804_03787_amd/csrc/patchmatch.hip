// Warped-patch costs: the cost refresh, the pixel lists of the restricted
// half-sweeps, and the half-sweep of a single call (msgpm_pm_halfsweep), which
// evaluates every candidate.  The passes of a whole solve, which evaluate only
// those that could win, are in search.h.
//
// Cost C(p, t, H): sum over the (2r+1)^2 taps d of the square patch of p of
//   sum_c w_c (F1_c(clamp(p + d)) - bilinear F2_c(t + Delta(d)))^2,
// Delta(d) = pi(H(p + d)) - pi(H p): the patch in the other frame is the square
// patch distorted by the plane's local motion around p (Sec. 3.1.3 compensates
// the plane distortion instead of enumerating distortions, Sec. 1).  The
// integer part of t + Delta is formed in integers, the fraction separately;
// bases below 0 or at/after the last pixel clamp with fraction 0.
//
// Work mapping (gfx950, wave64): a pixel is handled by 2r+1 adjacent lanes, lane
// j owning patch column dx = j - r for every candidate.  Each lane keeps its
// column's source features and tap geometry in registers.  A distorted tap
// needs the horizontal corner pairs of two rows, each fetched as one
// contiguous load (features are stored interleaved per pixel); integral
// geometries (identity, integer translations) fetch one pixel per tap.  Column
// partials are combined across the group in a fixed order, so every lane of the
// group takes the same decisions.  The single half-sweep evaluates identity-patch
// candidates in batches whose first rows are gathered together, each then finished
// on its own, and distorted-patch candidates one at a time; both with exact early
// rejections on partial sums (every schedule takes the decisions of a
// one-at-a-time loop).  Costs are accumulated in FP32; FP16 records are
// widened inside mixed-precision multiply-adds.
//
// PatchMatch (propagation + random search, as used by the paper for its NNF,
// Sec. 3.1) runs as red-black Jacobi half-sweeps: a pixel reads only the other
// colour's offsets, so a half-sweep is order-free.
#include "patch.h"
#include "search.h"

#pragma clang fp contract(off)

namespace msgpm {

// ---------------------------------------------------------------------------
// Cost refresh: cost[p] = C(p, p + v_p, H_p) for the selected pixels.
//
// A workgroup owns up to kCostSlots pixels: a tile of the frame (whose patches
// overlap), or a run of a list.  One lane per pixel takes its target and its
// plane's local motion (FP64) into LDS; then the lane groups take the selected
// pixels in turn, in rounds of 28 at r = 4, so that none sits idle for a pixel
// without a plane.
//
// Bound: dense frames by the gathers; few selected pixels by the latency of a
// workgroup, which waits for memory with every three rows of every round.  The
// selected pixels lie in clusters of whole windows, so that few workgroups have
// them all.  Refresh of the assigned pixels of a pair (mode 2, r = 4, FP32; 3 % and
// all assigned), in brackets with one lane group per pixel of a row and the motion
// computed by each of its lanes:
//    128x96  10 and 17 us (12, 19)     512x384  33 and 148 us (23, 163)
//   320x240  18 and 64 us (17, 70)    1024x436  46 and 331 us (51, 359)
//                                     2048x872 101 and 1277 us (187, 1413)
// ---------------------------------------------------------------------------
constexpr int kCostSlots = 168;

// Lane groups of a workgroup: the pixels of one round.
__host__ __device__ constexpr int cost_round(int r) { return kWave / (2 * r + 1) * (kBlock / kWave); }
__host__ __device__ constexpr int whole_rounds(int r, int pixels) {
  return (pixels + cost_round(r) - 1) / cost_round(r) * cost_round(r);
}
static_assert(whole_rounds(1, 128) <= kCostSlots && whole_rounds(2, 128) <= kCostSlots &&
                  whole_rounds(3, 128) <= kCostSlots && whole_rounds(4, 128) <= kCostSlots,
              "pixels of a workgroup");

// Tile of a workgroup.  Small frames: whole rounds, one or two, as a round of few
// pixels takes as long as a full one: of 64 pixels the third round is nearly empty
// (320x240 with 3 % assigned 22 us, with 56 pixels 18 us; 128x96 with 32 pixels 15
// us, with 28 10 us).  Larger frames: 128 pixels, which cost least where nothing
// is selected.  skew: by how many columns each row of tiles is turned on from the
// one above, so that the tiles of a column, which hold a cluster, are 9
// workgroups of an XCD apart (modulo its 32 compute units).  Without it the 32 or
// 64 tiles of a row of a 512 or 1024 pixels wide frame put a whole column on one
// compute unit: 42 instead of 33 us for 3 % of 512x384, 52 instead of 46 us of
// 1024x436.  Small frames lose by it (320x240 18 -> 20 us).
struct CostTile {
  int cols, rows, skew;
};
__host__ __device__ inline CostTile cost_tile(int r, int W, int H) {
  const int n = W * H;
  if (n >= 98304) return CostTile{16, 8, (((W + 15) >> 4) - 9) & 31};
  const int cols = r == 4 ? 14 : 12;  // which divide a round
  return CostTile{cols, whole_rounds(r, n < 32768 ? 28 : 56) / cols, 0};
}

// Pixels of a run of a list of cnt: one round until there are kCostRuns runs (of
// each of the four lists), then more rounds, up to what covers 128 pixels.  Runs of
// 32 to 128 pixels by the frame alone took 48 instead of 37 us for the 3 % unassigned
// pixels of a 1024x436 pair, 32 instead of 22 us at 512x384; all of them 361
// instead of 347 us.
constexpr int kCostRuns = 512;
__host__ __device__ inline int cost_run(int r, unsigned cnt) {
  const unsigned even = (cnt + kCostRuns - 1) / kCostRuns;
  return whole_rounds(r, even > 128u ? 128 : (even > 1u ? (int)even : 1));
}

struct CostLds {
  int pix[kCostSlots], tgt[kCostSlots];  // x | y << 16
  int valid[kCostSlots];                 // the plane has a motion there
  float motion[6][kCostSlots];
  float cost[kCostSlots];
  int n;
};

template <int R, int C, bool FP16, bool IDENT>
__device__ __forceinline__ void eval_cost_body(const DevParams& P, const Ws& w, Blk bk, int mode) {
  constexpr int G = 2 * R + 1, NG = kWave / G;
  __shared__ CostLds S;
  const int t = threadIdx.x, lane = t & (kWave - 1), wave = t / kWave;
  const int g = lane / G, j = lane - g * G, base = g * G;
  const int dir = bk.y;
  const int W = P.W, H = P.H;
  // this lane's pixel
  bool act = true;
  int x = 0, y = 0;
  if (mode == 1) {
    // the unassigned pixels, from the restricted pass's lists (both colours):
    // identity patches over the back lists (no region plane), distorted ones
    // over the front lists; each colour takes its own run of workgroups
    const unsigned c0 = w.act_count[2 * (2 * dir) + (IDENT ? 1 : 0)];
    const unsigned c1 = w.act_count[2 * (2 * dir + 1) + (IDENT ? 1 : 0)];
    const int run0 = cost_run(R, c0), run1 = cost_run(R, c1);
    const int nb0 = (int)((c0 + run0 - 1) / run0), nb1 = (int)((c1 + run1 - 1) / run1);
    if (bk.x >= nb0 + nb1) return;
    const int colour = bk.x < nb0 ? 0 : 1, run = colour ? run1 : run0;
    const unsigned i = (unsigned)xcd_remap(colour ? bk.x - nb0 : bk.x, colour ? nb1 : nb0) * run + t;
    act = t < run && i < (colour ? c1 : c0);
    const unsigned cap = (unsigned)((W + 1) >> 1) * (unsigned)H;
    const int q = act ? w.act[2 * dir + colour][IDENT ? cap - 1u - i : i] : 0;
    y = q / W;
    x = q - y * W;
  } else {
    const CostTile T = cost_tile(R, W, H);
    const int ntx = (W + T.cols - 1) / T.cols, b = xcd_remap(bk.x, bk.nx);
    const int row = b / ntx, col = (b - row * ntx + T.skew * row) % ntx;
    x = col * T.cols + t % T.cols;
    y = row * T.rows + t / T.cols;
    act = t < T.cols * T.rows && x < W && y < H;
  }
  const int p = y * W + x;
  int label = -1;
  if (act && !IDENT) {
    label = mode == 2 ? w.win[dir][p] : w.hlabel[dir][p];
    act = label >= 0;
  }
  if (t == 0) S.n = 0;
  __syncthreads();
  int slot = 0;
  if (wave < (kCostSlots + kWave - 1) / kWave) {
    const unsigned long long m = __ballot(act);
    int first = 0;
    if (lane == 0) first = atomicAdd(&S.n, __popcll(m));
    slot = __builtin_amdgcn_readfirstlane(first) + __popcll(m & ((1ull << lane) - 1ull));
    if (act) {
      const int32_t v = w.nnf[dir][p];
      S.pix[slot] = x | (y << 16);
      S.tgt[slot] = pack_off(x + off_dx(v), y + off_dy(v));
      if constexpr (!IDENT) {
        double qx, qy;
        float m6[6] = {};
        S.valid[slot] = plane_motion(w.planes[label].H, x, y, qx, qy, m6);
#pragma unroll
        for (int i = 0; i < 6; ++i) S.motion[i][slot] = m6[i];
      }
    }
  }
  __syncthreads();
  const int n = S.n;
  if (n == 0) {
    __syncthreads();  // a persistent launch clears S.n for its next workgroup
    return;
  }
  const Feat F1 = feat_buf<C, FP16>(w.feat[dir], W, H), F2 = feat_buf<C, FP16>(w.feat[1 - dir], W, H);
  for (int i0 = wave * NG; i0 < n; i0 += NG * (kBlock / kWave)) {
    const int i = i0 + g;
    if (g >= NG || i >= n) continue;
    const int px = S.pix[i] & 0xffff, py = (int)((unsigned)S.pix[i] >> 16);
    const int tx = off_dx(S.tgt[i]), ty = off_dy(S.tgt[i]);
    LaneCol<R, C, IDENT> L;
    int geo = 1;
    if constexpr (IDENT) {
      L.dx = j - R;
    } else {
      float m6[6];
#pragma unroll
      for (int q = 0; q < 6; ++q) m6[q] = S.motion[q][i];
      bool integral = false, ok = S.valid[i] != 0;
      if (ok) ok = tap_geometry<R, C>(L, m6, j - R, 4.0f * (float)(W > H ? W : H), integral);
      geo = group_geometry<G>(ok, integral, base);
    }
    float c = __builtin_huge_valf();
    if (geo != 2) {
      load_column<R, C, FP16, IDENT>(L, F1, W, H, px, py, j - R);
      bool rejected;
      unsigned rows = 0;
      if (IDENT || geo == 1)
        c = group_cost<R, C, FP16, IDENT, true, false>(L, F2, W, H, tx, ty, P.gw, base, 0.f, rejected, rows);
      else
        c = group_cost<R, C, FP16, IDENT, IDENT, false>(L, F2, W, H, tx, ty, P.gw, base, 0.f, rejected, rows);
    }
    if (j == 0) S.cost[i] = c;
  }
  __syncthreads();
  if (act) w.cost[dir][p] = S.cost[slot];
  if (t == 0)
    atomicAdd(&w.counters[(2 + dir) * kCounterStripes + (blockIdx.x & (kCounterStripes - 1))], (unsigned long long)n);
}

// Waves per SIMD the registers of distorted patches are held to: a final refresh
// of a 1024x436 pair with the outputs takes 182 us at the compiler's own choice of
// 2 (FP16 3: 116 us), 166 us at 3 (108 us at 4) and 227 us at 4, with spills.
constexpr int cost_waves(bool fp16, bool ident) { return ident ? 1 : (fp16 ? 4 : 3); }

template <int R, int C, bool FP16, bool IDENT>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(cost_waves(FP16, IDENT)))) void k_eval_cost(DevParams P, Ws w, int mode) {
  eval_cost_body<R, C, FP16, IDENT>(P, w, blk_here(), mode);
}

template <int R, int C, bool FP16, bool IDENT, bool LOOP>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(cost_waves(FP16, IDENT)))) void kb_eval_cost(const uint8_t* __restrict__ tab, int k, BArgs A) {
  const BatchView V = batch_view(tab, k);
  const PairDesc* __restrict__ pd = V.pd;
  const Item* __restrict__ it = V.it;
  const int n = V.n, total = V.total;
  for_each_item<true, LOOP>(it, n, total, [&](int i, Blk bk) {
    eval_cost_body<R, C, FP16, IDENT>(pd[it[i].pair].P, pd[it[i].pair].w, bk, A.a[0]);
  });
}

// Candidate loops of one pixel: the four neighbours' offsets (left, right, up,
// down), the plane candidate (restricted passes), then random search centred on
// the best offset after those; a candidate replaces the best only if strictly
// better.  Two schedules with identical decisions:
//  * identity patches (short per-candidate chain): candidates in batches of
//    NB; the first third of the rows of the batch is gathered together, then
//    each candidate still in the running is finished on its own, with exact
//    early rejections per lane group;
//  * distorted patches (long chain, register-heavy): one candidate at a time
//    with the exact early rejection of group_cost.

// Tap rows per load chunk of identity-patch batches: one (measured on MI355X, two
// or three rows per chunk take the kernel to 256 VGPRs and lose more than the
// longer chunks gain).
constexpr int kIdentRows = 1;
// Rows [T0, T) of NB identity-patch targets added to acc, in chunks of
// kIdentRows: each lane walks its column once, and the loads of a chunk (all
// candidates) are issued ahead of its arithmetic.
template <int R, int C, bool FP16, int NB, int T0, int T>
__device__ inline void ident_rows(float* acc, const LaneCol<R, C, true>& L, Feat F2, int W, int H, const int* tx,
                                  const int* ty, float gw) {
  IdentAddr<R, Px<C, FP16>::kBytes> A[NB] = {};
#pragma unroll
  for (int b = 0; b < NB; ++b) A[b] = IdentAddr<R, Px<C, FP16>::kBytes>(tx[b], ty[b], L.dx, W, H);
#pragma unroll
  for (int t0 = T0; t0 < T; t0 += kIdentRows) {
    constexpr int TC = kIdentRows;
    uint32_t v[TC][NB][Px<C, FP16>::kWords];
#pragma unroll
    for (int u = 0; u < TC; ++u)
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        if (t0 + u < T) Px<C, FP16>::raw1_at(F2, A[b].at(t0 + u), v[u][b]);
      }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < TC; ++u)
#pragma unroll
      for (int b = 0; b < NB; ++b)
        if (t0 + u < T) acc[b] += tap_sq_raw<C, FP16>(L.f1[t0 + u], v[u][b], gw);
    __builtin_amdgcn_sched_barrier(0);
  }
}

// Rows per step when one identity-patch candidate is finished, with an
// early-rejection check before each step.  Measured on MI355X at 1024x436
// (whole pipeline, r = 4, FP32 records): checks at rows 3 and 6 take 33.1 ms per
// pair, a check at row 3 only 33.9 ms, checks at rows 3, 5 and 7 33.8 ms,
// one at every row 38.2 ms; the batch-wide check this replaced took 37.3 ms.
constexpr int kIdentStep = 3;

// Rows [T0, T) of one identity-patch target in steps of kIdentStep rows, the
// group sum checked against bound before each step: false (and the rows
// computed added to rows) as soon as a partial sum is >= bound; otherwise a =
// the full lane partial and rows += T.
template <int R, int C, bool FP16, int T0>
__device__ inline bool ident_finish(float& a, float acc, const LaneCol<R, C, true>& L, Feat F2, int W, int H,
                                    int tx, int ty, float gw, int base, float bound, unsigned& rows) {
  constexpr int T = 2 * R + 1, T1 = T0 + kIdentStep < T ? T0 + kIdentStep : T;
  acc = ident_rows1<R, C, FP16, T0, T1>(acc, L, F2, W, H, tx, ty, gw);
  if constexpr (T1 == T) {
    a = acc;
    rows += T;
    return true;
  } else {
    if (!group_flag<T>(group_chain<T>(acc) < bound, base)) {
      rows += T1;
      return false;
    }
    return ident_finish<R, C, FP16, T1>(a, acc, L, F2, W, H, tx, ty, gw, base, bound, rows);
  }
}

// One identity-patch batch: NB targets, compared with the best in candidate
// order (a candidate replaces it only if strictly better), with the decisions
// of a one-at-a-time loop.  The first third of the rows of every target is
// gathered together; then each target still in the running is finished on its
// own, unless its partial sum is already >= the current best cost: taps are
// non-negative and FP32 addition is monotone, so its full cost could not be
// strictly lower, and its remaining rows are skipped.  The check is per lane
// group: the lanes of a dropped target sit out its remaining gathers, which
// is where the time goes (the cost of a gather scales with the lanes that
// take part in it).  A finished target is summed in the same order as a lone
// evaluation.  Every comparison is taken at the group's last lane, where the
// lane-order sum forms, and handed to the group by a ballot (group_flag), so
// the running best cost bc is exact at that lane only.  Both record formats
// use this form; with FP16 records (one load per tap) it was 3 % slower than
// gathering all rows of the batch and skipping the checks while the kernel's
// VALU work bound it, and after the per-target row offsets and the ballot
// decisions it is 7 % faster (measured on MI355X, 1024x436).
template <int R, int C, bool FP16, int NB>
__device__ inline void ident_batch(const LaneCol<R, C, true>& L, Feat F2, int W, int H, const int* tx,
                                   const int* ty, const bool* ok, float gw, int base, int& btx, int& bty, float& bc,
                                   unsigned& evals, unsigned& rows) {
  constexpr int T = 2 * R + 1, TE = T / 3;
  bool any = false;
#pragma unroll
  for (int b = 0; b < NB; ++b) any = any || ok[b];
  if (!any) return;
  float acc[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) acc[b] = 0.f;
  ident_rows<R, C, FP16, NB, 0, TE>(acc, L, F2, W, H, tx, ty, gw);
  float pre[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) pre[b] = group_chain<T>(acc[b]);
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    if (!ok[b]) continue;
    ++evals;
    if ((tx[b] == btx && ty[b] == bty) || !group_flag<T>(pre[b] < bc, base)) {
      rows += TE;
      continue;
    }
    float a;
    if (!ident_finish<R, C, FP16, TE>(a, acc[b], L, F2, W, H, tx[b], ty[b], gw, base, bc, rows)) continue;
    const float c = group_chain<T>(a);
    if (group_flag<T>(c < bc, base)) {
      bc = c;
      btx = tx[b];
      bty = ty[b];
    }
  }
}

// Random-search candidates k0 .. k0 + NB - 1 around (x + cdx, y + cdy), as one
// identity-patch batch.
template <int R, int C, bool FP16, int NB>
__device__ inline void random_batch(const LaneCol<R, C, true>& L, const DevParams& P, Feat F2, int x, int y,
                                    int cdx, int cdy, int k0, int base, const int* rox, const int* roy, int& btx,
                                    int& bty, float& bc, unsigned& evals, unsigned& rows) {
  constexpr int G = 2 * R + 1, NH = (16 + G - 1) / G;
  const int W = P.W, H = P.H;
  int tx[NB], ty[NB];
  bool ok[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    const int kk = k0 + b;
    const int src = base + (kk % G), slot_k = kk / G;
    int mx = rox[0], my = roy[0];
#pragma unroll
    for (int h = 1; h < NH; ++h) {
      mx = slot_k == h ? rox[h] : mx;
      my = slot_k == h ? roy[h] : my;
    }
    tx[b] = clampi(x + cdx + __shfl(mx, src), 0, W - 1);
    ty[b] = clampi(y + cdy + __shfl(my, src), 0, H - 1);
    ok[b] = !(tx[b] == btx && ty[b] == bty);
  }
  ident_batch<R, C, FP16, NB>(L, F2, W, H, tx, ty, ok, P.gw, base, btx, bty, bc, evals, rows);
}

// The last random-search batch, of rest < NB candidates (rest is the same for
// every lane).
template <int R, int C, bool FP16, int N>
__device__ inline void random_rest(int rest, const LaneCol<R, C, true>& L, const DevParams& P, Feat F2, int x, int y,
                                   int cdx, int cdy, int k0, int base, const int* rox, const int* roy, int& btx,
                                   int& bty, float& bc, unsigned& evals, unsigned& rows) {
  if constexpr (N > 0) {
    if (rest == N)
      random_batch<R, C, FP16, N>(L, P, F2, x, y, cdx, cdy, k0, base, rox, roy, btx, bty, bc, evals, rows);
    else
      random_rest<R, C, FP16, N - 1>(rest, L, P, F2, x, y, cdx, cdy, k0, base, rox, roy, btx, bty, bc, evals, rows);
  }
}

template <int R, int C, bool FP16>
__device__ inline void pm_candidates_ident(const LaneCol<R, C, true>& L, const DevParams& P, const Ws& w, int dir,
                                           int x, int y, int base, bool fresh, const int* rox, const int* roy,
                                           unsigned& evals, unsigned& rows) {
  constexpr int NB = 4;
  const int W = P.W, H = P.H, p = y * W + x;
  const Feat F2 = feat_buf<C, FP16>(w.feat[1 - dir], W, H);
  const int32_t* nnf = w.nnf[dir];
  const int32_t v0 = nnf[p];
  int btx = x + off_dx(v0), bty = y + off_dy(v0);
  float bc;
  if (fresh) {
    bool rejected;
    unsigned r0 = 0;
    bc = group_cost<R, C, FP16, true, true, false>(L, F2, W, H, btx, bty, P.gw, base, 0.f, rejected, r0);
  } else {
    bc = w.cost[dir][p];
  }
  {
    int tx[4], ty[4];
    bool ok[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int nx = x + (k == 0 ? -1 : (k == 1 ? 1 : 0));
      const int ny = y + (k == 2 ? -1 : (k == 3 ? 1 : 0));
      const bool inside = nx >= 0 && nx < W && ny >= 0 && ny < H;
      const int32_t v = nnf[clampi(ny, 0, H - 1) * W + clampi(nx, 0, W - 1)];
      tx[k] = clampi(x + off_dx(v), 0, W - 1);
      ty[k] = clampi(y + off_dy(v), 0, H - 1);
      ok[k] = inside && !(tx[k] == btx && ty[k] == bty);
    }
    ident_batch<R, C, FP16, 4>(L, F2, W, H, tx, ty, ok, P.gw, base, btx, bty, bc, evals, rows);
  }
  // random search in full batches, then one batch of the remaining radii (a
  // wave-uniform size, so no slot loads a patch for a radius that is not there)
  const int cdx = btx - x, cdy = bty - y;
  int k0 = 0;
  for (; k0 + NB <= P.nk; k0 += NB)
    random_batch<R, C, FP16, NB>(L, P, F2, x, y, cdx, cdy, k0, base, rox, roy, btx, bty, bc, evals, rows);
  random_rest<R, C, FP16, NB - 1>(P.nk - k0, L, P, F2, x, y, cdx, cdy, k0, base, rox, roy, btx, bty, bc, evals,
                                  rows);
  // the running best cost is exact at the group's last lane (group_flag)
  if (base + 2 * R == (int)(threadIdx.x & (kWave - 1))) {
    w.nnf[dir][p] = pack_off(btx - x, bty - y);
    w.cost[dir][p] = bc;
  }
}

template <int R, int C, bool FP16, bool IDENT, bool INTEGRAL>
__device__ inline void pm_candidates_serial(const LaneCol<R, C, IDENT>& L, const DevParams& P, const Ws& w, int dir, int x,
                                     int y, int base, bool fresh, bool has_plane, int ptx, int pty, const int* rox,
                                     const int* roy, unsigned& evals, unsigned& rows) {
  constexpr int G = 2 * R + 1, NH = (16 + G - 1) / G;
  constexpr bool EE = true;
  const int W = P.W, H = P.H, p = y * W + x;
  const Feat F2 = feat_buf<C, FP16>(w.feat[1 - dir], W, H);
  const int32_t* nnf = w.nnf[dir];
  const int32_t v0 = nnf[p];
  int btx = x + off_dx(v0), bty = y + off_dy(v0);
  float bc;
  if (fresh) {
    bool rejected;
    unsigned r0 = 0;
    bc = group_cost<R, C, FP16, IDENT, INTEGRAL, false>(L, F2, W, H, btx, bty, P.gw, base, 0.f, rejected, r0);
  } else {
    bc = w.cost[dir][p];
  }
  int cdx = 0, cdy = 0;
  for (int k = 0; k < 5 + P.nk; ++k) {
    int tx, ty;
    if (k < 4) {
      const int nx = x + (k == 0 ? -1 : (k == 1 ? 1 : 0));
      const int ny = y + (k == 2 ? -1 : (k == 3 ? 1 : 0));
      if (nx < 0 || nx >= W || ny < 0 || ny >= H) continue;
      const int32_t v = nnf[ny * W + nx];
      tx = clampi(x + off_dx(v), 0, W - 1);
      ty = clampi(y + off_dy(v), 0, H - 1);
    } else if (k == 4) {
      if (!has_plane) continue;
      tx = ptx;
      ty = pty;
    } else {
      if (k == 5) {
        cdx = btx - x;
        cdy = bty - y;
      }
      const int kk = k - 5;
      const int src = base + (kk % G), slot_k = kk / G;
      int mx = rox[0], my = roy[0];
#pragma unroll
      for (int h = 1; h < NH; ++h) {
        mx = slot_k == h ? rox[h] : mx;
        my = slot_k == h ? roy[h] : my;
      }
      tx = clampi(x + cdx + __shfl(mx, src), 0, W - 1);
      ty = clampi(y + cdy + __shfl(my, src), 0, H - 1);
    }
    if (tx == btx && ty == bty) continue;  // same target: same cost, never strictly better
    bool rejected;
    const float c = group_cost<R, C, FP16, IDENT, INTEGRAL, EE>(L, F2, W, H, tx, ty, P.gw, base, bc, rejected, rows);
    ++evals;
    if (!rejected && c < bc) {
      bc = c;
      btx = tx;
      bty = ty;
    }
  }
  if (base == (int)(threadIdx.x & (kWave - 1))) {
    w.nnf[dir][p] = pack_off(btx - x, bty - y);
    w.cost[dir][p] = bc;
  }
}

// ---------------------------------------------------------------------------
// Restricted half-sweeps update only the unassigned pixels of one colour.
// They are listed first, so that every lane group of the sweep has a pixel,
// in two lists sharing one buffer per direction: pixels with a region plane
// from the front (distorted patches), pixels without one from the back
// (identity patches: the update of the initial pass, without a plane
// candidate).  The first half of a direction's workgroups lists colour 0, the
// second colour 1.  Each workgroup appends the pixels of its span at
// positions taken from the two counters; the order of the spans varies between
// runs, and the update of a pixel does not depend on it.
// ---------------------------------------------------------------------------
__global__ void k_zero_active(Ws w) {
  if (threadIdx.x < 8) w.act_count[threadIdx.x] = 0u;
}

constexpr int kListSpan = 4;  // pixels of the colour per thread of k_active_list

__device__ __forceinline__ void active_list_body(const DevParams& P, const Ws& w, Blk bk) {
  constexpr int NS = kListSpan * (kBlock / kWave);
  __shared__ int s_cnt[2][NS];
  __shared__ unsigned s_base[2];
  const int dir = bk.y, half = bk.nx >> 1, colour = bk.x >= half ? 1 : 0;
  bk.x -= colour * half;
  const int W = P.W, H = P.H, Wh = (W + 1) >> 1, ntx = (W + 15) >> 4;
  const unsigned cap = (unsigned)Wh * (unsigned)H;
  const int t = threadIdx.x, lane = t & (kWave - 1), wave = t / kWave;
  int pixA[kListSpan], pixB[kListSpan];
  bool inA[kListSpan], inB[kListSpan];
  unsigned long long mA[kListSpan], mB[kListSpan];
#pragma unroll
  for (int k = 0; k < kListSpan; ++k) {
    // Pixels with a region plane row by row, the others (whose patches are
    // squares) by tiles of 16 x 8 pixels, 64 of the colour, so that a workgroup's
    // patches overlap: solves of 2048x872 FP16 pairs 73.1 ms -> 67.8 ms, of
    // 1024x436 16.2 ms -> 16.1 ms.  Tiles for both: 67.5 ms and 16.8 ms, as a
    // tile's distorted patches are alike in work and the long ones end up together.
    const int i = (bk.x * kListSpan + k) * kBlock + t, tile = i >> 6;
    const int ya = i / Wh, xa = 2 * (i - ya * Wh) + ((ya + colour) & 1);
    const int yb = tile / ntx * 8 + ((i >> 3) & 7), xb = tile % ntx * 16 + 2 * (i & 7) + ((yb + colour) & 1);
    pixA[k] = ya * W + xa;
    pixB[k] = yb * W + xb;
    inA[k] = xa < W && ya < H && w.win[dir][pixA[k]] < 0 && w.hlabel[dir][pixA[k]] >= 0;
    inB[k] = xb < W && yb < H && w.win[dir][pixB[k]] < 0 && w.hlabel[dir][pixB[k]] < 0;
    mA[k] = __ballot(inA[k]);
    mB[k] = __ballot(inB[k]);
    if (lane == 0) {
      s_cnt[0][k * (kBlock / kWave) + wave] = __popcll(mA[k]);
      s_cnt[1][k * (kBlock / kWave) + wave] = __popcll(mB[k]);
    }
  }
  __syncthreads();
  if (t < 2) {
    unsigned total = 0u;
    for (int k = 0; k < NS; ++k) total += s_cnt[t][k];
    s_base[t] = total ? atomicAdd(&w.act_count[2 * (2 * dir + colour) + t], total) : 0u;
  }
  __syncthreads();
  unsigned posA = s_base[0], posB = s_base[1];
  int done = 0;
  const unsigned long long lt = (1ull << lane) - 1ull;
#pragma unroll
  for (int k = 0; k < kListSpan; ++k) {
    const int mine = k * (kBlock / kWave) + wave;
    for (; done < mine; ++done) {
      posA += s_cnt[0][done];
      posB += s_cnt[1][done];
    }
    int32_t* list = w.act[2 * dir + colour];
    if (inA[k]) list[posA + __popcll(mA[k] & lt)] = pixA[k];
    if (inB[k]) list[cap - 1u - (posB + __popcll(mB[k] & lt))] = pixB[k];
  }
}

__global__ __launch_bounds__(kBlock) void k_active_list(DevParams P, Ws w) {
  active_list_body(P, w, blk_here());
}

__global__ __launch_bounds__(kBlock) void kb_active_list(const uint8_t* __restrict__ tab, int k, BArgs A) {
  const BatchView V = batch_view(tab, k);
  const PairDesc* __restrict__ pd = V.pd;
  const Item* __restrict__ it = V.it;
  const int n = V.n, total = V.total;
  for_each_item<true>(it, n, total, [&](int i, Blk bk) {
    active_list_body(pd[it[i].pair].P, pd[it[i].pair].w, bk);
  });
}

// ---------------------------------------------------------------------------
// One red-black half-sweep over the pixels of one colour, both directions
// (restricted: over the listed pixels).
// ---------------------------------------------------------------------------
// The distorted-patch form is held to 168 VGPRs (3 waves per SIMD): on MI355X
// the extra wave hides more gather latency than the few registers it costs.
// mode bit 0: restricted; bit 1 (fresh): the pixel's current cost is computed
// first, as the cost refresh of that pass computes it, instead of being read,
// so that the first half-sweep of each colour stands in for the refresh.
template <int R, int C, bool FP16, bool IDENT>
__device__ __forceinline__ void pm_halfsweep_body(const DevParams& P, const Ws& w, Blk bk, int colour, int iter,
                                                  int slot, int mode) {
  constexpr int G = 2 * R + 1, NG = kWave / G;
  const int restricted = mode & 1;
  const bool fresh = (mode & 2) != 0;
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int g = lane / G, j = lane - g * G, base = g * G;
  const int dir = bk.y;
  const int W = P.W, H = P.H, Wh = (W + 1) >> 1;
  bool act;
  int x, y;
  if (restricted) {
    // only the workgroups covering the list work; each XCD takes a contiguous
    // part.  Distorted patches: the front list; identity patches: the back one.
    const unsigned cnt = w.act_count[2 * (2 * dir + colour) + (IDENT ? 1 : 0)];
    constexpr unsigned per = NG * (kBlock / kWave);
    const int nb = (int)((cnt + per - 1) / per);
    if (bk.x >= nb) return;
    const long long i = ((long long)xcd_remap(bk.x, nb) * (kBlock / kWave) + wave) * NG + g;
    act = g < NG && i < (long long)cnt;
    const unsigned cap = (unsigned)Wh * (unsigned)H;
    const int q = act ? w.act[2 * dir + colour][IDENT ? cap - 1u - (unsigned)i : (unsigned)i] : 0;
    y = q / W;
    x = q - y * W;
  } else {
    const long long i = ((long long)xcd_remap(bk.x, bk.nx) * (kBlock / kWave) + wave) * NG + g;
    act = g < NG && i < (long long)Wh * H;
    y = act ? (int)(i / Wh) : 0;
    x = act ? 2 * (int)(i - (long long)y * Wh) + ((y + colour) & 1) : 0;
    act = act && x < W;
  }
  const int p = y * W + x;
  unsigned evals = 0, rows = 0, refreshed = 0;
  if (act) {
    const int label = restricted ? w.hlabel[dir][p] : -1;
    const double* Hp = plane_H(w, label);
    const float lim = 4.0f * (float)(W > H ? W : H);

    // random-search draws of this pixel, computed by the lanes of the group:
    // lane j holds radii k = j, j + G, j + 2G, ... (up to 16 radii)
    constexpr int NH = (16 + G - 1) / G;
    const uint64_t w3 = rng_word3(2, dir, slot, 0);
    int rox[NH], roy[NH];
#pragma unroll
    for (int h = 0; h < NH; ++h) {
      const int k = j + h * G;
      rox[h] = roy[h] = 0;
      if (k < P.nk) {
        const int Rk = P.R0 >> k;
        uint64_t c[4] = {(uint64_t)(uint32_t)p, (uint64_t)k, (uint64_t)iter, w3};
        philox4x64(c, P.seed, 0);
        rox[h] = draw_below(c[0], (uint32_t)(2 * Rk + 1)) - Rk;
        roy[h] = draw_below(c[1], (uint32_t)(2 * Rk + 1)) - Rk;
      }
    }

    LaneCol<R, C, IDENT> L;
    bool integral;
    const bool ok = setup_geometry<R, C, IDENT>(L, Hp, x, y, j - R, lim, integral);
    const int geo = group_geometry<G>(ok, integral, base);
    // a non-positive homogeneous coordinate makes every candidate +inf: no update
    if (geo != 2) {
      load_column<R, C, FP16, IDENT>(L, feat_buf<C, FP16>(w.feat[dir], W, H), W, H, x, y, j - R);
      // plane candidate: where the region plane sends p, rounded to the grid
      bool has_plane = false;
      int ptx = 0, pty = 0;
      if (restricted && Hp) {
        const double ww = Hp[6] * x + Hp[7] * y + Hp[8];
        if (ww > 0) {
          const double qx = (Hp[0] * x + Hp[1] * y + Hp[2]) / ww;
          const double qy = (Hp[3] * x + Hp[4] * y + Hp[5]) / ww;
          double rx = floor(qx + 0.5), ry = floor(qy + 0.5);
          const double dl = (double)lim;
          rx = rx < -dl ? -dl : (rx > dl ? dl : rx);
          ry = ry < -dl ? -dl : (ry > dl ? dl : ry);
          ptx = clampi((int)rx, 0, W - 1);
          pty = clampi((int)ry, 0, H - 1);
          has_plane = true;
        }
      }
      if constexpr (IDENT)
        pm_candidates_ident<R, C, FP16>(L, P, w, dir, x, y, base, fresh, rox, roy, evals, rows);
      else if (geo == 1)
        pm_candidates_serial<R, C, FP16, IDENT, true>(L, P, w, dir, x, y, base, fresh, has_plane, ptx, pty, rox, roy,
                                                      evals, rows);
      else
        pm_candidates_serial<R, C, FP16, IDENT, false>(L, P, w, dir, x, y, base, fresh, has_plane, ptx, pty, rox,
                                                       roy, evals, rows);
    } else if (fresh && j == 0) {
      w.cost[dir][p] = __builtin_huge_valf();
    }
    if (j != 0) evals = rows = 0;
    refreshed = fresh && j == 0 ? 1 : 0;
  }
  count_evals<IDENT>(w.counters, (restricted ? (IDENT ? 10 : 4) : 0) + dir, evals);
  count_evals<IDENT>(w.counters, (restricted ? (IDENT ? 12 : 8) : 6) + dir, rows);
  if (fresh) count_evals<IDENT>(w.counters, 2 + dir, refreshed);
}

template <int R, int C, bool FP16, bool IDENT>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(IDENT ? 4 : 3))) void k_pm_halfsweep(
    DevParams P, Ws w, int colour, int iter, int slot, int mode) {
  pm_halfsweep_body<R, C, FP16, IDENT>(P, w, blk_here(), colour, iter, slot, mode);
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
template <int R, int C, bool FP16, bool IDENT>
static hipError_t pm_launch(const DevParams& P, const Ws& w, int colour, int iter, int slot, int mode,
                            hipStream_t s) {
  constexpr int G = 2 * R + 1, NG = kWave / G;
  const long long n = (long long)((P.W + 1) >> 1) * P.H;
  const long long per = (long long)NG * (kBlock / kWave);
  const int nb = (int)((n + per - 1) / per);
  hipLaunchKernelGGL((k_pm_halfsweep<R, C, FP16, IDENT>), dim3(nb, 2), dim3(kBlock), 0, s, P, w, colour, iter, slot,
                     mode);
  return hipGetLastError();
}

// Restricted half-sweep over the lists of launch_pm_lists: the distorted-patch
// kernel over the front list or the identity-patch kernel over the back one
// (both read only the other colour, so their order does not matter).
template <int R, int C, bool FP16>
static hipError_t dispatch_restricted(const DevParams& P, const Ws& w, int colour, int iter, int slot, int ident,
                                      int fresh, hipStream_t s) {
  const int mode = 1 | (fresh ? 2 : 0);
  if (ident) return pm_launch<R, C, FP16, true>(P, w, colour, iter, slot, mode, s);
  return pm_launch<R, C, FP16, false>(P, w, colour, iter, slot, mode, s);
}

// Workgroups of k_active_list for both colours of a direction: the tiles cover
// no fewer pixels than the rows.
static int list_blocks(const DevParams& P) {
  const int tiles = ((P.W + 15) >> 4) * ((P.H + 7) >> 3), per = kListSpan * kBlock / 64;
  return 2 * ((tiles + per - 1) / per);
}

// The lists of both colours; they hold for every half-sweep of a restricted
// pass (assignment and region planes do not change during it).
// cleared: their counts are 0 already (k_nnf_update).
hipError_t launch_pm_lists(const DevParams& P, const Ws& w, bool cleared, hipStream_t s) {
  if (!cleared) {
    hipLaunchKernelGGL(k_zero_active, dim3(1), dim3(kWave), 0, s, w);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k_active_list, dim3(list_blocks(P), 2), dim3(kBlock), 0, s, P, w);
  return hipGetLastError();
}

// Workgroups of one direction of a cost refresh: tiles, or (mode 1) runs of both
// colours' lists.
static int cost_blocks(const DevParams& P, int mode) {
  if (mode == 1) {
    // a list has at most kCostRuns runs or, where those are of the most pixels, what covers it
    const int half = ((P.W + 1) >> 1) * P.H, one = whole_rounds(P.r, 1), most = whole_rounds(P.r, 128);
    const int short_runs = (half + one - 1) / one, long_runs = (half + most - 1) / most;
    const int few = short_runs < kCostRuns ? short_runs : kCostRuns;
    return 2 * (few > long_runs ? few : long_runs);
  }
  const CostTile T = cost_tile(P.r, P.W, P.H);
  return ((P.W + T.cols - 1) / T.cols) * ((P.H + T.rows - 1) / T.rows);
}

template <int R, int C, bool FP16, bool IDENT>
static hipError_t ec_launch(const DevParams& P, const Ws& w, int mode, hipStream_t s) {
  hipLaunchKernelGGL((k_eval_cost<R, C, FP16, IDENT>), dim3(cost_blocks(P, mode), 2), dim3(kBlock), 0, s, P, w, mode);
  return hipGetLastError();
}

template <int R, int C, bool FP16>
static hipError_t dispatch_pm(const DevParams& P, const Ws& w, int colour, int iter, int slot, int fresh,
                              hipStream_t s) {
  return pm_launch<R, C, FP16, true>(P, w, colour, iter, slot, fresh ? 2 : 0, s);
}

template <int R, int C, bool FP16>
static hipError_t dispatch_ec(const DevParams& P, const Ws& w, int mode, hipStream_t s) {
  if (mode == 0) return ec_launch<R, C, FP16, true>(P, w, mode, s);
  if (mode == 1) {
    hipError_t e = ec_launch<R, C, FP16, true>(P, w, mode, s);
    if (e != hipSuccess) return e;
  }
  return ec_launch<R, C, FP16, false>(P, w, mode, s);
}

hipError_t launch_pm_halfsweep(const DevParams& P, const Ws& w, int colour, int iter, int slot, int fresh,
                               hipStream_t s) {
  MSGPM_DISPATCH(dispatch_pm, P, w, colour, iter, slot, fresh, s);
}

hipError_t launch_pm_restricted(const DevParams& P, const Ws& w, int colour, int iter, int slot, int ident,
                                int fresh, hipStream_t s) {
  MSGPM_DISPATCH(dispatch_restricted, P, w, colour, iter, slot, ident, fresh, s);
}

hipError_t launch_eval_cost(const DevParams& P, const Ws& w, int mode, hipStream_t s) {
  MSGPM_DISPATCH(dispatch_ec, P, w, mode, s);
}

template <int R, int C, bool FP16, bool LOOP>
static void dispatch_batched_form(int kind, const uint8_t* tab, int k, dim3 grid, BArgs A, hipStream_t s) {
  const dim3 block(kBlock);
  if (kind == BK_EVAL_COST_IDENT)
    hipLaunchKernelGGL((kb_eval_cost<R, C, FP16, true, LOOP>), grid, block, 0, s, tab, k, A);
  else
    hipLaunchKernelGGL((kb_eval_cost<R, C, FP16, false, LOOP>), grid, block, 0, s, tab, k, A);
}

// persistent (loop over the virtual workgroups) or one-shot (grid >= total)
template <int R, int C, bool FP16>
static hipError_t dispatch_batched(int kind, const uint8_t* tab, int k, int ngrid, BArgs A, bool persist,
                                   hipStream_t s) {
  if (kind != BK_EVAL_COST_IDENT && kind != BK_EVAL_COST_PLANE) return hipErrorInvalidValue;
  if (persist)
    dispatch_batched_form<R, C, FP16, true>(kind, tab, k, dim3(ngrid, 2), A, s);
  else
    dispatch_batched_form<R, C, FP16, false>(kind, tab, k, dim3(ngrid, 2), A, s);
  return hipGetLastError();
}

hipError_t launch_batched_pm(int kind, const DevParams& P0, const uint8_t* tab, int k, int grid, BArgs A,
                             bool persist, hipStream_t s) {
  if (kind == BK_ACTIVE_LIST) {
    hipLaunchKernelGGL(kb_active_list, dim3(grid, 2), dim3(kBlock), 0, s, tab, k, A);
    return hipGetLastError();
  }
  const DevParams& P = P0;
  MSGPM_DISPATCH(dispatch_batched, kind, tab, k, grid, A, persist, s);
}

// Workgroups of the PatchMatch-side kernels for one pair (the single-pair
// launchers' grids).
int pm_batch_blocks(int kind, const DevParams& P, const int* a) {
  switch (kind) {
    case BK_EVAL_COST_IDENT:
    case BK_EVAL_COST_PLANE:
      return cost_blocks(P, a ? a[0] : 0);
    case BK_ACTIVE_LIST:
      return list_blocks(P);
    default:
      return search_batch_blocks(kind, P);
  }
}

// ---------------------------------------------------------------------------
// Self-check of the mixed-precision helpers of the FP16 records against
// widening first: thread i takes a word whose low half is FP16 pattern i (all
// 65536 patterns over the grid) and whose high half is another pattern, and
// compares every helper with the plain conversion-then-FP32 arithmetic for
// `rounds` partner words and FP32 operands drawn by an integer hash.  Results
// differ only where both are NaN (payloads are not compared).
// ---------------------------------------------------------------------------
__device__ inline uint32_t check_mix32(uint32_t x) {
  x ^= x >> 16;
  x *= 0x7feb352du;
  x ^= x >> 15;
  x *= 0x846ca68bu;
  x ^= x >> 16;
  return x;
}

__device__ inline float widen(uint32_t u, bool hi) {
  return (float)__builtin_bit_cast(_Float16, (uint16_t)(hi ? (u >> 16) : (u & 0xffffu)));
}

__device__ inline unsigned differs(float a, float b) {
  return (__float_as_uint(a) != __float_as_uint(b) && !(a != a && b != b)) ? 1u : 0u;
}

__global__ __launch_bounds__(kBlock) void k_check_fp16_arith(int rounds, unsigned long long* out) {
  const uint32_t i = blockIdx.x * kBlock + threadIdx.x;
  const uint32_t ua = (i & 0xffffu) | ((check_mix32(i) & 0xffffu) << 16);
  unsigned bad = 0;
  for (int j = 0; j < rounds; ++j) {
    const uint32_t ub = check_mix32(i * 131u + (uint32_t)j * 2654435761u);
    const uint32_t r = check_mix32(ub ^ 0x9e3779b9u);
    // FP32 operands over many magnitudes: a 24-bit mantissa scaled by 2^(e - 24)
    const float f = ldexpf((float)(int)(r & 0xffffffu) - 8388608.f, (int)((r >> 24) & 31u) - 36);
    const float w = ldexpf((float)(int)(check_mix32(r) & 0xffffffu) - 8388608.f, -23);
    const float a0 = widen(ua, false), a1 = widen(ua, true), b0 = widen(ub, false), b1 = widen(ub, true);
    bad += differs(sub_half<false>(f, ua), f - a0) + differs(sub_half<true>(f, ua), f - a1);
    bad += differs(sub_halves<false, false>(ua, ub), a0 - b0) + differs(sub_halves<true, true>(ua, ub), a1 - b1);
    bad += differs(sub_halves<true, false>(ua, ub), a1 - b0) + differs(sub_halves<false, true>(ua, ub), a0 - b1);
    bad += differs(sub_half_f32<false>(ua, f), a0 - f) + differs(sub_half_f32<true>(ua, f), a1 - f);
    bad += differs(fma_half<false>(ua, w, f), fmaf(a0, w, f)) + differs(fma_half<true>(ua, w, f), fmaf(a1, w, f));
    bad += differs(mul_half<false>(ua, w), a0 * w + 0.f) + differs(mul_half<true>(ua, w), a1 * w + 0.f);
  }
  if (bad) atomicAdd(out, (unsigned long long)bad);
}

__global__ void k_check_clear(unsigned long long* out) {
  if (threadIdx.x == 0) *out = 0ull;
}

hipError_t launch_check_fp16_arith(int rounds, unsigned long long* out, hipStream_t s) {
  hipLaunchKernelGGL(k_check_clear, dim3(1), dim3(64), 0, s, out);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_check_fp16_arith, dim3(65536 / kBlock), dim3(kBlock), 0, s, rounds, out);
  return hipGetLastError();
}

}  // namespace msgpm
