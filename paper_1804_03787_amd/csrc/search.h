// PatchMatch passes of the whole pipeline: half-sweeps that evaluate only the
// candidates that could win.
//
// A half-sweep gives every pixel the best of its current offset, its four
// neighbours' offsets, the plane candidate (distorted patches) and the random
// search around the best of those, a candidate replacing the best only if its
// FP32 cost (patch.h) is strictly lower.  Within a pass three exact
// arguments drop candidates before any of their patch is read:
//
//  * Unchanged neighbours.  A pixel keeps in its (otherwise constant) win entry
//    whether its last half-sweep changed its offset.  The offset of a
//    neighbour that did not change was offered in the pixel's previous
//    half-sweep of this pass and did not beat a best that has only fallen
//    since.  The plane candidate is the same all through a pass, so it is
//    evaluated in the first half-sweep alone.
//  * Targets tried before.  The same entry holds the positions of the 5x5
//    neighbourhood of the best that random search tried since the best was
//    set: the smallest radii draw them again and again.
//  * A lower bound from patch moments.  The SSD of two patches is at least the
//    squared distance of their projections on any orthonormal functions; here
//    the mean, the x and y slope and the x y term of the colour channels,
//    stored per pixel in 12 bytes (k_moments).  One 12-byte load per candidate,
//    made by one lane, stands in for the first rows of its patch: at 1024x436
//    it drops over nine tenths of the random targets at radii of 32 pixels and
//    more.  For a distorted patch the bound is lowered by what the distortion
//    can change, from a measure of the target's roughness kept beside the
//    moments.
//
// A pixel's candidate of the lowest bound is evaluated first, so that the others
// meet the lowest cost there is to be found; equal costs go to the candidate
// offered first, as in a one-at-a-time loop.
//
// What is left is evaluated by lane groups as everywhere else (a pixel by 2r+1
// lanes), so the accepted costs are the same bits.  A workgroup owns up to 64
// pixels: its lanes, one per candidate, propose and filter; then the pixels with
// work, sorted by their number of candidates so that the groups of a wave finish
// together, go to the lane groups of its four waves.  The two phases run twice,
// for propagation and for random search, and meet in LDS.
#pragma once

#include "patch.h"

#pragma clang fp contract(off)

namespace msgpm {

// win entry of an unassigned pixel during a pass: the sign, whether its last
// half-sweep changed its offset, and the tried positions around its best
// ((dy + 2) * 5 + dx + 2).  -1, the value outside passes, reads as changed.
constexpr unsigned kMemoSign = 0x80000000u, kMemoChanged = 1u << 25, kMemoTried = (1u << 25) - 1u;
static_assert((int32_t)(kMemoSign | kMemoChanged | kMemoTried) == kLastNote, "notes end at kLastNote");

constexpr int kTgtRows = 16;          // random-search radii: at most 15; neighbours and plane: 5
constexpr unsigned kRefresh = 1u << 31;  // in a candidate mask: the current cost first

constexpr int kSlots = 64;  // pixels of a workgroup

struct SearchLds {
  int tgt[kTgtRows][kSlots];  // random search: drawn offsets, then targets x | y << 16
  int ptgt[5][kSlots];        // propagation (and plane) targets
  uint16_t lb[kTgtRows][kSlots], plb[5][kSlots];  // their cost bounds (upper half of an FP32)
  unsigned mask[2][kSlots];   // candidates to evaluate, propagation and random search
  unsigned key[2][kSlots];    // the one of the lowest bound (its number in the low 4 bits)
  int pix[kSlots];            // x | y << 16, -1: no pixel
  int best0[kSlots], best[kSlots];  // best target before the half-sweep and now
  float bc[kSlots];           // its cost
  unsigned memo[kSlots];      // positions tried around best0 before
  unsigned tried[kSlots];     // positions tried around the best after propagation
  int won[kSlots];            // random search changed the best
  uint32_t src[3][kSlots];    // the pixel's moments
  float shift[kSlots];        // distorted patches: of the bound, and the plane's local motion
  float motion[6][kSlots];
  int order[kSlots];          // pixels with work, most candidates first
};

__device__ inline void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ inline int pack_xy(int x, int y) { return x | (y << 16); }
__device__ inline int xy_x(int v) { return v & 0xffff; }
__device__ inline int xy_y(int v) { return (int)((unsigned)v >> 16); }

// ---------------------------------------------------------------------------
// Patch moments
// ---------------------------------------------------------------------------
// Per pixel and colour channel the projections of its (border-clamped) patch
// on the orthonormal functions 1/T, x/sqrt(T n), y/sqrt(T n), x y/n (T = 2r+1,
// n = sum of x^2 over a row; the last not for blue), quantised to int8 in units
// of 1/scale: word c of a pixel holds channel c's.  The pixel values are first
// moved by the centre and cut to twice the half range of a sample of both
// frames, then the moments are cut to +-127 units; both cuts bring two values
// closer or leave their distance, so the bound below holds whatever the sample
// gave.  Rounding moves each component of a difference by at most 1 unit (FP32
// sums add under 0.01), so two patches whose stored vectors are D apart are at
// least (D - sqrt(11) - 0.01) / scale apart, and their SSD is at least the square.
//
// A distorted patch samples the target at d + a(d) instead of d.  With |a| <= 1
// along both axes, bilinear interpolation differs from the pixel at d by at
// most |ax| hx + |ay| hy per channel, hx the largest difference of horizontal
// neighbours at that pixel and at the rows above and below, hy that of its
// vertical ones.  So if |a(d)| <= b |d| at every tap, the sampled patch is at
// most b K from the undistorted one, K^2 the sum of |d|^2 (hx^2 + hy^2) over
// the patch.  The last byte of a pixel holds K, rounded up, in units of
// kRough / scale; 255: larger, or not known.
//
// That is the exact interpolation.  In FP32 (u = 2^-24) the four weights are off by
// at most 3u of their value, and the sums of four terms that stay within the
// largest corner M add 4u M, so that a sample is off by under 7.01u M, and the
// patch by sqrt(3) T as much.  In units that is kRounding M / half range, whatever
// T.  M is bounded by the centre and kFar half ranges; where a tap could read a
// pixel farther from the centre, K counts as not known.  On frames that span
// their range the term is under 0.003 units; past a level of 30000 half ranges
// it outgrows the other slack.
constexpr int kMomW = 32, kMomH = 8;  // pixels of a workgroup's tile
constexpr float kMomSlack = 3.3267f;  // sqrt(11) + 0.01
constexpr float kRough = 4.0f;
constexpr float kFar = 16.0f;
constexpr float kRounding = 1.15e-4f;  // 127 / 0.8 sqrt(3) 7.01 u

template <int R>
struct MomLds {
  static constexpr int TW = kMomW + 2 * R, TH = kMomH + 2 * R;
  float v[3][TH + 2][TW + 2];
  float h2[TH][TW];
  float s0[3][TH][kMomW], s1[3][TH][kMomW], q0[TH][kMomW], q2[TH][kMomW];
  float red[2][kBlock / kWave];
};

__device__ inline float rgb_value(const DevParams& P, const void* F, size_t i) {
  return P.fp16 ? __half2float(reinterpret_cast<const __half*>(F)[i]) : reinterpret_cast<const float*>(F)[i];
}

// Centre and half range of a fixed sample of both frames' colours, the same in
// every workgroup: half the threads read each frame.
__device__ inline void moment_range(const DevParams& P, const Ws& w, int stride, float (&red)[2][kBlock / kWave],
                                    float& centre, float& half) {
  const int t = threadIdx.x;
  const size_t p = (size_t)(((long long)P.W * P.H * (2 * (t & 127) + 1)) >> 8);
  float lo = __builtin_huge_valf(), hi = -__builtin_huge_valf();
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const float v = rgb_value(P, w.feat[t >> 7], p * stride + c);
    lo = fminf(lo, v);
    hi = fmaxf(hi, v);
  }
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    lo = fminf(lo, __shfl_xor(lo, o));
    hi = fmaxf(hi, __shfl_xor(hi, o));
  }
  if ((t & (kWave - 1)) == 0) {
    red[0][t / kWave] = lo;
    red[1][t / kWave] = hi;
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < kBlock / kWave; ++i) {
    lo = fminf(lo, red[0][i]);
    hi = fmaxf(hi, red[1][i]);
  }
  centre = 0.5f * (lo + hi);
  half = 0.5f * (hi - lo);
}

// bk.y = frame.  The moments of frame f go where the tentative assignment of
// direction f is kept, which is free during a PatchMatch pass: its labels and
// its losses lie one after the other, 12 bytes per pixel.
template <int R>
__device__ __forceinline__ void moments_body(const DevParams& P, const Ws& w, Blk bk) {
  constexpr int T = 2 * R + 1, TW = MomLds<R>::TW, TH = MomLds<R>::TH;
  __shared__ MomLds<R> S;
  const int f = bk.y, t = threadIdx.x, W = P.W, H = P.H;
  const int stride = P.fp16 ? (P.C == 3 ? 4 : 6) : P.C;
  float centre, half;
  moment_range(P, w, stride, S.red, centre, half);
  // 127 units reach 0.8 of the largest mean moment.  No usable range (a flat
  // sample, or values that are not finite): scale 0, which bounds nothing.
  const bool usable = half > 1e-15f && half < 1e15f;
  const float scale = usable ? 127.0f / (0.8f * (float)T * half) : 0.0f;
  if (bk.x == 0 && f == 0 && t == 0) {
    w.act_count[8] = __float_as_uint(scale);
    w.act_count[9] = __float_as_uint(usable ? kRounding * (fabsf(centre) / half + kFar) : 0.f);
  }
  const int ntx = (W + kMomW - 1) / kMomW;
  const int x0 = (bk.x % ntx) * kMomW, y0 = (bk.x / ntx) * kMomH;
  const float cut = 2.0f * half;
  for (int i = t; i < (TW + 2) * (TH + 2); i += kBlock) {
    const int ly = i / (TW + 2), lx = i - ly * (TW + 2);
    const size_t o = (size_t)(clampi(y0 + ly - R - 1, 0, H - 1) * W + clampi(x0 + lx - R - 1, 0, W - 1)) * stride;
#pragma unroll
    for (int c = 0; c < 3; ++c) S.v[c][ly][lx] = rgb_value(P, w.feat[f], o + c);
  }
  __syncthreads();
  for (int i = t; i < TW * TH; i += kBlock) {
    const int ly = i / TW + 1, lx = i % TW + 1;
    float e = 0.f, far = 0.f;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      float hx = 0.f;
#pragma unroll
      for (int d = -1; d <= 1; ++d) {
        const float m = S.v[c][ly + d][lx], l = S.v[c][ly + d][lx - 1], r = S.v[c][ly + d][lx + 1];
        hx = fmaxf(hx, fmaxf(fabsf(l - m), fabsf(r - m)));
        far = fmaxf(fmaxf(far, fabsf(m - centre)), fmaxf(fabsf(l - centre), fabsf(r - centre)));
      }
      const float m = S.v[c][ly][lx];
      const float hy = fmaxf(fabsf(S.v[c][ly - 1][lx] - m), fabsf(S.v[c][ly + 1][lx] - m));
      hx *= scale;
      e = fmaf(hx, hx, fmaf(hy * scale, hy * scale, e));
    }
    S.h2[ly - 1][lx - 1] = far > kFar * half ? __builtin_huge_valf() : e;
  }
  for (int i = t; i < 3 * TH * kMomW; i += kBlock) {
    const int lx = i % kMomW, ly = (i / kMomW) % TH, c = i / (kMomW * TH);
    float a = 0.f, b = 0.f;
#pragma unroll
    for (int d = 0; d < T; ++d) {
      const float v = fminf(fmaxf(S.v[c][ly + 1][lx + d + 1] - centre, -cut), cut) * scale;
      a += v;
      b = fmaf((float)(d - R), v, b);
    }
    S.s0[c][ly][lx] = a;
    S.s1[c][ly][lx] = b;
  }
  __syncthreads();
  for (int i = t; i < TH * kMomW; i += kBlock) {
    const int lx = i % kMomW, ly = i / kMomW;
    float a = 0.f, b = 0.f;
#pragma unroll
    for (int d = 0; d < T; ++d) {
      const float v = S.h2[ly][lx + d];
      a += v;
      b = fmaf((float)((d - R) * (d - R)), v, b);
    }
    S.q0[ly][lx] = a;
    S.q2[ly][lx] = b;
  }
  __syncthreads();
  const int lx = t % kMomW, ly = t / kMomW, x = x0 + lx, y = y0 + ly;
  if (x >= W || y >= H) return;
  constexpr float nx = (float)(R * (R + 1) * T) / 3.0f;
  const float k0 = 1.0f / (float)T, k1 = rsqrtf(nx * (float)T), k2 = 1.0f / nx;
  uint32_t word[3];
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    float m = 0.f, mx = 0.f, my = 0.f, mxy = 0.f;
#pragma unroll
    for (int d = 0; d < T; ++d) {
      const float a = S.s0[c][ly + d][lx], b = S.s1[c][ly + d][lx], yy = (float)(d - R);
      m += a;
      mx += b;
      my = fmaf(yy, a, my);
      mxy = fmaf(yy, b, mxy);
    }
    const float q[4] = {m * k0, mx * k1, my * k1, mxy * k2};
    uint32_t u = 0;
#pragma unroll
    for (int i = 0; i < (c < 2 ? 4 : 3); ++i)
      u |= ((uint32_t)(int)rintf(fminf(fmaxf(q[i], -127.f), 127.f)) & 0xffu) << (8 * i);
    word[c] = u;
  }
  float k2sum = 0.f;
#pragma unroll
  for (int d = 0; d < T; ++d)
    k2sum += fmaf((float)((d - R) * (d - R)), S.q0[ly + d][lx], S.q2[ly + d][lx]);
  const float rough = sqrtf(k2sum) * (1.0001f / kRough);
  word[2] |= (rough < 254.f ? (uint32_t)(int)ceilf(rough) : 255u) << 24;
  uint32_t* out = reinterpret_cast<uint32_t*>(w.twin[f]) + 3 * (size_t)(y * W + x);
  out[0] = word[0];
  out[1] = word[1];
  out[2] = word[2];
}

template <int R>
__global__ __launch_bounds__(kBlock) void k_moments(DevParams P, Ws w) {
  moments_body<R>(P, w, blk_here());
}

template <int R>
__global__ __launch_bounds__(kBlock) void kb_moments(const uint8_t* __restrict__ tab, int k) {
  const BatchView V = batch_view(tab, k);
  const PairDesc* __restrict__ pd = V.pd;
  const Item* __restrict__ it = V.it;
  const int n = V.n, total = V.total;
  for_each_item<true>(it, n, total, [&](int i, Blk bk) {
    moments_body<R>(pd[it[i].pair].P, pd[it[i].pair].w, bk);
  });
}

static int moments_blocks(const DevParams& P) {
  return ((P.W + kMomW - 1) / kMomW) * ((P.H + kMomH - 1) / kMomH);
}

// One frame's moments through a buffer resource: 32-bit byte offsets, unsigned, as
// the 12 bytes of each of at most 2^28 pixels (FP16 RGB records of 2 GiB) pass
// 2 GiB from pixel 178956971 on.
__host__ __device__ constexpr uint32_t moment_offset(int p) { return (uint32_t)p * 12u; }
static_assert(moment_offset((1 << 28) - 1) == 3221225460u, "offsets of the largest frame");
struct Moments {
  __amdgpu_buffer_rsrc_t r;
  __device__ inline u32x3 at(int p) const { return __builtin_amdgcn_raw_buffer_load_b96(r, (int)moment_offset(p), 0, 0); }
};
__device__ inline Moments moments_buf(const Ws& w, int f, int n) {
  return Moments{__builtin_amdgcn_make_buffer_rsrc(w.twin[f], (short)0, (int)moment_offset(n), 0x00020000)};
}

__device__ inline int dot4(uint32_t a, uint32_t b, int c) {
  return __builtin_amdgcn_sdot4((int)a, (int)b, c, false);
}
__device__ inline int moments_norm2(u32x3 a) { return dot4(a.x, a.x, dot4(a.y, a.y, dot4(a.z, a.z, 0))); }

// ---------------------------------------------------------------------------
// Half-sweep
// ---------------------------------------------------------------------------

// What bounds the costs of a pixel's candidates.
struct Bound {
  u32x3 src;    // the pixel's moments, without the last byte
  float shift;  // b of the pixel's distortion times kRough; infinite: no bound
  float round;  // units by which rounded samples may move a distorted patch
  float unit2;  // squared length of a unit, less what the cost may be under the exact SSD
};

// Largest |a(d)| / |d| of a distortion, a(d) = Delta(d) - d with Delta(d) = M d /
// (1 + g d): (|M - I| + |g| |d|) / (1 - |g| |d|) in the spectral norm, |d| at
// most sqrt(2) r; infinite where that does not keep |a| <= 1.
__device__ inline float distortion(const float (&m)[6], int r) {
  const float inf = __builtin_huge_valf();
  const float a = m[0] - 1.f, b = m[1], c = m[2], d = m[3] - 1.f;
  const float s = fmaf(a, a, b * b) + fmaf(c, c, d * d), det = a * d - b * c;
  const float norm = sqrtf(0.5f * (s + sqrtf(fmaxf(s * s - 4.f * det * det, 0.f))));
  const float reach = 1.4143f * (float)r, g = sqrtf(fmaf(m[4], m[4], m[5] * m[5])) * reach;
  if (!(g < 0.5f)) return inf;
  const float v = (norm + g) / (1.f - g) * 1.001f + 1e-4f;
  return v * reach < 1.f ? v : inf;
}

__device__ inline float bound_unit2(float scale) { return scale > 0.f ? 0.9999f / (scale * scale) : 0.f; }

// A cost that target p's cannot be below, or 0.
__device__ inline float cost_bound(const Bound& f, const Moments& M2, int p) {
  u32x3 t = M2.at(p);
  const uint32_t rough = t.z >> 24;
  t.z &= 0xffffffu;
  const int dot = dot4(f.src.x, t.x, dot4(f.src.y, t.y, dot4(f.src.z, t.z, 0)));
  const float d = sqrtf((float)(moments_norm2(f.src) + moments_norm2(t) - 2 * dot));
  const float less = f.shift > 0.f ? fmaf(f.shift, rough == 255u ? __builtin_huge_valf() : (float)rough, f.round) : 0.f;
  const float v = d - kMomSlack - less;
  return v > 0.f ? v * v * f.unit2 : 0.f;  // less infinite or not a number: 0
}

// Random-search offset k of pixel p.
__device__ inline int32_t draw_offset(const DevParams& P, int p, int k, int iter, uint64_t w3) {
  const int Rk = P.R0 >> k;
  uint64_t c[4] = {(uint64_t)(uint32_t)p, (uint64_t)k, (uint64_t)iter, w3};
  philox4x64(c, P.seed, 0);
  return pack_off(draw_below(c[0], (uint32_t)(2 * Rk + 1)) - Rk, draw_below(c[1], (uint32_t)(2 * Rk + 1)) - Rk);
}

// The bit of target (tx, ty) among the tried positions around (bx, by), 0 if outside.
__device__ inline unsigned tried_bit(int tx, int ty, int bx, int by) {
  const unsigned ux = (unsigned)(tx - bx + 2), uy = (unsigned)(ty - by + 2);
  return ux < 5u && uy < 5u ? 1u << (uy * 5u + ux) : 0u;
}
constexpr unsigned kTriedCentre = 1u << 12;

// A candidate's bound as kept in LDS, rounded down, and the key that orders a
// pixel's candidates by it.
__device__ inline uint16_t bound_bits(float v) { return (uint16_t)(__float_as_uint(v) >> 16); }
__device__ inline unsigned bound_key(float v, int k) { return (__float_as_uint(v) & ~15u) | (unsigned)k; }

// Lists the pixels with work in S.order, most candidates (at most `most`) first;
// returns their number.  Every wave makes the same list for itself.
__device__ inline int sort_by_work(SearchLds& S, int phase, int most) {
  const int lane = threadIdx.x & (kWave - 1);
  const int cnt = __popc(S.mask[phase][lane]);
  const unsigned long long lt = (1ull << lane) - 1ull;
  int n = 0;
  for (int c = most; c > 0; --c) {
    const unsigned long long m = __ballot(cnt == c);
    if (cnt == c) S.order[n + __popcll(m & lt)] = lane;
    n += __popcll(m);
  }
  wave_lds_fence();
  return n;
}

// Evaluates the candidates of a phase, one pixel per lane group at a time, the
// waves taking the list of pixels with work in turn; rows: tap rows computed
// (counted at the group's last lane).
template <int R, int C, bool FP16, bool IDENT>
__device__ inline void evaluate(const DevParams& P, const Ws& w, int dir, SearchLds& S, int phase, unsigned& rows_out) {
  constexpr int G = 2 * R + 1, NG = kWave / G;
  // rows of a distorted patch in flight: two of FP16 records fit 4 waves per SIMD
  constexpr int kChunk = FP16 ? 2 : 3;
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int g = lane / G, j = lane - g * G, base = g * G;
  const int W = P.W, H = P.H;
  const float gw = P.gw;
  const Feat F1 = feat_buf<C, FP16>(w.feat[dir], W, H), F2 = feat_buf<C, FP16>(w.feat[1 - dir], W, H);
  const int(*tgt)[kSlots] = phase ? S.tgt : S.ptgt;
  const uint16_t(*lbs)[kSlots] = phase ? S.lb : S.plb;
  const int n = sort_by_work(S, phase, phase ? P.nk : 6);
  for (int i0 = wave * NG; i0 < n; i0 += NG * (kBlock / kWave)) {
    const int i = i0 + g;
    if (g >= NG || i >= n) continue;
    const int sl = S.order[i];
    const int pix = S.pix[sl];
    const int x = xy_x(pix), y = xy_y(pix);
    int best = S.best[sl], kbest = -1;
    float bc = S.bc[sl];
    unsigned m = S.mask[phase][sl], rows = 0;
    LaneCol<R, C, IDENT> L;
    int geo = 1;
    if constexpr (IDENT) {
      L.dx = j - R;
    } else {
      float mo[6];
#pragma unroll
      for (int q = 0; q < 6; ++q) mo[q] = S.motion[q][sl];
      bool integral = false, ok = S.shift[sl] >= 0.f;
      if (ok) ok = tap_geometry<R, C>(L, mo, j - R, 4.0f * (float)(W > H ? W : H), integral);
      geo = group_geometry<G>(ok, integral, base);
    }
    // geo 2: a homogeneous coordinate is not positive, every cost is +inf
    if (geo != 2) load_column<R, C, FP16, IDENT>(L, F1, W, H, x, y, j - R);
    if (m & kRefresh) {
      bool rejected;
      unsigned r0 = 0;
      if (geo == 2)
        bc = __builtin_huge_valf();
      else if (IDENT || geo == 1)
        bc = group_cost<R, C, FP16, IDENT, true, false, kChunk>(L, F2, W, H, xy_x(best), xy_y(best), gw, base, 0.f, rejected, r0);
      else
        bc = group_cost<R, C, FP16, IDENT, IDENT, false, kChunk>(L, F2, W, H, xy_x(best), xy_y(best), gw, base, 0.f, rejected, r0);
    }
    m &= geo == 2 ? 0u : ~kRefresh;
    // the candidate of the lowest bound, then the others in order.  A cost equal
    // to the best one wins only before the candidate that holds it.
    int k = (int)(S.key[phase][sl] & 15u);
    while (m) {
      if (!((m >> k) & 1u)) k = __builtin_ctz(m);
      m &= ~(1u << k);
      const int t = tgt[k][sl];
      const float lb = __uint_as_float((unsigned)lbs[k][sl] << 16);
      const float top = k < kbest ? __uint_as_float(__float_as_uint(bc) + 1u) : bc;
      bool won;
      float c = 0.f;
      if constexpr (IDENT) {
        // comparisons at the group's last lane, where bc is exact
        won = group_flag<G>(lb < top, base) && t != best;
        if (won) {
          // all rows at once: a check on the way would drop few that the bound
          // has left (at 1024x436, after row 6 of 9, one in seven)
          c = group_chain<G>(ident_rows1<R, C, FP16, 0, G>(0.f, L, F2, W, H, xy_x(t), xy_y(t), gw));
          won = group_flag<G>(c < top, base);
          rows += G;
        }
      } else {
        won = lb < top && t != best;
        if (won) {
          bool rejected;
          if (geo == 1)
            c = group_cost<R, C, FP16, IDENT, true, true, kChunk>(L, F2, W, H, xy_x(t), xy_y(t), gw, base, top, rejected, rows);
          else
            c = group_cost<R, C, FP16, IDENT, IDENT, true, kChunk>(L, F2, W, H, xy_x(t), xy_y(t), gw, base, top, rejected, rows);
          won = !rejected && c < top;
        }
      }
      if (won) {
        bc = c;
        best = t;
        kbest = k;
      }
    }
    if (j == G - 1) {
      S.best[sl] = best;
      S.bc[sl] = bc;
      if (phase) S.won[sl] = kbest >= 0;
      rows_out += rows;
    }
  }
}

// Which pixel slot i of workgroup b has.
struct SlotMap {
  const int32_t* list;   // restricted: the list of pixels, from its front or its back
  int step;              // its direction
  int rows, ntx;         // tiles: rows of one, tiles per row of the frame
  int run, colour, W, H;
  unsigned b, cnt;
  __device__ inline bool at(int i, int& x, int& y) const {
    if (rows) {
      y = (int)(b / ntx) * rows + (i >> 3);
      x = (int)(b % ntx) * 16 + 2 * (i & 7) + ((y + colour) & 1);
      return x < W && y < H;
    }
    const unsigned q = b * run + i;
    if (q >= cnt) return false;
    if (list) {
      const int p = list[(long long)step * (int)q];
      y = p / W;
      x = p - y * W;
      return true;
    }
    const int Wh = (W + 1) >> 1;
    y = (int)(q / Wh);
    x = 2 * (int)(q - (unsigned)y * Wh) + ((y + colour) & 1);
    return x < W;
  }
};

// Opens slot sl and offers neighbour k's offset (0 left, 1 right, 2 up, 3 down);
// the lanes of k == 0 also load the pixel's own state.
template <int R, bool IDENT>
__device__ inline void open_slot(const DevParams& P, const Ws& w, int dir, SearchLds& S, const SlotMap& M, int sl, int k,
                                 bool first, const Moments& M1, const Moments& M2, float unit2, float round,
                                 unsigned& evals) {
  const int W = P.W, H = P.H;
  int x, y;
  if (!M.at(sl, x, y)) {
    if (k == 0) S.pix[sl] = -1;
    return;
  }
  const int p = y * W + x;
  const int nx = x + (k == 0 ? -1 : (k == 1 ? 1 : 0));
  const int ny = y + (k == 2 ? -1 : (k == 3 ? 1 : 0));
  const bool inside = nx >= 0 && nx < W && ny >= 0 && ny < H;
  const int q = inside ? ny * W + nx : p;
  const int32_t v0 = w.nnf[dir][p], v = w.nnf[dir][q];
  const int wq = w.win[dir][q];
  Bound f{};
  if (k == 0 || first) f.src = M1.at(p);
  f.unit2 = unit2;
  f.round = round;
  const int best0 = pack_xy(x + off_dx(v0), y + off_dy(v0));
  int tp = -1;
  if (k == 0) {
    S.pix[sl] = pack_xy(x, y);
    S.best0[sl] = best0;
    S.best[sl] = best0;
    S.bc[sl] = first ? 0.f : w.cost[dir][p];
    S.memo[sl] = first ? 0u : (unsigned)w.win[dir][p] & kMemoTried;
    S.won[sl] = 0;
    S.src[0][sl] = f.src.x;
    S.src[1][sl] = f.src.y;
    S.src[2][sl] = f.src.z & 0xffffffu;
  }
  f.src.z &= 0xffffffu;
  if constexpr (!IDENT) {
    // shift: negative where the plane has no motion (no cost is finite)
    if (k == 0 || first) {
      double qx, qy;
      float m[6] = {};
      f.shift = -1.f;
      if (plane_motion(plane_H(w, w.hlabel[dir][p]), x, y, qx, qy, m)) {
        f.shift = distortion(m, R) * kRough;
        // plane candidate: where the region plane sends the pixel, rounded to the grid
        const double dl = (double)(4.0f * (float)(W > H ? W : H));
        double rx = floor(qx + 0.5), ry = floor(qy + 0.5);
        rx = rx < -dl ? -dl : (rx > dl ? dl : rx);
        ry = ry < -dl ? -dl : (ry > dl ? dl : ry);
        tp = pack_xy(clampi((int)rx, 0, W - 1), clampi((int)ry, 0, H - 1));
      }
      if (k == 0) {
        S.shift[sl] = f.shift;
#pragma unroll
        for (int i = 0; i < 6; ++i) S.motion[i][sl] = m[i];
      }
    }
  }
  auto offer = [&](int kk, int t, bool need) {
    if (t == best0) return;
    ++evals;
    if (!need) return;
    // the bounds drop few of these candidates but in the first half-sweep,
    // where the best may still be a random one
    const float lb = first ? cost_bound(f, M2, xy_y(t) * W + xy_x(t)) : 0.f;
    S.ptgt[kk][sl] = t;
    S.plb[kk][sl] = bound_bits(lb);
    atomicMin(&S.key[0][sl], bound_key(lb, kk));
    atomicOr(&S.mask[0][sl], 1u << kk);
  };
  if (inside)
    offer(k, pack_xy(clampi(x + off_dx(v), 0, W - 1), clampi(y + off_dy(v), 0, H - 1)),
          first || (wq < 0 && (wq & (int)kMemoChanged)));
  if (!IDENT && k == 0 && tp != -1) offer(4, tp, first);
  if (k == 0 && first) atomicOr(&S.mask[0][sl], kRefresh);
}

// Random-search candidate k of slot sl, around the best after propagation; mine:
// the positions noted by this lane for the slot.
template <bool IDENT>
__device__ inline void offer_random(const DevParams& P, SearchLds& S, int sl, int k, const Moments& M2, float unit2,
                                    float round, unsigned& mine, unsigned& evals) {
  if (S.pix[sl] < 0) return;
  const int b = S.best[sl], bx = xy_x(b), by = xy_y(b);
  const int32_t v = S.tgt[k][sl];
  const int tx = clampi(bx + off_dx(v), 0, P.W - 1), ty = clampi(by + off_dy(v), 0, P.H - 1);
  const unsigned bit = tried_bit(tx, ty, bx, by);
  if (bit == kTriedCentre) return;
  ++evals;
  // Dropped: what earlier half-sweeps tried, and what this lane itself offered
  // under a lower number.  Radii that draw one position in different lanes come
  // here in any order, and the lowest must keep it (equal costs go by number): they
  // all stay, and evaluate() meets the lowest first, as their bounds are equal.
  if (bit & mine) return;
  mine |= bit;
  if (bit) {
    atomicOr(&S.tried[sl], bit);
    if (b == S.best0[sl] && (S.memo[sl] & bit)) return;
  }
  const Bound f{u32x3{S.src[0][sl], S.src[1][sl], S.src[2][sl]}, IDENT ? 0.f : S.shift[sl], round, unit2};
  const float lb = cost_bound(f, M2, ty * P.W + tx);
  if (lb >= S.bc[sl]) return;
  S.tgt[k][sl] = pack_xy(tx, ty);
  S.lb[k][sl] = bound_bits(lb);
  atomicMin(&S.key[1][sl], bound_key(lb, k));
  atomicOr(&S.mask[1][sl], 1u << k);
}

// Calls f(slot, k) for every slot < np and k < nk, the lanes of the workgroup
// taking the pairs in turn.  In a full workgroup a lane has one slot and a range of
// k in order, the same for all lanes of a wave (and scalar): the last wave that of
// the smallest radii, which often draw one position.  With the radii dealt out in
// turn, no repeat could be dropped there: 1.1 to 2 % more patch rows of a 1024x436
// pair, and solves 0.3 to 0.8 % slower.
template <class F>
__device__ inline void each_candidate(int np, int nk, F&& f) {
  if (np == kSlots) {
    constexpr int kWaves = kBlock / kSlots;
    const int per = (nk + kWaves - 1) / kWaves;
    const int end = nk - (kWaves - 1 - __builtin_amdgcn_readfirstlane(threadIdx.x / kSlots)) * per;
    for (int k = end > per ? end - per : 0; k < end; ++k) f((int)threadIdx.x % kSlots, k);
  } else {
    for (int i = threadIdx.x; i < np * nk; i += kBlock) {
      const int k = i / np;
      f(i - k * np, k);
    }
  }
}

// Rows of the 16-pixel wide tiles into which nx workgroups divide a frame, one
// per tile (8 pixels of a colour per row, whose patches overlap); 0: they do not.
__host__ __device__ inline int tile_rows(int W, int H, int nx) {
  for (int rows = 8; rows; rows >>= 1)
    if (((W + 15) >> 4) * ((H + rows - 1) / rows) == nx) return rows;
  return 0;
}

// mode: SM_* bits.  Unrestricted: the pixels of one colour, in tiles when the
// launch has a workgroup per tile, otherwise in runs.  Restricted: the listed
// pixels.
template <int R, int C, bool FP16, bool IDENT>
__device__ __forceinline__ void search_body(const DevParams& P, const Ws& w, SearchLds& S, Blk bk, int colour, int iter,
                                            int slot, int mode) {
  constexpr int G = 2 * R + 1, NG = kWave / G;
  const int t = threadIdx.x;
  const int dir = bk.y;
  const int W = P.W, H = P.H;
  const bool restricted = (mode & SM_RESTRICTED) != 0, first = (mode & SM_FIRST) != 0;
  const unsigned cap = (unsigned)((W + 1) >> 1) * (unsigned)H;
  SlotMap M;
  M.cnt = restricted ? w.act_count[2 * (2 * dir + colour) + (IDENT ? 1 : 0)] : cap;
  M.list = restricted ? w.act[2 * dir + colour] + (IDENT ? cap - 1u : 0u) : nullptr;
  M.step = IDENT ? -1 : 1;
  M.rows = restricted ? 0 : tile_rows(W, H, bk.nx);
  M.ntx = (W + 15) >> 4;
  M.run = M.rows ? 8 * M.rows : search_run(M.cnt, bk.nx, NG);
  M.colour = colour;
  M.W = W;
  M.H = H;
  const int nb = M.rows ? bk.nx : (int)((M.cnt + M.run - 1) / M.run), np = M.run;
  if (bk.x >= nb) return;
  M.b = xcd_remap(bk.x, nb);
  const float unit2 = bound_unit2(__uint_as_float(w.act_count[8])), round = __uint_as_float(w.act_count[9]);
  const Moments M1 = moments_buf(w, dir, W * H), M2 = moments_buf(w, 1 - dir, W * H);
  const uint64_t w3 = rng_word3(2, dir, slot, 0);
  unsigned evals = 0, tap_rows = 0;
  if (t < kSlots) {
    S.mask[0][t] = S.mask[1][t] = 0u;
    S.key[0][t] = S.key[1][t] = ~0u;
    S.tried[t] = 0u;
    S.pix[t] = -1;
  }
  __syncthreads();
  // the neighbours' candidates, and the draws while their loads are on the way
  each_candidate(np, 4, [&](int sl, int k) {
    open_slot<R, IDENT>(P, w, dir, S, M, sl, k, first, M1, M2, unit2, round, evals);
  });
  each_candidate(np, P.nk, [&](int sl, int k) {
    int x, y;
    if (M.at(sl, x, y)) S.tgt[k][sl] = draw_offset(P, y * W + x, k, iter, w3);
  });
  __syncthreads();
#pragma unroll 1
  for (int phase = 0; phase < 2; ++phase) {
    if (phase) {
      unsigned mine = 0;
      each_candidate(np, P.nk, [&](int sl, int k) {
        if (np != kSlots) mine = 0;  // another slot
        offer_random<IDENT>(P, S, sl, k, M2, unit2, round, mine, evals);
      });
      __syncthreads();
    }
    evaluate<R, C, FP16, IDENT>(P, w, dir, S, phase, tap_rows);
    __syncthreads();
  }
  const int pix = t < kSlots ? S.pix[t] : -1;
  if (pix >= 0) {
    const int x = xy_x(pix), y = xy_y(pix), p = y * W + x;
    const int best = S.best[t], best0 = S.best0[t];
    const bool changed = best != best0;
    if (changed) w.nnf[dir][p] = pack_off(xy_x(best) - x, xy_y(best) - y);
    if (changed || first) w.cost[dir][p] = S.bc[t];
    const unsigned tried = S.won[t] ? 0u : S.tried[t] | (changed ? 0u : S.memo[t]);
    w.win[dir][p] = mode & SM_LAST ? -1 : (int)(kMemoSign | (changed ? kMemoChanged : 0u) | tried);
  }
  count_evals<true>(w.counters, (restricted ? (IDENT ? 10 : 4) : 0) + dir, evals);
  count_evals<true>(w.counters, (restricted ? (IDENT ? 12 : 8) : 6) + dir, tap_rows);
  if (first) count_evals<true>(w.counters, 2 + dir, pix >= 0 ? 1u : 0u);
}

// Waves per SIMD the registers are held to.  Measured on MI355X at 1024x436, per
// pair: identity patches of FP16 records at 5 waves 6.8 ms, at 4 7.4 ms; of FP32
// records at 5 (with spills) 16.4 ms, at 4 10.3 ms.
// Both lists in one launch: FP16 records at 4 waves (distorted patches with two
// rows in flight) 14.6 ms, at 3 (with three) 15.1.
constexpr int search_waves(bool fp16, bool ident) { return ident ? (fp16 ? 5 : 4) : (fp16 ? 4 : 3); }

template <int R, int C, bool FP16, bool IDENT>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(search_waves(FP16, IDENT)))) void k_search(
    DevParams P, Ws w, int colour, int iter, int slot, int mode) {
  __shared__ SearchLds S;
  search_body<R, C, FP16, IDENT>(P, w, S, blk_here(), colour, iter, slot, mode);
}

// Both lists of a restricted half-sweep: the first half of a direction's workgroups
// (a multiple of kXcds) takes the pixels with a region plane, the second half
// the others, which then fill the tail that the first leave.  Two launches on
// two streams cost 12 us a half-sweep for their fork and join alone: 320x240
// FP32 5.48 -> 5.10 ms per pair, 1024x436 20.55 -> 19.5 (FP16 15.6 -> 15.1),
// 2048x872 81.1 -> 80.4 (71.9 -> 71.6).
template <int R, int C, bool FP16>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(search_waves(FP16, false)))) void k_search_lists(
    DevParams P, Ws w, int colour, int iter, int slot, int mode) {
  __shared__ SearchLds S;
  Blk bk = blk_here();
  bk.nx >>= 1;
  if (bk.x < bk.nx) {
    search_body<R, C, FP16, false>(P, w, S, bk, colour, iter, slot, mode);
  } else {
    bk.x -= bk.nx;
    search_body<R, C, FP16, true>(P, w, S, bk, colour, iter, slot, mode);
  }
}

template <int R, int C, bool FP16, bool LOOP>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(search_waves(FP16, true)))) void kb_search(
    const uint8_t* __restrict__ tab, int k, BArgs A) {
  const BatchView V = batch_view(tab, k);
  const PairDesc* __restrict__ pd = V.pd;
  const Item* __restrict__ it = V.it;
  const int n = V.n, total = V.total;
  __shared__ SearchLds S;
  for_each_item<true, LOOP>(it, n, total, [&](int i, Blk bk) {
    const Item& I = it[i];
    search_body<R, C, FP16, true>(pd[I.pair].P, pd[I.pair].w, S, bk, A.a[0], A.a[1], A.a[2], A.a[3]);
  });
}

template <int R, int C, bool FP16, bool LOOP>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(search_waves(FP16, false)))) void
kb_search_lists(const uint8_t* __restrict__ tab, int k, BArgs A) {
  const BatchView V = batch_view(tab, k);
  const PairDesc* __restrict__ pd = V.pd;
  const Item* __restrict__ it = V.it;
  const int n = V.n, total = V.total;
  __shared__ SearchLds S;
  for_each_item<true, LOOP>(it, n, total, [&](int i, Blk bk) {
    const Item& I = it[i];
    bk.nx >>= 1;
    if (bk.x < bk.nx) {
      search_body<R, C, FP16, false>(pd[I.pair].P, pd[I.pair].w, S, bk, A.a[0], A.a[1], A.a[2], A.a[3]);
    } else {
      bk.x -= bk.nx;
      search_body<R, C, FP16, true>(pd[I.pair].P, pd[I.pair].w, S, bk, A.a[0], A.a[1], A.a[2], A.a[3]);
    }
  });
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
// Workgroups of one direction of a half-sweep: one per tile of the most rows
// that still make kSearchGroups of them for both directions; smaller frames take
// runs of pixels, down to one per lane group of a wave.
static int search_blocks(const DevParams& P) {
  for (int rows = 8; rows; rows >>= 1) {
    const long long tiles = (long long)((P.W + 15) >> 4) * ((P.H + rows - 1) / rows);
    if (2 * tiles >= kSearchGroups) return (int)tiles;
  }
  const int n = ((P.W + 1) >> 1) * P.H;
  const int run = search_run((unsigned)n, n, kWave / (2 * P.r + 1));
  return (n + run - 1) / run;
}

// The same for both lists in one launch: twice that, each half a multiple of kXcds.
static int lists_blocks(const DevParams& P) { return 2 * ((search_blocks(P) + kXcds - 1) / kXcds * kXcds); }

template <int R, int C, bool FP16>
static hipError_t dispatch_search(const DevParams& P, const Ws& w, int colour, int iter, int slot, int mode, int ident,
                                  hipStream_t s) {
  const dim3 grid(search_blocks(P), 2);
  if (ident)
    hipLaunchKernelGGL((k_search<R, C, FP16, true>), grid, dim3(kBlock), 0, s, P, w, colour, iter, slot, mode);
  else
    hipLaunchKernelGGL((k_search<R, C, FP16, false>), grid, dim3(kBlock), 0, s, P, w, colour, iter, slot, mode);
  return hipGetLastError();
}

template <int R, int C, bool FP16>
static hipError_t dispatch_search_lists(const DevParams& P, const Ws& w, int colour, int iter, int slot, int mode,
                                        hipStream_t s) {
  hipLaunchKernelGGL((k_search_lists<R, C, FP16>), dim3(lists_blocks(P), 2), dim3(kBlock), 0, s, P, w, colour, iter,
                     slot, mode);
  return hipGetLastError();
}

template <int R, int C, bool FP16, bool LOOP>
static void dispatch_search_form(bool initial, const uint8_t* tab, int k, dim3 grid, BArgs A, hipStream_t s) {
  if (initial)
    hipLaunchKernelGGL((kb_search<R, C, FP16, LOOP>), grid, dim3(kBlock), 0, s, tab, k, A);
  else
    hipLaunchKernelGGL((kb_search_lists<R, C, FP16, LOOP>), grid, dim3(kBlock), 0, s, tab, k, A);
}

template <int R, int C, bool FP16>
static hipError_t dispatch_search_batched(bool initial, const uint8_t* tab, int k, int grid, BArgs A, bool persist,
                                          hipStream_t s) {
  if (persist)
    dispatch_search_form<R, C, FP16, true>(initial, tab, k, dim3(grid, 2), A, s);
  else
    dispatch_search_form<R, C, FP16, false>(initial, tab, k, dim3(grid, 2), A, s);
  return hipGetLastError();
}

hipError_t launch_search(const DevParams& P, const Ws& w, int colour, int iter, int slot, int mode, int ident,
                         hipStream_t s) {
  MSGPM_DISPATCH(dispatch_search, P, w, colour, iter, slot, mode, ident, s);
}

hipError_t launch_search_lists(const DevParams& P, const Ws& w, int colour, int iter, int slot, int mode,
                               hipStream_t s) {
  MSGPM_DISPATCH(dispatch_search_lists, P, w, colour, iter, slot, mode, s);
}

hipError_t launch_moments(const DevParams& P, const Ws& w, hipStream_t s) {
  const dim3 grid(moments_blocks(P), 2), block(kBlock);
  switch (P.r) {
    case 1: hipLaunchKernelGGL(k_moments<1>, grid, block, 0, s, P, w); break;
    case 2: hipLaunchKernelGGL(k_moments<2>, grid, block, 0, s, P, w); break;
    case 3: hipLaunchKernelGGL(k_moments<3>, grid, block, 0, s, P, w); break;
    case 4: hipLaunchKernelGGL(k_moments<4>, grid, block, 0, s, P, w); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_batched_search(int kind, const DevParams& P0, const uint8_t* tab, int k, int grid, BArgs A,
                                 bool persist, hipStream_t s) {
  const DevParams& P = P0;
  if (kind == BK_MOMENTS) {
    const dim3 g(grid, 2), block(kBlock);
    switch (P.r) {
      case 1: hipLaunchKernelGGL(kb_moments<1>, g, block, 0, s, tab, k); break;
      case 2: hipLaunchKernelGGL(kb_moments<2>, g, block, 0, s, tab, k); break;
      case 3: hipLaunchKernelGGL(kb_moments<3>, g, block, 0, s, tab, k); break;
      case 4: hipLaunchKernelGGL(kb_moments<4>, g, block, 0, s, tab, k); break;
      default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
  }
  MSGPM_DISPATCH(dispatch_search_batched, kind == BK_PM_INIT, tab, k, grid, A, persist, s);
}

int search_batch_blocks(int kind, const DevParams& P) {
  if (kind == BK_MOMENTS) return moments_blocks(P);
  return kind == BK_PM_INIT ? search_blocks(P) : lists_blocks(P);
}

}  // namespace msgpm
