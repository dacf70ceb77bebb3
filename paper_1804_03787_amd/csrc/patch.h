// Warped-patch SSD of one pixel's lane group: the device functions shared by the
// PatchMatch kernels of patchmatch.hip and search.h.
#pragma once

#include "common.h"

#include <hip/hip_fp16.h>

#pragma clang fp contract(off)

namespace msgpm {

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x3 __attribute__((ext_vector_type(3)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ inline float2 h2f(uint32_t u) { return __half22float2(__builtin_bit_cast(__half2, u)); }
__device__ inline float uf(uint32_t u) { return __uint_as_float(u); }

// Feature buffer of one frame, read through a buffer resource: offsets are
// 32-bit byte offsets (the host rejects frames whose features exceed 2 GiB), so
// an address costs one integer multiply-add instead of 64-bit arithmetic.
struct Feat {
  __amdgpu_buffer_rsrc_t r;
};
template <int C, bool FP16>
__device__ inline Feat feat_buf(const void* F, int W, int H) {
  constexpr int kBytes = FP16 ? (C == 3 ? 8 : 12) : 4 * C;
  // word 3 = 0x00020000: 32-bit data format, as raw dword buffer loads need on gfx9
  return Feat{__builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(F), (short)0, (W * H + 1) * kBytes, 0x00020000)};
}

// Feature access.  FP32: C floats per pixel; FP16: C=3 -> 4 halves, C=5 -> 6
// halves per pixel.  load1 reads pixel idx; raw2 pixels idx and idx + 1 with
// one contiguous access (the buffer is padded so idx + 1 always exists).
template <int C, bool FP16>
struct Px {
  static constexpr int kBytes = FP16 ? (C == 3 ? 8 : 12) : 4 * C;
  static __device__ inline void load1(Feat F, int idx, float* v) {
    const int o = idx * kBytes;
    if constexpr (!FP16) {
      if constexpr (C == 3) {
        const u32x3 a = __builtin_amdgcn_raw_buffer_load_b96(F.r, o, 0, 0);
        v[0] = uf(a.x); v[1] = uf(a.y); v[2] = uf(a.z);
      } else {
        const u32x4 a = __builtin_amdgcn_raw_buffer_load_b128(F.r, o, 0, 0);
        const uint32_t e = __builtin_amdgcn_raw_buffer_load_b32(F.r, o + 16, 0, 0);
        v[0] = uf(a.x); v[1] = uf(a.y); v[2] = uf(a.z); v[3] = uf(a.w); v[4] = uf(e);
      }
    } else {
      if constexpr (C == 3) {
        const u32x2 u = __builtin_amdgcn_raw_buffer_load_b64(F.r, o, 0, 0);
        const float2 a = h2f(u.x), b = h2f(u.y);
        v[0] = a.x; v[1] = a.y; v[2] = b.x;
      } else {
        const u32x3 u = __builtin_amdgcn_raw_buffer_load_b96(F.r, o, 0, 0);
        const float2 a = h2f(u.x), b = h2f(u.y), c = h2f(u.z);
        v[0] = a.x; v[1] = a.y; v[2] = b.x; v[3] = b.y; v[4] = c.x;
      }
    }
  }
  // The record of pixel idx as raw words (kWords of them), for tap_sq_raw.
  static constexpr int kWords = kBytes / 4;
  static __device__ inline void raw1(Feat F, int idx, uint32_t* u) { raw1_at(F, idx * kBytes, u); }
  // The same from the record's byte offset o.
  static __device__ inline void raw1_at(Feat F, int o, uint32_t* u) {
    if constexpr (kWords == 5) {
      const u32x4 a = __builtin_amdgcn_raw_buffer_load_b128(F.r, o, 0, 0);
      u[0] = a.x; u[1] = a.y; u[2] = a.z; u[3] = a.w;
      u[4] = __builtin_amdgcn_raw_buffer_load_b32(F.r, o + 16, 0, 0);
    } else if constexpr (kWords == 3) {
      const u32x3 a = __builtin_amdgcn_raw_buffer_load_b96(F.r, o, 0, 0);
      u[0] = a.x; u[1] = a.y; u[2] = a.z;
    } else {
      const u32x2 a = __builtin_amdgcn_raw_buffer_load_b64(F.r, o, 0, 0);
      u[0] = a.x; u[1] = a.y;
    }
  }
  // Records of pixels idx and idx + 1 as raw words (2 kWords), one access.
  static __device__ inline void raw2(Feat F, int idx, uint32_t* u) {
    const int o = idx * kBytes;
    if constexpr (kWords == 5) {
      const u32x4 a = __builtin_amdgcn_raw_buffer_load_b128(F.r, o, 0, 0);
      const u32x4 b = __builtin_amdgcn_raw_buffer_load_b128(F.r, o + 16, 0, 0);
      const u32x2 c = __builtin_amdgcn_raw_buffer_load_b64(F.r, o + 32, 0, 0);
      u[0] = a.x; u[1] = a.y; u[2] = a.z; u[3] = a.w; u[4] = b.x;
      u[5] = b.y; u[6] = b.z; u[7] = b.w; u[8] = c.x; u[9] = c.y;
    } else if constexpr (kWords == 3) {
      const u32x4 a = __builtin_amdgcn_raw_buffer_load_b128(F.r, o, 0, 0);
      const u32x2 b = __builtin_amdgcn_raw_buffer_load_b64(F.r, o + 16, 0, 0);
      u[0] = a.x; u[1] = a.y; u[2] = a.z; u[3] = a.w; u[4] = b.x; u[5] = b.y;
    } else {
      const u32x4 a = __builtin_amdgcn_raw_buffer_load_b128(F.r, o, 0, 0);
      u[0] = a.x; u[1] = a.y; u[2] = a.z; u[3] = a.w;
    }
  }
};

// Per-lane state of one pixel: the lane's patch column of source features and,
// for distorted patches, the tap geometry (integer offset + fraction of
// Delta(d)) of that column, all in registers for every candidate.  FP16
// records keep the column packed (the record's words in the first slots of
// each f1[t]; 27 registers instead of 45 for C = 5), which takes the
// distorted-patch kernel to 4 waves per SIMD without spills.
template <int R, int C, bool IDENT>
struct LaneCol {
  static constexpr int T = 2 * R + 1;
  static constexpr int TG = IDENT ? 1 : T;
  float f1[T][C];
  int dx;
  int o[TG];  // integer part of Delta: x in the low, y in the high 16 bits
  __device__ int ox(int t) const { return (int)(short)(o[t] & 0xffff); }
  __device__ int oy(int t) const { return o[t] >> 16; }
  float fx[TG], fy[TG];
};

// Local motion of plane H around pixel (x, y): Delta(d) = (A/w - q g^T) d /
// (1 + g.d) with q = pi(Hp), g = (h6, h7)/w; m = the 2x2 matrix by rows, then g.
// false when the homogeneous coordinate is not positive.
__device__ inline bool plane_motion(const double* H, int x, int y, double& qx, double& qy, float (&m)[6]) {
  const double w = H[6] * x + H[7] * y + H[8];
  if (!(w > 0)) return false;
  qx = (H[0] * x + H[1] * y + H[2]) / w;
  qy = (H[3] * x + H[4] * y + H[5]) / w;
  const double g0 = H[6] / w, g1 = H[7] / w;
  m[0] = (float)(H[0] / w - qx * g0);
  m[1] = (float)(H[1] / w - qx * g1);
  m[2] = (float)(H[3] / w - qy * g0);
  m[3] = (float)(H[4] / w - qy * g1);
  m[4] = (float)g0;
  m[5] = (float)g1;
  return true;
}

// Tap geometry of column dx under that motion.  Returns false when the
// homogeneous coordinate is not positive at some tap (cost = +inf); sets
// integral when every fraction of the column is 0.
template <int R, int C>
__device__ inline bool tap_geometry(LaneCol<R, C, false>& L, const float (&m)[6], int dx, float lim, bool& integral) {
  L.dx = dx;
  integral = true;
  bool ok = true;
  const float fdx = (float)dx;
#pragma unroll
  for (int t = 0; t < 2 * R + 1; ++t) {
    const float fdy = (float)(t - R);
    const float den = fmaf(m[5], fdy, fmaf(m[4], fdx, 1.0f));
    ok = ok && (den > 0.f);
    const float inv = 1.0f / den;
    float Dx = fmaf(m[1], fdy, m[0] * fdx) * inv;
    float Dy = fmaf(m[3], fdy, m[2] * fdx) * inv;
    Dx = fminf(fmaxf(Dx, -lim), lim);
    Dy = fminf(fmaxf(Dy, -lim), lim);
    const float flx = floorf(Dx), fly = floorf(Dy);
    // integer parts beyond +-32767 (frames are at most 32767 pixels) select
    // the same clamped border pixel with fraction 0, so they are cut there
    L.o[t] = pack_off((int)fminf(fmaxf(flx, -32767.f), 32767.f), (int)fminf(fmaxf(fly, -32767.f), 32767.f));
    L.fx[t] = Dx - flx;
    L.fy[t] = Dy - fly;
    integral = integral && (L.fx[t] == 0.f) && (L.fy[t] == 0.f);
  }
  return ok;
}

// The same from plane H at pixel (x, y) (H == nullptr: the identity).
template <int R, int C, bool IDENT>
__device__ inline bool setup_geometry(LaneCol<R, C, IDENT>& L, const double* H, int x, int y, int dx, float lim,
                                      bool& integral) {
  L.dx = dx;
  integral = true;
  if constexpr (IDENT) {
    return true;
  } else {
    if (H == nullptr) {
#pragma unroll
      for (int t = 0; t < 2 * R + 1; ++t) {
        L.o[t] = pack_off(dx, t - R);
        L.fx[t] = 0.f;
        L.fy[t] = 0.f;
      }
      return true;
    }
    double qx, qy;
    float m[6];
    if (!plane_motion(H, x, y, qx, qy, m)) return false;
    return tap_geometry(L, m, dx, lim, integral);
  }
}

template <int R, int C, bool FP16, bool IDENT>
__device__ inline void load_column(LaneCol<R, C, IDENT>& L, Feat F1, int W, int H, int x, int y, int dx) {
  const int cx = clampi(x + dx, 0, W - 1);
#pragma unroll
  for (int t = 0; t < 2 * R + 1; ++t) {
    const int cy = clampi(y + t - R, 0, H - 1);
    if constexpr (FP16) {
      // FP16 records stay packed: the column's words in the first slots of
      // f1[t] (bit copies), widened inside the tap arithmetic
      uint32_t u[Px<C, FP16>::kWords];
      Px<C, FP16>::raw1(F1, cy * W + cx, u);
#pragma unroll
      for (int k = 0; k < Px<C, FP16>::kWords; ++k) L.f1[t][k] = __builtin_bit_cast(float, u[k]);
    } else {
      Px<C, FP16>::load1(F1, cy * W + cx, L.f1[t]);
    }
  }
}

template <int C>
__device__ inline float tap_sq(const float* f1, const float* v, float gw) {
  float row = 0.f;
#pragma unroll
  for (int k = 0; k < C; ++k) {
    const float e = f1[k] - v[k];
    row = (k < 3) ? fmaf(e, e, row) : fmaf(gw * e, e, row);
  }
  return row;
}

// f - h for the FP16 value h in the low (HI = false) or high half of u: the
// half is widened exactly and the difference rounded once, as a conversion
// followed by an FP32 subtraction gives, but in one mixed-precision
// multiply-add (h * -1 + f) instead of two instructions.
template <bool HI>
__device__ inline float sub_half(float f, uint32_t u) {
  float e;
  if constexpr (HI)
    asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(e) : "v"(u), "v"(f));
  else
    asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel_hi:[1,0,0]" : "=v"(e) : "v"(u), "v"(f));
  return e;
}

// a - b for FP16 values a (half HA of ua) and b (half HB of ub), both widened
// exactly and the difference rounded once (b * -1 + a).
template <bool HA, bool HB>
__device__ inline float sub_halves(uint32_t ua, uint32_t ub) {
  float e;
  if constexpr (HA && HB)
    asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel:[1,0,1] op_sel_hi:[1,0,1]" : "=v"(e) : "v"(ub), "v"(ua));
  else if constexpr (HA)
    asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel:[0,0,1] op_sel_hi:[1,0,1]" : "=v"(e) : "v"(ub), "v"(ua));
  else if constexpr (HB)
    asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,1]" : "=v"(e) : "v"(ub), "v"(ua));
  else
    asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel_hi:[1,0,1]" : "=v"(e) : "v"(ub), "v"(ua));
  return e;
}

// a - v for the FP16 value a (half HA of ua) and an FP32 v: a widened exactly,
// the difference rounded once (v * -1 + a).
template <bool HA>
__device__ inline float sub_half_f32(uint32_t ua, float v) {
  float e;
  if constexpr (HA)
    asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel:[0,0,1] op_sel_hi:[0,0,1]" : "=v"(e) : "v"(v), "v"(ua));
  else
    asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel_hi:[0,0,1]" : "=v"(e) : "v"(v), "v"(ua));
  return e;
}

// h * w + acc and h * w + 0 for the FP16 value h in the low or high half of u,
// rounded once, with h widened exactly: the values a conversion followed by
// an FP32 multiply-add (or multiply) gives, up to the sign of an exact zero
// product, which no tap cost can tell apart (it only ever reaches a square).
template <bool HI>
__device__ inline float fma_half(uint32_t u, float w, float acc) {
  float r;
  if constexpr (HI)
    asm("v_fma_mix_f32 %0, %1, %2, %3 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(r) : "v"(u), "v"(w), "v"(acc));
  else
    asm("v_fma_mix_f32 %0, %1, %2, %3 op_sel_hi:[1,0,0]" : "=v"(r) : "v"(u), "v"(w), "v"(acc));
  return r;
}
template <bool HI>
__device__ inline float mul_half(uint32_t u, float w) {
  float r;
  if constexpr (HI)
    asm("v_fma_mix_f32 %0, %1, %2, 0 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(r) : "v"(u), "v"(w));
  else
    asm("v_fma_mix_f32 %0, %1, %2, 0 op_sel_hi:[1,0,0]" : "=v"(r) : "v"(u), "v"(w));
  return r;
}

// Channel k of the record whose raw words start at u (FP16: widened).
template <int C, bool FP16>
__device__ inline float chan(const uint32_t* u, int k) {
  if constexpr (FP16) {
    const uint32_t x = u[k >> 1];
    return (float)__builtin_bit_cast(_Float16, (uint16_t)((k & 1) ? (x >> 16) : (x & 0xffffu)));
  } else {
    return uf(u[k]);
  }
}

// tap_sq of a record in its raw words (Px::raw1): the same value.
template <int C, bool FP16>
__device__ inline float tap_sq_raw(const float* f1, const uint32_t* u, float gw) {
  float row = 0.f;
#pragma unroll
  for (int k = 0; k < C; ++k) {
    float e;
    if constexpr (FP16) {
      const uint32_t a = __builtin_bit_cast(uint32_t, f1[k >> 1]);
      e = (k & 1) ? sub_halves<true, true>(a, u[k >> 1]) : sub_halves<false, false>(a, u[k >> 1]);
    } else
      e = f1[k] - uf(u[k]);
    row = (k < 3) ? fmaf(e, e, row) : fmaf(gw * e, e, row);
  }
  return row;
}

// tap_sq with the source record packed (FP16 words, as load_column keeps them)
// and the target values in FP32: the same value as with the source widened first.
template <int C>
__device__ inline float tap_sq_packed(const float* f1, const float* v, float gw) {
  float row = 0.f;
#pragma unroll
  for (int k = 0; k < C; ++k) {
    const uint32_t a = __builtin_bit_cast(uint32_t, f1[k >> 1]);
    const float e = (k & 1) ? sub_half_f32<true>(a, v[k]) : sub_half_f32<false>(a, v[k]);
    row = (k < 3) ? fmaf(e, e, row) : fmaf(gw * e, e, row);
  }
  return row;
}

// G - 1 adds with the wave shifted right by one lane leave at lane l the sum
// ((v[l-G+1] + v[l-G+2]) + ...) + v[l]; at the group's last lane that is the
// group's G column partials in lane order.  Groups never straddle inactive
// lanes: a group is active or inactive as a whole.
template <int G>
__device__ inline float group_chain(float v) {
  float s = v;
#pragma unroll
  for (int k = 1; k < G; ++k) {
    const float sh =
        __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, s), 0x138, 0xf, 0xf, false));
    s = sh + v;
  }
  return s;
}

// Sum of the group's column partials in lane order, identical on every lane
// of the group: group_chain's value at the last lane, broadcast (by lane reads
// for up to nine groups: measured on MI355X, faster than a permute through
// LDS by 0.1 ms per pair with FP32 records and 1.6 ms with FP16 records).
template <int G>
__device__ inline float group_sum(float v, int base) {
  const float s = group_chain<G>(v);
  constexpr int NG = kWave / G;
  if constexpr (NG <= 9) {
    // few groups: read each group's last lane and select, no LDS round trip
    float r = 0.f;
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      const float t = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, s), g * G + G - 1));
      r = base == g * G ? t : r;
    }
    return r;
  } else {
    return __shfl(s, base + G - 1);
  }
}

// A decision taken at the group's last lane (where group_chain leaves the
// group's sum), handed to every lane of the group through one wave ballot:
// what a comparison of the broadcast sum would give on every lane, without
// the broadcast.  Values compared with such a sum (the running best cost of
// the identity-patch search) then need to be right only at the last lane.
template <int G>
__device__ inline bool group_flag(bool at_last, int base) {
  const unsigned long long m = __ballot(at_last);
  return (m >> (base + G - 1)) & 1ull;
}

__device__ inline const double* plane_H(const Ws& w, int label) {
  return label >= 0 ? w.planes[label].H : nullptr;
}

// Adds each group's count into counter `kind` with one atomic per wave;
// called by every lane of the wave (outside divergent code).  Spread over
// kCounterStripes copies (STRIPED) so that the waves of a launch do not
// serialise on one address, or all on copy 0: measured on MI355X, striping
// speeds the identity-patch and cost kernels (14.2 vs 14.4 ms and 1.4 vs 4.0
// ms per pipeline) while the distorted-patch kernel runs faster with one
// address (40.4 vs 51.3 ms); results are identical either way.
template <bool STRIPED>
__device__ inline void count_evals(unsigned long long* counters, int kind, unsigned v) {
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) v += __shfl_xor(v, o);
  const int stripe = STRIPED ? (blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave) & (kCounterStripes - 1) : 0;
  if ((threadIdx.x & (kWave - 1)) == 0 && v) atomicAdd(&counters[kind * kCounterStripes + stripe], (unsigned long long)v);
}

// Group-wide geometry status: 0 = usable, fractional taps; 1 = usable, all
// taps integral; 2 = some homogeneous coordinate not positive (cost +inf).
template <int G>
__device__ inline int group_geometry(bool ok, bool integral, int base) {
  const float bad = group_sum<G>(ok ? 0.f : 1.f, base);
  const float frac = group_sum<G>(integral ? 0.f : 1.f, base);
  return bad != 0.f ? 2 : (frac == 0.f ? 1 : 0);
}

// Adds the lane's taps of rows [T0, T1) for target (tx, ty) to acc, in row
// order.  Integral geometry: one pixel per tap.  Otherwise bilinear: the
// corner pairs of the tap's two rows, each one contiguous load.  Rows are
// taken CH at a time: all their loads are issued first and a scheduling
// barrier keeps them ahead of the arithmetic, so a wave has the gathers of
// CH rows in flight instead of waiting on each row in turn.
template <int R, int C, bool FP16, bool IDENT, bool INTEGRAL, int T0, int T1, int CH = 3>
__device__ inline float add_rows(float acc, const LaneCol<R, C, IDENT>& L, Feat F2, int W, int H,
                                 int tx, int ty, float gw) {
  if constexpr (T1 - T0 > CH) {
    acc = add_rows<R, C, FP16, IDENT, INTEGRAL, T0, T0 + CH, CH>(acc, L, F2, W, H, tx, ty, gw);
    return add_rows<R, C, FP16, IDENT, INTEGRAL, T0 + CH, T1, CH>(acc, L, F2, W, H, tx, ty, gw);
  } else if constexpr (IDENT || INTEGRAL) {
    constexpr int N = T1 - T0;
    uint32_t v[N][Px<C, FP16>::kWords];
#pragma unroll
    for (int n = 0; n < N; ++n) {
      const int t = T0 + n;
      int bx, by;
      if constexpr (IDENT) {
        bx = clampi(tx + L.dx, 0, W - 1);
        by = clampi(ty + t - R, 0, H - 1);
      } else {
        bx = clampi(tx + L.ox(t), 0, W - 1);
        by = clampi(ty + L.oy(t), 0, H - 1);
      }
      Px<C, FP16>::raw1(F2, by * W + bx, v[n]);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int n = 0; n < N; ++n) acc += tap_sq_raw<C, FP16>(L.f1[T0 + n], v[n], gw);
    return acc;
  } else {
    constexpr int N = T1 - T0, KW = Px<C, FP16>::kWords;
    uint32_t top[N][2 * KW], bot[N][2 * KW];
    float fx[N], fy[N];
#pragma unroll
    for (int n = 0; n < N; ++n) {
      const int t = T0 + n;
      // base pixel clamped into the frame; a fraction survives only where the
      // base and its right (lower) neighbour are both inside
      const int ux = tx + L.ox(t), uy = ty + L.oy(t);
      const int bx = min(max(ux, 0), W - 1), by = min(max(uy, 0), H - 1);
      fx[n] = (unsigned)ux < (unsigned)(W - 1) ? L.fx[t] : 0.f;
      fy[n] = (unsigned)uy < (unsigned)(H - 1) ? L.fy[t] : 0.f;
      const int i0 = by * W + bx;
      const int i1 = i0 + (by < H - 1 ? W : 0);
      Px<C, FP16>::raw2(F2, i0, top[n]);
      Px<C, FP16>::raw2(F2, i1, bot[n]);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int n = 0; n < N; ++n) {
      const float gx = 1.f - fx[n], gy = 1.f - fy[n];
      const float w00 = gx * gy, w01 = fx[n] * gy, w10 = gx * fy[n], w11 = fx[n] * fy[n];
      float v[C];
#pragma unroll
      for (int k = 0; k < C; ++k) {
        if constexpr (FP16) {
          // corners a, b (top pair) and c, d (bottom pair), widened inside the FMAs
          const int wi = k >> 1;
          if (k & 1)
            v[k] = fma_half<true>(bot[n][KW + wi], w11, fma_half<true>(bot[n][wi], w10,
                   fma_half<true>(top[n][KW + wi], w01, mul_half<true>(top[n][wi], w00))));
          else
            v[k] = fma_half<false>(bot[n][KW + wi], w11, fma_half<false>(bot[n][wi], w10,
                   fma_half<false>(top[n][KW + wi], w01, mul_half<false>(top[n][wi], w00))));
        } else {
          v[k] = fmaf(w11, chan<C, FP16>(bot[n] + KW, k),
                      fmaf(w10, chan<C, FP16>(bot[n], k),
                           fmaf(w01, chan<C, FP16>(top[n] + KW, k), w00 * chan<C, FP16>(top[n], k))));
        }
      }
      if constexpr (FP16)
        acc += tap_sq_packed<C>(L.f1[T0 + n], v, gw);
      else
        acc += tap_sq<C>(L.f1[T0 + n], v, gw);
    }
    return acc;
  }
}

// Group cost of target (tx, ty).  With EE the running group sum is compared
// with `bound` (the current best cost) after the first and second third of the
// rows: every tap adds a non-negative term and FP32 addition is monotone, so a
// prefix >= bound proves the full cost >= bound, and the candidate, which could
// never be strictly better, is dropped (rejected = true).  An accepted
// candidate is summed in the same order as without the checks.  rows returns
// the tap rows computed.
template <int R, int C, bool FP16, bool IDENT, bool INTEGRAL, bool EE, int CH = 3>
__device__ inline float group_cost(const LaneCol<R, C, IDENT>& L, Feat F2, int W, int H, int tx,
                                   int ty, float gw, int base, float bound, bool& rejected, unsigned& rows) {
  constexpr int T = 2 * R + 1, T1 = T / 3, T2 = (2 * T) / 3;
  rejected = false;
  if constexpr (!EE) {
    rows += T;
    return group_sum<T>(add_rows<R, C, FP16, IDENT, INTEGRAL, 0, T, CH>(0.f, L, F2, W, H, tx, ty, gw), base);
  } else {
    float acc = add_rows<R, C, FP16, IDENT, INTEGRAL, 0, T1, CH>(0.f, L, F2, W, H, tx, ty, gw);
    rows += T1;
    rejected = true;
    if (group_sum<T>(acc, base) >= bound) return 0.f;
    acc = add_rows<R, C, FP16, IDENT, INTEGRAL, T1, T2, CH>(acc, L, F2, W, H, tx, ty, gw);
    rows += T2 - T1;
    if (group_sum<T>(acc, base) >= bound) return 0.f;
    acc = add_rows<R, C, FP16, IDENT, INTEGRAL, T2, T, CH>(acc, L, F2, W, H, tx, ty, gw);
    rows += T - T2;
    rejected = false;
    return group_sum<T>(acc, base);
  }
}

// Byte offsets of the records of an identity-patch target (tx, ty) in a lane's
// column dx: record (clamp(tx + dx), clamp(ty + t - R)) of row t.  The row
// clamp commutes with the multiplication by the row pitch (positive), and a
// clamp commutes with adding the column's offset, so that a row costs one add
// of a wave-uniform term and one three-way median on a per-target base and
// bounds, instead of a clamp, a multiply-add and a multiply.
template <int R, int KB>
struct IdentAddr {
  int base, lo, hi, pitch;
  IdentAddr() = default;
  __device__ inline IdentAddr(int tx, int ty, int dx, int W, int H) {
    pitch = W * KB;
    lo = clampi(tx + dx, 0, W - 1) * KB;
    hi = lo + (H - 1) * pitch;
    base = lo + (ty - R) * pitch;
  }
  __device__ inline int at(int t) const {
    int o;
    asm("v_med3_i32 %0, %1, %2, %3" : "=v"(o) : "v"(base + t * pitch), "v"(lo), "v"(hi));
    return o;
  }
};

// Rows [T0, T) of one identity-patch target added to acc: the loads of all
// rows are issued ahead of their arithmetic.
template <int R, int C, bool FP16, int T0, int T>
__device__ inline float ident_rows1(float acc, const LaneCol<R, C, true>& L, Feat F2, int W, int H, int tx, int ty,
                                    float gw) {
  constexpr int N = T - T0;
  uint32_t v[N][Px<C, FP16>::kWords];
  const IdentAddr<R, Px<C, FP16>::kBytes> A(tx, ty, L.dx, W, H);
#pragma unroll
  for (int n = 0; n < N; ++n) Px<C, FP16>::raw1_at(F2, A.at(T0 + n), v[n]);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int n = 0; n < N; ++n) acc += tap_sq_raw<C, FP16>(L.f1[T0 + n], v[n], gw);
  return acc;
}

// Calls the instantiation FN<r, C, FP16> of P's parameters.
#define MSGPM_DISPATCH(FN, ...)                                                       \
  do {                                                                                \
    const bool h = P.fp16 != 0;                                                       \
    switch (P.r * 10 + P.C) {                                                         \
      case 13: return h ? FN<1, 3, true>(__VA_ARGS__) : FN<1, 3, false>(__VA_ARGS__); \
      case 15: return h ? FN<1, 5, true>(__VA_ARGS__) : FN<1, 5, false>(__VA_ARGS__); \
      case 23: return h ? FN<2, 3, true>(__VA_ARGS__) : FN<2, 3, false>(__VA_ARGS__); \
      case 25: return h ? FN<2, 5, true>(__VA_ARGS__) : FN<2, 5, false>(__VA_ARGS__); \
      case 33: return h ? FN<3, 3, true>(__VA_ARGS__) : FN<3, 3, false>(__VA_ARGS__); \
      case 35: return h ? FN<3, 5, true>(__VA_ARGS__) : FN<3, 5, false>(__VA_ARGS__); \
      case 43: return h ? FN<4, 3, true>(__VA_ARGS__) : FN<4, 3, false>(__VA_ARGS__); \
      case 45: return h ? FN<4, 5, true>(__VA_ARGS__) : FN<4, 5, false>(__VA_ARGS__); \
      default: return hipErrorInvalidValue;                                           \
    }                                                                                 \
  } while (0)

}  // namespace msgpm
