// Device helpers of the group evaluation (sl1m_wgroup.h): float16 operands split from
// float32, phasors, tapers.
#pragma once

#include "sl1m_device.h"
#include "sl1m_wgroup.h"

namespace sl1m {
namespace dev {

typedef _Float16 h2_t __attribute__((ext_vector_type(2)));
typedef _Float16 h8_t __attribute__((ext_vector_type(8)));
typedef float f2_t __attribute__((ext_vector_type(2)));
typedef float f4_t __attribute__((ext_vector_type(4)));

constexpr float kTwoPi = 6.28318530717958648f;

// exp(2 pi i a b) with the phase kept to 2^-24 turn (phasor: 2^-23) from FP64
// kMagicFine = kMagic / 2 on: two more instructions, for C_0, whose phase every
// entry of a group shares.
constexpr double kMagicFine = 0.5 * kMagic;
__device__ __forceinline__ void phasor_fine(double t, float& c, float& s) {
  const int32_t f = static_cast<int32_t>(static_cast<uint32_t>(__double2loint(t)) << 8);
  const float p = static_cast<float>(f) * 0x1.0p-32f;
  s = __builtin_amdgcn_sinf(p);
  c = __builtin_amdgcn_cosf(p);
}

// value = hi + lo in float16 (hi rounded to nearest, lo the rounded rest)
__device__ __forceinline__ void split2(float p, float q, h2_t& hi, h2_t& lo) {
  hi = __builtin_convertvector((f2_t{p, q}), h2_t);
  lo = __builtin_convertvector(
      (f2_t{p - static_cast<float>(hi[0]), q - static_cast<float>(hi[1])}), h2_t);
}

struct Op8 {
  h2_t v[4];
  __device__ __forceinline__ h8_t vec() const { return __builtin_bit_cast(h8_t, *this); }
};

__device__ __forceinline__ void split8(const float (&p)[8], Op8& hi, Op8& lo) {
#pragma unroll
  for (int j = 0; j < 4; ++j) split2(p[2 * j], p[2 * j + 1], hi.v[j], lo.v[j]);
}

__device__ __forceinline__ f4_t mma(h8_t a, h8_t b, f4_t c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ h8_t as_h8(uint4 v) { return __builtin_bit_cast(h8_t, v); }
__device__ __forceinline__ uint32_t as_u32(h2_t v) { return __builtin_bit_cast(uint32_t, v); }

__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}

// What a wavefront of a macro does: one of its row sets; with one set alone, a quarter of
// its visibility tiles (forward) or sign slots (adjoint).
struct WavePart {
  int set, lo, hi;  // visibility tiles [lo, hi)
  int mask;         // slots
  bool active;
};
__device__ __forceinline__ WavePart wave_part(int sets, int wv) {
  if (sets == 1) return {0, wv, wv + 1, 1 << wv, true};
  return {wv < sets ? wv : 0, 0, 4, 15, wv < sets};
}

__device__ __forceinline__ void store_slots(float4* __restrict__ o, int mask, float4 v) {
  if (mask == 15) {
    *o = v;
    return;
  }
  float* const f = &o->x;
  if (mask & 1) f[0] = v.x;
  if (mask & 2) f[1] = v.y;
  if (mask & 4) f[2] = v.z;
  if (mask & 8) f[3] = v.w;
}

// A slot's forward sum of one macro into its row, added where `add`.
__device__ __forceinline__ void store_row(float2* __restrict__ rows, int64_t at, bool add,
                                          float2 v) {
  if (add) {
    const float2 o = rows[at];
    v = make_float2(o.x + v.x, o.y + v.y);
  }
  rows[at] = v;
}

// What becomes of a slot's sum: times the gain, less the data (those given), into `out`
// and, times the conjugate gain, into the adjoint record `res`.
struct WgOut {
  const int32_t* order;
  const float* gain;
  const float2* data;
  float2* out;
  float2* res;
};
// slot t of visibility o / 2 (order), `acc` as for the caller's coordinates; returns the
// result, gain in gr, gi
__device__ __forceinline__ float2 wg_finish(const WgOut& w, int64_t t, int32_t o, float2 acc,
                                            float& gr, float& gi) {
  const int64_t k = o >> 1;
  gr = w.gain ? w.gain[2 * k] : 1.0f;
  gi = w.gain ? w.gain[2 * k + 1] : 0.0f;
  float re = acc.x, im = acc.y;
  if (w.gain) {
    re = gr * acc.x - gi * acc.y;
    im = gr * acc.y + gi * acc.x;
  }
  if (w.data) {
    re -= w.data[k].x;
    im -= w.data[k].y;
  }
  if (w.out) w.out[k] = make_float2(re, im);
  if (w.res) {
    const float ci = gr * im - gi * re;
    w.res[t] = make_float2(gr * re + gi * im, o & 1 ? -ci : ci);
  }
  return make_float2(re, im);
}

// log2 of the largest taper over +-[lo, hi] at baseline coordinate d
__device__ __forceinline__ float taper_top(float c1, float d, float w, float lo, float hi) {
  const float a = fmaf(-w, lo, d), b = fmaf(-w, hi, d), e = fmaf(w, lo, d), f = fmaf(w, hi, d);
  const float p = a * b <= 0.0f ? 0.0f : fminf(fabsf(a), fabsf(b));
  const float q = e * f <= 0.0f ? 0.0f : fminf(fabsf(e), fabsf(f));
  const float m = fminf(p, q);
  return c1 * (m * m);
}

// Sums (re, im) in units of k, a power of two: what is below one goes to the sums, which are
// large then (times a small taper it would be subnormal: 1.2e-5 instead of 4.9e-6 at tapers of
// 2^-113), the rest is returned for the taper (times the sums it could overflow).
__device__ __forceinline__ float scale_sums(float k, float& re, float& im) {
  const float s = fminf(k, 1.0f);
  re *= s;
  im *= s;
  return fmaxf(k, 1.0f);
}

// up 2^(c1 d^2 - top), at most up (padded positions may lie above the top).  Columns
// stand kGUp high: tapers down to 2^-28 of the largest are normal float16.  (The factor
// in the exponent would cost the exponent four bits.)
constexpr float kGUp = 0x1.0p14f, kGDown = 0x1.0p-14f;
__device__ __forceinline__ float taper(float c1, float d, float top, float up) {
  return up * __builtin_amdgcn_exp2f(fminf(fmaf(c1, d * d, -top), 0.0f));
}

}  // namespace dev
}  // namespace sl1m
