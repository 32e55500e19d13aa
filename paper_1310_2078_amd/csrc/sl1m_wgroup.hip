// Group evaluation of grid segments (sl1m_wgroup.h): kernels and launchers.
#include <cmath>

#include "sl1m_device.h"
#include "sl1m_wgroup.h"
#include "sl1m_wgroup_dev.h"

namespace sl1m {

// ---------------------------------------------------------------------------
// kernels
// ---------------------------------------------------------------------------

namespace {

using namespace dev;

constexpr int kParts = 5;  // column operand: hi, lo, x hi, x lo, x^2 / 2 (x = 2 pi s dw)

// Sums over the quads; lane L ends with visibility L.
__device__ __forceinline__ void quad_sum(const float (&vr)[4], const float (&vi)[4], int lane,
                                         float& sr, float& si) {
  const bool hi = (lane & 32) != 0, md = (lane & 16) != 0;
  float ar[2], ai[2];
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const float kr = hi ? vr[t + 2] : vr[t], ki = hi ? vi[t + 2] : vi[t];
    const float or_ = hi ? vr[t] : vr[t + 2], oi = hi ? vi[t] : vi[t + 2];
    ar[t] = kr + __shfl_xor(or_, 32, 64);
    ai[t] = ki + __shfl_xor(oi, 32, 64);
  }
  const float kr = md ? ar[1] : ar[0], ki = md ? ai[1] : ai[0];
  const float or_ = md ? ar[0] : ar[1], oi = md ? ai[0] : ai[1];
  sr = kr + __shfl_xor(or_, 16, 64);
  si = ki + __shfl_xor(oi, 16, 64);
}

// One step (16 columns) of one kind pair (re, im): the tile rows' values pr, pi
// (float32, this lane's row and four columns) times the column operands of the
// group's visibility tiles, with the series terms: D_re += x eta P_im,
// D_im -= x eta P_re (first order), D -= (x eta)^2 / 2 P (second).
template <int SER, bool FULL>
__device__ __forceinline__ void kind_pair(const float (&pr)[8], const float (&pi)[8],
                                          const float (&eta)[4], const uint4* __restrict__ col,
                                          const float (&hx)[4], int t0, int t1, f4_t (&dre)[4],
                                          f4_t (&dim)[4]) {
  Op8 rh, rl, ih, il, erh, erl, eih, eil;
  split8(pr, rh, rl);
  split8(pi, ih, il);
  if constexpr (SER >= 2) {
    float er[8], ei[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      er[j] = -eta[j / 2] * pr[j];
      ei[j] = eta[j / 2] * pi[j];
    }
    split8(er, erh, erl);
    split8(ei, eih, eil);
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const _Float16 e = static_cast<_Float16>(eta[j]);
      erh.v[j] = rh.v[j] * -(h2_t{e, e});
      eih.v[j] = ih.v[j] * h2_t{e, e};
    }
  }
  Op8 srh, sih;  // -eta^2 P_re, -eta^2 P_im
  if constexpr (SER >= 2) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float e = eta[j], e2 = -e * e;
      srh.v[j] = __builtin_convertvector((f2_t{e2 * pr[2 * j], e2 * pr[2 * j + 1]}), h2_t);
      sih.v[j] = __builtin_convertvector((f2_t{e2 * pi[2 * j], e2 * pi[2 * j + 1]}), h2_t);
    }
  } else if constexpr (SER == 1) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const _Float16 e = static_cast<_Float16>(eta[j]);
      srh.v[j] = erh.v[j] * h2_t{e, e};
      sih.v[j] = eih.v[j] * -(h2_t{e, e});
    }
  }
  Op8 trh, tih;
  if constexpr (SER == 3) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const _Float16 e = static_cast<_Float16>(eta[j]);
      trh.v[j] = sih.v[j] * h2_t{e, e};     // -eta^3 P_im
      tih.v[j] = srh.v[j] * -(h2_t{e, e});  // eta^3 P_re
    }
  }
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    if (!FULL && (t < t0 || t >= t1)) continue;
    const h8_t bh = as_h8(col[16 * t]), bl = as_h8(col[64 + 16 * t]), ch = as_h8(col[128 + 16 * t]);
    dre[t] = mma(rh.vec(), bh, dre[t]);
    dim[t] = mma(ih.vec(), bh, dim[t]);
    dre[t] = mma(rh.vec(), bl, dre[t]);
    dim[t] = mma(ih.vec(), bl, dim[t]);
    dre[t] = mma(rl.vec(), bh, dre[t]);
    dim[t] = mma(il.vec(), bh, dim[t]);
    dre[t] = mma(eih.vec(), ch, dre[t]);
    dim[t] = mma(erh.vec(), ch, dim[t]);
    if constexpr (SER >= 2) {
      const h8_t cl = as_h8(col[192 + 16 * t]);
      dre[t] = mma(eih.vec(), cl, dre[t]);
      dim[t] = mma(erh.vec(), cl, dim[t]);
      dre[t] = mma(eil.vec(), ch, dre[t]);
      dim[t] = mma(erl.vec(), ch, dim[t]);
    }
    if constexpr (SER > 0) {
      const h8_t sh = as_h8(col[256 + 16 * t]);
      dre[t] = mma(srh.vec(), sh, dre[t]);
      dim[t] = mma(sih.vec(), sh, dim[t]);
      if constexpr (SER == 3) {
        const h8_t th = sh * static_cast<_Float16>(hx[t]);  // x^3 / 6
        dre[t] = mma(trh.vec(), th, dre[t]);
        dim[t] = mma(tih.vec(), th, dim[t]);
      }
    }
  }
}

struct FwdAcc {
  f4_t cr[4], ci[4], sr[4], si[4];  // cos-row and sin-row sums (re, im) per visibility tile
};

// `e`: this lane's row and its four columns of every step.
template <int SER, bool FULL>
__device__ __forceinline__ void fwd_tile(int steps, double w0, const double* __restrict__ nu,
                                         const float4 (&e)[kWgSteps][4],
                                         const float (&eta)[kWgSteps][4],
                                         const uint4* __restrict__ col, const float (&hx)[4], int t0,
                                         int t1, FwdAcc& d) {
#pragma unroll
  for (int s = 0; s < kWgSteps; ++s) {
    if (!FULL && s >= steps) continue;
    float cc[4], cs[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) phasor_fine(fma(w0, nu[(s * 16 + j) * kWgRows], kMagicFine), cc[j], cs[j]);
    float pr[8], pi[8];
    const uint4* c = col + s * 4 * kParts * 64;
    // C = cc - i cs; cos row: bc (C e1), bs (-i C e3); sin row: bc (-i C e4), bs (C e2)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      pr[2 * j] = cc[j] * e[s][j].x;
      pr[2 * j + 1] = -cs[j] * e[s][j].z;
      pi[2 * j] = -cs[j] * e[s][j].x;
      pi[2 * j + 1] = -cc[j] * e[s][j].z;
    }
    kind_pair<SER, FULL>(pr, pi, eta[s], c, hx, t0, t1, d.cr, d.ci);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      pr[2 * j] = -cs[j] * e[s][j].w;
      pr[2 * j + 1] = cc[j] * e[s][j].y;
      pi[2 * j] = -cc[j] * e[s][j].w;
      pi[2 * j + 1] = -cs[j] * e[s][j].y;
    }
    kind_pair<SER, FULL>(pr, pi, eta[s], c, hx, t0, t1, d.sr, d.si);
  }
}

struct FwdLds {
  uint4 col[kWgSteps * 4 * kParts * 64];  // [step, quarter][part][visibility]: 4 columns (cos, sin)
  double nu[4][kWgCells];
  double la[4 * kWgRows], mb[kWgCols], u[kWgVis];
  float hx[kWgVis];                       // x / 3
  float2 red[4][kWgVis];
};

// Forward: block (groups x, x + gridDim.x, ..; macro y); row y of the partial sums holds the
// macro's sum per slot.  Bound by the vector instructions that form the operands (seven
// a product: C_0, its float16 splits, the rows' and columns' phasors), at two wavefronts
// per SIMD: 0.53 of the vector issue slots and 0.30 of the matrix cores' time at 256 x
// 256 x 97,536, 389 us (grid evaluation 511); 1024 x 1024 x 409,600: 10.2 ms (28.9).
// 16-row tiles of 32 columns: 32 x 32 products leave no registers for the group's 64
// visibilities (11.6 ms with groups of 32), 48 columns spill.
__global__ __launch_bounds__(kBlock, 2) void k_wg_fwd(
    const WgMacro* __restrict__ macros, int mac0, const float* __restrict__ xp,
    const float* __restrict__ pscale, const int4* __restrict__ slot, const double* __restrict__ nu,
    const float* __restrict__ eta, const double* __restrict__ la, const double* __restrict__ mb,
    const double* __restrict__ su, const double* __restrict__ sv, const float* __restrict__ sdw,
    const double* __restrict__ w0s, const float* __restrict__ hs, const int32_t* __restrict__ cnt,
    int n_groups, bool add, float2* __restrict__ rows) {
  __shared__ FwdLds lds;
  const int mac = mac0 + static_cast<int>(blockIdx.y);
  const ConstPtr<WgMacro> cm = as_const(macros) + mac;
  const int sets = cm->sets, steps = cm->steps;
  const float eta_max = cm->eta_max, xs = cm->xs;
  const int tid = threadIdx.x, lane = tid & 63, r16 = lane & 15, quad = lane >> 4;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const WavePart wp = wave_part(sets, wv);
  const bool active = wp.active;
  const float nu_t = cm->nu_t[wp.set];
  const int64_t cell0 = cm->cell_off + static_cast<int64_t>(wp.set) * kWgCells;
  if (tid < 4 * kWgRows) lds.la[tid] = la[cm->a_off + tid];
  if (tid < kWgCols) lds.mb[tid] = mb[cm->b_off + tid];
  const int64_t lane0 = cell0 + quad * 4 * kWgRows + r16;  // this lane's row, first column
  // sign combinations of the cells' amplitudes, times the power of two that
  // brings four times the tile's largest amplitude into [2^13, 2^14)
  for (int i = lane; i < kWgCells; i += 64) lds.nu[wv][i] = nu[cell0 + i];
  float4 e[kWgSteps][4];
  float et[kWgSteps][4];
  float mx = 0.0f;
#pragma unroll
  for (int s = 0; s < kWgSteps; ++s)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      et[s][j] = eta[lane0 + (s * 16 + j) * kWgRows];
      const int4 q = slot[lane0 + (s * 16 + j) * kWgRows];
      const float x0 = q.x >= 0 ? xp[q.x] * pscale[q.x] : 0.0f;
      const float x1 = q.y >= 0 ? xp[q.y] * pscale[q.y] : 0.0f;
      const float x2 = q.z >= 0 ? xp[q.z] * pscale[q.z] : 0.0f;
      const float x3 = q.w >= 0 ? xp[q.w] * pscale[q.w] : 0.0f;
      const float m = fmaxf(fmaxf(fabsf(x0), fabsf(x1)), fmaxf(fabsf(x2), fabsf(x3)));
      const float sum = (x0 + x1) + (x2 + x3);
      mx = fmaxf(mx, sum != sum ? __builtin_inff() : m);  // fmaxf drops a NaN
      e[s][j] = make_float4(sum, (x1 + x2) - (x0 + x3), (x0 + x1) - (x2 + x3),
                            (x0 - x1) + (x2 - x3));
    }
  const float c = 0.25f * op_scale(wave_max(mx)), sc = 1.0f / c;  // 4 mx may overflow
#pragma unroll
  for (int s = 0; s < kWgSteps; ++s)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      e[s][j].x *= c;
      e[s][j].y *= c;
      e[s][j].z *= c;
      e[s][j].w *= c;
    }
  const int g0 = static_cast<int>(blockIdx.x), gs = static_cast<int>(gridDim.x);
  const ConstPtr<double> cw0 = as_const(w0s);
  const ConstPtr<float> chs = as_const(hs);
  const ConstPtr<int32_t> ccnt = as_const(cnt);
  // each group's coordinates are loaded during the group before it
  double un_ = 0.0, vn = 0.0, w0n = 0.0;
  float dwn = 0.0f, hn = 0.0f;
  int cn = 0;
  auto load = [&](int g) {
    un_ = su[g * kWgVis + lane];
    vn = sv[g * kWgVis + lane];
    dwn = sdw[g * kWgVis + lane];
    w0n = cw0[g];
    hn = chs[g];
    cn = ccnt[g];
  };
  if (g0 < n_groups) load(g0);
  __syncthreads();
  for (int g = g0; g < n_groups; g += gs) {
    const float dw = dwn;
    const double w0 = w0n;
    const float xm = kTwoPi * hn * eta_max;
    const int ser = xm <= kWgXN ? 0 : xm <= kWgXM ? 1 : xm <= kWgXW ? 2 : 3;
    const bool wide = ser >= 2;
    const int nt = (cn + 15) >> 4;
    {
      const double v = vn;
      const float x = xs * dw;
      if (wv == 0) {
        lds.u[lane] = un_;
        lds.hx[lane] = 0.33333334f * x;
      }
      load(g + gs < n_groups ? g + gs : g);
      for (int un = wv; un < 4 * steps; un += 4) {
        uint4 o[kParts];
        uint32_t* const po = reinterpret_cast<uint32_t*>(o);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          float cb, sb;
          phasor(fma(v, lds.mb[un * 4 + j], kMagic), cb, sb);
          h2_t hi, lo, fh, fl;
          split2(cb, sb, hi, lo);
          po[j] = as_u32(hi);
          po[4 + j] = as_u32(lo);
          const float xc = x * cb, xsn = x * sb;
          if (ser > 0)
            po[16 + j] = as_u32(__builtin_convertvector((f2_t{0.5f * x * xc, 0.5f * x * xsn}), h2_t));
          if (wide) {
            split2(xc, xsn, fh, fl);
            po[12 + j] = as_u32(fl);
          } else {
            fh = __builtin_convertvector((f2_t{xc, xsn}), h2_t);
          }
          po[8 + j] = as_u32(fh);
        }
        uint4* dst = lds.col + un * kParts * 64 + lane;
        dst[0] = o[0];
        dst[64] = o[1];
        dst[128] = o[2];
        if (wide) dst[192] = o[3];
        if (ser > 0) dst[256] = o[4];
      }
    }
    __syncthreads();
    float re = 0.0f, im = 0.0f;
    if (active) {
      FwdAcc d;
#pragma unroll
      for (int t = 0; t < 4; ++t) d.cr[t] = d.ci[t] = d.sr[t] = d.si[t] = f4_t{0, 0, 0, 0};
      float hx[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) hx[t] = lds.hx[16 * t + r16];
      const uint4* col = lds.col + quad * kParts * 64 + r16;
      const double* nuw = &lds.nu[wv][quad * 4 * kWgRows + r16];
      const int t0 = wp.lo, t1 = nt < wp.hi ? nt : wp.hi;
      const bool full = steps == kWgSteps && t1 - t0 == 4;
      if (full && ser == 0)
        fwd_tile<0, true>(steps, w0, nuw, e, et, col, hx, t0, t1, d);
      else if (ser == 0)
        fwd_tile<0, false>(steps, w0, nuw, e, et, col, hx, t0, t1, d);
      else if (ser == 1)
        fwd_tile<1, false>(steps, w0, nuw, e, et, col, hx, t0, t1, d);
      else if (ser == 2)
        fwd_tile<2, false>(steps, w0, nuw, e, et, col, hx, t0, t1, d);
      else
        fwd_tile<3, false>(steps, w0, nuw, e, et, col, hx, t0, t1, d);
      // lane: visibility 16 t + r16, rows 4 quad + i
      float vr[4], vi[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        vr[t] = vi[t] = 0.0f;
        if (t < t0 || t >= t1) continue;
        const double u = lds.u[16 * t + r16];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          float ac, as;
          phasor(fma(u, lds.la[wp.set * kWgRows + quad * 4 + i], kMagic), ac, as);
          vr[t] = fmaf(ac, d.cr[t][i], vr[t]);
          vi[t] = fmaf(ac, d.ci[t][i], vi[t]);
          vr[t] = fmaf(as, d.sr[t][i], vr[t]);
          vi[t] = fmaf(as, d.si[t][i], vi[t]);
        }
      }
      float sr, si;
      quad_sum(vr, vi, lane, sr, si);
      const float th = dw * nu_t;
      const float ct = __builtin_amdgcn_cosf(th), st = __builtin_amdgcn_sinf(th);
      re = sc * fmaf(ct, sr, st * si);
      im = sc * fmaf(ct, si, -st * sr);
    }
    lds.red[wv][lane] = make_float2(re, im);
    __syncthreads();
    if (tid < kWgVis) {
      const float2 a = lds.red[0][tid], b = lds.red[1][tid], c2 = lds.red[2][tid],
                   d = lds.red[3][tid];
      store_row(rows, (static_cast<int64_t>(blockIdx.y) * n_groups + g) * kWgVis + tid, add,
                make_float2((a.x + b.x) + (c2.x + d.x), (a.y + b.y) + (c2.y + d.y)));
    }
  }
}

// Per-slot coordinates: the visibility's, negated where w < 0; w and w - w0, as far as they
// are read (padding: the group's w0, 0).
__global__ void k_wg_slots(const int32_t* __restrict__ order, const double* __restrict__ w0s,
                           const double* __restrict__ vu, const double* __restrict__ vv,
                           const double* __restrict__ vw, int64_t n, double* __restrict__ su,
                           double* __restrict__ sv, double* __restrict__ sw,
                           float* __restrict__ sdw) {
  const int64_t t = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (t >= n) return;
  const int32_t o = order[t];
  const double w0 = w0s[t / kWgVis];
  if (o < 0) {
    su[t] = sv[t] = 0.0;
    if (sw) sw[t] = w0;
    if (sdw) sdw[t] = 0.0f;
    return;
  }
  const int32_t k = o >> 1;
  const double sg = o & 1 ? -1.0 : 1.0;
  su[t] = sg * vu[k];
  sv[t] = sg * vv[k];
  const double w = sg * vw[k];
  if (sw) sw[t] = w;
  if (sdw) sdw[t] = static_cast<float>(w - w0);
}

// Slot t's visibility: the macros' rows, conjugated where w < 0, and the other
// segments' rows (indexed by visibility); gain, data and adjoint records as
// k_fwd_reduce.
__global__ void k_wg_fwd_reduce(const float2* __restrict__ part, int n_macros, int64_t n_slots,
                                const float2* __restrict__ rows, int n_rows, int64_t n_vis,
                                WgOut w, float2* __restrict__ rres,
                                const float* __restrict__ layerDs, int n_layers) {
  const int64_t t = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (t >= n_slots) return;
  const int32_t o = w.order[t];
  if (o < 0) {
    if (w.res) w.res[t] = make_float2(0.0f, 0.0f);
    return;
  }
  const int64_t k = o >> 1;
  float2 acc = make_float2(0.0f, 0.0f);
  strided_sum<float2>(part + t, n_macros, n_slots, acc);
  if (o & 1) acc.y = -acc.y;
  strided_sum<float2>(rows + k, n_rows, n_vis, acc);
  float gr, gi;
  const float2 v = wg_finish(w, t, o, acc, gr, gi);
  if (rres) write_res<float>(rres, layerDs, n_layers, n_vis, 1, k, 0, gr, gi, v.x, v.y);
}

// ---------------------------------------------------------------------------
// adjoint: per group and tile the sums over its visibilities
//   T_XY(a,b) = sum_k X_k(a) Y_k(b) rho_k, X, Y in {cos, sin}, rho the residual
//   times exp(2 pi i dw nuT),
// and the same with x_k, x_k^2 / 2, x_k^3 / 6 in front (T1, T2, T3; series in
// eta), are matrix products over k; then conj(C_0) and the series are applied
// once per cell:
//   Z = conj(C_0) (T + i eta T1 - eta^2 T2 - i eta^3 T3),
//   G1 += Re Z_cc, G2 += Re Z_ss, G3 += Im Z_cs, G4 += Im Z_sc  (sl1m_grid.h).
// ---------------------------------------------------------------------------

constexpr int kAdjPitch = 36;  // uint32 (visibility pairs) per column of an operand, padded

struct alignas(16) AdjLds {
  // [part][cos, sin][column][visibility pair]
  uint32_t col[kParts][2][kWgCols][kAdjPitch];
  uint32_t hx[kWgVis / 2];              // x / 3 of every pair
  double nu[4][4 * kWgSteps][64];       // by lane: column 16 c + lane % 16, row 4 (lane / 16) + i
  float eta[4][4 * kWgSteps][64];
  double la[4 * kWgRows], mb[kWgCols], u[kWgVis];
  float2 rho[4][kWgVis];
};

struct AdjOp {  // row operand of 32 visibilities: re and im, hi and lo
  Op8 rh, rl, ih, il;
};

// One kind X Y over the group, t = T and T1 (re, im each): `b`: this lane's column
// operand (part stride `ps`, column tile stride `cs`, in uint4).
template <int SER, bool FULL>
__device__ __forceinline__ void adj_low(const AdjOp (&a)[2], const uint4* __restrict__ b, int ps,
                                        int cs, f4_t (&t)[4][kWgSteps], int steps) {
#pragma unroll
  for (int c = 0; c < kWgSteps; ++c) {
#pragma unroll
    for (int o = 0; o < 4; ++o) t[o][c] = f4_t{0, 0, 0, 0};
    if (!FULL && c >= steps) continue;
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
      const uint4* q = b + c * cs + 4 * kb;
      const h8_t bh = as_h8(q[0]), bl = as_h8(q[ps]), ch = as_h8(q[2 * ps]);
      t[0][c] = mma(a[kb].rh.vec(), bh, t[0][c]);
      t[1][c] = mma(a[kb].ih.vec(), bh, t[1][c]);
      t[2][c] = mma(a[kb].rh.vec(), ch, t[2][c]);
      t[3][c] = mma(a[kb].ih.vec(), ch, t[3][c]);
      t[0][c] = mma(a[kb].rh.vec(), bl, t[0][c]);
      t[1][c] = mma(a[kb].ih.vec(), bl, t[1][c]);
      if constexpr (SER >= 2) {
        const h8_t cl = as_h8(q[3 * ps]);
        t[2][c] = mma(a[kb].rh.vec(), cl, t[2][c]);
        t[3][c] = mma(a[kb].ih.vec(), cl, t[3][c]);
      }
      t[0][c] = mma(a[kb].rl.vec(), bh, t[0][c]);
      t[1][c] = mma(a[kb].il.vec(), bh, t[1][c]);
      if constexpr (SER >= 2) {
        t[2][c] = mma(a[kb].rl.vec(), ch, t[2][c]);
        t[3][c] = mma(a[kb].il.vec(), ch, t[3][c]);
      }
    }
  }
}

// The same, t = T2 and (SER 3) T3; `hx`: x / 3 of this lane's visibilities.
template <int SER, bool FULL>
__device__ __forceinline__ void adj_high(const AdjOp (&a)[2], const uint4* __restrict__ b, int ps,
                                         int cs, const uint4* __restrict__ hx,
                                         f4_t (&t)[4][kWgSteps], int steps) {
#pragma unroll
  for (int c = 0; c < kWgSteps; ++c) {
#pragma unroll
    for (int o = 0; o < 4; ++o) t[o][c] = f4_t{0, 0, 0, 0};
    if (!FULL && c >= steps) continue;
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
      const h8_t sh = as_h8(b[c * cs + 4 * kb + 4 * ps]);
      t[0][c] = mma(a[kb].rh.vec(), sh, t[0][c]);
      t[1][c] = mma(a[kb].ih.vec(), sh, t[1][c]);
      if constexpr (SER == 3) {
        const h8_t th = sh * as_h8(hx[4 * kb]);  // x^3 / 6
        t[2][c] = mma(a[kb].rh.vec(), th, t[2][c]);
        t[3][c] = mma(a[kb].ih.vec(), th, t[3][c]);
      }
    }
  }
}

// G += Re (IM: Im) of conj(C) (T + i eta T1), or of conj(C) (-eta^2) (T2 + i eta T3)
// (HIGH; T3 there with SER 3 only).
template <int SER, bool IM, bool HIGH>
__device__ __forceinline__ void adj_fold(const f4_t (&t)[4][kWgSteps],
                                         const float (&cc)[kWgSteps][4],
                                         const float (&cs)[kWgSteps][4],
                                         const float* __restrict__ eta, float (&g)[kWgSteps][4]) {
#pragma unroll
  for (int c = 0; c < kWgSteps; ++c)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float e = eta[64 * (4 * c + i)];
      float zr = t[0][c][i], zi = t[1][c][i];
      if (!HIGH || SER == 3) {
        zr = fmaf(-e, t[3][c][i], zr);
        zi = fmaf(e, t[2][c][i], zi);
      }
      if constexpr (HIGH) {
        const float e2 = -e * e;
        zr *= e2;
        zi *= e2;
      }
      if constexpr (IM) {
        g[c][i] = fmaf(cc[c][i], zi, g[c][i]);
        g[c][i] = fmaf(cs[c][i], zr, g[c][i]);
      } else {
        g[c][i] = fmaf(cc[c][i], zr, g[c][i]);
        g[c][i] = fmaf(-cs[c][i], zi, g[c][i]);
      }
      // the sum is formed here: sunk below the next kinds it would keep their
      // accumulators and this one's alive together (256 registers and spills)
      asm volatile("" : "+v"(g[c][i]));
    }
}

// Row operands of the group from this lane's row phasor components (cos or sin)
// of its 16 visibilities.
__device__ __forceinline__ void adj_rows(const float (&ph)[2][8], const float2* __restrict__ rho,
                                         AdjOp (&a)[2]) {
#pragma unroll
  for (int kb = 0; kb < 2; ++kb)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float2 r0 = rho[32 * kb + 2 * j], r1 = rho[32 * kb + 2 * j + 1];
      const float p0 = ph[kb][2 * j], p1 = ph[kb][2 * j + 1];
      split2(p0 * r0.x, p1 * r1.x, a[kb].rh.v[j], a[kb].rl.v[j]);
      split2(p0 * r0.y, p1 * r1.y, a[kb].ih.v[j], a[kb].il.v[j]);
    }
}

template <int SER, bool FULL, bool IM>
__device__ __forceinline__ void adj_kind(const AdjOp (&a)[2], const uint4* __restrict__ b,
                                         const uint4* __restrict__ hx,
                                         const float (&cc)[kWgSteps][4],
                                         const float (&cs)[kWgSteps][4],
                                         const float* __restrict__ eta, int steps,
                                         float (&g)[kWgSteps][4]) {
  constexpr int kPart = 2 * kWgCols * kAdjPitch / 4, kTile = 16 * kAdjPitch / 4;
  f4_t t[4][kWgSteps];
  adj_low<SER, FULL>(a, b, kPart, kTile, t, steps);
  adj_fold<SER, IM, false>(t, cc, cs, eta, g);
  if constexpr (SER > 0) {
    adj_high<SER, FULL>(a, b, kPart, kTile, hx, t, steps);
    adj_fold<SER, IM, true>(t, cc, cs, eta, g);
  }
}

template <int SER, bool FULL>
__device__ __forceinline__ void adj_group(const float (&pc)[2][8], const float (&ps)[2][8],
                                          const float2* __restrict__ rho,
                                          const uint4* __restrict__ b, const uint4* __restrict__ hx,
                                          const float (&cc)[kWgSteps][4],
                                          const float (&cs)[kWgSteps][4],
                                          const float* __restrict__ eta, int steps, int mask,
                                          float (&g)[4][kWgSteps][4]) {
  constexpr int kType = kWgCols * kAdjPitch / 4;
  AdjOp a[2];
  if (mask & 5) adj_rows(pc, rho, a);
  if (mask & 1) adj_kind<SER, FULL, false>(a, b, hx, cc, cs, eta, steps, g[0]);
  if (mask & 4) adj_kind<SER, FULL, true>(a, b + kType, hx, cc, cs, eta, steps, g[2]);
  if (mask & 10) adj_rows(ps, rho, a);
  if (mask & 2) adj_kind<SER, FULL, false>(a, b + kType, hx, cc, cs, eta, steps, g[1]);
  if (mask & 8) adj_kind<SER, FULL, true>(a, b, hx, cc, cs, eta, steps, g[3]);
}

// Adjoint: block (groups x, x + gridDim.x, ..; macro y); part[x][cell] = (G1, G2,
// G3, G4) of its groups.  Bound as the forward (0.57 and 0.33 of the slots): 256 x 256 x
// 97,536 439 us (grid evaluation 601), 1024 x 1024 x 409,600 12.0 ms (27.4).
__global__ __launch_bounds__(kBlock, 2) void k_wg_adj(
    const WgMacro* __restrict__ macros, int mac0, const float2* __restrict__ res,
    const double* __restrict__ nu, const float* __restrict__ eta, const double* __restrict__ la,
    const double* __restrict__ mb, const double* __restrict__ su, const double* __restrict__ sv,
    const float* __restrict__ sdw, const double* __restrict__ w0s, const float* __restrict__ hs,
    int n_groups, int64_t cbase, int64_t cells, float4* __restrict__ part) {
  __shared__ AdjLds lds;
  const ConstPtr<WgMacro> cm = as_const(macros) + mac0 + blockIdx.y;
  const int sets = cm->sets, steps = cm->steps;
  const float eta_max = cm->eta_max, xs = cm->xs;
  const int tid = threadIdx.x, lane = tid & 63, r16 = lane & 15, quad = lane >> 4;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const WavePart wp = wave_part(sets, wv);
  const bool active = wp.active;
  const float nu_t = cm->nu_t[wp.set];
  const int64_t cell0 = cm->cell_off + static_cast<int64_t>(wp.set) * kWgCells;
  if (tid < 4 * kWgRows) lds.la[tid] = la[cm->a_off + tid];
  if (tid < kWgCols) lds.mb[tid] = mb[cm->b_off + tid];
  // this lane's cells: column 16 c + r16, rows 4 quad + i
  float g[4][kWgSteps][4];
#pragma unroll
  for (int c = 0; c < kWgSteps; ++c)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int64_t q = cell0 + (16 * c + r16) * kWgRows + quad * 4 + i;
      lds.nu[wv][4 * c + i][lane] = nu[q];
      lds.eta[wv][4 * c + i][lane] = eta[q];
#pragma unroll
      for (int o = 0; o < 4; ++o) g[o][c][i] = 0.0f;
    }
  const int g0 = static_cast<int>(blockIdx.x), gs = static_cast<int>(gridDim.x);
  const ConstPtr<double> cw0 = as_const(w0s);
  const ConstPtr<float> chs = as_const(hs);
  const int vp = tid & 31, c8 = tid >> 5;  // column operands: visibility pair, column
  // each group's coordinates and residuals are loaded during the group before it
  double2 vn = make_double2(0.0, 0.0);
  double un = 0.0, w0n = 0.0;
  float2 dwp = make_float2(0.0f, 0.0f), rn = make_float2(0.0f, 0.0f);
  float dwn = 0.0f, hn = 0.0f;
  auto load = [&](int gi) {
    vn = reinterpret_cast<const double2*>(sv)[gi * (kWgVis / 2) + vp];
    dwp = reinterpret_cast<const float2*>(sdw)[gi * (kWgVis / 2) + vp];
    un = su[gi * kWgVis + lane];
    dwn = sdw[gi * kWgVis + lane];
    rn = res[gi * kWgVis + lane];
    w0n = cw0[gi];
    hn = chs[gi];
  };
  if (g0 < n_groups) load(g0);
  __syncthreads();
  for (int gi = g0; gi < n_groups; gi += gs) {
    const double w0 = w0n;
    const float xm = kTwoPi * hn * eta_max;
    const int ser = xm <= kWgXN ? 0 : xm <= kWgXM ? 1 : xm <= kWgXW ? 2 : 3;
    // residuals times the tile's factor, scaled into float16's range
    const float th = dwn * nu_t;
    const float ct = __builtin_amdgcn_cosf(th), st = __builtin_amdgcn_sinf(th);
    const float rr = fmaf(ct, rn.x, -st * rn.y), ri = fmaf(ct, rn.y, st * rn.x);
    const float am = fmaxf(fabsf(rr), fabsf(ri));
    const float sc = op_scale(wave_max(rr != rr || ri != ri ? __builtin_inff() : am));
    lds.rho[wv][lane] = make_float2(rr * sc, ri * sc);
    const float inv = 1.0f / sc;
    if (wv == 0) lds.u[lane] = un;
    const double2 v = vn;
    const float x0 = xs * dwp.x, x1 = xs * dwp.y;
    if (tid < 32) lds.hx[vp] = as_u32(__builtin_convertvector((f2_t{0.33333334f * x0, 0.33333334f * x1}), h2_t));
    load(gi + gs < n_groups ? gi + gs : gi);
    for (int c = c8; c < 16 * steps; c += 8) {
      float a0, b0, a1, b1;
      const double m = lds.mb[c];
      phasor(fma(v.x, m, kMagic), a0, b0);
      phasor(fma(v.y, m, kMagic), a1, b1);
      h2_t hi, lo;
      split2(a0, a1, hi, lo);
      lds.col[0][0][c][vp] = as_u32(hi);
      lds.col[1][0][c][vp] = as_u32(lo);
      split2(b0, b1, hi, lo);
      lds.col[0][1][c][vp] = as_u32(hi);
      lds.col[1][1][c][vp] = as_u32(lo);
      a0 *= x0;
      a1 *= x1;
      b0 *= x0;
      b1 *= x1;
      if (ser > 0) {
        const float h0 = 0.5f * x0, h1 = 0.5f * x1;
        lds.col[4][0][c][vp] = as_u32(__builtin_convertvector((f2_t{h0 * a0, h1 * a1}), h2_t));
        lds.col[4][1][c][vp] = as_u32(__builtin_convertvector((f2_t{h0 * b0, h1 * b1}), h2_t));
      }
      if (ser >= 2) {
        split2(a0, a1, hi, lo);
        lds.col[2][0][c][vp] = as_u32(hi);
        lds.col[3][0][c][vp] = as_u32(lo);
        split2(b0, b1, hi, lo);
        lds.col[2][1][c][vp] = as_u32(hi);
        lds.col[3][1][c][vp] = as_u32(lo);
      } else {
        lds.col[2][0][c][vp] = as_u32(__builtin_convertvector((f2_t{a0, a1}), h2_t));
        lds.col[2][1][c][vp] = as_u32(__builtin_convertvector((f2_t{b0, b1}), h2_t));
      }
    }
    __syncthreads();
    if (active) {
      float pc[2][8], ps[2][8];
      const double l = lds.la[wp.set * kWgRows + r16];
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int j = 0; j < 8; ++j)
          phasor(fma(lds.u[32 * kb + 8 * quad + j], l, kMagic), pc[kb][j], ps[kb][j]);
      float cc[kWgSteps][4], cs[kWgSteps][4];
#pragma unroll
      for (int c = 0; c < kWgSteps; ++c)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          phasor_fine(fma(w0, lds.nu[wv][4 * c + i][lane], kMagicFine), cc[c][i], cs[c][i]);
          cc[c][i] *= inv;
          cs[c][i] *= inv;
        }
      const uint4* b = reinterpret_cast<const uint4*>(&lds.col[0][0][r16][4 * quad]);
      const uint4* hx = reinterpret_cast<const uint4*>(&lds.hx[4 * quad]);
      const float2* rho = &lds.rho[wv][8 * quad];
      if (ser == 0 && steps == kWgSteps)
        adj_group<0, true>(pc, ps, rho, b, hx, cc, cs, &lds.eta[wv][0][lane], steps, wp.mask,
                          g);
      else if (ser == 0)
        adj_group<0, false>(pc, ps, rho, b, hx, cc, cs, &lds.eta[wv][0][lane], steps, wp.mask,
                          g);
      else if (ser == 1)
        adj_group<1, false>(pc, ps, rho, b, hx, cc, cs, &lds.eta[wv][0][lane], steps, wp.mask,
                          g);
      else if (ser == 2)
        adj_group<2, false>(pc, ps, rho, b, hx, cc, cs, &lds.eta[wv][0][lane], steps, wp.mask,
                          g);
      else
        adj_group<3, false>(pc, ps, rho, b, hx, cc, cs, &lds.eta[wv][0][lane], steps, wp.mask,
                          g);
    }
    __syncthreads();
  }
  if (!active) return;
#pragma unroll
  for (int c = 0; c < kWgSteps; ++c)
#pragma unroll
    for (int i = 0; i < 4; ++i)
      store_slots(part + blockIdx.x * cells + cell0 - cbase + (16 * c + r16) * kWgRows +
                      quad * 4 + i,
                  wp.mask, make_float4(g[0][c][i], g[1][c][i], g[2][c][i], g[3][c][i]));
}

// ---------------------------------------------------------------------------
// Gaussian layers (completed-square form, sl1m_grid.h).  An entry is
//   D (1 + i s) exp(2 pi i (e0 - w kappa)) a_sign(|l|) b_sign(|m|),
//   a+- = T(u -+ w|l|) exp(2 pi i (+- A|l| + C l^2)), b+- the same of v, |m|, B,
// where C l^2 + C m^2 carries the phase's r^2 term; kappa (n - 1 + r^2 / 2) is alpha(l)
// + beta(m) + eta (append_segment), exp(-2 pi i w alpha) and exp(-2 pi i w beta) join
// the factors, and eta alone is left to the groups, whose series needs one order only
// (with kappa itself the coarse layers needed a second order and a split first one).
// Both factors are complex, so the products are twice as long.  Tapers are formed
// against the largest of the macro's columns and (adjoint) of the tile's rows per
// visibility, so that the float16 operands keep their precision where a whole
// baseline's taper is small.  Bound by the vector instructions around the products
// (C_0 and its splits, the rows' and columns' phasors and tapers), as for delta
// pixels.  512 x 512 pixels, 409,600 visibilities: forward 5.3 ms, adjoint 6.5 ms;
// the grid evaluation of the same layer took 13.2 and 14.9.  300 x 300 truncated,
// 100,003: 0.47 / 0.54 ms against 1.33 / 1.53.
// ---------------------------------------------------------------------------

struct alignas(16) FwdGLds {
  uint4 col[kWgCols / 2 * 4 * 64];  // [two columns][B1 hi, lo, B2 hi, lo][visibility]
  double la[4 * kWgRows], al[4 * kWgRows], mb[kWgCols], be[kWgCols];
  double A[kWgVis], C[kWgVis], w[kWgVis];
  float4 uw[kWgVis];                // u, w, c1, x
  float2 red[4][kWgVis];
};

// gamma x of one step of 8 columns for the two row signs: this lane's row, two
// columns of two signs, (re, im) each.
__device__ __forceinline__ void gauss_rows(double w0, const double (&kap)[2], const float4 (&x)[2],
                                           float (&pp)[8], float (&pm)[8]) {
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    float cc, cs;
    phasor_fine(fma(w0, kap[j], kMagicFine), cc, cs);
    pp[4 * j] = cc * x[j].x;
    pp[4 * j + 1] = -cs * x[j].x;
    pp[4 * j + 2] = cc * x[j].z;
    pp[4 * j + 3] = -cs * x[j].z;
    pm[4 * j] = cc * x[j].y;
    pm[4 * j + 1] = -cs * x[j].y;
    pm[4 * j + 2] = cc * x[j].w;
    pm[4 * j + 3] = -cs * x[j].w;
  }
}

__device__ __forceinline__ Op8 times_eta(const Op8& p, const float (&eta)[2]) {
  Op8 r;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const _Float16 e = static_cast<_Float16>(eta[j / 2]);
    r.v[j] = p.v[j] * h2_t{e, e};
  }
  return r;
}

// D (re, im; two row signs): sums over the tile's columns, SER 1 with the first
// order -i x eta.
struct GAcc {
  f4_t d[4][4];  // [+ re, + im, - re, - im][visibility tile]
};

template <int SER>
__device__ __forceinline__ void fwd_gauss_tile(int steps, double w0,
                                               const double (&kap)[2 * kWgSteps][2],
                                               const float4 (&x)[2 * kWgSteps][2],
                                               const float (&eta)[2 * kWgSteps][2],
                                               const uint4* __restrict__ col,
                                               const float (&xv)[4], int t0, int t1, GAcc& a) {
#pragma unroll
  for (int ks = 0; ks < 2 * kWgSteps; ++ks) {
    if (ks >= 2 * steps) continue;
    float pp[8], pm[8];
    gauss_rows(w0, kap[ks], x[ks], pp, pm);
    Op8 ph, pl, pe, mh, ml, me;
    split8(pp, ph, pl);
    split8(pm, mh, ml);
    if constexpr (SER > 0) {
      pe = times_eta(ph, eta[ks]);
      me = times_eta(mh, eta[ks]);
    }
    const uint4* q = col + ks * 4 * 4 * 64;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      if (t < t0 || t >= t1) continue;
      const h8_t b1h = as_h8(q[16 * t]), b1l = as_h8(q[64 + 16 * t]);
      const h8_t b2h = as_h8(q[128 + 16 * t]), b2l = as_h8(q[192 + 16 * t]);
      a.d[0][t] = mma(ph.vec(), b1h, a.d[0][t]);
      a.d[1][t] = mma(ph.vec(), b2h, a.d[1][t]);
      a.d[2][t] = mma(mh.vec(), b1h, a.d[2][t]);
      a.d[3][t] = mma(mh.vec(), b2h, a.d[3][t]);
      a.d[0][t] = mma(ph.vec(), b1l, a.d[0][t]);
      a.d[1][t] = mma(ph.vec(), b2l, a.d[1][t]);
      a.d[2][t] = mma(mh.vec(), b1l, a.d[2][t]);
      a.d[3][t] = mma(mh.vec(), b2l, a.d[3][t]);
      a.d[0][t] = mma(pl.vec(), b1h, a.d[0][t]);
      a.d[1][t] = mma(pl.vec(), b2h, a.d[1][t]);
      a.d[2][t] = mma(ml.vec(), b1h, a.d[2][t]);
      a.d[3][t] = mma(ml.vec(), b2h, a.d[3][t]);
      if constexpr (SER > 0) {
        const _Float16 xf = static_cast<_Float16>(xv[t]);
        const h8_t x2 = b2h * xf, x1 = b1h * -xf;
        a.d[0][t] = mma(pe.vec(), x2, a.d[0][t]);
        a.d[1][t] = mma(pe.vec(), x1, a.d[1][t]);
        a.d[2][t] = mma(me.vec(), x2, a.d[2][t]);
        a.d[3][t] = mma(me.vec(), x1, a.d[3][t]);
      }
    }
  }
}

__global__ __launch_bounds__(kBlock, 2) void k_wg_fwd_gauss(
    const WgMacro* __restrict__ macros, int mac0, const float* __restrict__ xp,
    const float* __restrict__ pscale, const int4* __restrict__ slot, const double* __restrict__ kap,
    const float* __restrict__ eta, const double* __restrict__ la, const double* __restrict__ mb,
    const double* __restrict__ alpha, const double* __restrict__ beta,
    const WgVisG* __restrict__ rec, const float* __restrict__ sdw, const double* __restrict__ w0s,
    const float* __restrict__ hs, const int32_t* __restrict__ cnt, int n_groups,
    bool add, float2* __restrict__ rows) {
  __shared__ FwdGLds lds;
  const int mac = mac0 + static_cast<int>(blockIdx.y);
  const ConstPtr<WgMacro> cm = as_const(macros) + mac;
  const int sets = cm->sets, steps = cm->steps;
  const float eta_max = cm->eta_max, xs = cm->xs, m_lo = cm->m_lo, m_hi = cm->m_hi;
  const int tid = threadIdx.x, lane = tid & 63, r16 = lane & 15, quad = lane >> 4;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const WavePart wp = wave_part(sets, wv);
  const bool active = wp.active;
  const int64_t cell0 = cm->cell_off + static_cast<int64_t>(wp.set) * kWgCells;
  if (tid < 4 * kWgRows) {
    lds.la[tid] = la[cm->a_off + tid];
    lds.al[tid] = alpha[cm->a_off + tid];
  }
  if (tid < kWgCols) {
    lds.mb[tid] = mb[cm->b_off + tid];
    lds.be[tid] = beta[cm->b_off + tid];
  }
  // amplitudes of this lane's row and its two columns of every 8, times the power
  // of two that brings the tile's largest into [2^13, 2^14)
  double kp[2 * kWgSteps][2];
  float4 x[2 * kWgSteps][2];
  float et[2 * kWgSteps][2];
  float mx = 0.0f;
#pragma unroll
  for (int s = 0; s < 2 * kWgSteps; ++s)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int64_t o = cell0 + (8 * s + 2 * quad + j) * kWgRows + r16;
      kp[s][j] = kap[o];
      et[s][j] = eta[o];
      const int4 q = slot[o];
      const float x0 = q.x >= 0 ? xp[q.x] * pscale[q.x] : 0.0f;
      const float x1 = q.y >= 0 ? xp[q.y] * pscale[q.y] : 0.0f;
      const float x2 = q.z >= 0 ? xp[q.z] * pscale[q.z] : 0.0f;
      const float x3 = q.w >= 0 ? xp[q.w] * pscale[q.w] : 0.0f;
      const float m = fmaxf(fmaxf(fabsf(x0), fabsf(x1)), fmaxf(fabsf(x2), fabsf(x3)));
      const float sum = (x0 + x1) + (x2 + x3);
      mx = fmaxf(mx, sum != sum ? __builtin_inff() : m);  // fmaxf drops a NaN
      x[s][j] = make_float4(x0, x1, x2, x3);
    }
  const float c = op_scale(wave_max(mx)), sc = 1.0f / c;
#pragma unroll
  for (int s = 0; s < 2 * kWgSteps; ++s)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      x[s][j].x *= c;
      x[s][j].y *= c;
      x[s][j].z *= c;
      x[s][j].w *= c;
    }
  const int g0 = static_cast<int>(blockIdx.x), gs = static_cast<int>(gridDim.x);
  const ConstPtr<double> cw0 = as_const(w0s);
  const ConstPtr<float> chs = as_const(hs);
  const ConstPtr<int32_t> ccnt = as_const(cnt);
  WgVisG rn = {};
  double w0n = 0.0;
  float dwn = 0.0f, hn = 0.0f;
  int cn = 0;
  auto load = [&](int g) {
    rn = rec[g * kWgVis + lane];
    dwn = sdw[g * kWgVis + lane];
    w0n = cw0[g];
    hn = chs[g];
    cn = ccnt[g];
  };
  if (g0 < n_groups) load(g0);
  __syncthreads();
  for (int g = g0; g < n_groups; g += gs) {
    const WgVisG r = rn;
    const float dw = dwn;
    const double w0 = w0n;
    const bool one = kTwoPi * hn * eta_max > kWgXZ;  // an order of the series
    const int nt = (cn + 15) >> 4;
    const double w = w0 + static_cast<double>(dw);
    if (wv == 0) {
      lds.A[lane] = r.A;
      lds.C[lane] = r.C;
      lds.w[lane] = w;
      lds.uw[lane] = make_float4(r.u, r.w, r.c1, xs * dw);
    }
    load(g + gs < n_groups ? g + gs : g);
    const float top = taper_top(r.c1, r.v, r.w, m_lo, m_hi);
    for (int un = wv; un < 8 * steps; un += 4) {
      uint4 o[4];
      uint32_t* const po = reinterpret_cast<uint32_t*>(o);
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const double m = lds.mb[un * 2 + j];
        const float mr = static_cast<float>(m);
        const double q = fma(r.C, m * m, -w * lds.be[un * 2 + j]);
        float cb, sb, cm_, sm_;
        phasor(fma(r.B, m, q) + kMagic, cb, sb);
        phasor(fma(-r.B, m, q) + kMagic, cm_, sm_);
        const float tp = taper(r.c1, fmaf(-r.w, mr, r.v), top, kGUp);
        const float tm = taper(r.c1, fmaf(r.w, mr, r.v), top, kGUp);
        h2_t hp, lp, hm, lm;
        split2(tp * cb, tp * sb, hp, lp);
        split2(tm * cm_, tm * sm_, hm, lm);
        // B1 = (re, -im), B2 = (im, re) of b+ and b-
        po[2 * j] = as_u32(h2_t{hp[0], -hp[1]});
        po[2 * j + 1] = as_u32(h2_t{hm[0], -hm[1]});
        po[4 + 2 * j] = as_u32(h2_t{lp[0], -lp[1]});
        po[4 + 2 * j + 1] = as_u32(h2_t{lm[0], -lm[1]});
        po[8 + 2 * j] = as_u32(hp.yx);
        po[8 + 2 * j + 1] = as_u32(hm.yx);
        po[12 + 2 * j] = as_u32(lp.yx);
        po[12 + 2 * j + 1] = as_u32(lm.yx);
      }
      uint4* dst = lds.col + un * 4 * 64 + lane;
#pragma unroll
      for (int q = 0; q < 4; ++q) dst[q * 64] = o[q];
    }
    __syncthreads();
    float re = 0.0f, im = 0.0f;
    if (active) {
      const int t0 = wp.lo, t1 = nt < wp.hi ? nt : wp.hi;
      GAcc d;
#pragma unroll
      for (int o = 0; o < 4; ++o)
#pragma unroll
        for (int t = 0; t < 4; ++t) d.d[o][t] = f4_t{0, 0, 0, 0};
      float xv[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) xv[t] = lds.uw[16 * t + r16].w;
      const uint4* col = lds.col + quad * 4 * 64 + r16;
      if (one)
        fwd_gauss_tile<1>(steps, w0, kp, x, et, col, xv, t0, t1, d);
      else
        fwd_gauss_tile<0>(steps, w0, kp, x, et, col, xv, t0, t1, d);
      float vr[4], vi[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        vr[t] = vi[t] = 0.0f;
        if (t < t0 || t >= t1) continue;
        const double A = lds.A[16 * t + r16], C = lds.C[16 * t + r16], W = lds.w[16 * t + r16];
        const float4 uw = lds.uw[16 * t + r16];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const double l = lds.la[wp.set * kWgRows + quad * 4 + i];
          const float lr = static_cast<float>(l);
          float cp, sp, cn_, sn_;
          const double q = fma(C, l * l, -W * lds.al[wp.set * kWgRows + quad * 4 + i]);
          phasor(fma(A, l, q) + kMagic, cp, sp);
          phasor(fma(-A, l, q) + kMagic, cn_, sn_);
          const float du = fmaf(-uw.y, lr, uw.x), dv = fmaf(uw.y, lr, uw.x);
          const float tp = pow2(uw.z * (du * du)), tm = pow2(uw.z * (dv * dv));
          const float apr = tp * cp, api = tp * sp, amr = tm * cn_, ami = tm * sn_;
          vr[t] = fmaf(apr, d.d[0][t][i], fmaf(-api, d.d[1][t][i], vr[t]));
          vi[t] = fmaf(apr, d.d[1][t][i], fmaf(api, d.d[0][t][i], vi[t]));
          vr[t] = fmaf(amr, d.d[2][t][i], fmaf(-ami, d.d[3][t][i], vr[t]));
          vi[t] = fmaf(amr, d.d[3][t][i], fmaf(ami, d.d[2][t][i], vi[t]));
        }
      }
      float sr, si;
      quad_sum(vr, vi, lane, sr, si);
      // visibility `lane`: D (1 + i s), e0, the columns' top
      const float ct = __builtin_amdgcn_cosf(r.e0), st = __builtin_amdgcn_sinf(r.e0);
      const float k = scale_sums(sc * kGDown, sr, si) * pow2(top);
      const float fr = k * fmaf(r.D, ct, -r.Ds * st), fi = k * fmaf(r.D, st, r.Ds * ct);
      re = fmaf(fr, sr, -fi * si);
      im = fmaf(fr, si, fi * sr);
    }
    lds.red[wv][lane] = make_float2(re, im);
    __syncthreads();
    if (tid < kWgVis) {
      const float2 a = lds.red[0][tid], b = lds.red[1][tid], c2 = lds.red[2][tid],
                   d = lds.red[3][tid];
      store_row(rows, (static_cast<int64_t>(blockIdx.y) * n_groups + g) * kWgVis + tid, add,
                make_float2((a.x + b.x) + (c2.x + d.x), (a.y + b.y) + (c2.y + d.y)));
    }
  }
}

constexpr int kGPitch = 68;  // uint32 (visibilities) per column of an operand, padded

struct alignas(16) AdjGLds {
  uint32_t col[2][4][kWgCols][kGPitch];  // [b+, b-][B1 hi, lo, B2 hi, lo][column][visibility]
  double la[4 * kWgRows], al[4 * kWgRows], mb[kWgCols], be[kWgCols];
  double A[kWgVis], C[kWgVis], w[kWgVis];
  float4 uw[kWgVis];                     // u, w, c1, x
  float2 rho[4][kWgVis];
  float top[4][kWgVis];
  uint32_t x[kWgVis];                    // (x, x) in float16
};

struct GOp {  // row operand of 16 visibilities: (re, im) each; hi, lo, and x times hi
  Op8 h, l, e;
};

// G of one sign pair += Re conj(C_0) (T + i eta T1), T1 with SER 1; `b`: this lane's
// column operand.
template <int SER>
__device__ __forceinline__ void adj_gauss_kind(const GOp (&a)[4], const uint4* __restrict__ b,
                                               const float (&cc)[kWgSteps][4],
                                               const float (&cs)[kWgSteps][4],
                                               const float (&eta)[kWgSteps][4], int steps,
                                               float (&g)[kWgSteps][4]) {
  constexpr int kPart = kWgCols * kGPitch / 4, kTile = 16 * kGPitch / 4;
  f4_t t[4][kWgSteps];
#pragma unroll
  for (int c = 0; c < kWgSteps; ++c) {
#pragma unroll
    for (int o = 0; o < 4; ++o) t[o][c] = f4_t{0, 0, 0, 0};
    if (c >= steps) continue;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint4* q = b + c * kTile + 4 * k;
      const h8_t b1h = as_h8(q[0]), b2h = as_h8(q[2 * kPart]);
      const h8_t b1l = as_h8(q[kPart]), b2l = as_h8(q[3 * kPart]);
      t[0][c] = mma(a[k].h.vec(), b1h, t[0][c]);
      t[1][c] = mma(a[k].h.vec(), b2h, t[1][c]);
      if constexpr (SER > 0) {
        t[2][c] = mma(a[k].e.vec(), b1h, t[2][c]);
        t[3][c] = mma(a[k].e.vec(), b2h, t[3][c]);
      }
      t[0][c] = mma(a[k].h.vec(), b1l, t[0][c]);
      t[1][c] = mma(a[k].h.vec(), b2l, t[1][c]);
      t[0][c] = mma(a[k].l.vec(), b1h, t[0][c]);
      t[1][c] = mma(a[k].l.vec(), b2h, t[1][c]);
    }
  }
#pragma unroll
  for (int c = 0; c < kWgSteps; ++c)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float e = eta[c][i];
      float zr = t[0][c][i], zi = t[1][c][i];
      if constexpr (SER > 0) {
        zr = fmaf(-e, t[3][c][i], zr);
        zi = fmaf(e, t[2][c][i], zi);
      }
      g[c][i] = fmaf(cc[c][i], zr, g[c][i]);
      g[c][i] = fmaf(-cs[c][i], zi, g[c][i]);
      asm volatile("" : "+v"(g[c][i]));  // formed here (adj_fold)
    }
}

struct GRow {  // this lane's row and the group's visibilities (LDS)
  float lr;
  double l, l2, al;
  const float4* uw;
  const double *A, *C, *w;
  const float2* rho;
  const float* top;
};

template <int SER>
__device__ __forceinline__ void adj_gauss_group(const GRow& r, int quad,
                                                const uint4* __restrict__ b,
                                                const uint4* __restrict__ x,
                                                const float (&cc)[kWgSteps][4],
                                                const float (&cs)[kWgSteps][4],
                                                const float (&eta)[kWgSteps][4], int steps,
                                                int mask, float (&g)[4][kWgSteps][4]) {
  constexpr int kSign = 4 * kWgCols * kGPitch / 4;
#pragma unroll
  for (int s = 0; s < 2; ++s) {  // row signs
    if (!(mask & (5 << s))) continue;
    GOp a[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const h8_t xk = as_h8(x[4 * k]);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int v = 16 * k + 4 * quad + j;
        const float4 uw = r.uw[v];
        const double A = s ? -r.A[v] : r.A[v];
        float ca, sa;
        phasor(fma(A, r.l, fma(r.C[v], r.l2, -r.w[v] * r.al)) + kMagic, ca, sa);
        const float t = taper(uw.z, fmaf(s ? uw.y : -uw.y, r.lr, uw.x), r.top[v], 1.0f);
        ca *= t;
        sa *= t;
        const float2 z = r.rho[v];
        const float yr = fmaf(ca, z.x, sa * z.y), yi = fmaf(ca, z.y, -sa * z.x);
        split2(yr, yi, a[k].h.v[j], a[k].l.v[j]);
      }
      if constexpr (SER > 0) a[k].e = __builtin_bit_cast(Op8, a[k].h.vec() * xk);
    }
    if (mask & (1 << s)) adj_gauss_kind<SER>(a, b, cc, cs, eta, steps, g[s]);
    if (mask & (4 << s)) adj_gauss_kind<SER>(a, b + kSign, cc, cs, eta, steps, g[2 + s]);
  }
}

// part[x][cell] = the four sign slots' sums
__global__ __launch_bounds__(kBlock, 2) void k_wg_adj_gauss(
    const WgMacro* __restrict__ macros, int mac0, const float2* __restrict__ res,
    const double* __restrict__ kap, const float* __restrict__ eta, const double* __restrict__ la,
    const double* __restrict__ mb, const double* __restrict__ alpha,
    const double* __restrict__ beta, const WgVisG* __restrict__ rec, const float* __restrict__ sdw,
    const double* __restrict__ w0s, const float* __restrict__ hs, int n_groups, int64_t cbase,
    int64_t cells, float4* __restrict__ part) {
  __shared__ AdjGLds lds;
  const ConstPtr<WgMacro> cm = as_const(macros) + mac0 + blockIdx.y;
  const int sets = cm->sets, steps = cm->steps;
  const float eta_max = cm->eta_max, xs = cm->xs, m_lo = cm->m_lo, m_hi = cm->m_hi;
  const int tid = threadIdx.x, lane = tid & 63, r16 = lane & 15, quad = lane >> 4;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const WavePart wp = wave_part(sets, wv);
  const bool active = wp.active;
  const float l_lo = cm->l_lo[wp.set], l_hi = cm->l_hi[wp.set];
  const int64_t cell0 = cm->cell_off + static_cast<int64_t>(wp.set) * kWgCells;
  if (tid < 4 * kWgRows) {
    lds.la[tid] = la[cm->a_off + tid];
    lds.al[tid] = alpha[cm->a_off + tid];
  }
  if (tid < kWgCols) {
    lds.mb[tid] = mb[cm->b_off + tid];
    lds.be[tid] = beta[cm->b_off + tid];
  }
  double kp[kWgSteps][4];
  float et[kWgSteps][4], g[4][kWgSteps][4];
#pragma unroll
  for (int c = 0; c < kWgSteps; ++c)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int64_t q = cell0 + (16 * c + r16) * kWgRows + quad * 4 + i;
      kp[c][i] = kap[q];
      et[c][i] = eta[q];
#pragma unroll
      for (int o = 0; o < 4; ++o) g[o][c][i] = 0.0f;
    }
  const int g0 = static_cast<int>(blockIdx.x), gs = static_cast<int>(gridDim.x);
  const ConstPtr<double> cw0 = as_const(w0s);
  const ConstPtr<float> chs = as_const(hs);
  WgVisG rn = {};
  float2 zn = make_float2(0.0f, 0.0f);
  double w0n = 0.0;
  float dwn = 0.0f, hn = 0.0f;
  auto load = [&](int gi) {
    rn = rec[gi * kWgVis + lane];
    zn = res[gi * kWgVis + lane];
    dwn = sdw[gi * kWgVis + lane];
    w0n = cw0[gi];
    hn = chs[gi];
  };
  if (g0 < n_groups) load(g0);
  __syncthreads();
  for (int gi = g0; gi < n_groups; gi += gs) {
    const WgVisG r = rn;
    const double w0 = w0n;
    const bool one = kTwoPi * hn * eta_max > kWgXZ;  // an order of the series
    // residual times conj of the visibility's factors, with both tops
    const float top = taper_top(r.c1, r.v, r.w, m_lo, m_hi);
    const float ltop = taper_top(r.c1, r.u, r.w, l_lo, l_hi);
    const double w = w0 + static_cast<double>(dwn);
    const float k = pow2(top + ltop);
    const float c0 = __builtin_amdgcn_cosf(r.e0), s0 = __builtin_amdgcn_sinf(r.e0);
    const float ct = k * fmaf(r.D, c0, -r.Ds * s0), st = k * fmaf(r.D, s0, r.Ds * c0);
    const float rr = fmaf(ct, zn.x, st * zn.y), ri = fmaf(ct, zn.y, -st * zn.x);
    const float am = fmaxf(fabsf(rr), fabsf(ri));
    // (at most 2^111: 1 / sc, which the cell factors take on, stays a normal number)
    const float sc = fminf(
        0.5f * op_scale(wave_max(rr != rr || ri != ri ? __builtin_inff() : am)), 0x1.0p111f);
    lds.rho[wv][lane] = make_float2(rr * sc, ri * sc);
    lds.top[wv][lane] = ltop;
    const float inv = kGDown / sc;
    if (wv == 0) {
      lds.A[lane] = r.A;
      lds.C[lane] = r.C;
      lds.w[lane] = w;
      const float x = xs * dwn;
      lds.uw[lane] = make_float4(r.u, r.w, r.c1, x);
      lds.x[lane] = as_u32(__builtin_convertvector((f2_t{x, x}), h2_t));
    }
    load(gi + gs < n_groups ? gi + gs : gi);
    for (int c = wv; c < 16 * steps; c += 4) {
      const double m = lds.mb[c];
      const float mr = static_cast<float>(m);
      const double q = fma(r.C, m * m, -w * lds.be[c]);
      float cp, sp, cn, sn;
      phasor(fma(r.B, m, q) + kMagic, cp, sp);
      phasor(fma(-r.B, m, q) + kMagic, cn, sn);
      const float tp = taper(r.c1, fmaf(-r.w, mr, r.v), top, kGUp);
      const float tm = taper(r.c1, fmaf(r.w, mr, r.v), top, kGUp);
      h2_t hi, lo;
      // conj(b): B1 = (re, im), B2 = (-im, re)
      split2(tp * cp, tp * sp, hi, lo);
      lds.col[0][0][c][lane] = as_u32(hi);
      lds.col[0][1][c][lane] = as_u32(lo);
      lds.col[0][2][c][lane] = as_u32(h2_t{-hi[1], hi[0]});
      lds.col[0][3][c][lane] = as_u32(h2_t{-lo[1], lo[0]});
      split2(tm * cn, tm * sn, hi, lo);
      lds.col[1][0][c][lane] = as_u32(hi);
      lds.col[1][1][c][lane] = as_u32(lo);
      lds.col[1][2][c][lane] = as_u32(h2_t{-hi[1], hi[0]});
      lds.col[1][3][c][lane] = as_u32(h2_t{-lo[1], lo[0]});
    }
    __syncthreads();
    if (active) {
      float cc[kWgSteps][4], cs[kWgSteps][4];
#pragma unroll
      for (int c = 0; c < kWgSteps; ++c)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          phasor_fine(fma(w0, kp[c][i], kMagicFine), cc[c][i], cs[c][i]);
          cc[c][i] *= inv;
          cs[c][i] *= inv;
        }
      const double l = lds.la[wp.set * kWgRows + r16], l2 = l * l;
      const float lr = static_cast<float>(l);
      const uint4* x = reinterpret_cast<const uint4*>(&lds.x[4 * quad]);
      const uint4* b = reinterpret_cast<const uint4*>(&lds.col[0][0][r16][4 * quad]);
      const GRow row{lr,    l,     l2,    lds.al[wp.set * kWgRows + r16], lds.uw, lds.A, lds.C,
                     lds.w, lds.rho[wv], lds.top[wv]};
      if (one)
        adj_gauss_group<1>(row, quad, b, x, cc, cs, et, steps, wp.mask, g);
      else
        adj_gauss_group<0>(row, quad, b, x, cc, cs, et, steps, wp.mask, g);
    }
    __syncthreads();
  }
  if (!active) return;
#pragma unroll
  for (int c = 0; c < kWgSteps; ++c)
#pragma unroll
    for (int i = 0; i < 4; ++i)
      store_slots(part + blockIdx.x * cells + cell0 - cbase + (16 * c + r16) * kWgRows +
                      quad * 4 + i,
                  wp.mask, make_float4(g[0][c][i], g[1][c][i], g[2][c][i], g[3][c][i]));
}

// Per-slot constants of a Gaussian layer (coordinates negated where w < 0).
__global__ void k_wg_slots_gauss(const int32_t* __restrict__ order, const double* __restrict__ vu,
                                 const double* __restrict__ vv, const double* __restrict__ vw,
                                 double sigma, int64_t n, WgVisG* __restrict__ rec) {
  const int64_t t = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (t >= n) return;
  WgVisG r = {};
  const int32_t o = order[t];
  if (o >= 0) {
    const int32_t k = o >> 1;
    const double sg = o & 1 ? -1.0 : 1.0;
    const double u = sg * vu[k], v = sg * vv[k], w = sg * vw[k];
    const double s2 = sigma * sigma, s = w * s2, D = 1.0 / (1.0 + s * s);
    r.A = -D * u;
    r.B = -D * v;
    r.C = 0.5 * D * w;
    r.u = static_cast<float>(u);
    r.v = static_cast<float>(v);
    r.w = static_cast<float>(w);
    r.c1 = static_cast<float>(-M_PI * s2 * D * 1.4426950408889634);
    const double e = -0.5 * D * w * s2 * s2 * (u * u + v * v);
    r.e0 = static_cast<float>(e - rint(e));
    r.D = static_cast<float>(D);
    r.Ds = static_cast<float>(D * s);
  }
  rec[t] = r;
}

// Chunk sums of every cell, combined into its sign slots (row 0 of the adjoint
// partials); SLOTS: they are the slots' sums themselves.  A block takes 16 cells, 16
// threads each every 16th chunk: small segments have few cells and many chunks (with
// one thread a cell 32 x 32 x 2,000 took 9.8 us instead of 4.4, and the adjoint of 256 x
// 256 pixels with three layers x 50,000 718 us instead of 433).
constexpr int kRedCells = 16, kRedSlices = kBlock / kRedCells;
template <bool SLOTS>
__global__ __launch_bounds__(kBlock) void k_wg_adj_reduce(const float4* __restrict__ part,
                                                          int n_chunks, int64_t cells,
                                                          const int4* __restrict__ slot,
                                                          float* __restrict__ out) {
  __shared__ float4 sh[kRedSlices][kRedCells];
  const int tid = static_cast<int>(threadIdx.x), ci = tid % kRedCells, sl = tid / kRedCells;
  const int64_t q = static_cast<int64_t>(blockIdx.x) * kRedCells + ci;  // cells: a multiple of 16
  float4 a = make_float4(0.0f, 0.0f, 0.0f, 0.0f), b = a;
  for (int c = sl; c < n_chunks; c += 2 * kRedSlices) {
    const float4 v = part[c * cells + q];
    a.x += v.x;
    a.y += v.y;
    a.z += v.z;
    a.w += v.w;
    if (c + kRedSlices < n_chunks) {
      const float4 w = part[(c + kRedSlices) * cells + q];
      b.x += w.x;
      b.y += w.y;
      b.z += w.z;
      b.w += w.w;
    }
  }
  sh[sl][ci] = make_float4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w);
  __syncthreads();
  // threads of a cell: component sl % 4, slices sl / 4, sl / 4 + 4, ..
  const float* f = &sh[0][0].x;
  float v = 0.0f;
#pragma unroll
  for (int i = 0; i < 4; ++i) v += f[((sl / 4 + 4 * i) * kRedCells + ci) * 4 + sl % 4];
  __syncthreads();
  float* w = &sh[0][0].x;
  w[(sl / 4 * kRedCells + ci) * 4 + sl % 4] = v;
  __syncthreads();
  if (sl != 0) return;
  const int4 s = slot[q];
  const float g1 = (sh[0][ci].x + sh[1][ci].x) + (sh[2][ci].x + sh[3][ci].x);
  const float g2 = (sh[0][ci].y + sh[1][ci].y) + (sh[2][ci].y + sh[3][ci].y);
  const float g3 = (sh[0][ci].z + sh[1][ci].z) + (sh[2][ci].z + sh[3][ci].z);
  const float g4 = (sh[0][ci].w + sh[1][ci].w) + (sh[2][ci].w + sh[3][ci].w);
  if constexpr (SLOTS) {
    if (s.x >= 0) out[s.x] = g1;
    if (s.y >= 0) out[s.y] = g2;
    if (s.z >= 0) out[s.z] = g3;
    if (s.w >= 0) out[s.w] = g4;
    return;
  }
  if (s.x >= 0) out[s.x] = g1 - g2 - g3 - g4;
  if (s.y >= 0) out[s.y] = g1 + g2 - g3 + g4;
  if (s.z >= 0) out[s.z] = g1 + g2 + g3 - g4;
  if (s.w >= 0) out[s.w] = g1 - g2 + g3 + g4;
}

// Adjoint records per slot from the caller's residual (k_adj_prep by slot).
__global__ void k_wg_adj_prep(const float2* __restrict__ r, const int32_t* __restrict__ order,
                              int64_t n_slots, int64_t n_vis, const float* __restrict__ gain,
                              float2* __restrict__ res, float2* __restrict__ rres,
                              const float* __restrict__ layerDs, int n_layers) {
  const int64_t t = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (t >= n_slots) return;
  const int32_t o = order[t];
  float2 z = make_float2(0.0f, 0.0f);
  if (o >= 0) {
    const int64_t k = o >> 1;
    const float gr = gain ? gain[2 * k] : 1.0f, gi = gain ? gain[2 * k + 1] : 0.0f;
    const float2 v = r[k];
    if (rres) write_res<float>(rres, layerDs, n_layers, n_vis, 1, k, 0, gr, gi, v.x, v.y);
    const float ci = gr * v.y - gi * v.x;
    z = make_float2(gr * v.x + gi * v.y, o & 1 ? -ci : ci);
  }
  res[t] = z;
}


static_assert(kWgCells % kRedCells == 0 && kFlatCells % kRedCells == 0, "whole blocks of cells");

inline unsigned blocks1(int64_t n) { return static_cast<unsigned>((n + kBlock - 1) / kBlock); }

}  // namespace

hipError_t launch_wg_setup(sl1m_plan* p, hipStream_t st) {
  const int64_t n = static_cast<int64_t>(p->wg_groups) * kWgVis;
  if (p->wg_n == 0 || n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_wg_slots, dim3(blocks1(n)), dim3(kBlock), 0, st, p->wg_order, p->wg_w0,
                     p->vu, p->vv, p->vw, n, p->wg_su, p->wg_sv, p->wg_sw, p->wg_dw);
  for (int i = 0; i < p->wg_n; ++i) {
    const GridSeg& g = p->grid_segs[i];
    if (g.kind != SL1M_PIX_DELTA)
      hipLaunchKernelGGL(k_wg_slots_gauss, dim3(blocks1(n)), dim3(kBlock), 0, st, p->wg_order,
                         p->vu, p->vv, p->vw, p->layer_sigma[g.layer], n,
                         p->wg_recg + g.layer * n);
  }
  return hipGetLastError();
}

hipError_t launch_wg_forward(sl1m_plan* p, const GridSeg& g, const void* xp, hipStream_t st) {
  const WgSeg& s = p->wg_segs[&g - p->grid_segs.data()];
  const float* x = static_cast<const float*>(xp);
  const float* scale = static_cast<const float*>(p->pscale);
  const int4* slot = reinterpret_cast<const int4*>(p->wg_slot);
  const bool delta = g.kind == SL1M_PIX_DELTA;
  return timed(p, delta ? T_GRID_FWD_DELTA : T_GRID_FWD_GAUSS, st, [&] {
    if (s.flat) return launch_flat_forward(p, g, s, x, st);
    return wg_passes(p, s, [&](int mac0, int macros, float2* rows, bool add) {
      const dim3 grid(static_cast<unsigned>(wg_chunks(macros, p->wg_groups)),
                      static_cast<unsigned>(macros));
      if (delta)
        hipLaunchKernelGGL(k_wg_fwd, grid, dim3(kBlock), 0, st, p->wg_mac, mac0, x, scale, slot,
                           p->wg_nu, p->wg_eta, p->wg_la, p->wg_mb, p->wg_su, p->wg_sv, p->wg_dw,
                           p->wg_w0, p->wg_h, p->wg_count, p->wg_groups, add, rows);
      else
        hipLaunchKernelGGL(k_wg_fwd_gauss, grid, dim3(kBlock), 0, st, p->wg_mac, mac0, x, scale,
                           slot, p->wg_nu, p->wg_eta, p->wg_la, p->wg_mb, p->wg_alpha, p->wg_beta,
                           p->wg_recg + static_cast<int64_t>(g.layer) * p->wg_groups * kWgVis,
                           p->wg_dw, p->wg_w0, p->wg_h, p->wg_count, p->wg_groups, add, rows);
      return hipGetLastError();
    });
  });
}

static bool wg_all_pixels(const sl1m_plan* p) {
  int64_t c = 0;
  for (int i = 0; i < p->wg_n; ++i) c += p->segs[p->grid_segs[i].seg].count;
  return c == p->n_pix;
}

// Residual records by visibility are for the segments outside the groups.
static float2* rres_of(const sl1m_plan* p) {
  return wg_all_pixels(p) ? nullptr : static_cast<float2*>(p->rres);
}

hipError_t launch_wg_forward_reduce(sl1m_plan* p, const void* data, void* out, bool recs,
                                    hipStream_t st) {
  const int64_t slots = static_cast<int64_t>(p->wg_groups) * kWgVis;
  const int skip = wg_skipped_rows(p);
  const float2* rows = static_cast<const float2*>(fwd_rows1(p)) + skip * p->n_vis;
  const WgOut w{p->wg_order, static_cast<const float*>(p->vgain), static_cast<const float2*>(data),
                static_cast<float2*>(out), recs ? p->wg_res : nullptr};
  hipLaunchKernelGGL(k_wg_fwd_reduce, dim3(blocks1(slots)), dim3(kBlock), 0, st,
                     static_cast<const float2*>(p->fpart), p->wg_mrows, slots, rows,
                     forward_rows(p, 1) - skip, p->n_vis, w, recs ? rres_of(p) : nullptr,
                     static_cast<const float*>(p->layerDs), p->n_layers);
  return hipGetLastError();
}

bool wg_single(const sl1m_plan* p) {
  return p->wg_n == 1 && wg_all_pixels(p) && p->wg_segs[0].flat && p->wg_segs[0].macros == 1;
}
int wg_single_chunks(const sl1m_plan* p) { return flat_chunks(1, p->wg_groups); }

hipError_t launch_wg_adjoint_prep(sl1m_plan* p, const void* r, hipStream_t st) {
  const int64_t slots = static_cast<int64_t>(p->wg_groups) * kWgVis;
  hipLaunchKernelGGL(k_wg_adj_prep, dim3(blocks1(slots)), dim3(kBlock), 0, st,
                     static_cast<const float2*>(r), p->wg_order, slots, p->n_vis,
                     static_cast<const float*>(p->vgain), p->wg_res, rres_of(p),
                     static_cast<const float*>(p->layerDs), p->n_layers);
  return hipGetLastError();
}

hipError_t launch_wg_adjoint(sl1m_plan* p, const GridSeg& g, hipStream_t st) {
  const WgSeg& s = p->wg_segs[&g - p->grid_segs.data()];
  const int chunks = (s.flat ? flat_chunks : wg_chunks)(s.macros, p->wg_groups);
  const dim3 grid(static_cast<unsigned>(chunks), static_cast<unsigned>(s.macros));
  const int4* slot = reinterpret_cast<const int4*>(p->wg_slot) + s.cell0;
  const bool delta = g.kind == SL1M_PIX_DELTA;
  hipError_t e = timed(p, delta ? T_GRID_ADJ_DELTA : T_GRID_ADJ_GAUSS, st, [&] {
    if (s.flat) return launch_flat_adjoint(p, g, s, st);
    if (delta)
      hipLaunchKernelGGL(k_wg_adj, grid, dim3(kBlock), 0, st, p->wg_mac, s.mac0, p->wg_res,
                         p->wg_nu, p->wg_eta, p->wg_la, p->wg_mb, p->wg_su, p->wg_sv, p->wg_dw,
                         p->wg_w0, p->wg_h, p->wg_groups, s.cell0, s.cells, p->wg_part);
    else
      hipLaunchKernelGGL(k_wg_adj_gauss, grid, dim3(kBlock), 0, st, p->wg_mac, s.mac0, p->wg_res,
                         p->wg_nu, p->wg_eta, p->wg_la, p->wg_mb, p->wg_alpha, p->wg_beta,
                         p->wg_recg + static_cast<int64_t>(g.layer) * p->wg_groups * kWgVis,
                         p->wg_dw, p->wg_w0, p->wg_h, p->wg_groups, s.cell0, s.cells, p->wg_part);
    return hipGetLastError();
  });
  if (e != hipSuccess || wg_single(p)) return e;
  float* out = static_cast<float*>(p->apart);
  const dim3 rb(static_cast<unsigned>(s.cells / kRedCells));
  if (delta && !s.flat)
    hipLaunchKernelGGL(k_wg_adj_reduce<false>, rb, dim3(kBlock), 0, st,
                       p->wg_part, chunks, s.cells, slot, out);
  else
    hipLaunchKernelGGL(k_wg_adj_reduce<true>, rb, dim3(kBlock), 0, st,
                       p->wg_part, chunks, s.cells, slot, out);
  return hipGetLastError();
}

}  // namespace sl1m
