// Flat segments of the group evaluation (sl1m_wgroup.h): no cell factors.
//
// Inside a macro, f(l, m) (nu, or kappa of a Gaussian layer) is alpha(l) + beta(m) + eta
// with eta = 0 along one row and one column, the mixed rest elsewhere.  exp(-2 pi i w
// alpha) and exp(-2 pi i w beta) go to the factors of l and m, and where |2 pi w eta|
// stays below kFlatX for every baseline a series of at most two terms in it is all that
// is left of the cells: their operands are the amplitudes themselves, real and the same
// for every group.  With a+- = t+- exp(2 pi i (+- A|l| + C l^2 - w alpha)) per visibility
// and row (t the taper, 1 for delta pixels) and b+- the same per column,
//   V = sum_a (a+ D+ + a- D-), D+ = sum_b (b+ x0 + b- x2), D- = sum_b (b+ x1 + b- x3),
//   gradient of slot (sa, sb) = sum_k Re(conj(a_sa) rho conj(b_sb)),
// half the products of the tiles with cell factors (Gaussian layers) and none of their
// phasors and splits, which leaves the rows' and columns' phasors as the main cost: the
// tiles are 64 columns wide, since a row's phasors serve all of them (at 32 columns the
// forward below takes 253 us, the adjoint 368).  Vector instructions and products do not
// overlap much at two wavefronts per SIMD, all that the operands' registers allow.
//
// 256 x 256 pixels over +-0.05, 100,000 visibilities: forward 210 us, adjoint 293 (grid
// evaluation 598, 667); 300 x 300 Gaussian pixels, 100,003: 302 and 435 us (tiles with
// cell factors 469, 540; grid evaluation 1333, 1528).
#include <algorithm>

#include "sl1m_wgroup_dev.h"

namespace sl1m {
namespace {

using namespace dev;

// A visibility as the kernels take it.
struct FlatVis {
  double A, B, C, w;
  float x;                           // 2 pi s w
  float u, v, wf, c1, e0, D, Ds;     // Gaussian
};

template <bool GAUSS>
struct FlatIn {
  const double* __restrict__ su;
  const double* __restrict__ sv;
  const WgVisG* __restrict__ rec;
  const double* __restrict__ sw;
  const float* __restrict__ sdw;
  const double* __restrict__ w0s;
  const float* __restrict__ hs;
  const int32_t* __restrict__ cnt;

  __device__ __forceinline__ FlatVis load(int g, int lane, float xs) const {
    FlatVis r = {};
    const int64_t t = static_cast<int64_t>(g) * kWgVis + lane;
    // The groups may be of any width: delta pixels take w itself (w n may be hundreds of
    // turns over the field, and float32 of w - w0 5e-5 rad off).  For Gaussian pixels what
    // is left to w, kappa, is below a turn, and the sum needs no second register.
    r.w = GAUSS ? as_const(w0s)[g] + static_cast<double>(sdw[t]) : sw[t];
    r.x = xs * static_cast<float>(r.w);
    if constexpr (GAUSS) {
      const WgVisG q = rec[t];
      r.A = q.A;
      r.B = q.B;
      r.C = q.C;
      r.u = q.u;
      r.v = q.v;
      r.wf = q.w;
      r.c1 = q.c1;
      r.e0 = q.e0;
      r.D = q.D;
      r.Ds = q.Ds;
    } else {
      r.A = -su[t];
      r.B = -sv[t];
    }
    return r;
  }
  // largest |w| of the group times 2 pi eta_max
  __device__ __forceinline__ int ser(int g, float eta_max) const {
    const float xm = kTwoPi * (static_cast<float>(as_const(w0s)[g]) + as_const(hs)[g]) * eta_max;
    return xm <= kWgXZ ? 0 : xm <= kFlatN ? 1 : 2;
  }
};

// exp(2 pi i (+- A l + C l^2 - w alpha))
template <bool GAUSS>
__device__ __forceinline__ void flat_phasors(double A, double C, double w, double l, double al,
                                             float& pc, float& ps, float& mc, float& ms) {
  double q = -w * al;  // kMagic comes last: one rounding to its grid
  if constexpr (GAUSS) q = fma(C, l * l, q);
  phasor(fma(A, l, q) + kMagic, pc, ps);
  phasor(fma(-A, l, q) + kMagic, mc, ms);
}

// b+ and b- of one column and visibility, (re, im) each
template <bool GAUSS>
__device__ __forceinline__ void flat_column(const FlatVis& r, double m, double be, float top,
                                            float (&re)[2], float (&im)[2]) {
  flat_phasors<GAUSS>(r.B, r.C, r.w, m, be, re[0], im[0], re[1], im[1]);
  if constexpr (GAUSS) {
    const float mr = static_cast<float>(m);
    const float tp = taper(r.c1, fmaf(-r.wf, mr, r.v), top, kGUp);
    const float tm = taper(r.c1, fmaf(r.wf, mr, r.v), top, kGUp);
    re[0] *= tp;
    im[0] *= tp;
    re[1] *= tm;
    im[1] *= tm;
  }
}

// ---------------------------------------------------------------------------
// forward
// ---------------------------------------------------------------------------

template <bool GAUSS>
struct alignas(16) FlatFwdLds {
  uint4 col[kFlatSteps * 4 * 4 * 64];  // [step, quarter][re hi, lo, im hi, lo][visibility]
  double la[4 * kWgRows], al[4 * kWgRows], mb[kFlatCols], be[kFlatCols];
  double A[kWgVis], w[kWgVis], C[GAUSS ? kWgVis : 1];
  float4 uw[GAUSS ? kWgVis : 1];     // u, w, c1, -
  float x[kWgVis];
  float2 red[4][kWgVis];
};

struct FlatRows {  // amplitude operands [row sign][step]: hi, lo, eta times
  Op8 h[2][kFlatSteps], l[2][kFlatSteps], e[2][kFlatSteps];
  h2_t eta[kFlatSteps][2];
};

// One step of 16 columns for one tile of 16 visibilities.
template <int SER>
__device__ __forceinline__ void flat_step(const FlatRows& a, int s, const uint4* __restrict__ q,
                                          f4_t (&d)[4], f4_t (&d1)[4], f4_t (&d2)[4]) {
  const h8_t bh[2] = {as_h8(q[0]), as_h8(q[128])}, bl[2] = {as_h8(q[64]), as_h8(q[192])};
#pragma unroll
  for (int i = 0; i < 4; ++i) d[i] = mma(a.h[i / 2][s].vec(), bh[i % 2], d[i]);
  if constexpr (SER > 0) {
#pragma unroll
    for (int i = 0; i < 4; ++i) d1[i] = mma(a.e[i / 2][s].vec(), bh[i % 2], d1[i]);
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) d[i] = mma(a.h[i / 2][s].vec(), bl[i % 2], d[i]);
  if constexpr (SER > 1) {
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      Op8 e2;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const _Float16 t = a.eta[s][j / 2][j % 2];
        e2.v[j] = a.e[k][s].v[j] * h2_t{t, t};
      }
#pragma unroll
      for (int o = 0; o < 2; ++o) d2[2 * k + o] = mma(e2.vec(), bh[o], d2[2 * k + o]);
    }
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) d[i] = mma(a.l[i / 2][s].vec(), bh[i % 2], d[i]);
}

// Sums over the columns for one tile of 16 visibilities (D+ re, im, D- re, im), series
// included.
template <int SER>
__device__ __forceinline__ void flat_sums(const FlatRows& a, const uint4* __restrict__ col,
                                          int steps, float x, f4_t (&d)[4]) {
  f4_t d1[4], d2[4];
#pragma unroll
  for (int o = 0; o < 4; ++o) d[o] = d1[o] = d2[o] = f4_t{0, 0, 0, 0};
  flat_step<SER>(a, 0, col, d, d1, d2);
#pragma unroll
  for (int s = 1; s < kFlatSteps; ++s)
    if (s < steps) flat_step<SER>(a, s, col + s * 4 * 4 * 64, d, d1, d2);
  if constexpr (SER > 0) {
    const float h = -0.5f * x * x;
#pragma unroll
    for (int k = 0; k < 4; k += 2)
#pragma unroll
      for (int i = 0; i < 4; ++i) {  // exp(-i x eta) = 1 - i x eta - (x eta)^2 / 2
        d[k][i] = fmaf(x, d1[k + 1][i], d[k][i]);
        d[k + 1][i] = fmaf(-x, d1[k][i], d[k + 1][i]);
        if constexpr (SER > 1) {
          d[k][i] = fmaf(h, d2[k][i], d[k][i]);
          d[k + 1][i] = fmaf(h, d2[k + 1][i], d[k + 1][i]);
        }
      }
  }
}

template <bool GAUSS>
__global__ __launch_bounds__(kBlock, 2) void k_flat_fwd(
    const WgMacro* __restrict__ macros, int mac0, const float* __restrict__ xp,
    const float* __restrict__ pscale, const int4* __restrict__ slot,
    const float* __restrict__ eta, const double* __restrict__ la, const double* __restrict__ mb,
    const double* __restrict__ alpha, const double* __restrict__ beta, FlatIn<GAUSS> in,
    int n_groups, WgOut fin, bool add, float2* __restrict__ rows) {
  __shared__ FlatFwdLds<GAUSS> lds;
  const int mac = mac0 + static_cast<int>(blockIdx.y);
  const ConstPtr<WgMacro> cm = as_const(macros) + mac;
  const int g0 = static_cast<int>(blockIdx.x), gs = static_cast<int>(gridDim.x);
  const int sets = cm->sets, steps = cm->steps;
  const float eta_max = cm->eta_max, xs = cm->xs, m_lo = cm->m_lo, m_hi = cm->m_hi;
  const int tid = threadIdx.x, lane = tid & 63, r16 = lane & 15, quad = lane >> 4;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  // one or two row sets: the wavefronts share a set's visibility tiles (the operands are
  // loaded once, so nothing is formed twice)
  const int set = sets == 1 ? 0 : sets == 2 ? wv >> 1 : wv;
  const int t_lo = sets == 1 ? wv : sets == 2 ? 2 * (wv & 1) : 0;
  const int t_hi = sets == 1 ? wv + 1 : sets == 2 ? t_lo + 2 : 4;
  const bool active = set < sets;
  const int64_t cell0 = cm->cell_off + static_cast<int64_t>(active ? set : 0) * kFlatCells;
  FlatVis rn = in.load(g0, lane, xs);
  int sn = in.ser(g0, eta_max), cn = as_const(in.cnt)[g0];
  if (tid < 4 * kWgRows) {
    lds.la[tid] = la[cm->a_off + tid];
    lds.al[tid] = alpha[cm->a_off + tid];
  }
  if (tid < kFlatCols) {
    lds.mb[tid] = mb[cm->b_off + tid];
    lds.be[tid] = beta[cm->b_off + tid];
  }
  // this lane's row, four columns of every step: amplitude operands, times the power
  // of two that brings the tile's largest into [2^13, 2^14)
  float e[kFlatSteps][4][4], et[kFlatSteps][4], mx = 0.0f;
#pragma unroll
  for (int s = 0; s < kFlatSteps; ++s)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int64_t o = cell0 + (16 * s + 4 * quad + j) * kWgRows + r16;
      et[s][j] = eta[o];
      const int4 q = slot[o];
      const float x0 = q.x >= 0 ? xp[q.x] * pscale[q.x] : 0.0f;
      const float x1 = q.y >= 0 ? xp[q.y] * pscale[q.y] : 0.0f;
      const float x2 = q.z >= 0 ? xp[q.z] * pscale[q.z] : 0.0f;
      const float x3 = q.w >= 0 ? xp[q.w] * pscale[q.w] : 0.0f;
      const float m = fmaxf(fmaxf(fabsf(x0), fabsf(x1)), fmaxf(fabsf(x2), fabsf(x3)));
      const float sum = (x0 + x1) + (x2 + x3);
      mx = fmaxf(mx, sum != sum ? __builtin_inff() : m);  // fmaxf drops a NaN
      e[s][j][0] = x0;
      e[s][j][1] = x2;
      e[s][j][2] = x1;
      e[s][j][3] = x3;
    }
  const float c = op_scale(wave_max(mx)), sc = 1.0f / c;
  FlatRows a;
#pragma unroll
  for (int s = 0; s < kFlatSteps; ++s)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float t = et[s][j];
      a.eta[s][j / 2][j % 2] = static_cast<_Float16>(t);
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const float p = c * e[s][j][2 * k], q = c * e[s][j][2 * k + 1];
        split2(p, q, a.h[k][s].v[j], a.l[k][s].v[j]);
        a.e[k][s].v[j] = __builtin_convertvector((f2_t{t * p, t * q}), h2_t);
      }
    }
  __syncthreads();
  for (int g = g0; g < n_groups; g += gs) {
    const FlatVis r = rn;
    const int ser = sn, nt = (cn + 15) >> 4;
    if (wv == 0) {
      lds.A[lane] = r.A;
      lds.w[lane] = r.w;
      lds.x[lane] = r.x;
      if constexpr (GAUSS) {
        lds.C[lane] = r.C;
        lds.uw[lane] = make_float4(r.u, r.wf, r.c1, 0.0f);
      }
    }
    const int gn = g + gs < n_groups ? g + gs : g;
    rn = in.load(gn, lane, xs);
    sn = in.ser(gn, eta_max);
    cn = as_const(in.cnt)[gn];
    const float top = GAUSS ? taper_top(r.c1, r.v, r.wf, m_lo, m_hi) : 0.0f;
    for (int un = wv; un < 4 * steps; un += 4) {
      uint4 o[4];
      uint32_t* const po = reinterpret_cast<uint32_t*>(o);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        float re[2], im[2];
        flat_column<GAUSS>(r, lds.mb[4 * un + j], lds.be[4 * un + j], top, re, im);
        h2_t hi, lo;
        split2(re[0], re[1], hi, lo);
        po[j] = as_u32(hi);
        po[4 + j] = as_u32(lo);
        split2(im[0], im[1], hi, lo);
        po[8 + j] = as_u32(hi);
        po[12 + j] = as_u32(lo);
      }
      uint4* dst = lds.col + un * 4 * 64 + lane;
#pragma unroll
      for (int q = 0; q < 4; ++q) dst[64 * q] = o[q];
    }
    __syncthreads();
    float re = 0.0f, im = 0.0f;
    if (active) {
      float sr = 0.0f, si = 0.0f;
#pragma unroll 1
      for (int t = t_lo; t < (nt < t_hi ? nt : t_hi); ++t) {
        const int v = 16 * t + r16;
        const uint4* col = lds.col + quad * 4 * 64 + v;
        f4_t d[4];
        if (ser == 0)
          flat_sums<0>(a, col, steps, 0.0f, d);
        else if (ser == 1)
          flat_sums<1>(a, col, steps, lds.x[v], d);
        else
          flat_sums<2>(a, col, steps, lds.x[v], d);
        const double A = lds.A[v], w = lds.w[v], C = GAUSS ? lds.C[GAUSS ? v : 0] : 0.0;
        float vr = 0.0f, vi = 0.0f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int row = set * kWgRows + quad * 4 + i;
          const double l = lds.la[row];
          float pc, ps, mc, ms;
          flat_phasors<GAUSS>(A, C, w, l, lds.al[row], pc, ps, mc, ms);
          if constexpr (GAUSS) {
            const float4 uw = lds.uw[v];
            const float lr = static_cast<float>(l);
            const float du = fmaf(-uw.y, lr, uw.x), dv = fmaf(uw.y, lr, uw.x);
            const float tp = pow2(uw.z * (du * du)), tm = pow2(uw.z * (dv * dv));
            pc *= tp;
            ps *= tp;
            mc *= tm;
            ms *= tm;
          }
          vr = fmaf(pc, d[0][i], fmaf(-ps, d[1][i], vr));
          vi = fmaf(pc, d[1][i], fmaf(ps, d[0][i], vi));
          vr = fmaf(mc, d[2][i], fmaf(-ms, d[3][i], vr));
          vi = fmaf(mc, d[3][i], fmaf(ms, d[2][i], vi));
        }
        vr += __shfl_xor(vr, 16, 64);
        vi += __shfl_xor(vi, 16, 64);
        vr += __shfl_xor(vr, 32, 64);
        vi += __shfl_xor(vi, 32, 64);
        sr = quad == t ? vr : sr;
        si = quad == t ? vi : si;
      }
      if constexpr (GAUSS) {
        const float ct = __builtin_amdgcn_cosf(r.e0), st = __builtin_amdgcn_sinf(r.e0);
        const float k = scale_sums(sc * kGDown, sr, si) * pow2(top);
        const float fr = k * fmaf(r.D, ct, -r.Ds * st), fi = k * fmaf(r.D, st, r.Ds * ct);
        re = fmaf(fr, sr, -fi * si);
        im = fmaf(fr, si, fi * sr);
      } else {
        re = sc * sr;
        im = sc * si;
      }
    }
    lds.red[wv][lane] = make_float2(re, im);
    __syncthreads();
    if (tid < kWgVis) {
      const float2 p = lds.red[0][tid], q = lds.red[1][tid], u = lds.red[2][tid],
                   v = lds.red[3][tid];
      float2 sum = make_float2((p.x + q.x) + (u.x + v.x), (p.y + q.y) + (u.y + v.y));
      const int64_t slot_g = static_cast<int64_t>(g) * kWgVis + tid;
      if (fin.order) {  // the plan's only macro: nothing to add up
        const int32_t o = fin.order[slot_g];
        if (o & 1) sum.y = -sum.y;
        float gr, gi;
        if (o >= 0)
          (void)wg_finish(fin, slot_g, o, sum, gr, gi);
        else if (fin.res)
          fin.res[slot_g] = make_float2(0.0f, 0.0f);
      } else {
        store_row(rows, static_cast<int64_t>(blockIdx.y) * n_groups * kWgVis + slot_g, add, sum);
      }
    }
  }
}

// ---------------------------------------------------------------------------
// adjoint
// ---------------------------------------------------------------------------

constexpr int kFlatPitch = 68;  // uint32 (visibilities) per column of an operand, padded

template <bool GAUSS>
struct alignas(16) FlatAdjLds {
  uint32_t col[2][2][kFlatCols][kFlatPitch];  // [b+, b-][hi, lo][column][visibility]: (re, im)
  double la[4 * kWgRows], al[4 * kWgRows], mb[kFlatCols], be[kFlatCols];
  double A[kWgVis], w[kWgVis], C[GAUSS ? kWgVis : 1];
  float4 uw[GAUSS ? kWgVis : 1];            // u, w, c1, -
  uint32_t x[kWgVis];                       // (x, x) in float16
  float2 rho[4][kWgVis];
  float top[GAUSS ? 4 : 1][kWgVis];
  float mx[4];
};

// One row sign of a group: G (two column signs) += the products' sums, the series in eta
// applied; two column tiles at a time (registers).  `h`, `l`: row operands of 4 x 16
// visibilities, (re, im) each; `b`: this lane's column operand.
template <int SER>
__device__ __forceinline__ void flat_adj_rows(const Op8 (&h)[4], const Op8 (&l)[4],
                                              const uint4* __restrict__ b,
                                              const uint4* __restrict__ x,
                                              const h2_t (&eta)[kFlatSteps][2], int steps,
                                              f4_t (&g0)[kFlatSteps], f4_t (&g1)[kFlatSteps]) {
  constexpr int kPart = kFlatCols * kFlatPitch / 4, kTile = 16 * kFlatPitch / 4;
  Op8 e[4], e2[4];
  if constexpr (SER > 0) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const Op8 xk = __builtin_bit_cast(Op8, as_h8(x[4 * k]));
#pragma unroll
      for (int j = 0; j < 4; ++j) {  // i x (re, im), -x^2 / 2 (re, im)
        e[k].v[j] = h2_t{-h[k].v[j][1], h[k].v[j][0]} * xk.v[j];
        if constexpr (SER > 1)
          e2[k].v[j] = h2_t{e[k].v[j][1], -e[k].v[j][0]} * (xk.v[j] * static_cast<_Float16>(-0.5f));
      }
    }
  }
#pragma unroll
  for (int cs = 0; cs < 2 * kFlatSteps; cs += 2) {  // column sign, two tiles
    const int sign = cs / kFlatSteps, c0 = cs % kFlatSteps;
    if (c0 >= steps) continue;
    f4_t t0[2], t1[2], t2[2];
#pragma unroll
    for (int c = 0; c < 2; ++c) t0[c] = t1[c] = t2[c] = f4_t{0, 0, 0, 0};
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
      for (int c = 0; c < 2; ++c) {  // a tile past `steps`: leftovers that no pixel reads
        const uint4* q = b + 4 * k + (c0 + c) * kTile + 2 * sign * kPart;
        const h8_t bh = as_h8(q[0]), bl = as_h8(q[kPart]);
        t0[c] = mma(h[k].vec(), bh, t0[c]);
        if constexpr (SER > 0) t1[c] = mma(e[k].vec(), bh, t1[c]);
        t0[c] = mma(h[k].vec(), bl, t0[c]);
        if constexpr (SER > 1) t2[c] = mma(e2[k].vec(), bh, t2[c]);
        t0[c] = mma(l[k].vec(), bh, t0[c]);
      }
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        float z = (sign ? g1[c0 + c][i] : g0[c0 + c][i]) + t0[c][i];
        if constexpr (SER > 0) {
          const float et = static_cast<float>(eta[c0 + c][i / 2][i % 2]);
          float y = t1[c][i];
          if constexpr (SER > 1) y = fmaf(et, t2[c][i], y);
          z = fmaf(et, y, z);
        }
        asm volatile("" : "+v"(z));  // formed here: the products' sums are not kept open
        (sign ? g1 : g0)[c0 + c][i] = z;
      }
  }
}

template <bool GAUSS>
__global__ __launch_bounds__(kBlock, 2) void k_flat_adj(
    const WgMacro* __restrict__ macros, int mac0, const float2* __restrict__ res,
    const float* __restrict__ eta, const double* __restrict__ la, const double* __restrict__ mb,
    const double* __restrict__ alpha, const double* __restrict__ beta, FlatIn<GAUSS> in,
    int n_groups, int64_t cbase, int64_t cells, float4* __restrict__ part) {
  __shared__ FlatAdjLds<GAUSS> lds;
  const ConstPtr<WgMacro> cm = as_const(macros) + mac0 + static_cast<int>(blockIdx.y);
  const int g0 = static_cast<int>(blockIdx.x), gs = static_cast<int>(gridDim.x);
  const int sets = cm->sets, steps = cm->steps;
  const float eta_max = cm->eta_max, xs = cm->xs, m_lo = cm->m_lo, m_hi = cm->m_hi;
  const int tid = threadIdx.x, lane = tid & 63, r16 = lane & 15, quad = lane >> 4;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool active = wv < sets;
  const float l_lo = cm->l_lo[wv], l_hi = cm->l_hi[wv];
  const int64_t cell0 = cm->cell_off + static_cast<int64_t>(active ? wv : 0) * kFlatCells;
  if (tid < 4 * kWgRows) {
    lds.la[tid] = la[cm->a_off + tid];
    lds.al[tid] = alpha[cm->a_off + tid];
  }
  if (tid < kFlatCols) {
    lds.mb[tid] = mb[cm->b_off + tid];
    lds.be[tid] = beta[cm->b_off + tid];
  }
  // One scale for the operands of the block's groups, of the residuals times their largest
  // taper (Gaussian; the wavefronts share the pass, over the rows of the whole macro).  Where
  // every baseline is tapered a scale of the bare residuals left the operands below float16's
  // range: relative errors of the gradient of 7e-6 at tapers of 2^-20, 0.05 at 2^-33.  (A
  // scale per group, folded into the sums, spills: 300 x 300 pixels x 100,003 550 us.)
  float mx = 0.0f;
  for (int g = g0 + wv * gs; g < n_groups; g += 4 * gs) {
    float2 z = res[static_cast<int64_t>(g) * kWgVis + lane];
    if constexpr (GAUSS) {
      const WgVisG* const q = in.rec + static_cast<int64_t>(g) * kWgVis + lane;
      const float k = pow2(taper_top(q->c1, q->v, q->w, m_lo, m_hi) +
                           taper_top(q->c1, q->u, q->w, cm->l_lo[0], cm->l_hi[sets - 1]));
      z.x *= k;  // |D (1 + i s)| <= 1
      z.y *= k;
    }
    const float m = fmaxf(fabsf(z.x), fabsf(z.y));
    mx = fmaxf(mx, z.x != z.x || z.y != z.y ? __builtin_inff() : m);
  }
  mx = wave_max(mx);
  if (lane == 0) lds.mx[wv] = mx;
  f4_t gr[4][kFlatSteps];
  h2_t et[kFlatSteps][2];
#pragma unroll
  for (int c = 0; c < kFlatSteps; ++c)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      gr[i][c] = f4_t{0, 0, 0, 0};
      et[c][i / 2][i % 2] = static_cast<_Float16>(eta[cell0 + (16 * c + r16) * kWgRows + quad * 4 + i]);
    }
  FlatVis rn = {};
  float2 zn = make_float2(0.0f, 0.0f);
  int sn = 0;
  if (g0 < n_groups) {
    rn = in.load(g0, lane, xs);
    zn = res[static_cast<int64_t>(g0) * kWgVis + lane];
    sn = in.ser(g0, eta_max);
  }
  __syncthreads();
  const float sc =
      0.5f * op_scale(fmaxf(fmaxf(lds.mx[0], lds.mx[1]), fmaxf(lds.mx[2], lds.mx[3])));
  for (int g = g0; g < n_groups; g += gs) {
    const FlatVis r = rn;
    const int ser = sn;
    const float top = GAUSS ? taper_top(r.c1, r.v, r.wf, m_lo, m_hi) : 0.0f;
    float2 z = zn;
    if constexpr (GAUSS) {
      // times conj D (1 + i s) exp(2 pi i e0), with both tops
      const float ltop = taper_top(r.c1, r.u, r.wf, l_lo, l_hi), k = pow2(top + ltop);
      const float c0 = __builtin_amdgcn_cosf(r.e0), s0 = __builtin_amdgcn_sinf(r.e0);
      const float ct = k * fmaf(r.D, c0, -r.Ds * s0), st = k * fmaf(r.D, s0, r.Ds * c0);
      const float zr = z.x;
      z.x = fmaf(ct, zr, st * z.y);
      z.y = fmaf(ct, z.y, -st * zr);
      lds.top[GAUSS ? wv : 0][lane] = ltop;
    }
    lds.rho[wv][lane] = make_float2(sc * z.x, sc * z.y);
    if (wv == 0) {
      lds.A[lane] = r.A;
      lds.w[lane] = r.w;
      lds.x[lane] = as_u32(__builtin_convertvector((f2_t{r.x, r.x}), h2_t));
      if constexpr (GAUSS) {
        lds.C[lane] = r.C;
        lds.uw[lane] = make_float4(r.u, r.wf, r.c1, 0.0f);
      }
    }
    const int gn = g + gs < n_groups ? g + gs : g;
    rn = in.load(gn, lane, xs);
    zn = res[static_cast<int64_t>(gn) * kWgVis + lane];
    sn = in.ser(gn, eta_max);
    for (int c = wv; c < 16 * steps; c += 4) {
      float re[2], im[2];
      flat_column<GAUSS>(r, lds.mb[c], lds.be[c], top, re, im);
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        h2_t hi, lo;
        split2(re[q], im[q], hi, lo);
        lds.col[q][0][c][lane] = as_u32(hi);
        lds.col[q][1][c][lane] = as_u32(lo);
      }
    }
    __syncthreads();
    if (active) {
      const int row = wv * kWgRows + r16;
      const double l = lds.la[row], al = lds.al[row];
      const float lr = static_cast<float>(l);
      const uint4* b = reinterpret_cast<const uint4*>(&lds.col[0][0][r16][4 * quad]);
      const uint4* x = reinterpret_cast<const uint4*>(&lds.x[4 * quad]);
#pragma unroll
      for (int s = 0; s < 2; ++s) {  // row signs
        Op8 h[4], lo[4];             // conj(a+-) rho of this lane's row, 16 visibilities
#pragma unroll
        for (int kb = 0; kb < 4; ++kb)
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const int v = 16 * kb + 4 * quad + j;
            double q = -lds.w[v] * al;
            if constexpr (GAUSS) q = fma(lds.C[GAUSS ? v : 0], l * l, q);
            float pc, ps;
            phasor(fma(s ? -lds.A[v] : lds.A[v], l, q) + kMagic, pc, ps);
            const float2 z = lds.rho[wv][v];
            float yr = fmaf(pc, z.x, ps * z.y), yi = fmaf(pc, z.y, -ps * z.x);
            if constexpr (GAUSS) {
              const float4 uw = lds.uw[v];
              const float t = taper(uw.z, fmaf(s ? uw.y : -uw.y, lr, uw.x),
                                    lds.top[GAUSS ? wv : 0][v], 1.0f);
              yr *= t;
              yi *= t;
            }
            split2(yr, yi, h[kb].v[j], lo[kb].v[j]);
          }
        if (ser == 0)
          flat_adj_rows<0>(h, lo, b, x, et, steps, gr[s], gr[2 + s]);
        else if (ser == 1)
          flat_adj_rows<1>(h, lo, b, x, et, steps, gr[s], gr[2 + s]);
        else
          flat_adj_rows<2>(h, lo, b, x, et, steps, gr[s], gr[2 + s]);
      }
    }
    __syncthreads();
  }
  if (!active) return;
  const float inv = GAUSS ? kGDown / sc : 1.0f / sc;
#pragma unroll
  for (int c = 0; c < kFlatSteps; ++c)
#pragma unroll
    for (int i = 0; i < 4; ++i)
      part[blockIdx.x * cells + cell0 - cbase + (16 * c + r16) * kWgRows + quad * 4 + i] =
          make_float4(inv * gr[0][c][i], inv * gr[1][c][i], inv * gr[2][c][i], inv * gr[3][c][i]);
}

}  // namespace

template <bool GAUSS>
static FlatIn<GAUSS> flat_in(const sl1m_plan* p, const GridSeg& g) {
  FlatIn<GAUSS> in;
  in.su = p->wg_su;
  in.sv = p->wg_sv;
  in.rec = GAUSS ? p->wg_recg + static_cast<int64_t>(g.layer) * p->wg_groups * kWgVis : nullptr;
  in.sw = p->wg_sw;
  in.sdw = p->wg_dw;
  in.w0s = p->wg_w0;
  in.hs = p->wg_h;
  in.cnt = p->wg_count;
  return in;
}

template <bool GAUSS>
static hipError_t flat_forward_t(sl1m_plan* p, const GridSeg& g, const WgSeg& s, const float* x,
                                 const WgOut& fin, hipStream_t st) {
  return wg_passes(p, s, [&](int mac0, int macros, float2* rows, bool add) {
    const dim3 grid(static_cast<unsigned>(flat_chunks(macros, p->wg_groups)),
                    static_cast<unsigned>(macros));
    hipLaunchKernelGGL(k_flat_fwd<GAUSS>, grid, dim3(kBlock), 0, st, p->wg_mac, mac0, x,
                       static_cast<const float*>(p->pscale),
                       reinterpret_cast<const int4*>(p->wg_slot), p->wg_eta, p->wg_la, p->wg_mb,
                       p->wg_alpha, p->wg_beta, flat_in<GAUSS>(p, g), p->wg_groups, fin, add,
                       rows);
    return hipGetLastError();
  });
}

hipError_t launch_flat_forward(sl1m_plan* p, const GridSeg& g, const WgSeg& s, const float* x,
                                  hipStream_t st) {
  const WgOut none{};
  return g.kind == SL1M_PIX_DELTA ? flat_forward_t<false>(p, g, s, x, none, st)
                                  : flat_forward_t<true>(p, g, s, x, none, st);
}

hipError_t launch_flat_single(sl1m_plan* p, const void* x, const void* data, void* out, bool recs,
                              hipStream_t st) {
  const GridSeg& g = p->grid_segs[0];
  const bool delta = g.kind == SL1M_PIX_DELTA;
  const WgOut fin{p->wg_order, static_cast<const float*>(p->vgain), static_cast<const float2*>(data),
                  static_cast<float2*>(out), recs ? p->wg_res : nullptr};
  const float* xf = static_cast<const float*>(x);
  return timed(p, delta ? T_GRID_FWD_DELTA : T_GRID_FWD_GAUSS, st, [&] {
    return delta ? flat_forward_t<false>(p, g, p->wg_segs[0], xf, fin, st)
                 : flat_forward_t<true>(p, g, p->wg_segs[0], xf, fin, st);
  });
}

template <bool GAUSS>
static hipError_t flat_adjoint_t(sl1m_plan* p, const GridSeg& g, const WgSeg& s, hipStream_t st) {
  const dim3 grid(static_cast<unsigned>(flat_chunks(s.macros, p->wg_groups)),
                  static_cast<unsigned>(s.macros));
  hipLaunchKernelGGL(k_flat_adj<GAUSS>, grid, dim3(kBlock), 0, st, p->wg_mac, s.mac0,
                     p->wg_res, p->wg_eta, p->wg_la, p->wg_mb, p->wg_alpha, p->wg_beta,
                     flat_in<GAUSS>(p, g), p->wg_groups, s.cell0, s.cells, p->wg_part);
  return hipGetLastError();
}

hipError_t launch_flat_adjoint(sl1m_plan* p, const GridSeg& g, const WgSeg& s, hipStream_t st) {
  return g.kind == SL1M_PIX_DELTA ? flat_adjoint_t<false>(p, g, s, st)
                                  : flat_adjoint_t<true>(p, g, s, st);
}

}  // namespace sl1m
