// Host tables of the group evaluation (sl1m_wgroup.h): tiles of the grids' cells, groups
// of the visibilities.  No device code.
#include <algorithm>
#include <cmath>
#include <cstring>

#include "sl1m_wgroup.h"

namespace sl1m {

// A hash of the bits instead of a sort of all values: a grid's axis has few (256 x 256
// pixels: 129 of 65,536; both axes 0.3 ms instead of 2.9, 16,384 scattered cells end after
// 1,281).
bool grid_axis(const double* v, int64_t n, int64_t most, std::vector<double>& values,
               std::vector<int32_t>& rank) {
  values.clear();
  rank.resize(n);
  int shift = 56;  // table of 2^(64 - shift)
  std::vector<int32_t> table(256, -1);
  // a free or its own place of x: from the product's top bits on
  auto find = [&](double x) -> int32_t& {
    uint64_t b;
    std::memcpy(&b, &x, sizeof(b));
    size_t h = (b ^ b >> 32) * 0x9E3779B97F4A7C15ull >> shift;
    while (table[h] >= 0 && values[table[h]] != x) h = (h + 1) & (table.size() - 1);
    return table[h];
  };
  double last = -1.0;
  int32_t id = -1;
  for (int64_t t = 0; t < n; ++t) {
    if (v[t] != last) {
      last = v[t];
      int32_t& place = find(last);
      id = place;
      if (id < 0) {
        if (static_cast<int64_t>(values.size()) >= most) return false;
        id = place = static_cast<int32_t>(values.size());
        values.push_back(last);
        if (2 * values.size() > table.size()) {
          shift -= 2;
          table.assign(4 * table.size(), -1);
          for (size_t i = 0; i < values.size(); ++i) find(values[i]) = static_cast<int32_t>(i);
        }
      }
    }
    rank[t] = id;
  }
  // first come, then ascending
  std::vector<int32_t> at(values.size()), to(values.size());
  for (size_t i = 0; i < at.size(); ++i) at[i] = static_cast<int32_t>(i);
  std::sort(at.begin(), at.end(), [&](int32_t i, int32_t j) { return values[i] < values[j]; });
  std::vector<double> sorted(values.size());
  for (size_t i = 0; i < at.size(); ++i) {
    sorted[i] = values[at[i]];
    to[at[i]] = static_cast<int32_t>(i);
  }
  values.swap(sorted);
  for (int32_t& r : rank) r = to[r];
  return true;
}

// Groups that hold few visibilities (sparse w, a wide field: the cut at kWgX ends
// them early) still cost C_0 and the float16 splits of every cell.  Measured on
// 256 x 256 pixels over +-0.3: 97,536 visibilities (1.19 times the full groups)
// take 0.66 of the grid evaluation's time, 20,000 (2.28 times) 0.98 of it forward
// and 1.17 adjoint; the line is drawn between.
int64_t wg_group_cap(int64_t n_vis) {
  const int64_t full = (n_vis + kWgVis - 1) / kWgVis;
  return full + full * 3 / 4 + 2;
}

// Blocks: two of 256 threads stay resident per compute unit (512 in all).  One round of
// them for few macros (each block loads its tiles' cells first, and the adjoint's chunk
// sums grow with the count), two for small grids, four for large ones, whose macros differ
// more in work.  Forward / adjoint in us at one, two (and four) rounds: 31 x 127 pixels x
// 20,000 visibilities (2 macros) 24.5 / 24.4, 27.5 / 29.7 (grid evaluation 24.5 / 41.4);
// 200 x 200 x 100,000 (8 macros) 152 / 165, 153 / 170; 256 x 256 x 100,000 (15) 268 / 294,
// 242 / 254; 1024 x 1024 x 409,600: 28.4 / 31.5 ms at two, 27.3 / 29.9 at four.
int wg_chunk_cap(int macros) {
  return std::max(1, (macros <= 8 ? 512 : macros <= 32 ? 1024 : 2048) / macros);
}
int wg_chunks(int macros, int groups) {
  return std::max(1, std::min(groups, wg_chunk_cap(macros)));
}

// Flat segments: one round of the blocks that stay resident (256 x 256 x 100,000: 210 /
// 293 us, two rounds 222 / 305; 300 x 300 Gaussian pixels x 100,003: 302 / 435, two
// rounds 316 / 446).
int flat_chunk_cap(int macros) { return std::max(1, 512 / macros); }
int flat_chunks(int macros, int groups) {
  return std::max(1, std::min(groups, flat_chunk_cap(macros)));
}

namespace {

// Macros and tile cells of a segment in tiles of up to `cs` column steps.
struct WgShape {
  int rsets, rmac, steps, cmac;
  bool lone;
  WgShape(const GridSeg& g, int cs)
      : rsets((g.na + kWgRows - 1) / kWgRows), rmac((rsets + 3) / 4), steps((g.nb + 15) / 16),
        cmac((steps + cs - 1) / cs), lone(cs == kWgSteps && rsets % 4 == 1 && rsets <= 9) {}
  // Evenly over the macros, but one set over (2^k pixels a side: 2^(k-1) + 1 |l| values)
  // has the last macro for itself, whose wavefronts share it, where that is much of the
  // grid: five sets 0.55 against 0.69 ms (128 x 128 Gaussian pixels x 409,600, forward),
  // nine sets 376 against 395 us (256 x 256 x 97,536); at 33 sets what the four form
  // each for themselves costs more (10.1 against 9.8 ms).  Flat segments form less and
  // are evaluated faster without (256 x 256 x 100,000: 210 against 217 us).
  int first_set(int ri) const {
    return lone ? std::min(4 * ri, rsets) : rsets * ri / rmac;
  }
  int macros() const { return rmac * cmac; }
  int64_t cells(int cs) const { return static_cast<int64_t>(rsets) * cmac * kWgRows * 16 * cs; }
};

// largest magnitude e as a power of two s: e / s in [1/2, 1), 1 for 0
double pow2_of(double e) {
  int ex = 0;
  (void)std::frexp(e, &ex);
  return e > 0.0 ? std::ldexp(1.0, ex) : 1.0;
}

// One segment's tables.  Flat segments and Gaussian ones: c = alpha(l) + beta(m) + eta,
// exact along the macro's middle row and column, each tile's eta centred by its rows'
// alpha (and nu holds eta); other delta segments, whose real factors of l and m have no
// place for alpha and beta: c = nu_t + eta.
// Row sets of kWgRows |l| values and column sets of up to `cs` steps of 16 |m| values,
// spread over the macros.
void append_segment(const GridSeg& g, const double* la, const double* mb, const double* c,
                    const int32_t* slot, bool flat, WgPlan& out) {
  const int na = g.na, nb = g.nb, cs = flat ? kFlatSteps : kWgSteps;
  const bool parts = flat || g.kind != SL1M_PIX_DELTA;
  const size_t tile = static_cast<size_t>(kWgRows) * 16 * cs;
  const WgShape sh(g, cs);
  WgSeg seg{};
  seg.mac0 = static_cast<int32_t>(out.macros.size());
  seg.cell0 = static_cast<int64_t>(out.nu.size());
  seg.flat = flat ? 1 : 0;
  double seg_eta = 0.0;
  auto cell = [&](int ia, int ib) {
    return (static_cast<int64_t>(ib / kGridNB) * na + ia) * kGridNB + ib % kGridNB;
  };
  for (int ri = 0; ri < sh.rmac; ++ri)
    for (int ci = 0; ci < sh.cmac; ++ci) {
      const int r0 = sh.first_set(ri), r1 = sh.first_set(ri + 1);
      const int s0 = sh.steps * ci / sh.cmac, s1 = sh.steps * (ci + 1) / sh.cmac;
      const int a0 = kWgRows * r0, a1 = std::min(kWgRows * r1, na);
      const int b0 = 16 * s0, b1 = std::min(16 * s1, nb);
      WgMacro m{};
      m.sets = r1 - r0;
      m.steps = s1 - s0;
      m.a_off = static_cast<int32_t>(out.la.size());
      m.b_off = static_cast<int32_t>(out.mb.size());
      m.cell_off = static_cast<int32_t>(out.nu.size());
      m.m_lo = static_cast<float>(mb[b0]);
      m.m_hi = static_cast<float>(mb[b1 - 1]);
      out.la.resize(out.la.size() + 4 * kWgRows, 0.0);
      out.alpha.resize(out.la.size(), 0.0);
      out.mb.resize(out.mb.size() + 16 * cs, 0.0);
      out.beta.resize(out.mb.size(), 0.0);
      double* const al = &out.alpha[m.a_off];
      double* const be = &out.beta[m.b_off];
      std::copy(la + a0, la + a1, &out.la[m.a_off]);
      std::copy(mb + b0, mb + b1, &out.mb[m.b_off]);
      if (parts) {
        const int ic = (a0 + a1) / 2, jc = (b0 + b1) / 2;
        for (int ia = a0; ia < a1; ++ia) al[ia - a0] = c[cell(ia, jc)] - c[cell(ic, jc)];
        for (int ib = b0; ib < b1; ++ib) be[ib - b0] = c[cell(ic, ib)];
      }
      double eta_max = 0.0;
      const size_t first = out.nu.size();
      out.nu.resize(first + m.sets * tile, 0.0);
      out.eta.resize(first + m.sets * tile, 0.0f);
      out.slot.resize(4 * (first + m.sets * tile), -1);
      std::vector<double> rest(m.sets * tile, 0.0);
      for (int w = 0; w < m.sets; ++w) {
        const int t0 = a0 + kWgRows * w, t1 = std::min(t0 + kWgRows, na);
        m.l_lo[w] = static_cast<float>(la[t0]);
        m.l_hi[w] = static_cast<float>(la[t1 - 1]);
        double lo = 1e300, hi = -1e300;
        for (int ib = b0; ib < b1; ++ib)
          for (int ia = t0; ia < t1; ++ia) {
            const double v = c[cell(ia, ib)] - al[ia - a0] - be[ib - b0];
            lo = std::min(lo, v);
            hi = std::max(hi, v);
          }
        // the tile's reference: in the rows' alpha, or as the kernels hold it (float32)
        double mid = 0.5 * (lo + hi);
        if (parts) {
          for (int ia = t0; ia < t1; ++ia) al[ia - a0] += mid;
          mid = 0.0;
        }
        m.nu_t[w] = static_cast<float>(mid);
        const double nt = static_cast<double>(m.nu_t[w]);
        for (int ib = b0; ib < b1; ++ib)
          for (int ia = t0; ia < t1; ++ia) {
            const int64_t q = cell(ia, ib);
            const size_t o = w * tile + static_cast<size_t>(ib - b0) * kWgRows + (ia - t0);
            rest[o] = c[q] - al[ia - a0] - be[ib - b0] - nt;
            out.nu[first + o] = parts ? rest[o] : c[q];
            eta_max = std::max(eta_max, std::fabs(rest[o]));
            for (int s = 0; s < 4; ++s) out.slot[4 * (first + o) + s] = slot[4 * q + s];
          }
      }
      // eta / s in [-1, 1] and x s (at most 2 kWgX) both lie in float16's range
      const double s = pow2_of(eta_max);
      for (size_t o = 0; o < rest.size(); ++o) out.eta[first + o] = static_cast<float>(rest[o] / s);
      m.xs = static_cast<float>(6.283185307179586 * s);
      m.eta_max = static_cast<float>(eta_max);
      seg_eta = std::max(seg_eta, eta_max);
      out.macros.push_back(m);
    }
  // a flat segment's groups may be of any width
  const float limit = g.kind == SL1M_PIX_DELTA ? kWgX : kWgXN;
  seg.width = flat ? 0.0f : static_cast<float>(seg_eta) / limit;
  seg.macros = static_cast<int32_t>(out.macros.size()) - seg.mac0;
  seg.cells = static_cast<int64_t>(out.nu.size()) - seg.cell0;
  out.segs.push_back(seg);
}

// Largest |eta| of the segment's flat tables.
double flat_eta(const GridSeg& g, const double* c) {
  const WgShape sh(g, kFlatSteps);
  auto at = [&](int ia, int ib) {
    return c[(static_cast<int64_t>(ib / kGridNB) * g.na + ia) * kGridNB + ib % kGridNB];
  };
  double top = 0.0;
  for (int ri = 0; ri < sh.rmac; ++ri)
    for (int ci = 0; ci < sh.cmac; ++ci) {
      const int a0 = kWgRows * sh.first_set(ri), b0 = 16 * (sh.steps * ci / sh.cmac);
      const int a1 = std::min(kWgRows * sh.first_set(ri + 1), g.na);
      const int b1 = std::min(16 * (sh.steps * (ci + 1) / sh.cmac), g.nb);
      const int ic = (a0 + a1) / 2, jc = (b0 + b1) / 2;
      for (int t0 = a0; t0 < a1; t0 += kWgRows) {
        const int t1 = std::min(t0 + kWgRows, a1);
        double lo = 1e300, hi = -1e300;
        for (int ib = b0; ib < b1; ++ib)
          for (int ia = t0; ia < t1; ++ia) {
            const double v = at(ia, ib) - (at(ia, jc) - at(ic, jc)) - at(ic, ib);
            lo = std::min(lo, v);
            hi = std::max(hi, v);
          }
        top = std::max(top, 0.5 * (hi - lo));
      }
    }
  return top;
}

}  // namespace

int wg_flat_macros(const GridSeg& g) { return WgShape(g, kFlatSteps).macros(); }

int wg_max_macros(const GridSeg& g) { return WgShape(g, kWgSteps).macros(); }

int64_t wg_max_cells(const GridSeg& g) {
  return std::max(WgShape(g, kWgSteps).cells(kWgSteps), WgShape(g, kFlatSteps).cells(kFlatSteps));
}

int wg_segments(const GridSeg* segs, int n_segs, int64_t n_vis) {
  if (n_vis >= int64_t{1} << 30) return 0;
  int64_t cells = 0, macros = 0;
  int n = 0;
  for (; n < n_segs; ++n) {
    const GridSeg& g = segs[n];
    const int64_t sets = (g.na + kWgRows - 1) / kWgRows, steps = (g.nb + 15) / 16;
    if (g.seg != segs[0].seg + n || 16 * kWgRows * sets * steps > int64_t{4} * g.na * g.nb) break;
    cells += wg_max_cells(g);
    macros += wg_max_macros(g);
    if (cells > INT32_MAX || macros > 65535) break;
  }
  return n;
}

size_t wg_part_bytes(const GridSeg& g, int64_t max_groups) {
  const WgShape a(g, kWgSteps), b(g, kFlatSteps);
  const int most = static_cast<int>(max_groups);
  return sizeof(float4) * std::max(a.cells(kWgSteps) * wg_chunks(a.macros(), most),
                                   b.cells(kFlatSteps) * flat_chunks(b.macros(), most));
}

void wg_build_tiles(const GridSeg& g, const double* la, const double* mb, const double* c,
                    const int32_t* slot, double w_max, WgPlan& out) {
  // Without cell factors where the series allows it: 1.9 times faster (disk baselines of
  // |w| < 250 over +-0.05, sl1m_wflat.hip), and closer: fewer phasors are rounded.
  const bool flat = 6.2831854 * w_max * flat_eta(g, c) <= 0.999 * kFlatX;
  append_segment(g, la, mb, c, slot, flat, out);
}

bool wg_build_groups(const std::vector<double>& w, float width, int64_t max_groups,
                     WgGroups& out) {
  const int64_t n = static_cast<int64_t>(w.size());
  double wm = 0.0;
  for (double x : w) {
    if (!std::isfinite(x)) return false;
    wm = std::max(wm, std::fabs(x));
  }
  if (wm >= 0x1.0p27) return false;  // phases below 2^27 turns (|nu| < 1): kMagicFine
  // order by |w| in 2^20 bins (two stable counting passes of 10 bits over (bin, index)
  // pairs); equal bins keep the caller's order
  const double scale = wm > 1e-290 ? 1048575.0 / wm : 0.0;
  std::vector<uint64_t> a(n), b(n);
  uint32_t at[2][1024] = {};
  for (int64_t k = 0; k < n; ++k) {
    const uint32_t key = static_cast<uint32_t>(std::fabs(w[k]) * scale);
    a[k] = static_cast<uint64_t>(key) << 32 | static_cast<uint32_t>(k);
    ++at[0][key & 1023u];
    ++at[1][key >> 10];
  }
  for (int pass = 0; pass < 2; ++pass) {
    uint32_t first = 0;
    for (uint32_t& c : at[pass]) {
      const uint32_t count = c;
      c = first;
      first += count;
    }
    const int sh = 32 + 10 * pass;
    for (int64_t i = 0; i < n; ++i) b[at[pass][(a[i] >> sh) & 1023u]++] = a[i];
    a.swap(b);
  }
  const double hmax = width > 0.0f ? 1.0 / (6.283185307179586 * width) : 1e300;
  const int64_t least = (n + kWgVis - 1) / kWgVis;
  out.order.reserve(kWgVis * least);
  out.w0.reserve(least);
  out.h.reserve(least);
  out.count.reserve(least);
  for (int64_t i = 0; i < n;) {
    if (static_cast<int64_t>(out.w0.size()) >= max_groups) return false;
    const size_t o = out.order.size();
    out.order.resize(o + kWgVis, -1);
    double lo = 1e300, hi = 0.0;
    int64_t j = i;
    for (const int64_t end = std::min(n, i + kWgVis); j < end; ++j) {
      const int32_t k = static_cast<int32_t>(static_cast<uint32_t>(a[j]));
      const double x = std::fabs(w[k]);
      const double l2 = std::min(lo, x), h2 = std::max(hi, x);
      if (j > i && h2 - l2 > 2.0 * hmax) break;
      lo = l2;
      hi = h2;
      out.order[o + (j - i)] = 2 * k + (w[k] < 0.0 ? 1 : 0);
    }
    out.w0.push_back(0.5 * (lo + hi));
    out.h.push_back(static_cast<float>(0.5 * (hi - lo)));
    out.count.push_back(static_cast<int32_t>(j - i));
    i = j;
  }
  return true;
}

int wg_fewer(const GridSeg& first, int n) {
  return n > 1 && first.kind == SL1M_PIX_DELTA ? 1 : 0;
}

namespace {

// Cuts the tables to the first n segments.
void keep_segments(WgPlan& t, int n) {
  if (n >= static_cast<int>(t.segs.size())) return;
  const int32_t mac0 = t.segs[n].mac0;
  const WgMacro m = t.macros[mac0];
  t.segs.resize(n);
  t.macros.resize(mac0);
  t.la.resize(m.a_off);
  t.alpha.resize(m.a_off);
  t.mb.resize(m.b_off);
  t.beta.resize(m.b_off);
  t.nu.resize(m.cell_off);
  t.eta.resize(m.cell_off);
  t.slot.resize(4 * static_cast<size_t>(m.cell_off));
}

}  // namespace

int wg_build(const GridSeg* segs, int n, const WgGrids& in, const std::vector<double>& w,
             int64_t max_groups, WgPlan& plan, WgGroups& groups) {
  double w_max = 0.0;
  for (double x : w) w_max = std::max(w_max, std::fabs(x));
  for (int i = 0; i < n; ++i) {
    const GridSeg& g = segs[i];
    wg_build_tiles(g, in.la + g.la_off, in.mb + g.mb_off,
                   (g.kind == SL1M_PIX_DELTA ? in.nu : in.kappa) + g.cell_off,
                   in.slot + 4 * g.cell_off, w_max, plan);
  }
  while (n) {
    groups = WgGroups();
    float width = 0.0f;
    for (int i = 0; i < n; ++i) width = std::max(width, plan.segs[i].width);
    if (wg_build_groups(w, width, max_groups, groups)) break;
    n = wg_fewer(segs[0], n);
    keep_segments(plan, n);
  }
  return n;
}

}  // namespace sl1m
