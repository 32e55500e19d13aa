// CPU checks of the group evaluation's host tables (sl1m_wgtables.hip).  Built and run by
// tests/test_groups_host.py with g++ (address/undefined sanitizers).
//
// stdin: segments, then per segment kind, |l| x |m| pixels, spacing; visibilities, their w.
// stdout: the segments kept and the groups; per kept segment whether it is evaluated
// without cell factors and how many (macro, group) pairs fall into each series class.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <random>

#include "sl1m_wgroup.h"

using namespace sl1m;

#define CHECK(c)                                                      \
  do {                                                                \
    if (!(c)) {                                                       \
      std::fprintf(stderr, "check failed at %d: %s\n", __LINE__, #c); \
      std::exit(1);                                                   \
    }                                                                 \
  } while (0)

struct Grids {
  std::vector<GridSeg> segs;
  std::vector<double> la, mb, nu, kappa;
  std::vector<int32_t> slot;
  WgGrids in() const { return {la.data(), mb.data(), nu.data(), kappa.data(), slot.data()}; }
};

// The |l|, |m| values of a centred grid of nl x nm pixels, cells as sl1m_api.hip lays them out.
static void add_segment(Grids& t, int kind, int nl, int nm, double d) {
  GridSeg g{};
  g.seg = static_cast<int32_t>(t.segs.size());
  g.kind = kind;
  g.na = nl / 2 + 1;
  g.nb = nm / 2 + 1;
  g.ng = (g.nb + kGridNB - 1) / kGridNB;
  g.cells = static_cast<int64_t>(g.ng) * kGridNB * g.na;
  g.la_off = static_cast<int64_t>(t.la.size());
  g.mb_off = static_cast<int64_t>(t.mb.size());
  g.cell_off = static_cast<int64_t>(t.nu.size());
  for (int i = 0; i < g.na; ++i) t.la.push_back(i * d);
  for (int i = 0; i < g.ng * kGridNB; ++i) t.mb.push_back(i < g.nb ? i * d : 0.0);
  t.nu.resize(g.cell_off + g.cells, 0.0);
  t.kappa.resize(g.cell_off + g.cells, 0.0);
  t.slot.resize(4 * (g.cell_off + g.cells), -1);
  for (int ib = 0; ib < g.nb; ++ib)
    for (int ia = 0; ia < g.na; ++ia) {
      const int64_t q = g.cell_off + (static_cast<int64_t>(ib / kGridNB) * g.na + ia) * kGridNB + ib % kGridNB;
      const double r2 = (ia * d) * (ia * d) + (ib * d) * (ib * d), n = std::sqrt(1.0 - r2);
      t.nu[q] = -r2 / (1.0 + n);
      if (kind == SL1M_PIX_GAUSS_WIDE) t.kappa[q] = -(r2 * r2) / (2.0 * (1.0 + n) * (1.0 + n));
      for (int s = 0; s < 4; ++s) t.slot[4 * q + s] = static_cast<int32_t>(4 * q + s);
    }
  t.segs.push_back(g);
}

// The limits of wg_segments: 32-bit slots, launch sizes, padding.
static void segment_checks() {
  auto seg = [](int na, int nb) {
    GridSeg g{};
    g.na = na;
    g.nb = nb;
    return g;
  };
  const int64_t most = (int64_t{1} << 30) - 1;
  const GridSeg small = seg(17, 17);
  CHECK(wg_segments(&small, 1, 1) == 1 && wg_segments(&small, 1, most) == 1);
  CHECK(wg_segments(&small, 1, most + 1) == 0 && wg_segments(&small, 1, INT32_MAX) == 0);
  // the slots of the most groups a plan of that many visibilities may have
  CHECK(wg_group_cap(most) * kWgVis <= INT32_MAX && 2 * (most - 1) + 1 <= INT32_MAX);
  // macros: 4 row sets x 32 columns each
  const GridSeg fits = seg(64, 32 * 65535), more = seg(64, 32 * 65535 + 1);
  CHECK(wg_segments(&fits, 1, 1000) == 1 && wg_segments(&more, 1, 1000) == 0);
  // a segment past the limit ends the run, and so does one that does not follow
  GridSeg three[3] = {small, more, small};
  three[1].seg = 1;
  three[2].seg = 2;
  CHECK(wg_segments(three, 3, 1000) == 1);
  three[1] = small;
  three[1].seg = 2;
  CHECK(wg_segments(three, 2, 1000) == 1);
  three[1].seg = 1;
  CHECK(wg_segments(three, 3, 1000) == 3);
  // padding: four columns of 16 fill a quarter, three do not
  const GridSeg four = seg(512, 4), three_c = seg(512, 3);
  CHECK(wg_segments(&four, 1, 1000) == 1 && wg_segments(&three_c, 1, 1000) == 0);
}

// grid_axis against a sort, at its limit and past it.
static void axis_checks() {
  std::mt19937 rng(3);
  for (int n : {0, 1, 2, 100, 5000})
    for (int distinct : {1, 2, 17, 130, 1000, 100000}) {
      std::vector<double> v(n);
      for (double& x : v) x = 1e-4 * static_cast<double>(rng() % distinct);
      if (n > 1) v[n / 2] = 1e-310;  // subnormal
      std::vector<double> want(v), got;
      std::sort(want.begin(), want.end());
      want.erase(std::unique(want.begin(), want.end()), want.end());
      std::vector<int32_t> rank;
      const int64_t most = static_cast<int64_t>(want.size());
      CHECK(grid_axis(v.data(), n, most, got, rank) && got == want);
      for (int t = 0; t < n; ++t) CHECK(got[rank[t]] == v[t]);
      if (n > 0) CHECK(!grid_axis(v.data(), n, most - 1, got, rank));
    }
}

int main() {
  segment_checks();
  axis_checks();
  int n = 0;
  CHECK(std::scanf("%d", &n) == 1);
  Grids t;
  for (int i = 0; i < n; ++i) {
    int kind, nl, nm;
    double d;
    CHECK(std::scanf("%d %d %d %lf", &kind, &nl, &nm, &d) == 4);
    add_segment(t, kind, nl, nm, d);
  }
  long nv = 0;
  CHECK(std::scanf("%ld", &nv) == 1);
  std::vector<double> w(nv);
  for (double& x : w) CHECK(std::scanf("%lf", &x) == 1);

  WgPlan p;
  WgGroups g;
  const int64_t cap = wg_group_cap(nv);
  const int kept = wg_build(t.segs.data(), n, t.in(), w, cap, p, g);
  std::printf("kept %d groups %zu\n", kept, kept ? g.w0.size() : size_t{0});

  // the tables hold the kept segments only and fit what a plan reserves for those
  size_t macros = 0, cells = 0;
  for (int i = 0; i < kept; ++i) {
    macros += static_cast<size_t>(wg_max_macros(t.segs[i]));
    cells += static_cast<size_t>(wg_max_cells(t.segs[i]));
  }
  CHECK(p.segs.size() == static_cast<size_t>(kept));
  CHECK(p.macros.size() <= macros && p.nu.size() <= cells && p.eta.size() == p.nu.size());
  CHECK(p.slot.size() == 4 * p.nu.size());
  CHECK(p.la.size() == 4 * kWgRows * p.macros.size() && p.alpha.size() == p.la.size());
  CHECK(p.mb.size() <= kFlatCols * macros && p.beta.size() == p.mb.size());
  // and are what building them alone gives
  WgPlan alone;
  double w_max = 0.0;
  for (double x : w) w_max = std::max(w_max, std::fabs(x));
  for (int i = 0; i < kept; ++i) {
    const GridSeg& s = t.segs[i];
    wg_build_tiles(s, t.la.data() + s.la_off, t.mb.data() + s.mb_off,
                   (s.kind == SL1M_PIX_DELTA ? t.nu : t.kappa).data() + s.cell_off,
                   t.slot.data() + 4 * s.cell_off, w_max, alone);
  }
  CHECK(alone.la == p.la && alone.mb == p.mb && alone.nu == p.nu && alone.eta == p.eta &&
        alone.slot == p.slot && alone.alpha == p.alpha && alone.beta == p.beta);
  if (!kept) return 0;

  // every visibility once, its group's w near its own
  CHECK(static_cast<int64_t>(g.w0.size()) <= cap);
  std::vector<char> seen(nv, 0);
  for (size_t i = 0; i < g.order.size(); ++i) {
    const int32_t o = g.order[i];
    const bool pad = static_cast<int>(i % kWgVis) >= g.count[i / kWgVis];
    CHECK(pad == (o < 0));
    if (o < 0) continue;
    CHECK(o / 2 < nv && !seen[o / 2] && (o % 2 == 1) == (w[o / 2] < 0.0));
    seen[o / 2] = 1;
    CHECK(std::fabs(std::fabs(w[o / 2]) - g.w0[i / kWgVis]) <= g.h[i / kWgVis] * (1.0 + 1e-6) + 1e-300);
  }
  for (char s : seen) CHECK(s);

  for (int i = 0; i < kept; ++i) {
    const WgSeg& s = p.segs[i];
    long cls[4] = {0, 0, 0, 0};
    for (int m = s.mac0; m < s.mac0 + s.macros; ++m)
      for (size_t k = 0; k < g.w0.size(); ++k) {
        const double tau = 6.283185307179586 * p.macros[m].eta_max;
        if (s.flat) {
          const double x = tau * (g.w0[k] + g.h[k]);
          CHECK(x <= kFlatX);
          ++cls[x <= kWgXZ ? 0 : x <= kFlatN ? 1 : 2];
        } else if (t.segs[i].kind == SL1M_PIX_DELTA) {
          const double x = tau * g.h[k];
          CHECK(x <= kWgX * 1.001);
          ++cls[x <= kWgXN ? 0 : x <= kWgXM ? 1 : x <= kWgXW ? 2 : 3];
        } else {
          const double x = tau * g.h[k];
          CHECK(x <= kWgXN * 1.001);
          ++cls[x <= kWgXZ ? 0 : 1];
        }
      }
    std::printf("segment %d flat %d classes %ld %ld %ld %ld\n", i, s.flat, cls[0], cls[1], cls[2], cls[3]);
  }
  return 0;
}
