// Group evaluation of grid segments on the matrix cores (gfx950, float32
// plans, one right-hand side): tables and launchers.
//
// The grid evaluation (sl1m_grid.h) factorises an entry into A_k(l) B_k(m) C_k(nu).
// C, the only factor that is no product of an l and an m part, depends on the
// visibility through w alone.  So the visibilities are ordered by |w| (w < 0
// folded onto w > 0: a real image has V(-u,-v,-w) = conj V) and cut into groups
// of at most 64 of nearly one w:
//   C_k(a,b) = C_0(a,b) exp(-2 pi i dw_k nu(a,b)),  dw_k = w_k - w_0 small.
// C_0 is formed once per (group, cell), and what is left of the sum over the
// columns of a tile of cells (forward) or over the visibilities of the group
// (adjoint) is a matrix product of real phasor components, which the matrix
// cores take.  Inside a tile nu(a,b) = nuT + eta(a,b): the factor of nuT is
// exact per visibility, that of eta a short series, whose argument 2 pi dw eta
// the cut of the groups keeps below kWgX radians.
//
// Gaussian layers (the completed-square form of sl1m_grid.h): gamma = exp(2 pi i
// (C r^2 - w kappa)) leaves the part of exp(-2 pi i w kappa) that does not separate alone
// to the groups; the rest goes to the factors of l and m, which are complex pairs a+-,
// b+- with their tapers.
//
// The operands are float32 values split into two float16 (value = hi + lo to
// 2^-22 of it), each product as hi hi + hi lo + lo hi with float32 sums.
#pragma once

#include <algorithm>

#include "sl1m_internal.h"

namespace sl1m {

constexpr int kWgVis = 64;      // visibilities per group
constexpr int kWgRows = 16;     // |l| values of a tile
constexpr int kWgSteps = 2;     // steps of 16 |m| values of a tile
constexpr int kWgCols = 16 * kWgSteps;
constexpr int kWgCells = kWgRows * kWgCols;
// series argument limits (radians), by the terms kept: up to kWgXN the first
// order in one float16 product, up to kWgXM the second order too, up to kWgXW the
// first order split like the zeroth, up to kWgX the third order too.  A unit pixel
// at the phase centre (every entry 1; 32 x 32 x 2,000) comes out within 4.3e-7,
// with limits of 1.5e-3, 3e-3, 2e-2 within 1.3e-6.
constexpr float kWgXN = 1.2e-3f;
constexpr float kWgXM = 2.5e-3f;
constexpr float kWgXW = 1.5e-2f;
constexpr float kWgX = 5.0e-2f;
// Gaussian segments: no series up to kWgXZ, one order up to kWgXN.
constexpr float kWgXZ = 5.0e-7f;
// Segments that need no cell factor (sl1m_wflat.hip): tiles twice as wide; the largest
// |2 pi w eta| of one: one order up to kFlatN, two up to kFlatX, in one float16 product
// each.
constexpr int kFlatSteps = 4;
constexpr int kFlatCols = 16 * kFlatSteps;
constexpr int kFlatCells = kWgRows * kFlatCols;
constexpr float kFlatN = 6.0e-4f;
constexpr float kFlatX = 2.5e-3f;

// Up to four tiles (one per wavefront) of neighbouring rows over the same columns.
struct WgMacro {
  int32_t a_off, b_off;        // first row / column position in wg_la / wg_mb
  int32_t sets, steps;         // row sets (tiles) and column steps
  int32_t cell_off;            // first cell of the first tile (kWgCells per tile)
  float eta_max, nu_t[4];      // largest |eta|; each tile's nuT
  float xs;                    // 2 pi s, s the power of two that the macro's eta are divided by
  float m_lo, m_hi;            // column positions' range; each tile's row positions' range
  float l_lo[4], l_hi[4];
};

// What a Gaussian layer holds per slot: entry = D (1 + i s) exp(2 pi i (A l + B m + C r^2
// - w kappa + e0)) 2^(c1 ((u - w l)^2 + (v - w m)^2)), all of the folded coordinates.
struct alignas(16) WgVisG {
  double A, B, C;
  float u, v, w, c1;
  float e0, D, Ds, pad;
};

// Where a segment's macros and cells lie in the tables.
struct WgSeg {
  int32_t mac0, macros;
  int64_t cell0, cells;
  int32_t flat;                // evaluated without cell factors (sl1m_wflat.hip)
  float width;                 // largest eta over its series limit
};

// Host-built tables of grid segments, one after the other.  Tile cells are numbered
// column * kWgRows + row, kWgCells or (flat segments) kFlatCells of a tile.
struct WgPlan {
  std::vector<WgSeg> segs;
  std::vector<WgMacro> macros;
  std::vector<double> la, mb;      // row / column positions of the macros
  std::vector<double> nu;          // per tile cell: nu, or eta where alpha and beta serve
  std::vector<float> eta;          // per tile cell, divided by the macro's s (below 1)
  std::vector<double> alpha, beta; // separable part at the positions (0: none)
  std::vector<int32_t> slot;       // [4 per tile cell] permuted pixel or -1
};

// Visibility groups: `order` holds per slot (kWgVis per group) 2 k + (1 where
// w_k < 0), -1 where padded (at a group's end).
struct WgGroups {
  std::vector<int32_t> order;
  std::vector<double> w0;
  std::vector<float> h;            // largest |dw| of the group
  std::vector<int32_t> count;      // visibilities of the group
};

// The distinct values among v[0, n) (finite, not negative) in ascending order and the rank of
// each; false where there are more than `most`.
bool grid_axis(const double* v, int64_t n, int64_t most, std::vector<double>& values,
               std::vector<int32_t>& rank);
// How many of a plan's grid segments, from the first on, groups of n_vis visibilities take:
// consecutive segments whose tiles hold at most four times their cells with padding (four
// |m| values in 16 columns, 1023 x 7 pixels x 20,000 visibilities: forward 32 us, adjoint 57;
// grid evaluation 59 and 63).  A few thin strips are slower forward alone, two launches'
// latency against the grid evaluation's one (33 x 127 pixels x 2,000: 22 and 17 us, grid 19
// and 29).  The tables number cells, slots (2 k + sign) and the launches' macros in 32 bits or fewer:
// none from 2^30 visibilities on, no more than 2^31 - 1 cells and 65,535 macros.
int wg_segments(const GridSeg* segs, int n_segs, int64_t n_vis);
// macros and tile cells of a segment, the larger of both kinds of tiles
int wg_max_macros(const GridSeg& g);
int64_t wg_max_cells(const GridSeg& g);
int wg_flat_macros(const GridSeg& g);
// bytes of the segment's adjoint chunk sums, of at most max_groups groups
size_t wg_part_bytes(const GridSeg& g, int64_t max_groups);
// appends a segment; `c`: nu or kappa per grid cell, `w_max`: largest |w|
void wg_build_tiles(const GridSeg& g, const double* la, const double* mb, const double* c,
                    const int32_t* slot, double w_max, WgPlan& out);
bool wg_build_groups(const std::vector<double>& w, float width, int64_t max_groups,
                     WgGroups& out);
// The grid tables that the segments' offsets (GridSeg) point into.
struct WgGrids {
  const double *la, *mb, *nu, *kappa;
  const int32_t* slot;
};
// The tables of the first n segments and the groups of the visibilities; those of fewer
// segments (wg_fewer) where their width makes more than max_groups.  Returns how many.
int wg_build(const GridSeg* segs, int n, const WgGrids& in, const std::vector<double>& w,
             int64_t max_groups, WgPlan& plan, WgGroups& groups);
// A plan whose visibilities make too many groups for n of its segments (Gaussian layers
// take narrower ones) tries the first, a delta grid's, alone, then goes without.
int wg_fewer(const GridSeg& first, int n);
// groups a plan reserves room for
int64_t wg_group_cap(int64_t n_vis);
// group chunks (blocks per macro) of the operator kernels, at most wg_chunk_cap()
int wg_chunks(int macros, int groups);
int wg_chunk_cap(int macros);
int flat_chunks(int macros, int groups);
int flat_chunk_cap(int macros);

hipError_t launch_wg_setup(sl1m_plan* p, hipStream_t st);
hipError_t launch_wg_forward(sl1m_plan* p, const GridSeg& g, const void* xp, hipStream_t st);
// the forward reduction (launch_forward_reduce) of a plan with groups, one side
hipError_t launch_wg_forward_reduce(sl1m_plan* p, const void* data, void* out, bool adj_records,
                                    hipStream_t st);
// adjoint records of a plan with groups, one side (launch_adjoint_prep)
hipError_t launch_wg_adjoint_prep(sl1m_plan* p, const void* r, hipStream_t st);
// the segment's gradient sums into row 0 of the adjoint partials (its only row)
hipError_t launch_wg_adjoint(sl1m_plan* p, const GridSeg& g, hipStream_t st);

// A segment's forward in passes over its macros: `launch`(first macro, macros, their rows of
// sums [macro][group][visibility], whether an earlier pass has left sums there).
template <typename F>
hipError_t wg_passes(const sl1m_plan* p, const WgSeg& s, F&& launch) {
  hipError_t e = hipSuccess;
  for (int m = s.mac0, end = s.mac0 + s.macros; m < end && e == hipSuccess;) {
    const int row = m % p->wg_mrows, n = std::min(end - m, p->wg_mrows - row);
    float2* const rows = static_cast<float2*>(p->fpart) +
                         static_cast<int64_t>(row) * p->wg_groups * kWgVis;
    e = launch(m, n, rows, m >= p->wg_mrows);
    m += n;
  }
  return e;
}

// sl1m_wflat.hip: flat segments (the adjoint: its chunk sums)
hipError_t launch_flat_forward(sl1m_plan* p, const GridSeg& g, const WgSeg& s, const float* x,
                               hipStream_t st);
// wg_single: forward and reduction at once
hipError_t launch_flat_single(sl1m_plan* p, const void* x, const void* data, void* out,
                              bool adj_records, hipStream_t st);
hipError_t launch_flat_adjoint(sl1m_plan* p, const GridSeg& g, const WgSeg& s, hipStream_t st);

}  // namespace sl1m
