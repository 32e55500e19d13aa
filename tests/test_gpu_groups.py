"""Group evaluation of grids (visibilities in groups of nearly one w, the sums on
the matrix cores): operators against the FP64 oracle at the FP32 operator tolerance and
the element-wise bound (tests/elementwise.py), at the sizes where its tiles (16 |l|
values by 32 |m| values, 64 without cell factors, four tiles to a block), its groups (64
visibilities, tiles of 16) and its series (argument classes set by the spread of w in a
group, or by the largest w) end.

A plan of one side takes it, a plan of two sides the grid evaluation for the same calls,
so results that differ in their bits show that it ran.
"""
import ctypes

import numpy as np
import pytest
import torch

import elementwise as E
import oracle as O
from paper_1310_2078_amd import sl1m
from paper_1310_2078_amd import workloads as W

pytestmark = pytest.mark.gpu

TOL = 1e-5


def rel(a, b):
    return float(np.linalg.norm(np.asarray(a) - np.asarray(b)) / np.linalg.norm(np.asarray(b)))


def _grid(nl, nm, d):
    L, M = np.meshgrid((np.arange(nl) - nl // 2) * d, (np.arange(nm) - nm // 2) * d)
    return L.ravel(), M.ravel()


# name: |l| x |m| pixels, spacing, visibilities, w spread, gains, pixels kept (fraction)
CASES = {
    "one_group": (40, 40, 2e-3, 64, 1.0, False, 1.0),          # a full group, narrow
    "one_more": (40, 40, 2e-3, 65, 1.0, False, 1.0),           # and a group of one
    "odd_17_tiles": (33, 33, 2e-3, 1023, 2.0, False, 1.0),     # 17 x 17 cells: padded tiles
    "exact_tiles": (63, 127, 1e-3, 3200, 5.0, True, 1.0),      # 32 x 64 cells: no padding
    "columns_129": (40, 256, 1e-3, 2500, 10.0, False, 1.0),    # nine steps, a lone one
    "rows_five_sets": (150, 34, 1.5e-3, 2111, 10.0, True, 1.0),
    "wide_field": (48, 48, 6e-3, 6000, 30.0, True, 1.0),       # split first order, groups cut
    "third_order": (40, 40, 6e-3, 3001, 40.0, False, 1.0),
    "w_zero": (36, 36, 2e-3, 1500, 0.0, False, 1.0),           # one w: no series
    "many_groups": (40, 40, 4e-3, 30000, 30.0, False, 1.0),    # cell factors, one order
    "flat_65": (129, 129, 1e-3, 500, 20.0, True, 1.0),         # 65 x 65 cells, one order
    "flat_two_orders": (150, 34, 1.5e-3, 700, 150.0, False, 1.0),
    "flat_one_visibility": (40, 40, 2e-3, 1, 1.0, False, 1.0),
    "cut_off": (70, 70, 1e-3, 2700, 20.0, True, 0.55),         # truncated mid-row, shuffled
}


def _case(name):
    nl, nm, d, nv, ws, gains, keep = CASES[name]
    seed = 40 + sorted(CASES).index(name)
    wl = W.small_random(seed, 10, nv, uv_radius=700.0, w_sigma=ws, with_gains=gains)
    l, m = _grid(nl, nm, d)
    rng = np.random.default_rng(seed)
    if keep < 1.0:
        n = int(keep * l.size)
        sel = rng.permutation(n)
        l, m = l[:n][sel], m[:n][sel]
    wl.l, wl.m = l, m
    wl.sigma, wl.kind = np.zeros(l.size), np.zeros(l.size, np.uint8)
    wl.x_true = None
    x = rng.standard_normal(l.size)
    r = rng.standard_normal(nv) + 1j * rng.standard_normal(nv)
    return wl, x, r


@pytest.mark.parametrize("name", list(CASES))
def test_group_operators(name):
    print(f"[case] groups {name}", flush=True)
    wl, x, r = _case(name)
    p = O.Problem.from_workload(wl)
    Vo, go = O.forward(p, x), O.adjoint(p, r)
    plan = sl1m.Plan.from_workload(wl)
    other = sl1m.Plan.from_workload(wl, max_rhs=2, grid="require")
    V, g = plan.forward(x).cpu().numpy(), plan.adjoint(r).cpu().numpy()
    V2, g2 = other.forward(x).cpu().numpy(), other.adjoint(r).cpu().numpy()
    wf = E.worst_ratio(V, Vo, E.abs_forward_rows(p, x), wl.n_pix)
    wa = E.worst_ratio(g, go, E.abs_adjoint_cols(p, r), wl.n_vis)
    print(f"    forward {rel(V, Vo):.3e} adjoint {rel(g, go):.3e} element-wise {wf:.3e} {wa:.3e} "
          f"grid evaluation {rel(V2, Vo):.3e} {rel(g2, go):.3e}", flush=True)
    assert not np.array_equal(V, V2) and not np.array_equal(g, g2), "the groups did not run"
    assert rel(V, Vo) <= TOL and rel(g, go) <= TOL
    assert wf <= 1.0 and wa <= 1.0
    # the same bits again, whatever ran in between
    plan.forward(2.0 * x), plan.adjoint(r.conj())
    assert np.array_equal(plan.forward(x).cpu().numpy(), V)
    assert np.array_equal(plan.adjoint(r).cpu().numpy(), g)


def test_scales_zeros_and_non_finite():
    """Operands far from 1 are scaled by powers of two, exactly; zero inputs give zero;
    a NaN reaches every output."""
    wl, x, r = _case("odd_17_tiles")
    plan = sl1m.Plan.from_workload(wl)
    V, g = plan.forward(x).cpu().numpy(), plan.adjoint(r).cpu().numpy()
    for s in (2.0 ** -60, 2.0 ** 60):
        assert np.array_equal(plan.forward(x * s).cpu().numpy(), V * np.float32(s))
        assert np.array_equal(plan.adjoint(r * s).cpu().numpy(), g * np.float32(s))
    assert not plan.forward(0 * x).cpu().numpy().any()
    assert not plan.adjoint(0 * r).cpu().numpy().any()
    x[5] = np.nan
    r[7] = np.nan
    assert not np.isfinite(plan.forward(x).cpu().numpy()).any()
    assert not np.isfinite(plan.adjoint(r).cpu().numpy()).any()


@pytest.mark.parametrize("name", ["many_groups", "odd_17_tiles"])
def test_amplitudes_near_the_largest_float(name):
    """One pixel or one visibility of 2^120 (exact: powers of two) and of 2^126."""
    wl, x, r = _case(name)
    plan = sl1m.Plan.from_workload(wl)
    x, r = 0 * x, 0 * r
    x[7], r[9] = 1.0, 1.0
    for f, v in ((plan.forward, x), (plan.adjoint, r)):
        a, b = f(v).cpu().numpy(), f(v * 2.0 ** 120).cpu().numpy()
        assert np.array_equal(b, a * np.float32(2.0 ** 120))
        c = f(v * 2.0 ** 126).cpu().numpy()
        assert np.isfinite(c).all() and rel(c / np.float32(2.0 ** 126), a) <= TOL


# name: |l| x |m| pixels, spacing, sigma (spacings), kind, visibilities, w spread, with a
# delta grid of twice the resolution
GAUSS = {
    "no_series": (40, 40, 1e-3, 2.0, W.PIX_GAUSS_WIDE, 1000, 5.0, False),
    "paraxial_odd": (33, 35, 2e-3, 1.0, W.PIX_GAUSS_PARAXIAL, 65, 20.0, False),
    "one_order": (64, 130, 4e-3, 1.0, W.PIX_GAUSS_WIDE, 2047, 12.0, False),
    "flat_two_orders": (64, 130, 4e-3, 1.0, W.PIX_GAUSS_WIDE, 700, 1.0, False),
    "wide": (48, 48, 1.2e-2, 0.5, W.PIX_GAUSS_WIDE, 2500, 40.0, False),
    "layer_and_delta": (34, 40, 8e-3, 1.0, W.PIX_GAUSS_WIDE, 3001, 60.0, True),
    "steep_taper": (40, 40, 5e-3, 3.0, W.PIX_GAUSS_WIDE, 1500, 60.0, False),
}


def _gauss_case(name):
    nl, nm, d, sig, kind, nv, ws, delta = GAUSS[name]
    seed = 70 + sorted(GAUSS).index(name)
    wl = W.small_random(seed, 10, nv, uv_radius=300.0, w_sigma=ws, with_gains=True)
    l, m = _grid(nl, nm, d)
    wl.sigma, wl.kind = np.full(l.size, sig * d), np.full(l.size, kind, np.uint8)
    if delta:
        l2, m2 = _grid(2 * nl, 2 * nm, d / 2)
        wl.sigma = np.concatenate([np.zeros(l2.size), wl.sigma])
        wl.kind = np.concatenate([np.zeros(l2.size, np.uint8), wl.kind])
        l, m = np.concatenate([l2, l]), np.concatenate([m2, m])
    wl.l, wl.m, wl.x_true = l, m, None
    rng = np.random.default_rng(seed)
    return wl, rng.standard_normal(l.size), (rng.standard_normal(nv)
                                             + 1j * rng.standard_normal(nv))


@pytest.mark.parametrize("name", list(GAUSS))
def test_group_gaussians(name):
    print(f"[case] gaussian groups {name}", flush=True)
    wl, x, r = _gauss_case(name)
    p = O.Problem.from_workload(wl)
    Vo, go = O.forward(p, x), O.adjoint(p, r)
    plan = sl1m.Plan.from_workload(wl)
    V, g = plan.forward(x).cpu().numpy(), plan.adjoint(r).cpu().numpy()
    wf = E.worst_ratio(V, Vo, E.abs_forward_rows(p, x), wl.n_pix)
    wa = E.worst_ratio(g, go, E.abs_adjoint_cols(p, r), wl.n_vis)
    print(f"    forward {rel(V, Vo):.3e} adjoint {rel(g, go):.3e} element-wise {wf:.3e} {wa:.3e}",
          flush=True)
    assert rel(V, Vo) <= TOL and rel(g, go) <= TOL
    assert wf <= 1.0 and wa <= 1.0
    # one pixel, far from the largest taper of its tile: its entries alone
    j = wl.n_pix - 1
    e = np.zeros(wl.n_pix)
    e[j] = 1.0
    V1, Vo1 = plan.forward(e).cpu().numpy(), O.forward(p, e)
    assert rel(V1, Vo1) <= TOL
    # the same bits again; a NaN reaches every output
    assert np.array_equal(plan.forward(x).cpu().numpy(), V)
    assert np.array_equal(plan.adjoint(r).cpu().numpy(), g)
    x[-1], r[-1] = np.nan, np.nan
    assert not np.isfinite(plan.forward(x).cpu().numpy()).any()
    assert not np.isfinite(plan.adjoint(r).cpu().numpy()[wl.kind != 0]).any()


# name: delta pixels a side, spacing, pixels a side and spacing of a wide Gaussian layer
# around them (sigma one spacing), visibilities, w spread; segments in groups, those without
# cell factors (bits)
LAYERS = {
    "both": (40, 5e-3, 96, 0.5 / 96, 6000, 60.0, 2, 0),
    "both_delta_flat": (40, 2.5e-3, 96, 0.5 / 96, 3000, 6.0, 2, 1),
    "delta_alone": (40, 5e-3, 96, 0.5 / 96, 3000, 60.0, 1, 0),       # too many groups for both
    "delta_alone_flat": (40, 2.5e-3, 96, 0.5 / 96, 3000, 100.0, 1, 1),
}


def _layer_case(name):
    dn, dd, gn, gd, nv, ws = LAYERS[name][:6]
    seed = 90 + sorted(LAYERS).index(name)
    wl = W.small_random(seed, 10, nv, uv_radius=200.0, w_sigma=ws, with_gains=True)
    l, m = _grid(dn, dn, dd)
    l2, m2 = _grid(gn, gn, gd)
    wl.l, wl.m, wl.x_true = np.concatenate([l, l2]), np.concatenate([m, m2]), None
    wl.sigma = np.concatenate([np.zeros(l.size), np.full(l2.size, gd)])
    wl.kind = np.concatenate([np.zeros(l.size, np.uint8),
                              np.full(l2.size, W.PIX_GAUSS_WIDE, np.uint8)])
    rng = np.random.default_rng(seed)
    return wl, rng.standard_normal(wl.l.size), (rng.standard_normal(nv)
                                                + 1j * rng.standard_normal(nv))


@pytest.mark.parametrize("name", list(LAYERS))
def test_delta_grid_inside_a_layer(name):
    """Both segments in groups, or the delta grid alone beside the layer's grid evaluation."""
    print(f"[case] groups and layers {name}", flush=True)
    wl, x, r = _layer_case(name)
    p = O.Problem.from_workload(wl)
    Vo, go = O.forward(p, x), O.adjoint(p, r)
    plan = sl1m.Plan.from_workload(wl)
    info = plan.info()
    assert (info["grid"], info["grid_groups"], info["grid_flat"]) == (2, *LAYERS[name][6:])
    V, g = plan.forward(x).cpu().numpy(), plan.adjoint(r).cpu().numpy()
    wf = E.worst_ratio(V, Vo, E.abs_forward_rows(p, x), wl.n_pix)
    wa = E.worst_ratio(g, go, E.abs_adjoint_cols(p, r), wl.n_vis)
    print(f"    forward {rel(V, Vo):.3e} adjoint {rel(g, go):.3e} element-wise {wf:.3e} {wa:.3e}",
          flush=True)
    assert rel(V, Vo) <= TOL and wf <= 1.0 and wa <= 1.0
    for k in (0, W.PIX_GAUSS_WIDE):       # the pixels of either kind on their own
        assert rel(g[wl.kind == k], go[wl.kind == k]) <= TOL
    r[-1] = np.nan
    assert not np.isfinite(plan.adjoint(r).cpu().numpy()).any()


@pytest.mark.parametrize("name", list(GAUSS))
def test_gaussian_cases_evaluation(name):
    """Which evaluation the Gaussian cases take: all but two whose visibilities make too many
    groups for any segment take the groups, with cell factors where the series asks for them."""
    plan = sl1m.Plan.from_workload(_gauss_case(name)[0])
    info = plan.info()
    want = {"no_series": (1, 1), "paraxial_odd": (1, 1), "one_order": (1, 0),
            "flat_two_orders": (1, 1), "steep_taper": (1, 0)}.get(name, (0, 0))
    assert (info["grid_groups"], info["grid_flat"]) == want


@pytest.mark.parametrize("reach", [0.5, 2.1, 2.4, 2.7, 3.0, 3.3])
def test_gaussian_baselines_all_tapered(reach):
    """Every visibility on long baselines (sigma |(u, v)| = reach, tapers of 2^-1 to 2^-49),
    w = 0: no cell factors.  The adjoint keeps the forward's relative accuracy."""
    print(f"[case] tapered ring {reach}", flush=True)
    d, nv = 1.5e-3, 700
    rng = np.random.default_rng(120)
    wl = W.small_random(120, 10, nv, with_gains=True)
    wl.l, wl.m = _grid(40, 70, d)
    wl.sigma, wl.kind = np.full(wl.l.size, 2.0 * d), np.full(wl.l.size, W.PIX_GAUSS_WIDE, np.uint8)
    wl.x_true = None
    phi, rho = rng.uniform(0, 2 * np.pi, nv), reach / (2.0 * d) * rng.uniform(0.98, 1.0, nv)
    wl.u, wl.v, wl.w = rho * np.cos(phi), rho * np.sin(phi), np.zeros(nv)
    x = rng.standard_normal(wl.l.size)
    r = rng.standard_normal(nv) + 1j * rng.standard_normal(nv)
    p = O.Problem.from_workload(wl)
    plan = sl1m.Plan.from_workload(wl)
    info = plan.info()
    assert (info["grid_groups"], info["grid_flat"]) == (1, 1)
    Vo, go = O.forward(p, x), O.adjoint(p, r)
    V, g = plan.forward(x).cpu().numpy(), plan.adjoint(r).cpu().numpy()
    print(f"    forward {rel(V, Vo):.3e} adjoint {rel(g, go):.3e}", flush=True)
    assert rel(V, Vo) <= TOL and rel(g, go) <= TOL
    s = r.astype(np.complex128)
    dirty = plan.dirty_image(s).cpu().numpy()
    assert np.isfinite(dirty).all() and dirty.any()


def test_spread_w_without_cell_factors():
    """A narrow field with one group of visibilities of widely spread w (hundreds of turns of
    w n over the field): entries of single pixels within the element-wise bound's entry error,
    which takes the phase as float64 until it is reduced."""
    n, nv = 256, 64
    d = 0.012 / n
    wl = W.small_random(130, 10, nv, uv_radius=3000.0)
    wl.l, wl.m = _grid(n, n, d)
    wl.sigma, wl.kind, wl.x_true = np.zeros(n * n), np.zeros(n * n, np.uint8), None
    wl.w = np.random.default_rng(130).uniform(-1e7, 1e7, nv)
    plan = sl1m.Plan.from_workload(wl)
    info = plan.info()
    assert (info["grid_groups"], info["grid_flat"]) == (1, 1)
    p = O.Problem.from_workload(wl)
    worst = 0.0
    for j in (0, n - 1, n * (n - 1), n * n - 1, n * (n // 2)):
        e = np.zeros(n * n)
        e[j] = 1.0
        V, Vo = plan.forward(e).cpu().numpy(), O.forward(p, e)
        worst = max(worst, float(np.max(np.abs(V - Vo) / np.abs(Vo))))
    print(f"    largest entry error {worst:.3e}", flush=True)
    assert worst <= E.E_ENTRY["fp32"]


# name: delta pixels a side, extent, pixels a side of a wide Gaussian layer over them (0: none),
# visibilities, w spread; segments in groups, those without cell factors
MANY = {
    "cell_factors": (1024, 0.3, 0, 3_000_000, 60.0, 1, 0),     # 153 macros: 6.4 GB of rows
    "delta_and_layer": (768, 0.3, 384, 3_500_000, 60.0, 2, 0),  # 91 + 28 macros: 5.8 GB
    "flat": (2048, 0.01, 0, 1_200_000, 300.0, 1, 1),           # 289 macros: 4.9 GB
}


@pytest.mark.parametrize("name", list(MANY))
def test_macros_sharing_rows(name):
    """More macros than the plan's rows of forward sums: passes that add to them.  The
    workspace stays below 4 GiB, or a quarter above what it is without groups (no more than
    that of two sides, which has none); sampled visibilities against the oracle and all of
    them against the grid evaluation (a plan of two sides)."""
    n, ext, ng, nv, ws, groups, flat = MANY[name]
    print(f"[case] shared rows {name}", flush=True)
    wl = W.small_random(140, 10, nv, uv_radius=400.0, w_sigma=ws)
    l, m = _grid(n, n, 2 * ext / n)
    sig = np.zeros(l.size)
    if ng:
        l2, m2 = _grid(ng, ng, 2 * ext / ng)
        l, m = np.concatenate([l, l2]), np.concatenate([m, m2])
        sig = np.concatenate([sig, np.full(l2.size, 2 * ext / ng)])
    wl.l, wl.m, wl.sigma, wl.x_true = l, m, sig, None
    wl.kind = np.where(sig > 0, W.PIX_GAUSS_WIDE, W.PIX_DELTA).astype(np.uint8)
    x = np.random.default_rng(140).standard_normal(l.size)
    plan = sl1m.Plan.from_workload(wl)
    info = plan.info()
    assert (info["grid_groups"], info["grid_flat"]) == (groups, flat)
    V = plan.forward(x).cpu().numpy()
    print(f"    workspace {plan.workspace_bytes / 1e9:.2f} GB", flush=True)
    ks = np.arange(0, nv, nv // 40)
    p = O.Problem.from_workload(wl)
    Vo = sum(O.matrix_block(p, ks, np.arange(b, min(b + 65536, l.size))) @ x[b:b + 65536]
             for b in range(0, l.size, 65536))
    assert rel(V[ks], Vo) <= TOL
    again = plan.forward(x).cpu().numpy()
    plan.close()
    assert np.array_equal(again, V)
    other = sl1m.Plan.from_workload(wl, max_rhs=2)
    V2 = other.forward(x).cpu().numpy()
    print(f"    oracle {rel(V[ks], Vo):.3e}, grid evaluation {rel(V, V2):.3e}, its workspace "
          f"{other.workspace_bytes / 1e9:.2f} GB", flush=True)
    assert plan.workspace_bytes <= max(4 << 30, 1.25 * other.workspace_bytes)
    assert rel(V, V2) <= TOL
    other.close()


@pytest.mark.parametrize("name", ["flat_65", "one_group", "wide_field"])
def test_timing_counts_one_launch_an_operator(name):
    """The delta kinds of sl1m_timing, with and without cell factors, one macro or more."""
    wl, x, r = _case(name)
    plan = sl1m.Plan.from_workload(wl)
    plan.timing_begin(16)
    for _ in range(3):
        plan.forward(x), plan.adjoint(r)
    tim = plan.timing_end()
    for kind in ("forward", "adjoint", "grid_fwd_delta", "grid_adj_delta"):
        assert tim[kind][0] == 3 and tim[kind][1] > 0.0, (kind, tim)


# name: |l| x |m| pixels, spacing, visibilities, w spread; without cell factors
STRIPS = {
    "one_row_set": (31, 127, 4e-3, 3000, 15.0, 0),         # 16 |l| values: a lone set a macro
    "one_row_set_flat": (31, 255, 5e-4, 900, 60.0, 1),
    "two_row_sets": (33, 127, 4e-3, 3000, 15.0, 0),        # 17 values: 15 of 32 rows padded
    "four_columns": (1023, 7, 4e-4, 700, 60.0, 1),         # 12 of 16 columns padded
    "four_columns_two_orders": (319, 7, 1.8e-3, 3000, 600.0, 1),
}


@pytest.mark.parametrize("name", list(STRIPS))
def test_strips(name):
    nl, nm, d, nv, ws, flat = STRIPS[name]
    print(f"[case] strip {name}", flush=True)
    seed = 150 + sorted(STRIPS).index(name)
    wl = W.small_random(seed, 10, nv, uv_radius=400.0, w_sigma=ws, with_gains=True)
    wl.l, wl.m = _grid(nl, nm, d)
    wl.sigma, wl.kind, wl.x_true = np.zeros(wl.l.size), np.zeros(wl.l.size, np.uint8), None
    rng = np.random.default_rng(seed)
    x = rng.standard_normal(wl.l.size)
    r = rng.standard_normal(nv) + 1j * rng.standard_normal(nv)
    p = O.Problem.from_workload(wl)
    Vo, go = O.forward(p, x), O.adjoint(p, r)
    plan = sl1m.Plan.from_workload(wl)
    info = plan.info()
    V, g = plan.forward(x).cpu().numpy(), plan.adjoint(r).cpu().numpy()
    wf = E.worst_ratio(V, Vo, E.abs_forward_rows(p, x), wl.n_pix)
    wa = E.worst_ratio(g, go, E.abs_adjoint_cols(p, r), nv)
    print(f"    {info['grid_groups']} {info['grid_flat']} forward {rel(V, Vo):.3e} adjoint "
          f"{rel(g, go):.3e} element-wise {wf:.3e} {wa:.3e}", flush=True)
    assert (info["grid_groups"], info["grid_flat"]) == (1, flat)
    assert rel(V, Vo) <= TOL and rel(g, go) <= TOL
    assert wf <= 1.0 and wa <= 1.0


@pytest.mark.parametrize("n,nv,ext", [(40, 2000, 0.05), (40, 20_000, 0.3), (97, 20_000, 0.05),
                                      (97, 100_000, 0.3)])
def test_noalloc_is_the_plans_forward(n, nv, ext):
    """sl1m_forward_noalloc gives the plan's forward bit for bit where the plan evaluates in
    groups, up to plans that share rows to fit its scratch (the last)."""
    print(f"[case] noalloc groups {n} {nv} {ext}", flush=True)
    wl = W.small_random(160, 10, nv, uv_radius=400.0, w_sigma=60.0, with_gains=True)
    wl.l, wl.m = _grid(n, n, 2 * ext / n)
    wl.sigma, wl.kind, wl.x_true = np.zeros(n * n), np.zeros(n * n, np.uint8), None
    x = torch.as_tensor(np.random.default_rng(160).standard_normal(n * n), dtype=torch.float32,
                        device="cuda")
    plan = sl1m.Plan.from_workload(wl)
    assert plan.info()["grid_groups"] == 1 and plan.workspace_bytes <= 64 << 20
    V = plan.forward(x)
    lib = sl1m.lib()
    lib.sl1m_forward_noalloc.argtypes = [ctypes.POINTER(sl1m.Problem)] + 3 * [ctypes.c_void_p]
    lib.sl1m_forward_noalloc.restype = ctypes.c_int
    out = torch.full_like(V, float("nan"))
    for _ in range(2):
        st = lib.sl1m_forward_noalloc(ctypes.byref(plan._prob), ctypes.c_void_p(x.data_ptr()),
                                      ctypes.c_void_p(out.data_ptr()),
                                      ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
        assert st == sl1m.OK
        assert torch.equal(torch.view_as_real(out), torch.view_as_real(V))
    other = sl1m.Plan.from_workload(wl, max_rhs=2)
    assert rel(V.cpu().numpy(), other.forward(x).cpu().numpy()) <= TOL


@pytest.mark.parametrize("w_sigma,d,nv,flat", [(0.0, 1.5e-3, 700, 1), (20.0, 1.5e-3, 700, 1),
                                               (30.0, 4e-3, 6000, 0)])
def test_tapers_near_the_smallest_float(w_sigma, d, nv, flat):
    """Tapers of 2^-113: no further from a float64 plan than the grid evaluation (a plan of two
    sides), whose float32 exponents have the same rounding, times 1.3 for chance."""
    rng = np.random.default_rng(170)
    wl = W.small_random(170, 10, nv, with_gains=True)
    wl.l, wl.m = _grid(40, 70, d)
    wl.sigma, wl.kind = np.full(wl.l.size, 2.0 * d), np.full(wl.l.size, W.PIX_GAUSS_WIDE, np.uint8)
    wl.x_true = None
    phi, rho = rng.uniform(0, 2 * np.pi, nv), 5.0 / (2.0 * d) * rng.uniform(0.98, 1.0, nv)
    wl.u, wl.v, wl.w = rho * np.cos(phi), rho * np.sin(phi), w_sigma * rng.standard_normal(nv)
    x = rng.standard_normal(wl.l.size).astype(np.float32)
    r = (rng.standard_normal(nv) + 1j * rng.standard_normal(nv)).astype(np.complex64)
    plan = sl1m.Plan.from_workload(wl)
    info = plan.info()
    assert (info["grid_groups"], info["grid_flat"]) == (1, flat)
    other = sl1m.Plan.from_workload(wl, max_rhs=2, grid="require")
    exact = sl1m.Plan.from_workload(wl, precision="fp64")
    for f, v in (("forward", x), ("adjoint", r)):
        ref = getattr(exact, f)(v).cpu().numpy()
        e, eg = (rel(getattr(p, f)(v).cpu().numpy(), ref) for p in (plan, other))
        print(f"    {f} {e:.3e}, grid evaluation {eg:.3e}", flush=True)
        assert e <= 1.3 * eg


@pytest.mark.parametrize("name", ["no_series", "one_order"])
def test_gaussian_amplitudes_near_the_largest_float(name):
    """One pixel or one visibility of 2^100 (exact: powers of two) and of 2^126."""
    wl, x, r = _gauss_case(name)
    plan = sl1m.Plan.from_workload(wl)
    x, r = 0 * x, 0 * r
    x[7], r[9] = 1.0, 1.0
    for f, v in ((plan.forward, x), (plan.adjoint, r)):
        a, b = f(v).cpu().numpy(), f(v * 2.0 ** 100).cpu().numpy()
        assert np.array_equal(b, a * np.float32(2.0 ** 100))
        c = f(v * 2.0 ** 126).cpu().numpy()
        assert np.isfinite(c).all() and rel(c / np.float32(2.0 ** 126), a) <= TOL
