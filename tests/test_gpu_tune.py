"""Autotuning of launch shapes (sl1m_tune) and explicit lane counts, through
the C ABI.  A tuned plan computes the same operator (oracle tolerance); the
tuner's choice is never slower than the default it timed beside it."""
import ctypes
import sys
import time

import numpy as np
import pytest

import oracle as O
from paper_1310_2078_amd import sl1m
from paper_1310_2078_amd import workloads as W

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def rel(a, b):
    return float(np.linalg.norm(np.asarray(a) - np.asarray(b)) / np.linalg.norm(np.asarray(b)))


@pytest.mark.parametrize("name", ["config1", "irregular", "config1_gauss_layers"])
def test_tuned_plan_matches_oracle(name):
    if name == "config1":
        wl = W.config1()
    elif name == "irregular":
        wl = W.small_random(31, 3001, 2503, kind=W.PIX_GAUSS_WIDE, sigma=2e-3, with_gains=True)
    else:
        wl = W.config1()
        wl.kind = np.full(wl.n_pix, W.PIX_GAUSS_WIDE, np.uint8)
        wl.sigma = np.full(wl.n_pix, 2e-3)
    say(f"[case] tune {name} n_pix={wl.n_pix} n_vis={wl.n_vis}")
    base = sl1m.Plan.from_workload(wl)
    t = base.tune(reps=3)
    base.close()
    say(f"    tuning {t}")
    assert t["candidates"] >= 2
    assert t["forward_ms"] + t["adjoint_ms"] <= t["default_forward_ms"] + t["default_adjoint_ms"]
    plan = sl1m.Plan.from_workload(wl, tuning=t)
    p = O.Problem.from_workload(wl)
    rng = np.random.default_rng(1)
    x = rng.standard_normal(wl.n_pix)
    r = rng.standard_normal(wl.n_vis) + 1j * rng.standard_normal(wl.n_vis)
    ef = rel(plan.forward(x).cpu().numpy(), O.forward(p, x))
    ea = rel(plan.adjoint(r).cpu().numpy(), O.adjoint(p, r))
    say(f"    tuned plan forward {ef:.3e} adjoint {ea:.3e}")
    assert ef <= 1e-5 and ea <= 1e-5


@pytest.mark.parametrize("vpl,ppl", [(1, 1), (2, 4), (4, 2)])
def test_explicit_lane_counts(vpl, ppl):
    """Direct kernels with every lane count the tuner may pick, on irregular
    pixels of two kinds with gains (ragged sizes)."""
    wl = W.small_random(32, 2777, 3101, with_gains=True)
    rng = np.random.default_rng(2)
    wl.kind = rng.choice([W.PIX_DELTA, W.PIX_GAUSS_WIDE], wl.n_pix).astype(np.uint8)
    wl.sigma = np.where(wl.kind == W.PIX_DELTA, 0.0, 2.5e-3)
    say(f"[case] lanes vpl={vpl} ppl={ppl}")
    plan = sl1m.Plan(wl.l, wl.m, wl.u, wl.v, wl.w, sigma=wl.sigma, kind=wl.kind, ant_p=wl.ant_p,
                     ant_q=wl.ant_q, ant_gain=wl.ant_gain, ant_fwhm=wl.ant_fwhm, grid="off",
                     fwd_vpl=vpl, adj_ppl=ppl)
    info = plan.info()
    assert info["fwd_vpl"] == vpl and info["adj_ppl"] == ppl
    p = O.Problem.from_workload(wl)
    x = rng.standard_normal(wl.n_pix)
    r = rng.standard_normal(wl.n_vis) + 1j * rng.standard_normal(wl.n_vis)
    ef = rel(plan.forward(x).cpu().numpy(), O.forward(p, x))
    ea = rel(plan.adjoint(r).cpu().numpy(), O.adjoint(p, r))
    say(f"    forward {ef:.3e} adjoint {ea:.3e}")
    assert ef <= 1e-5 and ea <= 1e-5


def test_tuning_several_sides_times_their_kernels():
    """A plan of one side evaluates this grid (16 x 512 values of |l| and |m|) in groups of
    visibilities, about three times as fast as the grid evaluation that plans of several
    sides run: tuning times the kernels of the plan it is asked about."""
    l, m = np.meshgrid((np.arange(31) - 15) * 5e-5, (np.arange(1023) - 511) * 5e-5)
    wl = W.small_random(33, 10, 100_000, uv_radius=2000.0, w_sigma=300.0)
    wl.l, wl.m, wl.x_true = l.ravel(), m.ravel(), None
    wl.sigma, wl.kind = np.zeros(l.size), np.zeros(l.size, np.uint8)
    ms = []
    for sides in (1, 2):
        plan = sl1m.Plan.from_workload(wl, max_rhs=sides)
        assert plan.info()["grid"] == 1 and plan.info()["grid_groups"] == (sides == 1)
        t = plan.tune(reps=5)
        say(f"[case] tune {sides} side(s): {t}")
        ms.append(t["default_forward_ms"])
        plan.close()
    assert ms[1] > 1.5 * ms[0]


def test_float64_plans_are_analysed_once():
    """The finer chunks of small float64 plans do not cost large ones a second analysis: the
    workspace of a float64 problem that is past the no-allocation scratch either way takes
    about as long to work out as that of the same float32 problem off the grid."""
    n = 512
    wl = W.small_random(34, 10, 50_000)
    l, m, _ = W.grid_pixels(n, 0.2)
    rng = np.random.default_rng(34)
    wl.l, wl.m, wl.x_true = l, m, None
    wl.sigma = np.where(rng.random(l.size) < 0.5, 0.0, 1e-3)
    wl.kind = np.where(wl.sigma > 0, W.PIX_GAUSS_WIDE, W.PIX_DELTA).astype(np.uint8)
    best = {}
    for prec in ("fp32", "fp64"):
        plan = sl1m.Plan.from_workload(wl, precision=prec, grid="off")
        assert plan.workspace_bytes > 64 << 20 or prec == "fp32"
        nbytes = ctypes.c_size_t()
        times = []
        for _ in range(15):
            t = time.perf_counter()
            assert sl1m.lib().sl1m_plan_workspace_bytes(ctypes.byref(plan._prob),
                                                        ctypes.byref(nbytes)) == 0
            times.append(time.perf_counter() - t)
        best[prec] = min(times)
        plan.close()
    say(f"[case] analysis {best}")
    assert best["fp64"] <= 1.5 * best["fp32"]
