"""CPU checks of the group evaluation's host tables: the tables of a plan hold the segments
that it evaluates in groups and no others, and the cases of the GPU tests run what their
names say (tiles without cell factors, the series classes)."""
import os
import shutil
import subprocess

import pytest

import test_gpu_groups as G
from paper_1310_2078_amd import workloads as W

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1310_2078_amd", "csrc")


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path_factory.mktemp("groups") / "groups_check")
    subprocess.run([gxx, "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined",
                    "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", CSRC,
                    "-x", "c++", os.path.join(CSRC, "sl1m_wgtables.hip"),
                    os.path.join(ROOT, "tests", "groups_check.cpp"), "-o", exe],
                   check=True, capture_output=True, text=True)

    def run(segments, w):
        text = "\n".join([str(len(segments))] + ["%d %d %d %r" % s for s in segments]
                         + [str(len(w))] + [repr(float(x)) for x in w])
        out = subprocess.run([exe], input=text, capture_output=True, text=True, timeout=120)
        assert out.returncode == 0, out.stderr
        lines = [ln.split() for ln in out.stdout.splitlines()]
        segs = [(int(ln[3]), [int(c) for c in ln[5:9]]) for ln in lines[1:]]
        return int(lines[0][1]), int(lines[0][3]), segs
    return run


# case: without cell factors, the series classes that occur (test_gpu_groups.CASES, GAUSS)
DELTA = {
    "one_group": (1, {1}), "one_more": (1, {1}), "odd_17_tiles": (1, {0, 1}),
    "exact_tiles": (1, {0, 1}), "columns_129": (1, {0, 1}), "rows_five_sets": (1, {0, 1}),
    "wide_field": (0, {0, 2, 3}), "third_order": (0, {0, 2, 3}), "w_zero": (1, {0}),
    "many_groups": (0, {0, 1, 2, 3}), "flat_65": (1, {1}), "flat_two_orders": (1, {1, 2}),
    "flat_one_visibility": (1, {1}),
}
GAUSS = {
    "no_series": (1, {0, 1}), "paraxial_odd": (1, {0}), "one_order": (0, {1}),
    "flat_two_orders": (1, {1, 2}), "steep_taper": (0, {1}),
}


def _ran(seg):
    flat, cls = seg
    return flat, {i for i in range(4) if cls[i]}


@pytest.mark.parametrize("name", list(DELTA))
def test_delta_cases_run_what_they_name(check, name):
    nl, nm, d = G.CASES[name][:3]
    wl, _, _ = G._case(name)
    kept, groups, segs = check([(W.PIX_DELTA, nl, nm, d)], wl.w)
    assert kept == 1 and groups >= (wl.n_vis + 63) // 64
    assert _ran(segs[0]) == DELTA[name]


@pytest.mark.parametrize("name", list(GAUSS))
def test_gaussian_cases_run_what_they_name(check, name):
    nl, nm, d, _, kind = G.GAUSS[name][:5]
    wl, _, _ = G._gauss_case(name)
    kept, _, segs = check([(kind, nl, nm, d)], wl.w)
    assert kept == 1
    assert _ran(segs[0]) == GAUSS[name]


@pytest.mark.parametrize("name", list(G.LAYERS))
def test_tables_hold_the_segments_kept(check, name):
    """Where the Gaussian layer makes too many groups, the delta grid's tables alone (the
    larger layer's would reach past the regions reserved for them)."""
    dn, dd, gn, gd, _, _, n, flat = G.LAYERS[name]
    wl = G._layer_case(name)[0]
    kept, _, segs = check([(W.PIX_DELTA, dn, dn, dd), (W.PIX_GAUSS_WIDE, gn, gn, gd)], wl.w)
    assert kept == n
    assert sum(f << i for i, (f, _) in enumerate(segs)) == flat
