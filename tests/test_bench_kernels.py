"""bench.py prices the operator kernels that a plan reports it runs."""
import bench


def test_operator_kernels_follow_the_plan():
    names = bench.operator_kernels({"grid_groups": 4, "grid_flat": 0})
    assert names == {"grid_fwd_delta": "k_wg_fwd", "grid_adj_delta": "k_wg_adj",
                     "grid_fwd_gauss": "k_wg_fwd_gauss", "grid_adj_gauss": "k_wg_adj_gauss"}
    # the layers outside the groups, the delta grid without cell factors
    names = bench.operator_kernels({"grid_groups": 1, "grid_flat": 1})
    assert names["grid_adj_delta"] == "k_flat_adj"
    assert names["grid_adj_gauss"] == "k_grid_adj_gauss_multi"
    names = bench.operator_kernels({"grid_groups": 0, "grid_flat": 0})
    assert names["grid_fwd_delta"] == "k_grid_fwd_delta_pairs"
    for info in ({"grid_groups": g, "grid_flat": f} for g in range(5) for f in range(1 << g)):
        assert set(bench.operator_kernels(info).values()) <= set(bench.EXEC_FLOP_PER_EVAL)


def test_dominant_kernel_counts_a_layer_or_all():
    tim = {"grid_fwd_delta": (2, 2.0), "grid_adj_gauss": (3, 9.0)}
    info = {"grid_groups": 4, "grid_flat": 0}
    assert bench.dominant_kernel(info, tim, 100, 30, 10, 3) == \
        ("k_wg_adj_gauss", 3.0, 100.0, "grid_adj_gauss")
    info = {"grid_groups": 1, "grid_flat": 0}
    assert bench.dominant_kernel(info, tim, 100, 30, 10, 3) == \
        ("k_grid_adj_gauss_multi", 3.0, 300, "grid_adj_gauss")
