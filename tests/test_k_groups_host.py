"""ucl_tuning.k_groups names a kernel where there is one and is never a reason to refuse a call: the word was reserved and
ignored before it had a meaning (host only)."""
import pytest

import paper_2603_29010_amd as ucl
from paper_2603_29010_amd.binding import Tuning, UclError

PROBLEM = dict(M=200, N=136, K=1992)


@pytest.mark.parametrize("k_groups", [-1, 1, 2, 3, 4, 7, 1 << 30])
def test_served_whatever_it_holds(k_groups):
    for dt in ("bf16", "f16", "e4m3"):
        problem = dict(PROBLEM, K=2000)
        for tile in ((), (64, 64, 64, 4), (128, 128, 64, 2)):
            assert ucl.ucl_workspace_size("gemm", dt, "bf16", Tuning(*tile, k_groups=k_groups), **problem) == (0, 1)
    conv = (2, 9, 7, 40, 72, 3, 3, 1, 1, 1, 1, 1, 1)
    for op in ("conv2d_fprop", "conv2d_dgrad", "conv2d_wgrad"):
        assert ucl.ucl_workspace_size(op, "bf16", "bf16", Tuning(k_groups=k_groups), conv=conv) == (0, 1)


@pytest.mark.parametrize("mode", ["serial", "parallel"])
def test_split_k_does_not_look_at_it(mode):
    for tile in ((), (64, 64, 64, 4)):
        for dt_out in ("bf16", "f32"):
            plain = ucl.ucl_workspace_size("gemm", "bf16", dt_out, Tuning(*tile, split_k=mode), M=200, N=136, K=30000)
            assert plain[1] > 1
            assert ucl.ucl_workspace_size("gemm", "bf16", dt_out, Tuning(*tile, split_k=mode, k_groups=2), M=200, N=136, K=30000) == plain


def test_shapes_built_with_k_groups_only_serve_no_split():
    conv = (2, 9, 7, 40, 72, 3, 3, 1, 1, 1, 1, 1, 1)
    assert ucl.ucl_workspace_size("conv2d_fprop", "bf16", "bf16", Tuning(128, 64, 64, 3), conv=conv) == (0, 1)
    for tile in ((16, 32, 64, 1), (32, 32, 64, 1)):
        assert ucl.ucl_workspace_size("gemm", "bf16", "bf16", Tuning(*tile), **PROBLEM) == (0, 1)
        with pytest.raises(UclError) as e:
            ucl.ucl_workspace_size("gemm", "bf16", "bf16", Tuning(*tile, split_k="parallel", slices=4), **PROBLEM)
        assert e.value.status == "UCL_ERR_UNSUPPORTED"


@pytest.mark.parametrize("kw,few_rows", [
    (dict(op="grouped_gemm", dt="e4m3", M_g=[20, 4, 27, 30], N=304, K=704), True), (dict(op="grouped_gemm", dt="bf16", M_g=[21, 20], N=616, K=640), True),
    (dict(op="grouped_gemm", dt="e4m3", M_g=[(7 * g) % 33 for g in range(64)], N=2048, K=1024), False),
    (dict(op="grouped_gemm", dt="bf16", M_g=[30] * 49, N=2400, K=576), False),
    (dict(op="gemm", dt="e4m3", M=25, N=21, K=608), True), (dict(op="gemm", dt="bf16", M=55, N=101, K=296), True), (dict(op="gemm", dt="bf16", M=256, N=256, K=256), False)])
def test_where_the_few_row_kernels_begin(kw, few_rows):
    kw = dict(kw)
    assert (ucl.ucl_select_tuning(kw.pop("op"), kw.pop("dt"), "bf16", **kw)["stages"] == 1) == few_rows


@pytest.mark.parametrize("dt", ["bf16", "f16"])
def test_small_products_of_transposed_operands_take_small_tiles(dt):
    for (M, N, K) in ((8, 8, 2048), (8, 24, 7168), (64, 64, 4096), (40, 512, 3000)):
        t = ucl.ucl_select_tuning("gemm", dt, "f32", M=M, N=N, K=K, a_layout="mn", b_layout="mn")
        assert (t["tile_m"], t["tile_n"], t["tile_k"], t["k_groups"]) == (64, 64, 64, 2)


def test_data_gradients_of_few_taps_have_nothing_for_k_groups():
    for conv in ((9, 5, 5, 24, 32, 3, 3, 1, 1, 1, 1, 1, 1), (3, 24, 24, 24, 24, 3, 3, 1, 1, 1, 1, 1, 1)):
        assert ucl.ucl_select_tuning("conv2d_dgrad", "bf16", "bf16", conv=conv)["k_groups"] == 1
