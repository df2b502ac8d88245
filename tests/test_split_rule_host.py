"""Split-K calls that leave the slices to the library: what the size query answers for them (host only)."""
import pytest

import paper_2603_29010_amd as ucl
from paper_2603_29010_amd.binding import Tuning


def query(op, dt_in, dt_out, mode, tile=(), **kw):
    return ucl.ucl_workspace_size(op, dt_in, dt_out, tune=Tuning(*tile, split_k=mode), **kw)


@pytest.mark.parametrize("dt_out,mode,M,N,K,layouts", [
    ("bf16", "serial", 4096, 512, 16384, "kk"), ("bf16", "serial", 136, 12696, 5376, "kk"), ("bf16", "serial", 5952, 664, 14040, "kk"),
    ("f32", "serial", 72, 9800, 7472, "mm"), ("f32", "serial", 1056, 1512, 6168, "mk")])
def test_no_split_where_the_tiles_fill_the_chip(dt_out, mode, M, N, K, layouts):
    # split and unsplit launches are priced by the same model: there are tiles enough for every CU
    a, b = ("mn" if c == "m" else "k" for c in layouts)
    assert query("gemm", "bf16", dt_out, mode, M=M, N=N, K=K, a_layout=a, b_layout=b) == (0, 1)


def test_split_where_the_model_splits():
    # (few large tiles: a split pays, though a launch of whole tiles looks cheap to the model that unsplit calls are priced by)
    assert query("gemm", "bf16", "f32", "parallel", M=4096, N=1000, K=32768, a_layout="mn", b_layout="mn")[1] == 4
