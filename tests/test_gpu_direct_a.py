"""A contiguous along M through the transpose reads, with the smallest tiles: their ring holds two A fragments, and a k-step that is
not behind a barrier has to wait for the one that the k-step before requested last.  Exact on integers, every such kernel."""
import pytest

import paper_2603_29010_amd as ucl
from paper_2603_29010_amd import synth
from paper_2603_29010_amd.binding import Tuning

import parity

pytestmark = pytest.mark.gpu


def _kernels():
    return [v for v in map(ucl.ucl_variant, range(ucl.ucl_num_variants()))
            if v["mode"] == 0 and v["a_path"] == 5 and v["tile_m"] == 64 and not v["scheduler"]]


@pytest.mark.parametrize("v", _kernels(), ids=lambda v: f"{v['dt']}-{v['tile_k']}x{v['stages']}-b{v['b_path']}-kg{v['k_groups']}")
def test_exact(v):
    tune = Tuning(v["tile_m"], v["tile_n"], v["tile_k"], v["stages"], k_groups=v["k_groups"])
    for (M, N, K) in ((64, 64, 64), (1096, 1032, 2056), (2048, 2048, 1024)):
        spec = synth.gemm_spec(M, N, K, dt_in=v["dt"], dt_out="f32", a_layout="col", b_layout="row" if v["b_layout"] else "col",
                               epilogue=(), integer=True)
        parity.check_exact(spec, tune, label=f"{M}x{N}x{K}")
