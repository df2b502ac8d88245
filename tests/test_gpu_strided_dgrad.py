"""Data gradient of strided convolutions: rows are taken residue class by residue class with the taps each class meets.
Exact against the oracle for classes with all, some and no taps, ragged classes, and every built gather kernel."""
import pytest

from paper_2603_29010_amd import synth
from paper_2603_29010_amd.binding import Tuning

import paper_2603_29010_amd as ucl
import parity

pytestmark = pytest.mark.gpu

GEOMS = [
    dict(Nb=2, H=14, W=14, C=24, Ko=40, R=3, S=3, pad=(1, 1), stride=(2, 2)),
    dict(Nb=3, H=13, W=11, C=72, Ko=16, R=3, S=3, pad=(1, 1), stride=(2, 2)),           # ragged classes
    dict(Nb=2, H=9, W=12, C=8, Ko=24, R=1, S=1, pad=(0, 0), stride=(2, 2)),             # three classes without a tap
    dict(Nb=1, H=17, W=10, C=16, Ko=136, R=3, S=5, pad=(1, 2), stride=(3, 2)),
    dict(Nb=2, H=12, W=9, C=16, Ko=8, R=3, S=3, pad=(0, 1), stride=(1, 4)),             # stride wider than the filter
    dict(Nb=2, H=15, W=15, C=16, Ko=24, R=3, S=3, pad=(2, 2), stride=(2, 2), dil=(2, 2)),  # odd residues meet no tap
    dict(Nb=2, H=15, W=16, C=16, Ko=24, R=4, S=3, pad=(3, 1), stride=(2, 3), dil=(3, 2)),
    dict(Nb=2, H=4, W=5, C=8, Ko=8, R=2, S=2, pad=(1, 1), stride=(7, 6)),               # stride beyond the image
    dict(Nb=2, H=4, W=5, C=8, Ko=16, R=3, S=3, pad=(1, 1), stride=((1 << 32), 2)),      # strides beyond 32 bits: one output row
    dict(Nb=2, H=4, W=5, C=8, Ko=16, R=3, S=3, pad=(2, 1), stride=((1 << 31) + 3, 1 << 40)),
    dict(Nb=1, H=1, W=33, C=8, Ko=64, R=1, S=3, pad=(0, 1), stride=(1, 2)),
]


def tilings():
    out = []
    for i in range(ucl.ucl_num_variants()):
        v = ucl.ucl_variant(i)
        if (v["mode"], v["dt"], v["a_path"]) == (3, "bf16", 2):
            out.append(Tuning(v["tile_m"], v["tile_n"], v["tile_k"], v["stages"], 0, 1, k_groups=v["k_groups"]))
    return out


@pytest.mark.parametrize("geom", GEOMS, ids=lambda g: "x".join(map(str, (g["H"], g["W"], g["R"], g["S"]))) + "s%d%d" % g["stride"])
def test_exact(geom):
    spec = synth.conv_grad_spec("dgrad", dt_out="f32", integer=True, **geom)
    for tune in tilings():
        parity.check_exact(spec, tune, label=f"{geom} {tune.as_dict()}")
    parity.check_exact(spec, None, label="table choice")


@pytest.mark.parametrize("chain", [("bias", "aux_load", "relu"), ("per_row_scale", "bias", "silu"), ("column_broadcast", "aux_load")])
def test_chains_see_the_pixels_of_their_rows(chain):
    spec = synth.conv_grad_spec("dgrad", dt_out="bf16", epilogue=chain, **GEOMS[1])
    parity.check(spec, None, label=str(chain))
    parity.check(spec, Tuning(128, 128, 32, 4, 0, 1), label=str(chain))
