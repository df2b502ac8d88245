"""Parallel split-K weight gradients that leave kernel and slices to the library: exact whatever is chosen, in the workspace
that ucl_workspace_size() names and in a larger one, tile named or not (less workspace: test_gpu_split_choice.py)."""
import pytest
import torch

import paper_2603_29010_amd as ucl
from paper_2603_29010_amd import synth
from paper_2603_29010_amd.binding import Tuning

import parity

pytestmark = pytest.mark.gpu

GEOMS = [dict(Nb=2, H=28, W=28, C=64, Ko=128, R=3, S=3, pad=(1, 1)), dict(Nb=3, H=7, W=9, C=8, Ko=24, R=1, S=1, pad=(0, 0)),
         dict(Nb=5, H=13, W=11, C=40, Ko=72, R=3, S=3, pad=(1, 1), stride=(2, 2)), dict(Nb=1, H=2, W=3, C=8, Ko=8, R=1, S=1, pad=(0, 0))]


@pytest.mark.parametrize("dt", ["bf16", "f16"])
@pytest.mark.parametrize("geom", GEOMS, ids=lambda g: f"{g['Nb']}x{g['H']}x{g['W']}")
def test_chosen_slices(geom, dt):
    spec = synth.conv_grad_spec("wgrad", dt_in=dt, dt_out="f32", integer=True, **geom)
    s = geom.get("stride", (1, 1))
    conv = (geom["Nb"], geom["H"], geom["W"], geom["C"], geom["Ko"], geom["R"], geom["S"], *geom["pad"], *s, 1, 1)
    sizes = {"named": ucl.ucl_workspace_size("conv2d_wgrad", dt, "f32", tune=Tuning(split_k="parallel"), conv=conv)[0]}
    sizes["large"] = 64 << 20
    for what, nbytes in sizes.items():
        ws = torch.empty(max(nbytes, 1 << 16), dtype=torch.uint8, device="cuda")
        ucl.ucl_workspace_init(ws.data_ptr(), ws.numel(), torch.cuda.current_stream().cuda_stream)
        parity.check_exact(spec, Tuning(split_k="parallel", workspace=ws.data_ptr(), workspace_bytes=ws.numel()), label=f"{geom} {dt} {what}")
        for tile in ((64, 64, 32, 3), (128, 128, 32, 4)):
            if what == "large":
                parity.check_exact(spec, Tuning(*tile, split_k="parallel", workspace=ws.data_ptr(), workspace_bytes=ws.numel()), label=f"{geom} {dt} {tile}")
