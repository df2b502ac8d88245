"""Kernels with K groups (two groups of four wavefronts share a tile, each multiplying its own part of K): exact on
integers for every such kernel, at the sizes where the split of K can go wrong, and in fixed order."""
import numpy as np
import pytest
import torch

import paper_2603_29010_amd as ucl
from paper_2603_29010_amd import synth
from paper_2603_29010_amd.binding import Tuning
from paper_2603_29010_amd.workload import DeviceWorkload

import parity

pytestmark = pytest.mark.gpu

VARIANTS = [v for v in (ucl.ucl_variant(i) for i in range(ucl.ucl_num_variants())) if v["k_groups"] > 1]
NAMES = {0: "gemm", 2: "fprop", 3: "dgrad", 4: "wgrad"}


def tuning(v, **kw):
    return Tuning(v["tile_m"], v["tile_n"], v["tile_k"], v["stages"], 0, 1 if v["mode"] in (2, 3) else 0, k_groups=v["k_groups"], **kw)


def ident(v):
    return f"{NAMES[v['mode']]}-{v['dt']}-{v['tile_m']}x{v['tile_n']}x{v['tile_k']}x{v['stages']}-a{v['a_path']}b{v['b_path']}"


@pytest.mark.parametrize("v", VARIANTS, ids=ident)
def test_exact(v):
    dt = v["dt"]
    step = 16 if dt in ("e4m3", "e5m2") else 8
    if v["mode"] == 0:
        la, lb = "col" if v["a_layout"] else "row", "row" if v["b_layout"] else "col"
        # one K group without any k, both with part of a k-tile, a ragged tail in either, several tiles each way
        for (M, N, K) in ((72, 136, step), (136, 72, 64), (136, 200, 5 * 64 + step), (264, 136, 9 * 64 - step), (64, 64, 2048)):
            spec = synth.gemm_spec(M, N, K, dt_in=dt, dt_out="f32", a_layout=la, b_layout=lb, epilogue=(), integer=True)
            parity.check_exact(spec, tuning(v), label=f"{ident(v)} {M}x{N}x{K}")
        return
    for g in (dict(Nb=2, H=9, W=7, C=40, Ko=72, R=3, S=3, pad=(1, 1)), dict(Nb=1, H=6, W=6, C=8, Ko=8, R=1, S=1, pad=(0, 0)),
              dict(Nb=1, H=11, W=10, C=136, Ko=64, R=3, S=3, pad=(1, 1), stride=(2, 2))):
        if v["mode"] == 2:
            spec = synth.conv_spec(dt_in=dt, dt_out="f32", epilogue=(), integer=True, **g)
        else:
            spec = synth.conv_grad_spec(NAMES[v["mode"]], dt_in=dt, dt_out="f32", integer=True, **g)
        parity.check_exact(spec, tuning(v), label=f"{ident(v)} {g}")


@pytest.mark.parametrize("v", [v for v in VARIANTS if v["mode"] == 4], ids=ident)
@pytest.mark.parametrize("mode", ["serial", "parallel"])
def test_weight_gradient_with_split_k(v, mode):
    # split-K cuts K into slices, K groups cut every slice again
    spec = synth.conv_grad_spec("wgrad", dt_in=v["dt"], dt_out="f32", integer=True, Nb=3, H=13, W=11, C=24, Ko=40, R=3, S=3, pad=(1, 1))
    ws = torch.empty(16 << 20, dtype=torch.uint8, device="cuda")
    ucl.ucl_workspace_init(ws.data_ptr(), ws.numel(), torch.cuda.current_stream().cuda_stream)
    for slices in (2, 3, 5):
        parity.check_exact(spec, tuning(v, split_k=mode, slices=slices, workspace=ws.data_ptr(), workspace_bytes=ws.numel()),
                           label=f"{ident(v)} {mode} x{slices}")


def test_repeated_runs_give_the_same_bits():
    spec = synth.gemm_spec(200, 136, 1992, dt_out="f32", epilogue=("bias", "silu"))
    v = next(v for v in VARIANTS if v["mode"] == 0 and v["dt"] == "bf16")
    w = DeviceWorkload(spec)
    first = None
    for _ in range(8):
        w.run(tune=tuning(v))
        got = w.result_bits().copy()
        first = got if first is None else first
        assert np.array_equal(got, first)
    parity.check(spec, tuning(v), label="K groups, bias + SiLU")


def test_a_workspace_that_served_without_k_groups_goes_on_serving():
    # the weight gradient's own choice takes K groups only where the caller's workspace holds their partial tiles
    conv = dict(Nb=8, H=28, W=28, C=128, Ko=128, R=3, S=3, pad=(1, 1))
    spec = synth.conv_grad_spec("wgrad", dt_out="f32", integer=True, **conv)
    geom = (8, 28, 28, 128, 128, 3, 3, 1, 1, 1, 1, 1, 1)
    small, _ = ucl.ucl_workspace_size("conv2d_wgrad", "bf16", "f32", tune=Tuning(split_k="parallel", k_groups=1), conv=geom)
    ws = torch.empty(small, dtype=torch.uint8, device="cuda")
    ucl.ucl_workspace_init(ws.data_ptr(), small, torch.cuda.current_stream().cuda_stream)
    parity.check_exact(spec, Tuning(split_k="parallel", workspace=ws.data_ptr(), workspace_bytes=small), label="smaller workspace")
