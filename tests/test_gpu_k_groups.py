"""Kernels with K groups (two groups of four wavefronts, or in the few-row kernels four single wavefronts, share a tile, each
multiplying its own part of K): exact on integers for every such kernel, at the sizes where the split of K can go wrong, and in fixed order."""
import numpy as np
import pytest
import torch

import paper_2603_29010_amd as ucl
from paper_2603_29010_amd import synth
from paper_2603_29010_amd.binding import Tuning
from paper_2603_29010_amd.workload import DeviceWorkload

import parity

pytestmark = pytest.mark.gpu

def _all_variants():
    i = 0
    while True:
        try:
            yield ucl.ucl_variant(i)
        except ucl.UclError:
            return
        i += 1


VARIANTS = [v for v in _all_variants() if v["k_groups"] > 1]         # (the few-row kernels among them)
NAMES = {0: "gemm", 1: "grouped", 2: "fprop", 3: "dgrad", 4: "wgrad"}


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
    if v["mode"] == 1:
        for (rows, N, K) in (([0, 1, 16, 17, 33], 72, step), ([70, 0, 5, 128], 136, 5 * 64 + step), ([3], 264, 1024)):
            spec = synth.grouped_spec(rows, N, K, dt_in=dt, dt_out="f32", epilogue=(), integer=True)
            parity.check_exact(spec, tuning(v), label=f"{ident(v)} {rows} {N}x{K}")
        return
    for g in (dict(Nb=2, H=9, W=7, C=40, Ko=72, R=3, S=3, pad=(1, 1)), dict(Nb=1, H=6, W=6, C=8, Ko=8, R=1, S=1, pad=(0, 0)),
              dict(Nb=1, H=11, W=10, C=136, Ko=64, R=3, S=3, pad=(1, 1), stride=(2, 2))):
        if v["mode"] == 2:
            g = dict(g)
            spec = synth.conv_spec(dt_in=dt, dt_out="f32", epilogue=(), integer=True, **g)
        else:
            spec = synth.conv_grad_spec(NAMES[v["mode"]], dt_in=dt, dt_out="f32", integer=True, **g)
        parity.check_exact(spec, tuning(v), label=f"{ident(v)} {g}")


@pytest.mark.parametrize("mode,slices", [("serial", 4), ("parallel", 2), ("parallel", 5)])
def test_named_k_groups_leave_split_k_alone(mode, slices):
    # split-K has kernels without K groups only: the one of the named shape runs
    spec = synth.gemm_spec(200, 136, 1992, dt_out="f32", epilogue=(), integer=True)
    ws = torch.empty(64 << 20, dtype=torch.uint8, device="cuda")
    ucl.ucl_workspace_init(ws.data_ptr(), ws.numel(), torch.cuda.current_stream().cuda_stream)
    tune = Tuning(64, 64, 64, 4, split_k=mode, slices=slices, k_groups=2, workspace=ws.data_ptr(), workspace_bytes=ws.numel())
    parity.check_exact(spec, tune, label=f"{mode} x{slices}")


def test_few_row_kernels_refuse_split_k():
    v = next(v for v in VARIANTS if v["stages"] == 1 and v["mode"] == 0)
    spec = synth.gemm_spec(16, 64, 4096, dt_in=v["dt"])
    with pytest.raises(ucl.UclError) as e:
        parity.gpu_result(spec, tuning(v, split_k="parallel", slices=4, workspace=4096, workspace_bytes=1 << 30))
    assert e.value.status == "UCL_ERR_UNSUPPORTED"


@pytest.mark.parametrize("chain", [("bias", "aux_load", "gelu_tanh"), ("per_row_scale", "bias", "silu"), ("column_broadcast", "aux_load", "relu")])
@pytest.mark.parametrize("dt", ["bf16", "f16", "e4m3"])
def test_few_row_kernels_run_the_chain(chain, dt):
    spec = synth.gemm_spec(21, 1003, 1200, dt_in=dt, dt_out="f16" if dt == "f16" else "bf16", epilogue=chain)
    for v in VARIANTS:
        if v["stages"] == 1 and v["mode"] == 0 and v["dt"] == dt:
            parity.check(spec, tuning(v), label=f"{ident(v)} {chain}")


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
