"""Filter gradients of 3x3 convolutions whose slices are left to the library, on the kernel that multiplies all taps of a pixel: exact over
partial tiles of filters and channels, odd extents, both strides, narrow and wide rows and images; the calls beside it are not its."""
import numpy as np
import pytest
import torch

import paper_2603_29010_amd as ucl
from paper_2603_29010_amd import synth
from paper_2603_29010_amd.binding import Tuning
from paper_2603_29010_amd.workload import DeviceWorkload

import oracle
import parity
from oracle import run_spec as orc_run

pytestmark = pytest.mark.gpu


def geom(n, h, w, c, ko, stride=1, r=3, pad=1):
    return dict(Nb=n, H=h, W=w, C=c, Ko=ko, R=r, S=r, pad=(pad, pad), stride=(stride, stride))


def open_split(nbytes=64 << 20):
    ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    ucl.ucl_workspace_init(ws.data_ptr(), ws.numel(), torch.cuda.current_stream().cuda_stream)
    return Tuning(split_k="parallel", workspace=ws.data_ptr(), workspace_bytes=ws.numel()), ws


def kernels_of(spec, tune):
    w = DeviceWorkload(spec)
    w.run(tune=tune)
    torch.cuda.synchronize()
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as p:
        w.run(tune=tune)
        torch.cuda.synchronize()
    return [e.name for e in p.events() if "ucl" in e.name]


# tiles are 64 filters x 32 channels; k-tiles 128 padded pixels (stride 2: 64)
@pytest.mark.parametrize("dt", ["bf16", "f16"])
@pytest.mark.parametrize("g", [geom(24, 28, 28, 72, 136), geom(40, 7, 7, 264, 200), geom(3, 62, 62, 136, 72), geom(70, 60, 2, 128, 136),
                               geom(500, 1, 9, 256, 264), geom(33, 29, 27, 136, 200, 2), geom(8, 124, 123, 72, 104, 2),
                               geom(64, 14, 15, 264, 200, 2)], ids=lambda g: f"{g['Nb']}x{g['H']}x{g['W']}x{g['C']}-{g['Ko']}s{g['stride'][0]}")
def test_exact(g, dt):
    spec = synth.conv_grad_spec("wgrad", dt_in=dt, dt_out="f32", integer=True, **g)
    tune, ws = open_split()
    assert any("wgrad_taps_kernel" in k for k in kernels_of(spec, tune))
    parity.check_exact(spec, tune, label=f"{g} {dt}")
    conv = (g["Nb"], g["H"], g["W"], g["C"], g["Ko"], 3, 3, 1, 1, *g["stride"], 1, 1)
    need, slices = ucl.ucl_workspace_size("conv2d_wgrad", dt, "f32", Tuning(split_k="parallel"), conv=conv)
    tune, ws = open_split(max(need, 1 << 16))
    assert any("wgrad_taps_kernel" in k for k in kernels_of(spec, tune)) and slices >= 1
    parity.check_exact(spec, tune, label=f"{g} {dt}, the workspace that the query names")


# (the last, with 16-bit results: whole sums in one workgroup, stored without a second launch)
@pytest.mark.parametrize("dt", ["bf16", "f16"])
@pytest.mark.parametrize("g", [geom(24, 28, 28, 72, 136), geom(40, 7, 7, 264, 200), geom(500, 1, 9, 256, 264), geom(33, 29, 27, 136, 200, 2),
                               geom(64, 14, 14, 264, 200, 2), geom(16, 62, 60, 72, 104, 2), geom(2, 28, 28, 304, 440)],
                         ids=lambda g: f"{g['Nb']}x{g['H']}x{g['W']}x{g['C']}-{g['Ko']}s{g['stride'][0]}")
def test_special_values_stay_where_their_taps_are(g, dt):
    # infinities and NaN in the first and last rows, columns and images of x, a channel each: a tap that would meet one outside the image stays finite
    spec = synth.conv_grad_spec("wgrad", dt_in=dt, dt_out=dt if g["Ko"] == 440 else "f32", integer=True, **g)
    n, h, w, x = g["Nb"], g["H"], g["W"], spec["x"]
    inf, nan, sign = (0x7f80, 0x7fc0, 0x8000) if dt == "bf16" else (0x7c00, 0x7e00, 0x8000)
    for c, (at, bits) in enumerate([((0, 0, 0), inf), ((0, 0, w - 1), nan), ((n - 1, h - 1, 0), nan), ((n - 1, h - 1, w - 1), inf), ((0, h - 1, w // 2), inf | sign),
                                    ((n // 2, h // 2, w - 1), inf), ((n // 2, h // 2, 0), nan), ((1, 0, w // 2), inf)]):
        x[at + (c * 9 - c % 3,)] = bits
    want = orc_run.run(spec)
    want = oracle.round_to(want, spec["dt_out"]).reshape(want.shape)
    assert np.isfinite(want).any() and not np.isfinite(want).all()
    tune, ws = open_split()
    assert any("wgrad_taps_kernel" in k for k in kernels_of(spec, tune))
    for t in (tune, Tuning(64, 64, 32, 3, split_k="parallel", workspace=ws.data_ptr(), workspace_bytes=ws.numel())):
        got = parity.gpu_result(spec, t)[0].reshape(want.shape)
        assert np.array_equal(got, want, equal_nan=True), np.argwhere(~((got == want) | (np.isnan(got) & np.isnan(want))))[:4]


def test_the_tallest_image():
    # (its row indexes come out of fp32 products; |sums| stay far below 2^24)
    spec = synth.conv_grad_spec("wgrad", dt_in="bf16", dt_out="f32", integer=True, **geom(1, (1 << 20) - 1, 1, 32, 40))
    tune, ws = open_split()
    assert any("wgrad_taps_kernel" in k for k in kernels_of(spec, tune))
    parity.check_exact(spec, tune, label="tallest")


@pytest.mark.parametrize("dt", ["bf16", "f16"])
def test_other_outputs(dt):
    tune, ws = open_split()
    for g in (geom(24, 28, 28, 72, 136), geom(40, 7, 7, 264, 200)):
        for out, chain in ((dt, ()), ("f32", (("scale", 0.25),)), (dt, (("scale", 0.25),))):
            spec = synth.conv_grad_spec("wgrad", dt_in=dt, dt_out=out, epilogue=chain, **g)
            assert any("wgrad_taps_kernel" in k for k in kernels_of(spec, tune))
            parity.check(spec, tune, label=f"{g} {dt} -> {out} {chain}")


def test_what_stays_with_the_tile_kernel():
    tune, ws = open_split()
    g = geom(24, 28, 28, 72, 136)
    for other, tn, chain in ((dict(g, pad=(0, 0)), tune, ()), (dict(g, stride=(2, 1)), tune, ()), (dict(g, Ko=32), tune, ()), (geom(24, 28, 28, 72, 136, r=1, pad=0), tune, ()),
                             (geom(2, 70, 70, 72, 136), tune, ()), (g, tune, ("relu",)), (g, None, ()),
                             (g, Tuning(64, 64, 32, 3, split_k="parallel", workspace=ws.data_ptr(), workspace_bytes=ws.numel()), ())):
        spec = synth.conv_grad_spec("wgrad", dt_in="bf16", dt_out="f32", epilogue=chain, integer=True, **other)
        assert not any("wgrad_taps_kernel" in k for k in kernels_of(spec, tn)), other
        parity.check_exact(spec, tn, label=f"{other} {chain}")


def test_graph_replays():
    spec = synth.conv_grad_spec("wgrad", dt_in="bf16", dt_out="f32", integer=True, **geom(24, 28, 28, 72, 136))
    tune, ws = open_split()
    w = DeviceWorkload(spec)
    w.run(tune=tune)
    torch.cuda.synchronize()
    want = w.D.clone()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        w.run(tune=tune)
    for _ in range(3):
        w.D.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(w.D, want)
