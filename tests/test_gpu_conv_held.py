"""3x3 convolutions at stride 1 and 2 and data gradients at stride 1 on the kernel that holds the filter in registers: bit for bit the rounded integer sums over odd images,
partial strips, bands and tiles of channels, every number of wave groups, several passes over the channels, pairs of narrow images; the chain's parts."""
import numpy as np
import pytest
import torch

import oracle
import parity
from oracle import run_spec as orc_run
from paper_2603_29010_amd import synth
from paper_2603_29010_amd.binding import Tuning
from paper_2603_29010_amd.workload import DeviceWorkload

pytestmark = pytest.mark.gpu


def geom(n, h, w, c, ko, stride=1):
    return dict(Nb=n, H=h, W=w, C=c, Ko=ko, R=3, S=3, stride=(stride, stride))


def name(g):
    return f"{g['Nb']}x{g['H']}x{g['W']}x{g['C']}-{g['Ko']}s{g['stride'][0]}"


def kernels_of(spec, tune=None):
    w = DeviceWorkload(spec)
    w.run(tune=tune)
    torch.cuda.synchronize()
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as p:
        w.run(tune=tune)
        torch.cuda.synchronize()
    return [e.name for e in p.events() if "ucl" in e.name]


def check_rounded(spec, prepare=lambda w: None):
    """Whole numbers: the sums are exact in fp32, so the results are theirs rounded once."""
    assert DeviceWorkload(spec).kernel() == {"unnamed": "conv_held"}
    assert any("conv_held_kernel" in k for k in kernels_of(spec)), kernels_of(spec)
    w = DeviceWorkload(spec)
    prepare(w)
    w.run()
    got, want = w.result(), oracle.round_to(orc_run.run(spec), spec["dt_out"])
    wrong = np.argwhere(got.reshape(want.shape) != want)
    assert wrong.size == 0, f"{len(wrong)} of {want.size} wrong, first at {wrong[0]}"


# (channels of one pass: 64, 128 and 256 in one, two and four wave groups; filters in tiles of 32, 64 and 128; images of up to 7 columns in pairs,
# the last one without a partner; one, three and five rows per workgroup, by one or more waves; rows of more than one strip, and of a strip and one column; rows of up to 225 pixels, by one wave and by several; one-pixel and one-row images)
FPROP = [geom(5, 28, 28, 64, 128), geom(2, 56, 56, 64, 72), geom(3, 13, 17, 40, 136), geom(6, 28, 28, 128, 128), geom(4, 9, 33, 104, 40),
         geom(9, 14, 14, 256, 72), geom(2, 15, 16, 136, 264), geom(31, 7, 7, 256, 64), geom(3, 5, 7, 64, 32), geom(7, 1, 1, 64, 64), geom(2, 1, 60, 32, 64),
         geom(40, 6, 3, 128, 24),
         geom(4, 56, 56, 64, 128, 2), geom(3, 27, 33, 40, 72, 2), geom(2, 30, 28, 128, 64, 2), geom(5, 28, 27, 256, 72, 2), geom(9, 14, 13, 128, 264, 2),
         geom(40, 14, 14, 256, 64), geom(70, 9, 17, 128, 64), geom(14, 18, 18, 128, 256, 2), geom(90, 7, 7, 256, 128), geom(85, 14, 14, 128, 64),
         geom(2, 112, 112, 64, 64), geom(1, 100, 225, 64, 200), geom(1, 40, 200, 64, 264), geom(2, 60, 81, 40, 264), geom(1, 60, 72, 128, 264), geom(1, 40, 100, 128, 264),
         geom(1, 60, 112, 64, 72, 2), geom(1, 160, 160, 64, 264, 2), geom(1, 100, 200, 40, 200, 2), geom(1, 1, 81, 72, 8, 2),
         geom(7, 15, 2, 104, 40, 2), geom(3, 1, 30, 64, 64, 2), geom(2, 32, 63, 64, 48, 2), geom(33, 14, 14, 256, 64, 2), geom(6, 27, 25, 104, 128, 2)]
DGRAD = [geom(5, 28, 28, 128, 64), geom(2, 56, 56, 72, 64), geom(3, 13, 17, 136, 40), geom(6, 28, 28, 128, 128), geom(4, 9, 33, 32, 104),
         geom(9, 14, 14, 72, 256), geom(5, 15, 16, 264, 136), geom(31, 7, 7, 64, 256), geom(3, 5, 7, 32, 64), geom(2, 14, 14, 64, 512), geom(9, 7, 7, 136, 520),
         geom(1, 60, 225, 264, 64), geom(1, 20, 200, 264, 64), geom(2, 64, 65, 128, 128), geom(1, 60, 72, 264, 72), geom(1, 30, 100, 264, 72), geom(1, 100, 160, 264, 32),
         geom(2, 8, 8, 72, 1024), geom(40, 14, 14, 64, 256), geom(90, 9, 17, 64, 128), geom(10, 25, 25, 40, 136), geom(43, 14, 14, 64, 128)]


@pytest.mark.parametrize("dt", ["bf16", "f16"])
@pytest.mark.parametrize("g", FPROP, ids=name)
def test_forward(g, dt):
    check_rounded(synth.conv_spec(dt_in=dt, dt_out=dt, integer=True, **g))


@pytest.mark.parametrize("dt", ["bf16", "f16"])
@pytest.mark.parametrize("g", DGRAD, ids=name)
def test_data_gradient(g, dt):
    check_rounded(synth.conv_grad_spec("dgrad", dt_in=dt, dt_out=dt, integer=True, **g))


@pytest.mark.parametrize("chain", [(), ("bias",), ("aux_load",), ("relu",), ("bias", "relu"), ("bias", "aux_load")])
def test_parts_of_the_chain(chain):
    check_rounded(synth.conv_spec(dt_in="f16", dt_out="f16", integer=True, epilogue=chain, **geom(3, 14, 14, 128, 64)))
    check_rounded(synth.conv_grad_spec("dgrad", dt_in="f16", dt_out="f16", integer=True, epilogue=chain, **geom(3, 14, 14, 64, 320)))


# (sums are read from registers where channels are not shared out, else from where waves' parts meet, with several passes from what is kept)
LAYERS = [("fprop", geom(3, 14, 14, 64, 64)), ("fprop", geom(3, 14, 14, 128, 64)), ("fprop", geom(3, 14, 14, 256, 72)), ("fprop", geom(4, 28, 28, 64, 64, 2)),
          ("fprop", geom(5, 28, 27, 256, 72, 2)), ("dgrad", geom(3, 14, 14, 64, 64)), ("dgrad", geom(3, 14, 14, 64, 256)), ("dgrad", geom(3, 14, 14, 72, 520))]


def layer(op, g, epilogue, dt="f16"):
    make = synth.conv_spec if op == "fprop" else lambda **k: synth.conv_grad_spec("dgrad", **k)
    return make(dt_in=dt, dt_out=dt, integer=True, epilogue=epilogue, **g)


@pytest.mark.parametrize("op,g", LAYERS, ids=lambda v: v if isinstance(v, str) else name(v))
def test_factors_and_the_types_of_the_bias(op, g):
    check_rounded(layer(op, g, (("scale", 0.5), "bias", ("aux_load", -0.5), "relu")))
    check_rounded(layer(op, g, (("scale", -0.25), ("aux_load", 3.0)), "bf16"))
    # fp32 with bits that 16-bit types don't hold, and at an address of 4 bytes' alignment; 16-bit at one of 2 bytes'
    spec = layer(op, g, ("bias", "aux_load"), "bf16")
    key = spec["epilogue"][0][1]
    small = synth.bits_to_f64(*spec["tensors"][key])
    spec["tensors"][key] = ((small * 1.25 + 2.0 ** -12).astype(np.float32), "f32")
    keep = []

    def shift(w):
        t = w.keep[0]
        keep.append(torch.empty(t.numel() + 1, dtype=t.dtype, device=t.device))
        keep[-1][1:].copy_(t)
        w.epi.c.steps[0].ptr = keep[-1][1:].data_ptr()

    check_rounded(spec)
    check_rounded(spec, shift)
    check_rounded(layer(op, g, ("bias", "relu")), shift)


@pytest.mark.parametrize("op,g", LAYERS, ids=lambda v: v if isinstance(v, str) else name(v))
def test_nan_and_infinities_under_the_chain_as_in_the_tile_kernel(op, g):
    for epilogue in (("relu",), ("bias", "relu"), ("bias",)):
        spec = layer(op, g, epilogue)
        x = spec["x" if op == "fprop" else "dy"]
        x[1, 4, 7, 3], x[0, 2, 5, 60], x[2, 9, 1, 17] = synth.to_bits(np.array([np.nan, np.inf, -np.inf]), "f16")
        held = DeviceWorkload(spec)
        assert "unnamed" in held.kernel()
        held.run()
        tile = DeviceWorkload(spec)
        tile.run(tune=Tuning(iterator=1))
        assert np.array_equal(held.result(), tile.result(), equal_nan=True)
        assert epilogue[-1] == "relu" or np.isnan(held.result()).any()


def test_other_chains_and_named_kernels_stay_where_they_were():
    g = geom(3, 14, 14, 128, 64)
    assert "unnamed" not in DeviceWorkload(synth.conv_spec(integer=True, epilogue=("silu",), **g)).kernel(), "what is reported runs"
    assert not any("held" in k for k in kernels_of(synth.conv_spec(integer=True, epilogue=("silu",), **g)))
    assert not any("held" in k for k in kernels_of(synth.conv_spec(integer=True, dt_out="f32", **g)))
    for tune in (Tuning(tile_m=64, tile_n=64, tile_k=64, stages=4), Tuning(raster=4), Tuning(iterator=1)):
        assert not any("held" in k for k in kernels_of(synth.conv_spec(integer=True, **g), tune))


def test_normal_inputs_and_repeated_launches():
    for spec in (synth.conv_spec(**geom(8, 56, 56, 64, 128)), synth.conv_grad_spec("dgrad", **geom(8, 28, 28, 128, 128))):
        assert any("conv_held_kernel" in k for k in kernels_of(spec))
        parity.check(spec)
        first, w = parity.gpu_result(spec)
        for _ in range(20):
            w.run()
        torch.cuda.synchronize()
        again, _ = parity.gpu_result(spec)
        assert np.array_equal(first, again)


def test_infinities_and_nan_stay_with_the_pixels_that_meet_them():
    spec = synth.conv_spec(integer=True, epilogue=(), dt_in="f16", dt_out="f16", **geom(2, 9, 20, 64, 64))
    want = orc_run.run(spec)
    spec["x"][1, 4, 7, 3], spec["x"][0, 8, 19, 60] = synth.to_bits(np.array([np.nan, np.inf]), "f16")
    got = parity.gpu_result(spec)[0].reshape(2, 9, 20, 64)
    near = np.zeros((2, 9, 20), bool)
    near[1, 3:6, 6:9] = near[0, 7:9, 18:20] = True
    assert np.array_equal(got[~near], want.reshape(got.shape)[~near]) and not np.isfinite(got[near]).all()
    assert np.isnan(got[1, 3:6, 6:9]).all()
