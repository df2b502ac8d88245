"""Few-row kernels on either side of a tile for each CU: with more tiles the launch takes the ones with one stage buffer per wave (gemm, batched),
and grouped calls have variants of their own; exact over ragged rows, columns and K, K shorter than the waves, batches and the library's choice."""
import pytest

import paper_2603_29010_amd as ucl
from paper_2603_29010_amd import synth
from paper_2603_29010_amd.binding import Tuning

import parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile", [(16, 16), (16, 32), (32, 32), (32, 64)], ids=lambda t: "%dx%d" % t)
@pytest.mark.parametrize("dt", ["bf16", "f16", "e4m3", "e5m2"])
def test_both_depths(dt, tile):
    tune, unit = Tuning(*tile, 64, 1, k_groups=4), 2 if dt in ("e4m3", "e5m2") else 1
    # one row of 256 and 257 tiles, two rows of tiles with ragged edges; fewer steps of K than waves, one more, a ragged last one
    for M, N, K in ((5, 256 * tile[1], 64 * unit), (tile[0], 256 * tile[1] + 3, 5 * 64 * unit), (tile[0] + 1, 200 * tile[1] - 5, (9 * 64 - 8) * unit),
                    (3 * tile[0], 130 * tile[1] + 8, 16)):
        spec = synth.gemm_spec(M, N, K, dt_in=dt, dt_out="f32", epilogue=(), integer=True)
        parity.check_exact(spec, tune, label=f"{dt} {tile} {M}x{N}x{K}")
    spec = synth.batched_spec(90, 2 * tile[0] - 3, 3 * tile[1] - 8, 328 * unit, dt_in=dt, dt_out="f32", epilogue=(), integer=True)
    parity.check_exact(spec, tune, label=f"{dt} {tile} batched")
    spec = synth.gemm_spec(tile[0] - 1, 259 * tile[1] + 5, 600 * unit - 600 * unit % 16, dt_in=dt, dt_out="f16" if dt == "f16" else "bf16", epilogue=("bias", "aux_load", "silu"))
    parity.check(spec, tune, label=f"{dt} {tile} chain")


@pytest.mark.parametrize("dt", ["bf16", "f16", "e4m3", "e5m2"])
def test_grouped_choice(dt):
    # experts that decode: the one-buffer variants are chosen, and named again they are the same
    rows = [(7 * g) % 33 for g in range(64)]
    spec = synth.grouped_spec(rows, 1096, 1040, dt_in=dt, dt_out="f32", epilogue=(), integer=True)
    t = ucl.ucl_select_tuning("grouped_gemm", dt, "f32", M_g=rows, N=1096, K=1040)
    assert (t["tile_m"], t["stages"], t["k_groups"]) == (32, 4, 4)
    parity.check_exact(spec, None, label=f"{dt} chosen")
    parity.check_exact(spec, Tuning(**t), label=f"{dt} named")


@pytest.mark.parametrize("dt", ["bf16", "f16", "e4m3", "e5m2"])
@pytest.mark.parametrize("batch,M,N,K", [(64, 16, 520, 336), (20, 25, 1000, 400), (9, 65, 700, 400)], ids=lambda v: str(v))
def test_batches_and_more_rows_chosen(batch, M, N, K, dt):
    # batches of more tiles than CUs, as the library chooses: exact, and a chain over them
    unit = 2 if dt in ("e4m3", "e5m2") else 1
    t = ucl.ucl_select_tuning("batched_gemm", dt, "f32", batch=batch, M=M, N=N, K=K * unit)
    assert t["stages"] == 1 and t["k_groups"] == 4 and batch * -(-M // t["tile_m"]) * -(-N // t["tile_n"]) > 256
    parity.check_exact(synth.batched_spec(batch, M, N, K * unit, dt_in=dt, dt_out="f32", epilogue=(), integer=True), None, label=f"{dt} chosen")
    parity.check(synth.batched_spec(batch, M, N, K * unit, dt_in=dt, dt_out="f16" if dt == "f16" else "bf16", epilogue=("bias", "aux_load", "silu")), None, label=f"{dt} chain")


@pytest.mark.parametrize("rows", [9, 10, 11, 17, 21])
def test_even_bands(rows):
    # rows of 64-row tiles in one, two and three bands, the last one shorter where they do not divide
    spec = synth.gemm_spec(64 * rows - 7, 840, 1032, dt_in="bf16", dt_out="f32", epilogue=(), integer=True)
    for tile in ((64, 64, 64, 4), (64, 64, 32, 4)):
        parity.check_exact(spec, Tuning(*tile), label=f"{rows} rows of tiles {tile}")
