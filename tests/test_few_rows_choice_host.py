"""Which kernels and bands are chosen for problems around a tile per CU, as measured (host only): calls that a cost row or a line once sent to a slower kernel."""
import pytest

import paper_2603_29010_amd as ucl


def chosen(M, N, K, dt, batch=0, out=None):
    kw = dict(M=M, N=N, K=K, **({"batch": batch} if batch else {}))
    return ucl.ucl_select_tuning("batched_gemm" if batch else "gemm", dt, out or ("bf16" if dt == "e4m3" else dt), **kw)


@pytest.mark.parametrize("M,N,K,dt,tile", [(40, 3664, 2752, "bf16", (32, 32)),        # 9.6 us, 16x32 tiles 10.3
                                           (58, 2744, 1984, "bf16", (32, 32)),        # 7.8 us, 16x32 tiles 8.3
                                           (39, 3184, 2016, "f16", (32, 32))])        # 8.0 us, 16x32 tiles 8.9
def test_somewhat_more_tiles_than_cus(M, N, K, dt, tile):
    t = chosen(M, N, K, dt)
    assert (t["tile_m"], t["tile_n"], t["stages"]) == (*tile, 1)


@pytest.mark.parametrize("batch,M,N,K,dt", [(64, 16, 512, 1024, "bf16"), (32, 24, 1024, 768, "f16"), (16, 40, 2048, 1024, "e4m3"), (100, 8, 256, 512, "bf16")])
def test_batches_are_priced_by_what_they_run(batch, M, N, K, dt):
    # more than 256 tiles at any tile of up to 32 rows, and those run with one stage buffer per wave, 0.5 to 0.9 of the time of several
    t = chosen(M, N, K, dt, batch, "f32")
    assert t["stages"] == 1 and t["tile_m"] <= 32


@pytest.mark.parametrize("M,N,K,dt", [(35, 7304, 8016, "bf16"), (36, 8120, 5376, "f16"), (33, 7296, 7552, "bf16")])
def test_64_rows_of_eight_waves_need_tiles_for_half_of_the_cus(M, N, K, dt):
    # 52, 26 and 37 us on the 64x64 kernel of eight waves, 40, 20 and 28 us on the 32x64 one
    assert chosen(M, N, K, dt)["tile_m"] == 32


@pytest.mark.parametrize("M,N,K,dt,bands", [(610, 2024, 5408, "f16", 10), (591, 1776, 3104, "bf16", 10), (673, 1520, 4736, "bf16", 6), (863, 1248, 3088, "bf16", 7)])
def test_bands_of_64_row_tiles_are_even(M, N, K, dt, bands):
    t = chosen(M, N, K, dt)
    assert t["tile_m"] == 64 and t["raster"] == bands
