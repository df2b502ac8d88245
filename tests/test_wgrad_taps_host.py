"""Which filter gradients the kernel with all taps in one workgroup may serve, asked of the size query (host only)."""
import numpy as np
import pytest

import paper_2603_29010_amd as ucl
from paper_2603_29010_amd.binding import Epilogue, Tuning


def slices(conv, dt_out="bf16", epi=None):
    return ucl.ucl_workspace_size("conv2d_wgrad", "bf16", dt_out, tune=Tuning(split_k="parallel"), conv=conv, epi=epi)


def tall(H, stride=1):
    return (1, H, 1, 32, 56, 3, 3, 1, 1, stride, stride, 1, 1)


def test_row_indexes_are_exact_as_far_as_it_is_chosen():
    # the kernel's fp32 step, (vp + 1/2) * (1 / (P + 1)), at both sides of every multiple of P + 1 that vp = p0 + wq - 2 + P + 1 reaches (p0 <= P,
    # wq <= (127 + 3 (Q + 1)) / (Q + 1) < 68), for every P that is admitted
    rows = np.arange(2, (1 << 20) + 1, dtype=np.int64)
    rcp = np.float32(1) / rows.astype(np.float32)
    for k in range(1, 68):
        for side in (-1, 0):
            vp = k * rows + side
            use = vp <= 2 * rows + 66
            got = ((vp.astype(np.float32) + np.float32(.5)) * rcp).astype(np.int64)
            assert np.array_equal(got[use], (vp // rows)[use]), (k, side)


@pytest.mark.parametrize("H,stride", [(8483559, 1), (9320585, 1), (1 << 20, 1), (1 << 21, 2)])
def test_taller_images_stay_with_the_tile_kernel(H, stride):
    # (a chain with a ReLU is the tile kernel's at any size)
    assert slices(tall(H, stride)) == slices(tall(H, stride), epi=Epilogue([("relu",)]))


def test_the_tallest_image_it_serves():
    assert slices(tall((1 << 20) - 1)) != slices(tall((1 << 20) - 1), epi=Epilogue([("relu",)]))
