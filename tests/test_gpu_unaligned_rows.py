"""Outputs and epilogue tensors whose rows start at any element: every residue of the last columns (pieces of 4, 2 and 1
elements), base pointers off 16 bytes, odd leading strides; exact on integers, and nothing outside the rows is touched."""
import numpy as np
import pytest
import torch

import paper_2603_29010_amd as ucl
from paper_2603_29010_amd.binding import Epilogue, Tuning

pytestmark = pytest.mark.gpu

TORCH = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}
GUARD = 99.0


@pytest.mark.parametrize("dt_out", ["bf16", "f16", "f32"])
@pytest.mark.parametrize("chain", ["fused", "steps"])
@pytest.mark.parametrize("tile", [(64, 64, 32, 3), (128, 128, 32, 4), (256, 128, 32, 3), (64, 64, 64, 4, 2), (16, 16, 64, 1), (16, 32, 64, 1),
                                  (32, 32, 64, 1), (32, 64, 64, 1)])
def test_rows_at_any_alignment(dt_out, chain, tile):
    g = torch.Generator().manual_seed(7)
    M, K, off = 70, 64, 1
    ints = lambda *s: torch.randint(-2, 3, s, generator=g).float()  # noqa: E731
    for N in list(range(1, 18)) + [63, 64, 65, 71, 130, 133]:
        ld = N + 3
        A, B, R, bias = ints(M, K), ints(N, K), ints(M, ld), ints(N)
        want = A.double() @ B.double().t() + bias.double() + 2.0 * R[:, :N].double()
        cuda = lambda t, dt: t.to(TORCH[dt]).cuda()  # noqa: E731
        a, b = cuda(A, "bf16"), cuda(B, "bf16")
        res = torch.zeros(off + M * ld, dtype=TORCH[dt_out], device="cuda")
        res[off:] = cuda(R.reshape(-1), dt_out)
        bs = torch.zeros(off + N, dtype=TORCH[dt_out], device="cuda")
        bs[off:] = cuda(bias, dt_out)
        out = torch.full((off + M * ld + 8,), GUARD, dtype=TORCH[dt_out], device="cuda")
        aux = torch.full((off + M * ld + 8,), GUARD, dtype=TORCH[dt_out], device="cuda")
        at = lambda t: t.data_ptr() + off * t.element_size()  # noqa: E731
        steps = [("bias", at(bs), dt_out), ("aux_load", at(res), dt_out, ld, 0, 2.0)]
        if chain == "steps":
            steps.append(("aux_store", at(aux), dt_out, ld))
        ucl.ucl_gemm(M, N, K, a.data_ptr(), "bf16", K, 1, b.data_ptr(), "bf16", 1, K, at(out), dt_out, ld, 1, Epilogue(steps),
                     Tuning(*tile[:4], k_groups=sum(tile[4:])),
                     torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        for name, t in (("D", out), ("aux", aux))[:2 if chain == "steps" else 1]:
            t = t.double().cpu()
            rows = t[off:off + M * ld].view(M, ld)
            assert torch.equal(rows[:, :N], want), (name, N, np.argwhere((rows[:, :N] != want).numpy())[:4])
            assert (rows[:, N:] == GUARD).all() and t[0] == GUARD and (t[off + M * ld:] == GUARD).all(), (name, N)
