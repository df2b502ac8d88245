"""Parallel split-K GEMMs that leave the slices to the library: exact on integers whichever way the choice goes (not split, tiles
of 64 or of 128), in the workspace that ucl_workspace_size() names and in smaller and larger ones, and replayed from a graph; the
output type that keeps its slices; a leading stride that only the smaller tiles can address."""
import pytest
import torch

import paper_2603_29010_amd as ucl
from paper_2603_29010_amd import synth
from paper_2603_29010_amd.binding import Tuning
from paper_2603_29010_amd.workload import DeviceWorkload

import parity

pytestmark = pytest.mark.gpu
COUNTERS = 65536


def workspace(nbytes):
    ws = torch.empty(max(nbytes, COUNTERS), dtype=torch.uint8, device="cuda")
    ucl.ucl_workspace_init(ws.data_ptr(), ws.numel(), torch.cuda.current_stream().cuda_stream)
    return ws


def tuning(ws):
    return Tuning(split_k="parallel", workspace=ws.data_ptr(), workspace_bytes=ws.numel())


@pytest.mark.parametrize("dt_out", ["same", "f32"])
@pytest.mark.parametrize("M,N,K", [(72, 136, 4096), (33, 40, 8192), (33, 40, 8200), (200, 72, 5 * 64 + 8), (264, 264, 20040), (512, 512, 40008),
                                   (1, 8, 72)])
def test_exact(M, N, K, dt_out):
    for dt in ("bf16", "f16"):
        out = dt if dt_out == "same" else dt_out
        spec = synth.gemm_spec(M, N, K, dt_in=dt, dt_out=out, epilogue=(), integer=True)
        need, slices = ucl.ucl_workspace_size("gemm", dt, out, Tuning(split_k="parallel"), M=M, N=N, K=K)
        general = ucl.ucl_workspace_size("gemm", dt, out, Tuning(64, 64, 32, 3, split_k="parallel"), M=M, N=N, K=K)[0]
        assert slices > 1 or out != "f32" or general == 0, "fp32 sums stay in slices"
        check = parity.check_exact if out == "f32" else parity.check      # (16-bit outputs round)
        for nbytes in (need, 512 << 20):
            ws = workspace(nbytes)
            check(spec, tuning(ws), label=f"{dt} -> {out}, {slices} slices, {nbytes} bytes")
        ws = workspace(general)
        try:
            check(spec, tuning(ws), label=f"{dt} -> {out}, {general} bytes")
        except ucl.UclError as e:
            assert e.status == "UCL_ERR_WORKSPACE" and general < need


def test_graph_replays():
    for (M, N, K) in ((88, 160, 4200), (256, 256, 16384)):
        w = DeviceWorkload(synth.gemm_spec(M, N, K, dt_in="bf16", dt_out="bf16", epilogue=("bias", "relu")))
        ws = workspace(64 << 20)
        tune = tuning(ws)
        w.run(tune=tune)
        torch.cuda.synchronize()
        first = w.result_bits().copy()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            w.run(tune=tune)
        for _ in range(3):
            w.D.zero_()
            g.replay()
            torch.cuda.synchronize()
            assert (w.result_bits() == first).all()


def test_leading_stride_beyond_the_large_tiles():
    # 64 rows of 8.5 M elements are just addressable in 32 bits, the 128 rows that this size would be given are not
    M, N, K, lda = 512, 2048, 1024, 8_500_000
    A = torch.empty((M - 1) * lda + K, dtype=torch.bfloat16, device="cuda")
    a = A.as_strided((M, K), (lda, 1))
    a.copy_(torch.randint(-3, 4, (M, K), device="cuda"))
    B = torch.randint(-3, 4, (N, K), device="cuda").to(torch.bfloat16)
    D = torch.empty(M, N, dtype=torch.float32, device="cuda")
    ucl.ucl_gemm(M, N, K, A.data_ptr(), "bf16", lda, 1, B.data_ptr(), "bf16", 1, K, D.data_ptr(), "f32", N, 1, None, None,
                 torch.cuda.current_stream().cuda_stream)
    assert torch.equal(D, a.float().contiguous() @ B.float().t())
