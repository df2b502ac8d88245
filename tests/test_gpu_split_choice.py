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
        serial = ucl.ucl_workspace_size("gemm", dt, out, Tuning(split_k="serial"), M=M, N=N, K=K)[1]
        assert slices > 1 or out != "f32" or serial == 1, "fp32 sums stay in slices"
        check = parity.check_exact if out == "f32" else parity.check      # (16-bit outputs round)
        for nbytes in (need, 512 << 20):
            ws = workspace(nbytes)
            check(spec, tuning(ws), label=f"{dt} -> {out}, {slices} slices, {nbytes} bytes")


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


def served(spec, tune, label):
    check = parity.check_exact if spec["dt_out"] == "f32" else parity.check
    check(spec, tune, label=label)


@pytest.mark.parametrize("what", ["none", "off 16 bytes", "counters only"])
def test_calls_that_need_no_workspace_by_the_general_rule_run_without_one(what):
    # the choice would split these, the general rule does not: they always ran with any workspace, or none
    ws = torch.empty(1 << 20, dtype=torch.uint8, device="cuda")
    given = {"none": dict(workspace=0, workspace_bytes=0), "off 16 bytes": dict(workspace=ws.data_ptr() + 8, workspace_bytes=ws.numel() - 8),
             "counters only": dict(workspace=ws.data_ptr(), workspace_bytes=COUNTERS)}[what]
    tune = Tuning(split_k="parallel", **given)
    for dt in ("bf16", "f16"):
        gemm = synth.gemm_spec(1152, 952, 3128, dt_in=dt, dt_out=dt, epilogue=(), integer=True)
        assert ucl.ucl_workspace_size("gemm", dt, dt, Tuning(split_k="parallel"), M=1152, N=952, K=3128)[1] > 1
        served(gemm, tune, f"gemm {dt}, {what}")
        wgrad = synth.conv_grad_spec("wgrad", dt_in=dt, dt_out="f32", integer=True, Nb=2, H=37, W=37, C=8, Ko=832, R=5, S=5, pad=(2, 2), stride=(3, 3))
        assert ucl.ucl_workspace_size("conv2d_wgrad", dt, "f32", Tuning(split_k="parallel"), conv=(2, 37, 37, 8, 832, 5, 5, 2, 2, 3, 3, 1, 1))[1] > 1
        served(wgrad, tune, f"wgrad {dt}, {what}")


def test_a_workspace_that_holds_the_general_rule_serves_it():
    # bytes of the general rule's partial tiles, fewer than those of the slices that would be chosen
    spec = synth.gemm_spec(8, 8, 9488, dt_in="f16", dt_out="f16", epilogue=(), integer=True)
    assert ucl.ucl_workspace_size("gemm", "f16", "f16", Tuning(split_k="parallel"), M=8, N=8, K=9488)[0] > 557056
    ws = workspace(557056)
    served(spec, tuning(ws), "gemm")
    spec = synth.conv_grad_spec("wgrad", dt_in="bf16", dt_out="f32", integer=True, Nb=7, H=40, W=40, C=8, Ko=40, R=1, S=1, pad=(0, 0), stride=(3, 3))
    assert ucl.ucl_workspace_size("conv2d_wgrad", "bf16", "f32", Tuning(split_k="parallel"), conv=(7, 40, 40, 8, 40, 1, 1, 0, 0, 3, 3, 1, 1))[0] > 147456
    ws = workspace(147456)
    served(spec, tuning(ws), "wgrad")
    with pytest.raises(ucl.UclError) as e:           # less than either needs: refused, as it always was
        served(spec, tuning(ws[:147440]), "wgrad")
    assert e.value.status == "UCL_ERR_WORKSPACE"
