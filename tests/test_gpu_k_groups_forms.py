"""Kernels with K groups, the few-row kernels among them, each by name over the forms of a call beside packed operands: padded
leading and batch strides with NaN in the padding, tensors that the chain stores, chains over groups, infinities and NaN."""
import numpy as np
import pytest
import torch

import paper_2603_29010_amd as ucl
from paper_2603_29010_amd import synth
from paper_2603_29010_amd.binding import Epilogue, Tuning
from paper_2603_29010_amd.workload import DeviceWorkload

import parity
from test_gpu_k_groups import VARIANTS, ident, tuning

pytestmark = pytest.mark.gpu

TORCH = {"bf16": torch.bfloat16, "f16": torch.float16, "e4m3": torch.float8_e4m3fn, "e5m2": torch.float8_e5m2}
GUARD = 99.0


def of_modes(*modes):
    return [v for v in VARIANTS if v["mode"] in modes]


def _ints(g, *shape):
    return torch.randint(-2, 3, shape, generator=g).double()


def _padded(x, dt, lead, batch_stride):
    """x [batch, rows, contiguous] in a buffer with the given strides, NaN wherever x is not; returns (buffer, view)."""
    b, r, c = x.shape
    buf = torch.full((b * batch_stride,), float("nan")).to(TORCH[dt])
    raw = buf.view(torch.uint8) if buf.element_size() == 1 else buf.view(torch.int16)
    raw.as_strided((b, r, c), (batch_stride, lead, 1)).copy_(x.to(TORCH[dt]).view(raw.dtype))
    return buf.cuda()


@pytest.mark.parametrize("v", of_modes(0), ids=ident)
def test_padded_strides_and_stored_tensors(v):
    g, dt = torch.Generator().manual_seed(11), v["dt"]
    unit = 16 if dt in ("e4m3", "e5m2") else 8
    stream = torch.cuda.current_stream().cuda_stream
    for (b, M, N, K) in ((3, 40, 72, 5 * 64 + unit), (2, 72, 136, unit), (2, 16, 200, 64 * 9 - unit)):
        A, B = _ints(g, b, M, K), _ints(g, b, N, K)
        want = A @ B.transpose(1, 2)
        a, w = (A.transpose(1, 2), (K, M)) if v["a_layout"] else (A, (M, K)), (B.transpose(1, 2), (K, N)) if v["b_layout"] else (B, (N, K))
        lda, ldb = a[1][1] + unit, w[1][1] + 2 * unit
        abs_, bbs = a[1][0] * lda + unit, w[1][0] * ldb + unit
        da, db = _padded(a[0].contiguous(), dt, lda, abs_), _padded(w[0].contiguous(), dt, ldb, bbs)
        ldd, lds = N + 3, N + 5
        D = torch.full((b * (M * ldd + 7),), GUARD, device="cuda")
        S = torch.full((b * (M * lds + 9),), GUARD, device="cuda")
        a_st = (1, lda) if v["a_layout"] else (lda, 1)
        b_st = (ldb, 1) if v["b_layout"] else (1, ldb)
        epi = Epilogue([("scale", 2.0), ("aux_store", S.data_ptr(), "f32", lds, M * lds + 9), ("relu",)])
        ucl.ucl_batched_gemm(b, M, N, K, da.data_ptr(), dt, *a_st, abs_, db.data_ptr(), dt, *b_st, bbs, D.data_ptr(), "f32", ldd, 1, M * ldd + 7,
                             epi, tuning(v), stream)
        torch.cuda.synchronize()
        for name, t, ld, bs, ref in (("D", D, ldd, M * ldd + 7, (2 * want).clamp(min=0)), ("stored", S, lds, M * lds + 9, 2 * want)):
            t = t.cpu()
            rows = t.as_strided((b, M, N), (bs, ld, 1))
            assert torch.equal(rows.double(), ref), (ident(v), name, b, M, N, K)
            rows.fill_(GUARD)
            assert (t == GUARD).all(), f"{ident(v)}: {name} written outside its rows"


@pytest.mark.parametrize("chain", [("bias", "aux_load", "silu"), ("per_row_scale", "bias", ("aux_store", "kept", "f32"), "relu"),
                                   ("column_broadcast", "per_col_scale", "gelu_tanh")])
@pytest.mark.parametrize("v", of_modes(1), ids=ident)
def test_chains_over_groups(v, chain):
    spec = synth.grouped_spec([0, 1, 16, 33, 0, 70], 136, 1200, dt_in=v["dt"], dt_out="f16" if v["dt"] == "f16" else "bf16", epilogue=chain)
    if not any(st[0] == "aux_store" for st in spec["epilogue"]):
        parity.check(spec, tuning(v), label=f"{ident(v)} {chain}")
        return
    w = DeviceWorkload(spec)
    w.run(tune=tuning(v))
    plain, upto = dict(spec, epilogue=[st for st in spec["epilogue"] if st[0] != "aux_store"]), dict(spec, epilogue=spec["epilogue"][:2], dt_out="f32")
    for got, s in ((w.result(), plain), (w.aux_result("kept"), upto)):
        ref, absacc = parity.oracle_result(s)
        parity.compare(got.reshape(ref.shape), ref, absacc, s, f"{ident(v)} {chain}")


def _same_specials(got, want, what):
    assert np.array_equal(np.isnan(got), np.isnan(want)), f"{what}: NaN in other places"
    assert np.array_equal(np.isposinf(got), np.isposinf(want)) and np.array_equal(np.isneginf(got), np.isneginf(want)), f"{what}: infinities"
    ok = np.isfinite(want)
    assert np.array_equal(got[ok], want[ok]), f"{what}: finite values beside them"


@pytest.mark.parametrize("v", of_modes(0), ids=ident)
def test_infinities_and_nan(v):
    # (e4m3 has no infinity)
    dt = v["dt"]
    g = torch.Generator().manual_seed(5)
    unit = 16 if dt in ("e4m3", "e5m2") else 8
    for (M, N, K) in ((40, 72, 5 * 64 + unit), (16, 40, unit)):
        A, B = _ints(g, M, K), _ints(g, N, K)
        special = float("nan") if dt == "e4m3" else float("inf")
        A[3, K - 1] = special
        A[5, 0] = float("nan")
        B[7, K // 2] = -special
        want = (A[:, None, :] * B[None, :, :]).sum(-1).numpy()
        a, b = (A.t() if v["a_layout"] else A).contiguous().to(TORCH[dt]).cuda(), (B.t() if v["b_layout"] else B).contiguous().to(TORCH[dt]).cuda()
        D = torch.empty(M, N, device="cuda")
        ucl.ucl_gemm(M, N, K, a.data_ptr(), dt, *((1, M) if v["a_layout"] else (K, 1)), b.data_ptr(), dt, *((N, 1) if v["b_layout"] else (1, K)),
                     D.data_ptr(), "f32", N, 1, None, tuning(v), torch.cuda.current_stream().cuda_stream)
        _same_specials(D.double().cpu().numpy(), want, f"{ident(v)} {M}x{N}x{K}")


@pytest.mark.parametrize("v", of_modes(2), ids=ident)
def test_nan_pixels_stay_where_their_taps_are(v):
    dt = v["dt"]
    g = torch.Generator().manual_seed(6)
    N, H, W, C, Ko = 2, 9, 7, 40, 72
    x, w = _ints(g, N, H, W, C), _ints(g, Ko, 3, 3, C)
    x[0, 0, 0, 5], x[1, 8, 6, 0], x[1, 4, 3, 39] = float("nan"), float("inf"), float("nan")
    want = torch.nn.functional.conv2d(torch.where(torch.isfinite(x), x, torch.zeros_like(x)).permute(0, 3, 1, 2), w.permute(0, 3, 1, 2), padding=1)
    want = want.permute(0, 2, 3, 1).contiguous()
    for n, h, q, c in ((0, 0, 0, 5), (1, 8, 6, 0), (1, 4, 3, 39)):
        for r in range(3):
            for s in range(3):
                p_, q_ = h + 1 - r, q + 1 - s
                if 0 <= p_ < H and 0 <= q_ < W:
                    want[n, p_, q_] += x[n, h, q, c] * w[:, r, s, c]
    dx, dw = x.to(TORCH[dt]).cuda(), w.to(TORCH[dt]).cuda()
    D = torch.empty(N, H, W, Ko, device="cuda")
    ucl.ucl_conv2d_fprop(N, H, W, C, Ko, 3, 3, 1, 1, 1, 1, 1, 1, dx.data_ptr(), dt, dw.data_ptr(), dt, D.data_ptr(), "f32", None, tuning(v),
                         torch.cuda.current_stream().cuda_stream)
    _same_specials(D.double().cpu().numpy(), want.numpy(), ident(v))
