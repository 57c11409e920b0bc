"""The linear with float activations on both sides of its one-launch route (32x32 tiles, at most 256 of them, K % 64 == 0,
K <= 1024): bit for bit the quantizer followed by the linear on codes, which the oracle's tests hold to the paper."""
import numpy as np
import pytest

import oracle
from helpers import RTOL, assert_codes_match_with_tie_band, assert_float_close, to_dev, to_np

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mkq():
    import torch
    assert torch.cuda.is_available()
    import paper_2203_13483_amd as m
    m.load()
    return m


@pytest.mark.parametrize("dtype", [np.float32, np.float16])
@pytest.mark.parametrize("M,N,K", [(1, 1, 64), (1, 32, 1024), (31, 33, 128), (33, 40, 704), (128, 768, 768), (70, 2312, 832),
                                   (256, 1024, 1024), (257, 1000, 768), (40, 64, 1088), (40, 64, 96)])
def test_one_launch_equals_quantizer_and_linear(mkq, M, N, K, dtype):
    import torch
    rng = np.random.default_rng(M + N + K)
    x = rng.standard_normal((M, K)).astype(np.float32)
    x[rng.random((M, K)) < 0.01] *= 8
    s_x = np.float32(1.0 / 3)
    x.flat[:3] = (np.nan, np.inf, -np.inf)
    x.flat[3:40] = (rng.integers(-9, 9, 37) + 0.5) * s_x  # exact and near ties
    x = x.astype(dtype)
    Wc = rng.integers(-8, 8, (N, K), dtype=np.int8)
    s_w = rng.uniform(0.001, 0.05, N).astype(np.float32)
    bias = rng.normal(0, 0.5, N).astype(np.float32)
    res = rng.normal(0, 1, (M, N)).astype(np.float16)
    codes = oracle.quantize(x.astype(np.float32), s_x)
    w = mkq.mkq_pack_codes_int4(to_dev(Wc)).reshape(-1)
    ws = torch.zeros(mkq.mkq_linear_int4_workspace_bytes(M, N, K, mkq.MKQ_F32), dtype=torch.uint8, device="cuda")
    args = (to_dev(x), float(s_x), w, to_dev(s_w), to_dev(bias), N, K)
    ref = oracle.linear_int4(codes, s_x, Wc, s_w, bias)
    r = mkq.mkq_linear_int4(*args, mkq.MKQ_F32, want_acc=True, workspace=ws)
    assert np.array_equal(to_np(r["acc"]), ref["acc"]) and np.array_equal(to_np(r["out"]), ref["y"])
    assert np.array_equal(to_np(ws)[: M * K // 2].reshape(M, K // 2), oracle.pack_nibbles(codes))
    ref = oracle.linear_int4(codes, s_x, Wc, s_w, bias, residual=res.astype(np.float32), out_dtype=oracle.F16)
    r = mkq.mkq_linear_int4(*args, mkq.MKQ_F16, residual=to_dev(res), workspace=ws)
    assert np.array_equal(to_np(r["out"]).astype(np.float32), ref["y"])
    if N % 2 == 0:
        ref = oracle.linear_int4(codes, s_x, Wc, s_w, bias, s_next=0.7)
        r = mkq.mkq_linear_int4(*args, mkq.MKQ_I4, s_next=0.7, workspace=ws)
        assert np.array_equal(to_np(r["out"]), oracle.pack_nibbles(ref["q"]))


def test_output_in_place_of_the_activations(mkq):
    """out over a: the activations are read by every workgroup, so such a call keeps its quantizer launch."""
    import torch
    rng = np.random.default_rng(3)
    M = N = K = 256
    x = rng.standard_normal((M, K)).astype(np.float32)
    Wc = rng.integers(-8, 8, (N, K), dtype=np.int8)
    s_w = rng.uniform(0.001, 0.05, N).astype(np.float32)
    ref = oracle.linear_int4(oracle.quantize(x, np.float32(0.3)), np.float32(0.3), Wc, s_w, None)
    xd = to_dev(x)
    mkq.mkq_linear_int4(xd, 0.3, mkq.mkq_pack_codes_int4(to_dev(Wc)).reshape(-1), to_dev(s_w), None, N, K, mkq.MKQ_F32, out=xd)
    assert np.array_equal(to_np(xd), ref["y"])


@pytest.mark.parametrize("M,N,K", [(64, 32, 1024), (64, 64, 832)])
def test_output_over_the_workspace(mkq, M, N, K):
    """out over the workspace at sizes that the GEMM's own launch serves with a single workgroup, which reads every code
    before it writes: such a call keeps its quantizer launch (in one launch, the codes of one 32-row tile would race with
    the results of the other)."""
    import torch
    rng = np.random.default_rng(K)
    x = rng.standard_normal((M, K)).astype(np.float32)
    Wc = rng.integers(-8, 8, (N, K), dtype=np.int8)
    s_w = rng.uniform(0.001, 0.05, N).astype(np.float32)
    ref = oracle.linear_int4(oracle.quantize(x, np.float32(0.3)), np.float32(0.3), Wc, s_w, None)
    ws = torch.zeros(mkq.mkq_linear_int4_workspace_bytes(M, N, K, mkq.MKQ_F32), dtype=torch.uint8, device="cuda")
    out = ws[: M * N * 4].view(torch.float32).reshape(M, N)
    mkq.mkq_linear_int4(to_dev(x), 0.3, mkq.mkq_pack_codes_int4(to_dev(Wc)).reshape(-1), to_dev(s_w), None, N, K, mkq.MKQ_F32,
                        out=out, workspace=ws)
    assert np.array_equal(to_np(out), ref["y"])


@pytest.mark.parametrize("dtype", [np.float32, np.float16])
@pytest.mark.parametrize("M,N,K", [(1, 8, 64), (33, 40, 704), (70, 200, 832), (128, 768, 768)])
def test_every_output_of_the_general_epilogue(mkq, M, N, K, dtype):
    """GELU, codes beside a float output, and code rows with a pitch (zero codes behind the last channel), with float
    activations; only codes behind a GELU may fall either way at a tie."""
    import torch
    rng = np.random.default_rng(M * N + K)
    x = rng.standard_normal((M, K)).astype(dtype)
    Wc = rng.integers(-8, 8, (N, K), dtype=np.int8)
    s_w = rng.uniform(0.001, 0.05, N).astype(np.float32)
    bias = rng.normal(0, 0.5, N).astype(np.float32)
    s_x = np.float32(0.34)
    codes = oracle.quantize(x.astype(np.float32), s_x)
    args = (to_dev(x), float(s_x), mkq.mkq_pack_codes_int4(to_dev(Wc)).reshape(-1), to_dev(s_w), to_dev(bias), N, K)
    pitch = N + 24
    pad = np.zeros((M, 24), np.int8)
    ref = oracle.linear_int4(codes, s_x, Wc, s_w, bias, s_next=0.7)
    q = torch.full((M, pitch // 2), 255, dtype=torch.uint8, device="cuda")
    r = mkq.mkq_linear_int4(*args, mkq.MKQ_F32, s_next=0.7, q_out=q, q_pitch=pitch)
    assert np.array_equal(to_np(r["out"]), ref["y"])
    assert np.array_equal(oracle.unpack_nibbles(to_np(q), pitch), np.hstack([ref["q"], pad]))
    r = mkq.mkq_linear_int4(*args, mkq.MKQ_I4, s_next=0.7, q_pitch=pitch)
    assert np.array_equal(oracle.unpack_nibbles(to_np(r["out"]), pitch), np.hstack([ref["q"], pad]))
    refg = oracle.linear_int4(codes, s_x, Wc, s_w, bias, act=oracle.ACT_GELU, s_next=0.7)
    r = mkq.mkq_linear_int4(*args, mkq.MKQ_F32, act=mkq.MKQ_ACT_GELU, s_next=0.7, want_q=True)
    assert_float_close(to_np(r["out"]), refg["y"], RTOL[0], "GELU")
    assert_codes_match_with_tie_band(oracle.unpack_nibbles(to_np(r["q"]), N), refg["q"], refg["y"], 0.7, what="GELU codes")
