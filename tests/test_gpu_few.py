"""The linears of few tokens and small linears (csrc/gemm_few.hip) against the oracle: every tile of the rule, one piece of a row and
fewer pieces than waves, pieces that do not divide evenly over the waves, ragged tokens and channels, the accumulator extremes.
Integer sums and correctly rounded binary32 epilogues: exact; only codes behind a GELU may fall either way at a tie."""
import numpy as np
import pytest

import oracle
from helpers import assert_codes_match_with_tie_band, to_dev, to_np

pytestmark = pytest.mark.gpu

# (M, N, bytes of a row), one line per tile of the 4-bit rule: 16x16, 16x32, 32x32, 32x64 and 64x64 channels x tokens, then the long
# rows.  (8 bits take the persistent kernels for some.)
SHAPES = [(1, 8, 64), (16, 40, 128), (7, 130, 576),
          (17, 200, 192), (32, 24, 64),
          (33, 72, 320), (100, 768, 384), (24, 8200, 64),
          (600, 1000, 192), (640, 1040, 64),
          (1000, 600, 1024), (650, 1000, 1088),
          (5, 42, 2048), (20, 104, 2176), (40, 200, 4096), (300, 1000, 2048), (1000, 600, 2048), (61, 16500, 2048)]


@pytest.fixture(scope="module")
def mkq():
    import torch
    assert torch.cuda.is_available()
    import paper_2203_13483_amd as m
    m.load()
    return m


@pytest.mark.parametrize("bits", [4, 8])
@pytest.mark.parametrize("M,N,row", SHAPES)
def test_tiles(mkq, bits, M, N, row):
    K = row * 8 // bits
    rng = np.random.default_rng(M + N + K)
    q = 1 << (bits - 1)
    A = rng.integers(-q, q, (M, K), dtype=np.int8)
    Wc = rng.integers(-q, q, (N, K), dtype=np.int8)
    A[0], Wc[0] = -q, -q  # the largest sum
    s_w = rng.uniform(0.001, 0.05, N).astype(np.float32) / (1 if bits == 4 else 256)
    s_x, bias = np.float32(0.02), rng.normal(0, 0.5, N).astype(np.float32)
    res = rng.normal(0, 1, (M, N)).astype(np.float16)
    clamp = dict(qmin=-128, qmax=127) if bits == 8 else {}
    a, w = (to_dev(A), to_dev(Wc)) if bits == 8 else (mkq.mkq_pack_codes_int4(to_dev(A)), mkq.mkq_pack_codes_int4(to_dev(Wc)).reshape(-1))

    def run(out_dtype, **kw):
        if bits == 8:
            return mkq.mkq_linear_int8(a, float(s_x), w, to_dev(s_w), to_dev(bias), out_dtype, **kw)
        return mkq.mkq_linear_int4(a, float(s_x), w, to_dev(s_w), to_dev(bias), N, K, out_dtype, **kw)

    ref = oracle.linear_int4(A, s_x, Wc, s_w, bias, **clamp)
    r = run(mkq.MKQ_F32, want_acc=True)
    assert np.array_equal(to_np(r["acc"]), ref["acc"]) and np.array_equal(to_np(r["out"]), ref["y"])
    ref = oracle.linear_int4(A, s_x, Wc, s_w, bias, residual=res.astype(np.float32), out_dtype=oracle.F16, **clamp)
    assert np.array_equal(to_np(run(mkq.MKQ_F16, residual=to_dev(res))["out"]).astype(np.float32), ref["y"])
    if N % 2:
        return
    codes = mkq.MKQ_I4 if bits == 4 else mkq.MKQ_I8
    ref = oracle.linear_int4(A, s_x, Wc, s_w, bias, s_next=0.9, **clamp)
    got = to_np(run(codes, s_next=0.9)["out"])
    assert np.array_equal(got, oracle.pack_nibbles(ref["q"]) if bits == 4 else ref["q"])
    # (the tie bands of the other GELU tests, which derive from the two erf forms)
    s_next, band = (0.9, {}) if bits == 4 else (0.05, dict(band=2.0 ** -7, max_frac=2e-3))
    ref = oracle.linear_int4(A, s_x, Wc, s_w, bias, act=oracle.ACT_GELU, s_next=s_next, **clamp)
    got = to_np(run(codes, act=mkq.MKQ_ACT_GELU, s_next=s_next)["out"])
    assert_codes_match_with_tie_band(oracle.unpack_nibbles(got, N) if bits == 4 else got, ref["q"], ref["y"], s_next, what="GELU", **band)
