"""The tile kernels with stages of 128-byte rows against the oracle: 4- and 8-bit configurations by number, at one stage
per tile, ragged edges, more tiles than resident workgroups, and every kind of epilogue; the binary16 linear at sizes
on every side of its tile choice.  Everything is exact: integer sums, correctly rounded binary32 epilogues, and for
binary16 small integer operands, whose sums binary32 holds exactly in any order; only codes behind a GELU may fall
either way at a tie."""
import numpy as np
import pytest

import oracle
from helpers import RTOL, assert_codes_match_with_tie_band, assert_float_close, to_dev, to_np

pytestmark = pytest.mark.gpu
GROUPS4 = {46: 2, 47: 2, 48: 2, 51: 2}  # wave groups that share the k loop
GROUPS8 = {47: 2}


@pytest.fixture(scope="module")
def mkq():
    import torch
    assert torch.cuda.is_available()
    import paper_2203_13483_amd as m
    m.load()
    return m


def _case(M, N, K, bits, seed):
    rng = np.random.default_rng(seed)
    q = 1 << (bits - 1)
    A = rng.integers(-q, q, (M, K), dtype=np.int8)
    Wc = rng.integers(-q, q, (N, K), dtype=np.int8)
    s_w = rng.uniform(0.001, 0.05, N).astype(np.float32) / (1 if bits == 4 else 256)
    res = rng.normal(0, 1, (M, N)).astype(np.float16)
    return A, Wc, s_w, np.float32(0.02), rng.normal(0, 0.5, N).astype(np.float32), res


# one stage per tile; several stages and ragged edges; N % 8 != 0 (the general epilogue); more tiles than any
# configuration keeps resident
@pytest.mark.parametrize("M,N,stages", [(300, 520, 1), (257, 136, 5), (330, 522, 3), (1500, 1104, 2), (8200, 2312, 1)])
@pytest.mark.parametrize("bits,cfg", [(4, c) for c in (*range(43, 50), 51)] + [(8, c) for c in (43, 44, 46, 47, 51, 52)])
def test_configurations(mkq, bits, cfg, M, N, stages):
    K = stages * (1024 // bits) * (GROUPS4 if bits == 4 else GROUPS8).get(cfg, 1)
    A, Wc, s_w, s_x, bias, res = _case(M, N, K, bits, cfg + M + K)
    clamp = dict(qmin=-128, qmax=127) if bits == 8 else {}

    def run(out_dtype, **kw):
        if bits == 8:
            return mkq.mkq_linear_int8(to_dev(A), float(s_x), to_dev(Wc), to_dev(s_w), to_dev(bias), out_dtype, config=cfg, **kw)
        return mkq.mkq_linear_int4(mkq.mkq_pack_codes_int4(to_dev(A)), float(s_x), mkq.mkq_pack_codes_int4(to_dev(Wc)).reshape(-1),
                                   to_dev(s_w), to_dev(bias), N, K, out_dtype, config=cfg, **kw)

    ref = oracle.linear_int4(A, s_x, Wc, s_w, bias, out_dtype=oracle.BF16, s_next=0.9, **clamp)
    assert np.array_equal(to_np(run(mkq.MKQ_BF16)["out"]).astype(np.float32), ref["y"])
    codes = to_np(run(mkq.MKQ_I4 if bits == 4 else mkq.MKQ_I8, s_next=0.9)["out"])
    assert np.array_equal(codes, oracle.pack_nibbles(ref["q"]) if bits == 4 else ref["q"])
    ref = oracle.linear_int4(A, s_x, Wc, s_w, bias, residual=res.astype(np.float32), out_dtype=oracle.F16, **clamp)
    assert np.array_equal(to_np(run(mkq.MKQ_F16, residual=to_dev(res))["out"]).astype(np.float32), ref["y"])
    ref = oracle.linear_int4(A, s_x, Wc, s_w, bias, **clamp)
    assert np.array_equal(to_np(run(mkq.MKQ_F32)["out"]), ref["y"])
    # GELU and codes behind it (the tie bands of the other GELU tests, which derive from the two erf forms)
    s_next, band = (0.9, {}) if bits == 4 else (0.05, dict(band=2.0 ** -7, max_frac=2e-3))
    refg = oracle.linear_int4(A, s_x, Wc, s_w, bias, act=oracle.ACT_GELU, s_next=s_next, **clamp)
    g = to_np(run(mkq.MKQ_I4 if bits == 4 else mkq.MKQ_I8, act=mkq.MKQ_ACT_GELU, s_next=s_next)["out"])
    assert_codes_match_with_tie_band(oracle.unpack_nibbles(g, N) if bits == 4 else g, refg["q"], refg["y"], s_next, what="GELU", **band)
    if M < 1000:
        r = run(mkq.MKQ_F32, want_acc=True)
        assert np.array_equal(to_np(r["acc"]), ref["acc"]) and np.array_equal(to_np(r["out"]), ref["y"])
        r = run(mkq.MKQ_F16)
        assert np.array_equal(to_np(r["out"]).astype(np.float32), oracle.round_storage(ref["y"], oracle.F16))


def test_configurations_need_whole_stages(mkq):
    A, Wc, s_w, s_x, bias, _ = _case(64, 64, 384, 4, 0)
    a, w = mkq.mkq_pack_codes_int4(to_dev(A)), mkq.mkq_pack_codes_int4(to_dev(Wc)).reshape(-1)
    for cfg in (*range(43, 50), 51):
        with pytest.raises(mkq.MkqError):
            mkq.mkq_linear_int4(a, float(s_x), w, to_dev(s_w), to_dev(bias), 64, 384, mkq.MKQ_F16, config=cfg)


# one shape per tile choice, in its order, with one and with several stages; a ragged N takes the general epilogue
@pytest.mark.parametrize("M,N,K", [(100, 72, 256), (1, 8, 64), (70, 136, 192), (33, 77, 128), (1500, 1544, 64), (1500, 1540, 320),
                                   (2100, 2056, 128), (2100, 2056, 64), (4100, 2312, 192), (8200, 2312, 64), (8200, 2312, 192)]
                         # the last tile of 96 and of 192 channels of one and of all columns; 128x128, deep and shallow; 256x256
                         + [(1100, 2209, 64), (1030, 2304, 256), (3850, 2497, 64), (4097, 2112, 128), (2100, 1800, 128), (6000, 2312, 64), (8192, 2048, 64)])
def test_linear_fp16_tile_choices(mkq, M, N, K):
    import torch
    rng = np.random.default_rng(M + K)
    a, W = (rng.integers(-8, 8, s).astype(np.float16) for s in ((M, K), (N, K)))
    b, res = (rng.integers(-64, 64, s).astype(np.float32) for s in ((N,), (M, N)))
    ref = a.astype(np.float32) @ W.astype(np.float32).T + b
    args = [to_dev(a), to_dev(W), to_dev(b)]
    assert np.array_equal(to_np(mkq.mkq_linear_fp16(*args, mkq.MKQ_F32)), ref)
    assert np.array_equal(to_np(mkq.mkq_linear_fp16(*args, mkq.MKQ_F16)), ref.astype(np.float16))
    got = mkq.mkq_linear_fp16(*args, mkq.MKQ_F16, mkq.MKQ_ACT_NONE, to_dev(res.astype(np.float16)))
    assert np.array_equal(to_np(got), (ref + res).astype(np.float16))
    small = [to_dev(a * np.float16(2.0 ** -6)), args[1], to_dev(b * np.float32(2.0 ** -6))]
    got = to_np(mkq.mkq_linear_fp16(*small, mkq.MKQ_F16, mkq.MKQ_ACT_GELU))
    want = torch.nn.functional.gelu(torch.from_numpy(ref.astype(np.float64) * 2.0 ** -6)).numpy()
    assert_float_close(got, want, RTOL[1], "GELU")


def test_linear_fp16_long_rows(mkq):
    """Rows of 256 MiB and more, whose bytes times eight pass 2^31: a few whole numbers in rows of zeros, exact."""
    import torch
    K = (1 << 27) + 64
    at = torch.tensor([0, 63, 64, (1 << 26) + 5, (1 << 27) - 1, 1 << 27, K - 1], device="cuda")
    a, W = (torch.zeros((rows, K), dtype=torch.float16, device="cuda") for rows in (2, 3))
    a[:, at] = torch.arange(14, device="cuda").reshape(2, 7).half()
    W[:, at] = torch.arange(-10, 11, device="cuda").reshape(3, 7).half()
    ref = a[:, at].cpu().float() @ W[:, at].cpu().float().T
    assert np.array_equal(to_np(mkq.mkq_linear_fp16(a, W, None, mkq.MKQ_F32)), ref.numpy())
