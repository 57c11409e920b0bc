"""GPU parity: LayerNorm, attention core, binary16 baseline linear, and the W4A4 /
binary16 encoder layers vs the CPU oracle.  Integer stages are checked
"teacher-forced": the oracle is fed the GPU's own upstream codes, so accumulators
and binary16 outputs must match bit for bit regardless of upstream float wobble;
codes decided from LayerNorm / softmax / GELU outputs may differ by one step only
inside a narrow band around a rounding boundary."""
import numpy as np
import pytest

import oracle
from paper_2203_13483_amd import workloads as wl
from helpers import RTOL, assert_codes_match_with_tie_band, assert_float_close, to_dev, to_np
from layer_checks import LayerBuffers, attention_code_band, check_layer_stagewise, codes_match

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mkq():
    import torch
    assert torch.cuda.is_available()
    import paper_2203_13483_amd as m
    m.load()
    return m


def _f16(a):
    return np.asarray(a, np.float32).astype(np.float16)


@pytest.mark.parametrize("M,D", [(128, 768), (37, 1024), (5, 64), (64, 3072), (16, 8192)])
def test_layernorm(mkq, M, D):
    rng = np.random.default_rng(D + M)
    x = _f16(rng.normal(0.2, 1.5, (M, D)))
    g = rng.normal(1, 0.2, D).astype(np.float32)
    b = rng.normal(0, 0.2, D).astype(np.float32)
    s_next = 0.3
    y, q = mkq.mkq_layernorm(to_dev(x), to_dev(g), to_dev(b), 1e-12, s_next=s_next, want_q=True)
    ref = oracle.layernorm(x.astype(np.float32), g, b, 1e-12)
    assert_float_close(to_np(y).astype(np.float32), oracle.round_storage(ref, oracle.F16), RTOL[1], "layernorm")
    got = oracle.unpack_nibbles(to_np(q), D)
    assert_codes_match_with_tie_band(got, oracle.quantize(ref, s_next), ref, s_next, what="layernorm codes")
    # gamma = beta = None means 1 and 0
    y0, _ = mkq.mkq_layernorm(to_dev(x), None, None, 1e-5)
    assert_float_close(to_np(y0).astype(np.float32), oracle.layernorm(x.astype(np.float32), eps=1e-5), RTOL[1], "ln plain")


@pytest.mark.parametrize("M,D", [(9, 8), (65, 64), (513, 512), (1025, 1024), (1031, 1032), (2047, 312), (2049, 312), (2049, 256), (2049, 768), (2050, 520),
                                 (2051, 1024), (4097, 4096)])
def test_layernorm_counts_every_lane_once(mkq, M, D):
    """Rows with one value that is not zero, in every place: a lane that a reduction missed or counted twice moves mean and
    variance of its rows by as much as they are.  Binary32 sums of exact zeros and one value, one binary16 rounding."""
    import torch
    x = torch.zeros(M, D, dtype=torch.float16, device="cuda")
    at = torch.arange(M, device="cuda")
    x[at, at % D] = 8.0
    y, _ = mkq.mkq_layernorm(x, None, None, 1e-5)
    xd = x.double()
    want = torch.nn.functional.layer_norm(xd, (D,), eps=1e-5)
    assert bool(((y.double() - want).abs() <= (2.0 ** -11 + 4e-6) * want.abs() + 2.0 ** -24).all())


def test_layernorm_of_more_rows_than_fit_a_launch_four_to_a_workgroup(mkq):
    """2^26 rows: the codes of 4096 rows over and over are those of these rows alone."""
    import torch
    D, rows, M = 264, 4096, 2 ** 26
    g = torch.Generator(device="cuda").manual_seed(D)
    base = torch.randn((rows, D), generator=g, device="cuda").half()
    x = torch.empty((M, D), dtype=torch.float16, device="cuda")
    x.view(M // rows, rows, D).copy_(base)
    few, q = (mkq.mkq_layernorm(t, None, None, 1e-5, s_next=0.3, want_y=False, want_q=True)[1] for t in (base, x))
    q = q.view(M // rows, rows, D // 2)
    for part in q.split(1024):
        assert bool((part == q[0]).all())
    # means and variances over half waves and over whole waves are sums in another order: a value at a rounding boundary may
    # fall the other way, and codes are 0.3 wide where the sums differ by 1e-6
    assert float((q[0] != few).float().mean()) < 1e-4


@pytest.mark.parametrize("B,S,heads", [(2, 128, 12), (3, 64, 2), (1, 32, 1), (2, 96, 4)])
def test_attention(mkq, B, S, heads):
    H = heads * 64
    rng = np.random.default_rng(S + heads)
    qkv = _f16(rng.normal(0, 1.0, (B * S, 3 * H)))
    s_next = 0.05
    ctx, q = mkq.mkq_attention(to_dev(qkv), B, S, H, heads, s_next=s_next, want_q=True)
    ref = oracle.attention(qkv.astype(np.float32), B, S, H, heads, p_dtype=oracle.F16)
    assert_float_close(to_np(ctx).astype(np.float32), ref, RTOL[1], "attention")
    got = oracle.unpack_nibbles(to_np(q), H)
    for b in range(B):  # the band of every element: what one binary16 unit of every probability can move it
        rows = slice(b * S, (b + 1) * S)
        codes_match(got[rows], oracle.quantize(ref[rows], s_next), ref[rows], s_next,
                    attention_code_band(qkv[rows].astype(np.float32), S, H, heads, s_next), "attention codes")
    # the probabilities of one query sum to one: with v = 1 the context is 1
    ones = qkv.copy()
    ones[:, 2 * H:] = 1.0
    ctx1, _ = mkq.mkq_attention(to_dev(ones), B, S, H, heads)
    assert np.abs(to_np(ctx1).astype(np.float32) - 1.0).max() < 2e-3


# head sizes other than 64 (the 4-layer student: 312 / 12 = 26) and sequences longer than one key block
@pytest.mark.parametrize("B,S,heads,dk", [(2, 512, 16, 64), (1, 512, 12, 26), (3, 200, 12, 26), (2, 128, 12, 26),
                                          (2, 130, 4, 32), (2, 77, 2, 48), (1, 129, 1, 64), (2, 384, 3, 64),
                                          (1, 40, 4, 2), (1, 300, 4, 62)])
def test_attention_any_head_size_and_length(mkq, B, S, heads, dk):
    H = heads * dk
    rng = np.random.default_rng(S + heads + dk)
    qkv = _f16(rng.normal(0, 1.0, (B * S, 3 * H)))
    s_next = 0.05
    ctx, q = mkq.mkq_attention(to_dev(qkv), B, S, H, heads, s_next=s_next, want_q=True)
    ref = oracle.attention(qkv.astype(np.float32), B, S, H, heads, p_dtype=oracle.F16)
    assert_float_close(to_np(ctx).astype(np.float32), ref, RTOL[1], "attention")
    got = oracle.unpack_nibbles(to_np(q), H)
    for b in range(B):
        rows = slice(b * S, (b + 1) * S)
        codes_match(got[rows], oracle.quantize(ref[rows], s_next), ref[rows], s_next,
                    attention_code_band(qkv[rows].astype(np.float32), S, H, heads, s_next), "attention codes")
    ctx8, q8 = mkq.mkq_attention_int8(to_dev(qkv), B, S, H, heads, s_next=s_next / 16)
    assert np.array_equal(to_np(ctx8), to_np(ctx))
    for b in range(B):
        rows = slice(b * S, (b + 1) * S)
        codes_match(to_np(q8)[rows], oracle.quantize(ref[rows], s_next / 16, qmin=-128, qmax=127), ref[rows],
                    s_next / 16, attention_code_band(qkv[rows].astype(np.float32), S, H, heads, s_next / 16),
                    "attention codes, 8 bits")
    # a sharply peaked softmax (one key far above the rest) and the probabilities summing to one
    peaked = qkv.copy()
    peaked[:, :2 * H] *= 6.0
    ctxp, _ = mkq.mkq_attention(to_dev(peaked), B, S, H, heads)
    assert_float_close(to_np(ctxp).astype(np.float32),
                       oracle.attention(peaked.astype(np.float32), B, S, H, heads, p_dtype=oracle.F16), RTOL[1], "peaked")
    ones = qkv.copy()
    ones[:, 2 * H:] = 1.0
    ctx1, _ = mkq.mkq_attention(to_dev(ones), B, S, H, heads)
    assert np.abs(to_np(ctx1).astype(np.float32) - 1.0).max() < 4e-3


@pytest.mark.parametrize("S,dk", [(1, 26), (33, 32), (64, 26), (65, 8), (128, 26), (129, 64), (160, 26), (191, 48),
                                  (193, 32), (256, 64), (257, 64), (320, 26), (448, 32), (449, 64), (512, 64), (512, 26),
                                  (513, 62), (700, 32), (1000, 64)])
@pytest.mark.parametrize("scores", ["rising", "falling", "equal", "far apart"])
def test_attention_at_the_edges_of_its_key_groups(mkq, S, dk, scores):
    """Scores that put the maximum of a row first, last or nowhere, at the edges of the kernels' groups of keys, against the
    softmax in binary64.  Every probability is rounded to binary16 once (2^-11 of it, or 2^-25 below the smallest normal
    number), the sums are binary32 and the result is binary16."""
    import torch
    H = 4 * dk
    g = torch.Generator().manual_seed(S + dk)
    qkv = torch.randn(S, 3 * H, generator=g) * 0.3
    t = torch.arange(S) / S
    lift = {"rising": 40.0 * t, "falling": -40.0 * t, "equal": 0.0 * t,
            "far apart": 25.0 * (torch.arange(S) % 97 == 5).float() + 60.0 * (torch.arange(S) == S - 1).float()}[scores]
    for h in range(4):  # q = (c, noise), k = (lift, noise): scores about lift
        qkv[:, h * dk] = dk ** 0.5
        qkv[:, H + h * dk] = lift
    qkv = qkv.half()
    ctx, _ = mkq.mkq_attention(qkv.cuda(), 1, S, H, 4)
    q, k, v = (x.double().reshape(S, 4, dk).transpose(0, 1) for x in qkv.chunk(3, dim=1))
    p = torch.softmax(q @ k.transpose(1, 2).contiguous() / dk ** 0.5, dim=2)
    want = (p @ v).transpose(0, 1).reshape(S, H).numpy()
    mass = (p @ v.abs()).transpose(0, 1).reshape(S, H).numpy()
    got = to_np(ctx).astype(np.float64)
    small = S * 2.0 ** -25 * float(v.abs().max())
    assert np.all(np.abs(got - want) <= (2.0 ** -11 + 2.0 ** -14) * mass + small + 2.0 ** -11 * np.abs(want) + 2.0 ** -24)


@pytest.mark.parametrize("batch", [2 ** 20 - 1, 2 ** 20])
def test_attention_of_a_million_one_token_sequences(mkq, batch):
    """As many heads as workgroups of 512 threads can be launched for, and more: the context of one token is its v."""
    import torch
    heads, H = 8, 64
    g = torch.Generator(device="cuda").manual_seed(batch)
    qkv = torch.randn((batch, 3 * H), generator=g, device="cuda").half()
    ctx, _ = mkq.mkq_attention(qkv, batch, 1, H, heads)
    assert torch.equal(ctx, qkv[:, 2 * H:])


def test_attention_with_rows_beyond_32_bit_offsets(mkq):
    """One sequence whose rows of qkv reach over 4 GiB: the first and the last heads against the softmax in binary64."""
    import torch
    S, dk, heads, few = 512, 64, 21952, 4
    H = heads * dk
    assert S * 6 * H > 2 ** 32
    g = torch.Generator(device="cuda").manual_seed(5)
    qkv = torch.empty((S, 3, heads, dk), dtype=torch.float16, device="cuda")
    for r in range(0, S, 64):
        qkv[r: r + 64] = torch.randn((64, 3, heads, dk), generator=g, device="cuda", dtype=torch.float16)
    ctx, _ = mkq.mkq_attention(qkv.view(S, 3 * H), 1, S, H, heads)
    ctx = ctx.view(S, heads, dk)
    for sl in (slice(0, few), slice(heads - few, heads)):
        q, k, v = (qkv[:, i, sl].double().transpose(0, 1).contiguous().cpu() for i in range(3))
        p = torch.softmax(q @ k.transpose(1, 2).contiguous() / dk ** 0.5, dim=2)
        want = (p @ v).transpose(0, 1).numpy()
        assert_float_close(to_np(ctx[:, sl]).astype(np.float32), want, RTOL[1], f"heads {sl}")


@pytest.mark.parametrize("batch,total,max_seq,heads,dk", [(5, 2300, 512, 4, 64), (5, 700, 300, 12, 26),
                                                          (4, 9, 512, 2, 64), (3, 520, 512, 2, 32)])
def test_attention_over_long_ragged_sequences(mkq, batch, total, max_seq, heads, dk):
    H = heads * dk
    lens = _lengths(total, batch, max_seq, seed=total)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    rng = np.random.default_rng(total + heads)
    qkv = _f16(rng.normal(0, 1.0, (total, 3 * H)))
    s_next = 0.05
    ctx, q = mkq.mkq_attention_varlen(to_dev(qkv), to_dev(cu), max_seq, H, heads, s_next=s_next, q_bits=4)
    got, codes = to_np(ctx).astype(np.float32), oracle.unpack_nibbles(to_np(q), H)
    for b in range(batch):
        rows = slice(cu[b], cu[b + 1])
        if lens[b] == 0:
            continue
        ref = oracle.attention(qkv[rows].astype(np.float32), 1, int(lens[b]), H, heads, p_dtype=oracle.F16)
        assert_float_close(got[rows], ref, RTOL[1], f"sequence {b} of length {lens[b]}")
        codes_match(codes[rows], oracle.quantize(ref, s_next), ref, s_next,
                    attention_code_band(qkv[rows].astype(np.float32), int(lens[b]), H, heads, s_next), "context codes")


def _attention_bound(qkv, heads):
    """The softmax attention of one sequence in binary64 and its bound: every probability is rounded to binary16 once (2^-11 of
    it, or 2^-25 below the smallest normal number), the sums are binary32 and the result is binary16."""
    import torch
    n, dk = qkv.shape[0], qkv.shape[1] // (3 * heads)
    q, k, v = (x.double().reshape(n, heads, dk).transpose(0, 1) for x in qkv.cpu().chunk(3, dim=1))
    p = torch.softmax(q @ k.transpose(1, 2).contiguous() / dk ** 0.5, dim=2)
    want = (p @ v).transpose(0, 1).reshape(n, heads * dk).numpy()
    mass = (p @ v.abs()).transpose(0, 1).reshape(n, heads * dk).numpy()
    return want, (2.0 ** -11 + 2.0 ** -14) * mass + n * 2.0 ** -25 * float(v.abs().max()) + 2.0 ** -11 * np.abs(want) + 2.0 ** -24


# batch * heads well above what the device runs at a time (several blocks of 128 queries per workgroup), and as many as that
@pytest.mark.parametrize("batch,max_seq,heads,dk", [(48, 200, 16, 64), (48, 300, 12, 26), (45, 384, 12, 32), (16, 500, 16, 64),
                                                    (48, 512, 12, 48), (200, 500, 4, 26), (24, 256, 32, 8), (40, 700, 8, 64)])
@pytest.mark.parametrize("longest", ["uniform", "one", "a quarter", "most"])
def test_attention_of_many_sequences_is_that_of_each_alone(mkq, batch, max_seq, heads, dk, longest):
    """Bit for bit, context and codes of both widths: what a query's result is does not depend on which workgroup has its block, nor
    on how the sequences are dealt.  Some of them against binary64."""
    import torch
    H = heads * dk
    g = np.random.default_rng(batch * max_seq + dk)
    lens = g.integers(1, max_seq - 127, batch)
    lens[:6] = [0, 1, 127, min(128, max_seq), min(129, max_seq), min(257, max_seq - 100)]
    share = {"uniform": batch, "one": 1, "a quarter": batch // 4, "most": batch - 8}[longest]
    lens[batch - share:] = g.integers(max_seq - max_seq % 128 + 1 if max_seq % 128 else max_seq - 127, max_seq + 1, share)
    lens[-1] = max_seq
    if longest == "uniform":
        lens[:] = max_seq
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    gen = torch.Generator(device="cuda").manual_seed(int(cu[-1]))
    qkv = torch.randn((int(cu[-1]), 3 * H), generator=gen, device="cuda").half()
    s_next = 0.02
    if longest == "uniform":
        ctx, q4 = mkq.mkq_attention(qkv, batch, max_seq, H, heads, s_next=s_next, want_q=True)
        _, q8 = mkq.mkq_attention_int8(qkv, batch, max_seq, H, heads, s_next=s_next / 16)
    else:
        ctx, q4 = mkq.mkq_attention_varlen(qkv, to_dev(cu), max_seq, H, heads, s_next=s_next, q_bits=4)
        _, q8 = mkq.mkq_attention_varlen(qkv, to_dev(cu), max_seq, H, heads, s_next=s_next / 16, q_bits=8)
    checked = {2, 3, 5, batch // 2, batch - 1}
    for b, n in enumerate(int(v) for v in lens):
        if n == 0:
            continue
        rows = slice(int(cu[b]), int(cu[b]) + n)
        one = to_dev(np.array([0, n], np.int32))
        c1, a4 = mkq.mkq_attention_varlen(qkv[rows].contiguous(), one, max_seq, H, heads, s_next=s_next, q_bits=4)
        _, a8 = mkq.mkq_attention_varlen(qkv[rows].contiguous(), one, max_seq, H, heads, s_next=s_next / 16, q_bits=8)
        assert torch.equal(ctx[rows], c1) and torch.equal(q4[rows], a4) and torch.equal(q8[rows], a8), (b, n)
        if b in checked:
            want, bound = _attention_bound(qkv[rows], heads)
            assert np.all(np.abs(to_np(ctx[rows]).astype(np.float64) - want) <= bound), (b, n)


@pytest.mark.parametrize("batch,seq,ragged", [(48, 128, True), (48, 300, True), (22, 512, True), (48, 300, False), (5, 520, True)])
def test_layer_context_codes_with_a_row_pitch(mkq, batch, seq, ragged):
    """The context codes inside a layer of hidden size 312 (rows of 384 codes): those of the attention alone on the layer's own
    q, k, v, and zeros behind them, for more sequences than the device runs at a time."""
    import torch
    H, heads, F = 312, 12, 1200
    g = torch.Generator(device="cuda").manual_seed(batch * seq)
    rng = np.random.default_rng(batch + seq)
    lens = rng.integers(1, seq + 1, batch) if ragged else np.full(batch, seq)
    lens[-1] = seq
    cu = to_dev(np.concatenate([[0], np.cumsum(lens)]).astype(np.int32))
    M = int(lens.sum())
    h = torch.randn((M, H), generator=g, device="cuda").half()
    weights = {}
    for nm, K, N in (("qkv", H, 3 * H), ("ao", H, H), ("up", H, F), ("down", F, H)):
        W = torch.randn((N, K), generator=g, device="cuda") * 0.05
        weights[nm] = mkq.mkq_pack_weights_int4_padded(W) + (torch.zeros(N, device="cuda"),)
    ln = {k: torch.full((H,), float(k.endswith("gamma")), device="cuda") for k in ("ln1_gamma", "ln1_beta", "ln2_gamma", "ln2_beta")}
    sx = {"qkv": 0.3, "ao": 0.05, "up": 0.3, "down": 0.05}
    layer = mkq.BertLayerInt4(batch, seq, H, heads, F, weights, sx, ln, 1e-12, cu_seqlens=cu if ragged else None,
                              total_tokens=M if ragged else 0)
    ws = torch.full((layer.workspace_bytes(),), 0x5A, dtype=torch.uint8, device="cuda")
    layer(h, ws)
    pitch = mkq.mkq_padded_k(H) // 2
    qkv = ws[layer.layout.qkv: layer.layout.qkv + M * 3 * H * 2].view(torch.float16).reshape(M, 3 * H).contiguous()
    codes = ws[layer.layout.c1: layer.layout.c1 + M * pitch].reshape(M, pitch)
    _, alone = mkq.mkq_attention_varlen(qkv, cu, seq, H, heads, s_next=sx["ao"], q_bits=4)
    assert torch.equal(codes[:, : H // 2], alone) and not codes[:, H // 2:].any()


@pytest.mark.parametrize("S,dk", [(64, 26), (130, 64), (512, 32), (511, 64)])
def test_attention_passes_nan_and_infinities_on(mkq, S, dk):
    """A NaN or an infinite score makes its query's row NaN; every other row keeps its bits.  A key of -inf (scores of -inf
    for queries with positive first dimension) has probability 0: the row is that of the sequence without the key."""
    import torch
    heads, H = 4, 4 * dk
    g = torch.Generator().manual_seed(S * dk)
    base = torch.randn((S, 3 * H), generator=g).half()
    base[:, 0] = base[:, 0].abs() + 0.5       # q, head 0, first dimension: positive
    clean = mkq.mkq_attention(base.cuda(), 1, S, H, heads)[0].cpu()
    for row in (0, S // 2, S - 1):
        for bad in (float("nan"), float("inf"), float("-inf")):
            x = base.clone()
            x[row, 1] = bad                   # one query, head 0
            got = mkq.mkq_attention(x.cuda(), 1, S, H, heads)[0].cpu()
            assert torch.isnan(got[row, :dk]).all(), (row, bad)
            other = torch.ones(S, heads, dtype=torch.bool)
            other[row, 0] = False
            assert torch.equal(got.reshape(S, heads, dk)[other], clean.reshape(S, heads, dk)[other])
        x = base.clone()
        x[row, H] = float("-inf")             # one key, head 0: out of every row's sum
        got = mkq.mkq_attention(x.cuda(), 1, S, H, heads)[0].cpu()
        keep = [r for r in range(S) if r != row]
        q, k, v = (base[:, i * H: i * H + dk].double() for i in range(3))
        p = torch.softmax(q @ k[keep].t().contiguous() / dk ** 0.5, dim=1)
        want, mass = (p @ v[keep]).numpy(), (p @ v[keep].abs()).numpy()
        bound = (2.0 ** -11 + 2.0 ** -14) * mass + S * 2.0 ** -25 * float(v.abs().max()) + 2.0 ** -11 * np.abs(want) + 2.0 ** -24
        assert np.all(np.abs(to_np(got[:, :dk]).astype(np.float64) - want) <= bound), row
        x = base.clone()
        x[row, 2 * H] = float("nan")          # one value: a column of head 0
        got = mkq.mkq_attention(x.cuda(), 1, S, H, heads)[0].cpu()
        assert torch.isnan(got[:, 0]).all() and torch.equal(got[:, 1:], clean[:, 1:])


@pytest.mark.parametrize("M,N,K", [(128, 768, 768), (200, 328, 192), (1024, 2304, 768), (77, 64, 3072)])
@pytest.mark.parametrize("variant", ["plain", "gelu", "residual_f32out"])
def test_linear_fp16_baseline(mkq, M, N, K, variant):
    import torch
    rng = np.random.default_rng(M + N)
    a = _f16(rng.normal(0, 1, (M, K)))
    W = _f16(rng.normal(0, 0.05, (N, K)))
    b = rng.normal(0, 0.1, N).astype(np.float32)
    res = _f16(rng.normal(0, 1, (M, N)))
    act = mkq.MKQ_ACT_GELU if variant == "gelu" else mkq.MKQ_ACT_NONE
    use_res = variant == "residual_f32out"
    out_dtype = mkq.MKQ_F32 if use_res else mkq.MKQ_F16
    y = mkq.mkq_linear_fp16(to_dev(a), to_dev(W), to_dev(b), out_dtype, act, to_dev(res) if use_res else None)
    ref = oracle.linear_float(a.astype(np.float32), W.astype(np.float32), b,
                              residual=res.astype(np.float32) if use_res else None,
                              act=oracle.ACT_GELU if variant == "gelu" else oracle.ACT_NONE,
                              out_dtype=oracle.F32 if use_res else oracle.F16)
    assert_float_close(to_np(y).astype(np.float32), ref, RTOL[0] if use_res else RTOL[1], "fp16 linear")


def _layer_case(seed, B, S, hidden, heads, ffn):
    p = wl.bert_layer_weights(hidden, heads, ffn, seed)
    rng = np.random.default_rng(seed + 7)
    for ln in ("ln1", "ln2"):
        p[ln + "_gamma"] = rng.normal(1, 0.1, hidden).astype(np.float32)
        p[ln + "_beta"] = rng.normal(0, 0.1, hidden).astype(np.float32)
    h = _f16(wl.hidden_states(B, S, hidden, seed + 1))
    return p, h


def _quantized_params(p, h, B, S):
    """Oracle-side weight codes and activation steps (calibrated on the float layer)."""
    H, F, heads = p["hidden"], p["ffn"], p["heads"]
    hf = h.astype(np.float32)
    qkv = oracle.linear_float(hf, p["W_qkv"], p["b_qkv"])
    ctx = oracle.attention(qkv, B, S, H, heads)
    u = oracle.linear_float(ctx, p["W_ao"], p["b_ao"], residual=hf)
    h1 = oracle.layernorm(u, p["ln1_gamma"], p["ln1_beta"], p["ln_eps"])
    g = oracle.linear_float(h1, p["W_up"], p["b_up"], act=oracle.ACT_GELU)
    q = {k: p[k] for k in ("hidden", "heads", "ffn", "ln_eps", "ln1_gamma", "ln1_beta", "ln2_gamma", "ln2_beta")}
    q["batch"], q["seq"] = B, S
    for nm, act_in in (("qkv", hf), ("ao", ctx), ("up", h1), ("down", g)):
        q["w_" + nm], q["sw_" + nm] = oracle.quantize_weights(p["W_" + nm])
        q["b_" + nm] = p["b_" + nm]
        q["sx_" + nm] = float(np.float32(oracle.absmax_scale(act_in) * 0.5))  # a learned step clips the tails
    return q


@pytest.mark.parametrize("B,S,hidden,heads,ffn", [(2, 64, 128, 2, 256), (2, 128, 768, 12, 3072)])
def test_bert_layer_int4_stagewise_and_end_to_end(mkq, B, S, hidden, heads, ffn):
    import torch
    p, h = _layer_case(31, B, S, hidden, heads, ffn)
    q = _quantized_params(p, h, B, S)
    M = B * S
    packed, sx = {}, {}
    for nm in ("qkv", "ao", "up", "down"):
        Wq, s_w = mkq.mkq_pack_weights_int4(to_dev(p["W_" + nm]))
        assert np.array_equal(to_np(s_w), q["sw_" + nm])
        packed[nm] = (Wq, s_w, to_dev(p["b_" + nm]))
        sx[nm] = q["sx_" + nm]
    ln = {k: to_dev(p[k]) for k in ("ln1_gamma", "ln1_beta", "ln2_gamma", "ln2_beta")}
    s_out_next = 0.4
    layer = mkq.BertLayerInt4(B, S, hidden, heads, ffn, packed, sx, ln, p["ln_eps"], s_out_next)
    ws = torch.zeros(layer.workspace_bytes(), dtype=torch.uint8, device="cuda")
    q_next = torch.empty((M, hidden // 2), dtype=torch.uint8, device="cuda")
    h_out = layer(to_dev(h), ws, q_out_next=q_next)
    torch.cuda.synchronize()

    L = layer.layout
    wsn = to_np(ws)

    def codes(off, cols):
        return oracle.unpack_nibbles(wsn[off: off + M * cols // 2], cols)

    def f16buf(off, cols):
        return wsn[off: off + M * cols * 2].view(np.float16).reshape(M, cols).astype(np.float32)

    hf = h.astype(np.float32)
    c0, c1, c2, c3 = codes(L.c0, hidden), codes(L.c1, hidden), codes(L.c2, hidden), codes(L.c3, ffn)
    qkv, u, h1, d = f16buf(L.qkv, 3 * hidden), f16buf(L.u, hidden), f16buf(L.h1, hidden), f16buf(L.d, hidden)

    # stage by stage, each fed the GPU's own inputs
    assert np.array_equal(c0, oracle.quantize(hf, q["sx_qkv"]))
    r = oracle.linear_int4(c0, q["sx_qkv"], q["w_qkv"], q["sw_qkv"], q["b_qkv"], out_dtype=oracle.F16)
    assert np.array_equal(qkv, r["y"])
    ctx_ref = oracle.attention(qkv, B, S, hidden, heads, p_dtype=oracle.F16)
    for b in range(B):
        rows = slice(b * S, (b + 1) * S)
        codes_match(c1[rows], oracle.quantize(ctx_ref[rows], q["sx_ao"]), ctx_ref[rows], q["sx_ao"],
                    attention_code_band(qkv[rows], S, hidden, heads, q["sx_ao"]), "context codes")
    r = oracle.linear_int4(c1, q["sx_ao"], q["w_ao"], q["sw_ao"], q["b_ao"], residual=hf, out_dtype=oracle.F16)
    assert np.array_equal(u, r["y"])
    h1_ref = oracle.layernorm(u, p["ln1_gamma"], p["ln1_beta"], p["ln_eps"])
    assert_float_close(h1, oracle.round_storage(h1_ref, oracle.F16), RTOL[1], "h1")
    assert_codes_match_with_tie_band(c2, oracle.quantize(h1_ref, q["sx_up"]), h1_ref, q["sx_up"], what="h1 codes")
    r = oracle.linear_int4(c2, q["sx_up"], q["w_up"], q["sw_up"], q["b_up"], act=oracle.ACT_GELU, s_next=q["sx_down"])
    assert_codes_match_with_tie_band(c3, r["q"], r["y"], q["sx_down"], what="ffn codes")
    r = oracle.linear_int4(c3, q["sx_down"], q["w_down"], q["sw_down"], q["b_down"], residual=h1, out_dtype=oracle.F16)
    assert np.array_equal(d, r["y"])
    out_ref = oracle.layernorm(d, p["ln2_gamma"], p["ln2_beta"], p["ln_eps"])
    got_out = to_np(h_out).astype(np.float32)
    assert_float_close(got_out, oracle.round_storage(out_ref, oracle.F16), RTOL[1], "layer out (teacher-forced)")
    assert_codes_match_with_tie_band(oracle.unpack_nibbles(to_np(q_next), hidden), oracle.quantize(out_ref, s_out_next),
                                     out_ref, s_out_next, what="next-layer codes")

    # end to end against the oracle's own layer: codes may flip near boundaries upstream,
    # so only closeness is asked, and most codes must agree
    ref_out, it = oracle.bert_layer_int4(q, hf, act_dtype=oracle.F16)
    assert (c3 != it["c3"]).mean() < 0.02
    err = np.abs(got_out - ref_out)
    assert np.sqrt((err ** 2).mean()) < 0.03 * np.sqrt((ref_out ** 2).mean())

    # the caller may hand in the input codes instead of having them computed
    h_out2 = layer(to_dev(h), ws, q_in=to_dev(oracle.pack_nibbles(c0)), q_out_next=q_next)
    assert np.array_equal(to_np(h_out2), to_np(h_out))


@pytest.mark.parametrize("B,S,hidden,heads,ffn", [(2, 64, 128, 2, 256), (2, 128, 768, 12, 3072), (1, 300, 512, 16, 1024), (1, 512, 256, 4, 512)])
def test_bert_layer_fp16_baseline(mkq, B, S, hidden, heads, ffn):
    import torch
    p, h = _layer_case(41, B, S, hidden, heads, ffn)
    weights, ref_params = {}, {k: p[k] for k in ("hidden", "heads", "ffn", "ln_eps", "ln1_gamma", "ln1_beta",
                                                  "ln2_gamma", "ln2_beta")}
    ref_params["batch"], ref_params["seq"] = B, S
    for nm in ("qkv", "ao", "up", "down"):
        W16 = _f16(p["W_" + nm])
        weights[nm] = (to_dev(W16), to_dev(p["b_" + nm]))
        ref_params["w_" + nm] = W16.astype(np.float32)
        ref_params["b_" + nm] = p["b_" + nm]
    ln = {k: to_dev(p[k]) for k in ("ln1_gamma", "ln1_beta", "ln2_gamma", "ln2_beta")}
    layer = mkq.BertLayerFp16(B, S, hidden, heads, ffn, weights, ln, p["ln_eps"])
    ws = torch.empty(layer.workspace_bytes(), dtype=torch.uint8, device="cuda")
    out = to_np(layer(to_dev(h), ws)).astype(np.float32)
    ref = oracle.bert_layer_float(ref_params, h.astype(np.float32), act_dtype=oracle.F16)
    assert_float_close(out, oracle.round_storage(ref, oracle.F16), RTOL[1], "fp16 layer")


# The 4-layer student of section 5.2 (hidden 312, 12 heads of 26, FFN 1200: no reduction length is a multiple
# of 32, every code buffer is stored padded) and a BERT-large layer on 512-token sequences.
@pytest.mark.parametrize("B,S,hidden,heads,ffn", [(2, 128, 312, 12, 1200), (3, 50, 312, 12, 1200),
                                                  (1, 512, 1024, 16, 4096), (2, 200, 768, 12, 3072)])
def test_bert_layer_int4_other_head_sizes_and_long_sequences(mkq, B, S, hidden, heads, ffn):
    import torch
    from layer_checks import code_row_pitch
    p, h = _layer_case(47, B, S, hidden, heads, ffn)
    q = _quantized_params(p, h, B, S)
    M = B * S
    padded = hidden % 32 != 0
    packed, sx = {}, {}
    for nm in ("qkv", "ao", "up", "down"):
        pack = mkq.mkq_pack_weights_int4_padded if padded else mkq.mkq_pack_weights_int4
        Wq, s_w = pack(to_dev(p["W_" + nm]))
        assert np.array_equal(to_np(s_w), q["sw_" + nm])
        packed[nm] = (Wq, s_w, to_dev(p["b_" + nm]))
        sx[nm] = q["sx_" + nm]
    ln = {k: to_dev(p[k]) for k in ("ln1_gamma", "ln1_beta", "ln2_gamma", "ln2_beta")}
    s_out_next = 0.4
    layer = mkq.BertLayerInt4(B, S, hidden, heads, ffn, packed, sx, ln, p["ln_eps"], s_out_next)
    ws = torch.full((layer.workspace_bytes(),), 0x5A, dtype=torch.uint8, device="cuda")  # stale contents
    pitch = code_row_pitch(hidden)
    q_next = torch.full((M, pitch // 2), 0x5A, dtype=torch.uint8, device="cuda")
    h_out = layer(to_dev(h), ws, q_out_next=q_next)
    torch.cuda.synchronize()
    buf = LayerBuffers(to_np(ws), layer.layout, M, hidden, ffn, 4)
    qn = oracle.unpack_nibbles(to_np(q_next), pitch)
    assert not qn[:, hidden:].any()
    check_layer_stagewise(buf, q, h.astype(np.float32), to_np(h_out).astype(np.float32),
                          [(b * S, S) for b in range(B)], q_next=qn[:, :hidden], s_out_next=s_out_next,
                          what=f"layer {hidden}/{heads}/{ffn}")
    # end to end against the oracle's own layer
    ref_out, it = oracle.bert_layer_int4(q, h.astype(np.float32), act_dtype=oracle.F16)
    assert (buf.codes(layer.layout.c3, ffn) != it["c3"]).mean() < 0.02
    err = np.abs(to_np(h_out).astype(np.float32) - ref_out)
    assert np.sqrt((err ** 2).mean()) < 0.03 * np.sqrt((ref_out ** 2).mean())
    # handing in the (padded) input codes gives the same result
    c0 = torch.from_numpy(buf.ws[layer.layout.c0: layer.layout.c0 + M * pitch // 2].copy()).cuda()
    h_out2 = layer(to_dev(h), ws, q_in=c0, q_out_next=q_next)
    assert np.array_equal(to_np(h_out2), to_np(h_out))


# --- padding-free batches (the "valid tokens" of Table 2) ----------------------------------

_lengths = wl.ragged_lengths


@pytest.mark.parametrize("batch,total,max_seq,heads", [(16, 440, 128, 12), (5, 200, 70, 2), (3, 96, 32, 1), (4, 7, 128, 2)])
def test_attention_over_ragged_sequences(mkq, batch, total, max_seq, heads):
    import torch
    H = heads * 64
    lens = _lengths(total, batch, min(max_seq, 128), seed=total)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    rng = np.random.default_rng(total + heads)
    qkv = _f16(rng.normal(0, 1.0, (total, 3 * H)))
    s_next = 0.05
    ctx, q = mkq.mkq_attention_varlen(to_dev(qkv), to_dev(cu), max_seq, H, heads, s_next=s_next, q_bits=4)
    got, codes = to_np(ctx).astype(np.float32), oracle.unpack_nibbles(to_np(q), H)
    for b in range(batch):
        rows = slice(cu[b], cu[b + 1])
        ref = oracle.attention(qkv[rows].astype(np.float32), 1, int(lens[b]), H, heads, p_dtype=oracle.F16)
        assert_float_close(got[rows], ref, RTOL[1], f"sequence {b} of length {lens[b]}")
        codes_match(codes[rows], oracle.quantize(ref, s_next), ref, s_next,
                    attention_code_band(qkv[rows].astype(np.float32), int(lens[b]), H, heads, s_next), "context codes")
    # equal lengths that are a multiple of 32 reproduce the fixed-length entry point exactly
    S = 64
    qkv2 = _f16(rng.normal(0, 1.0, (3 * S, 3 * H)))
    cu2 = np.arange(4, dtype=np.int32) * S
    a, _ = mkq.mkq_attention_varlen(to_dev(qkv2), to_dev(cu2), S, H, heads)
    b_, _ = mkq.mkq_attention(to_dev(qkv2), 3, S, H, heads)
    assert torch.equal(a, b_)


@pytest.mark.parametrize("kind", ["int4", "int8", "fp16"])
def test_layers_on_a_padding_free_batch(mkq, kind):
    """Sequences do not interact: each sequence's rows of the layer output equal the oracle's layer run on
    that sequence alone (batch 1, its own length)."""
    import torch
    batch, total, hidden, heads, ffn = 6, 230, 128, 2, 256
    lens = _lengths(total, batch, 100, seed=5)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    p, _ = _layer_case(81, 1, 32, hidden, heads, ffn)
    h = _f16(np.random.default_rng(82).standard_normal((total, hidden)))
    ln = {k: to_dev(p[k]) for k in ("ln1_gamma", "ln1_beta", "ln2_gamma", "ln2_beta")}
    cud = to_dev(cu)
    base = {k: p[k] for k in ("hidden", "heads", "ffn", "ln_eps", "ln1_gamma", "ln1_beta", "ln2_gamma", "ln2_beta")}
    if kind == "fp16":
        weights = {}
        for nm in ("qkv", "ao", "up", "down"):
            W16 = _f16(p["W_" + nm])
            weights[nm] = (to_dev(W16), to_dev(p["b_" + nm]))
            base["w_" + nm], base["b_" + nm] = W16.astype(np.float32), p["b_" + nm]
        layer = mkq.BertLayerFp16(batch, 100, hidden, heads, ffn, weights, ln, p["ln_eps"], cu_seqlens=cud,
                                  total_tokens=total)
    else:
        qr = dict(qmin=-8, qmax=7) if kind == "int4" else dict(qmin=-128, qmax=127)
        scale = 1.0 if kind == "int4" else 7.0 / 127.0
        packed, sx = {}, {}
        for nm, st in (("qkv", 0.34), ("ao", 0.05), ("up", 0.34), ("down", 0.05)):
            base["w_" + nm], base["sw_" + nm] = oracle.quantize_weights(p["W_" + nm], **qr)
            base["b_" + nm] = p["b_" + nm]
            base["sx_" + nm] = sx[nm] = float(np.float32(st * scale))
            pack = mkq.mkq_pack_weights_int4 if kind == "int4" else mkq.mkq_pack_weights_int8
            packed[nm] = pack(to_dev(p["W_" + nm])) + (to_dev(p["b_" + nm]),)
        cls = mkq.BertLayerInt4 if kind == "int4" else mkq.BertLayerInt8
        layer = cls(batch, 100, hidden, heads, ffn, packed, sx, ln, p["ln_eps"], cu_seqlens=cud, total_tokens=total)
    ws = torch.zeros(layer.workspace_bytes(), dtype=torch.uint8, device="cuda")
    out = to_np(layer(to_dev(h), ws)).astype(np.float32)
    assert out.shape == (total, hidden)
    if kind != "fp16":
        # every stage of every sequence against the oracle fed the GPU's own previous stage: a wrong row range
        # at a sequence seam or one bad head shows in the stage where it happens
        buf = LayerBuffers(to_np(ws), layer.layout, total, hidden, ffn, 4 if kind == "int4" else 8)
        check_layer_stagewise(buf, base, h.astype(np.float32), out, [(int(cu[b]), int(lens[b])) for b in range(batch)],
                              what=kind + " ragged")
    for b in range(batch):
        rows = slice(cu[b], cu[b + 1])
        q = dict(base, batch=1, seq=int(lens[b]))
        x = h[rows].astype(np.float32)
        if kind == "fp16":
            ref = oracle.bert_layer_float(q, x, act_dtype=oracle.F16)
            assert_float_close(out[rows], oracle.round_storage(ref, oracle.F16), RTOL[1], f"sequence {b}")
        else:
            ref, _ = oracle.bert_layer_int4(q, x, act_dtype=oracle.F16, **qr)
            err = out[rows] - ref
            assert np.sqrt((err ** 2).mean()) < 0.04 * np.sqrt((ref ** 2).mean()), (b, int(lens[b]))


@pytest.mark.parametrize("heads,dk,max_seq", [(2, 64, 512), (12, 26, 300), (2, 64, 128)])
def test_attention_with_empty_and_one_token_sequences(mkq, heads, dk, max_seq):
    """A padding-free batch may hold empty sequences (skipped) and sequences of one token (softmax of one score)."""
    H = heads * dk
    lens = np.array([5, 0, 1, min(max_seq, 290), 0, 33])
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    total = int(lens.sum())
    rng = np.random.default_rng(heads + dk)
    qkv = _f16(rng.normal(0, 1.0, (total, 3 * H)))
    ctx, q = mkq.mkq_attention_varlen(to_dev(qkv), to_dev(cu), max_seq, H, heads, s_next=0.05, q_bits=4)
    got, codes = to_np(ctx).astype(np.float32), oracle.unpack_nibbles(to_np(q), H)
    for b, n in enumerate(lens):
        if n == 0:
            continue
        rows = slice(cu[b], cu[b + 1])
        ref = oracle.attention(qkv[rows].astype(np.float32), 1, int(n), H, heads, p_dtype=oracle.F16)
        assert_float_close(got[rows], ref, RTOL[1], f"sequence {b} of length {n}")
        codes_match(codes[rows], oracle.quantize(ref, 0.05), ref, 0.05,
                    attention_code_band(qkv[rows].astype(np.float32), int(n), H, heads, 0.05), "context codes")
    one = slice(cu[2], cu[3])  # one token: the context is that token's v
    assert np.array_equal(got[one], qkv[one, 2 * H:].astype(np.float32))


# Layers of small hidden size (launch_rules.h, small_layer_*): q, k, v with the attention in one launch, and what follows it in another.
# Smallest and largest of token tiles (1, 16, 17, 32, 33, 64, 65, 128), of heads (2 to 32, even and multiples of 8), of hidden rows (one and a
# half 256-code units among them) and of FFN chunks (one column group, ragged, whole, several of both widths); tokens past one round.
_SMALL = [(1, 1, 312, 12, 1200, None), (3, 17, 312, 12, 1200, None), (1, 32, 128, 4, 512, None), (3, 33, 384, 12, 1536, None), (2, 64, 256, 8, 8, None),
          (2, 65, 376, 47, 1320, None), (2, 128, 384, 192, 2560, None), (1, 128, 104, 4, 768, None), (4, 20, 128, 2, 776, None), (2, 130, 256, 16, 1288, None),
          (7, 128, 312, 12, 1200, (128, 0, 1, 32, 33, 64, 65)), (5, 40, 384, 48, 904, (40, 0, 16, 17, 1)), (34, 128, 312, 12, 1200, (128,) * 31 + (1, 127, 1))]


@pytest.mark.parametrize("batch,seq,hidden,heads,ffn,lens", _SMALL)
@pytest.mark.parametrize("bias", [True, False])
def test_layers_of_small_hidden_size(mkq, batch, seq, hidden, heads, ffn, lens, bias):
    import torch
    from layer_checks import code_row_pitch
    p, _ = _layer_case(batch + hidden, 1, 8, hidden, heads, ffn)
    lens = [seq] * batch if lens is None else list(lens)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    M = int(cu[-1])
    h = _f16(np.random.default_rng(hidden + M).standard_normal((M, hidden)))
    ln = {k: to_dev(p[k]) for k in ("ln1_gamma", "ln1_beta", "ln2_gamma", "ln2_beta")}
    base = {k: p[k] for k in ("hidden", "heads", "ffn", "ln_eps", "ln1_gamma", "ln1_beta", "ln2_gamma", "ln2_beta")}
    packed, sx = {}, {}
    for nm, step in (("qkv", 0.34), ("ao", 0.05), ("up", 0.34), ("down", 0.05)):
        base["w_" + nm], base["sw_" + nm] = oracle.quantize_weights(p["W_" + nm])
        base["b_" + nm] = p["b_" + nm] if bias else np.zeros_like(p["b_" + nm])
        base["sx_" + nm] = sx[nm] = float(np.float32(step))
        pack = mkq.mkq_pack_weights_int4 if p["W_" + nm].shape[1] % 32 == 0 else mkq.mkq_pack_weights_int4_padded
        packed[nm] = pack(to_dev(p["W_" + nm])) + (to_dev(p["b_" + nm]),)
    next_bits, s_next = (8, 0.03) if hidden % 64 == 0 else (4, 0.4)
    uniform = len(set(lens)) == 1
    layer = mkq.BertLayerInt4(batch, seq, hidden, heads, ffn, packed, sx, ln, p["ln_eps"], s_next, next_bits,
                              cu_seqlens=None if uniform else to_dev(cu), total_tokens=0 if uniform else M)
    if not bias:
        for nm in ("qkv", "ao", "up", "down"):
            setattr(layer.params, "b_" + nm, None)
    ws = torch.full((layer.workspace_bytes(),), 0x5A, dtype=torch.uint8, device="cuda")  # stale contents
    pitch = code_row_pitch(hidden)
    q_next = torch.full((M, hidden if next_bits == 8 else pitch // 2), 0x5A, dtype=torch.uint8, device="cuda")
    x = to_dev(h)
    h_out = layer(x, ws, q_out_next=q_next)
    torch.cuda.synchronize()
    qn = to_np(q_next).view(np.int8) if next_bits == 8 else oracle.unpack_nibbles(to_np(q_next), pitch)
    assert not qn[:, hidden:].any()
    some = range(batch) if M < 1000 else (0, 1, 30, 31, 32, batch - 1) if batch > 30 else range(batch)
    check_layer_stagewise(LayerBuffers(to_np(ws), layer.layout, M, hidden, ffn, 4), base, h.astype(np.float32), to_np(h_out).astype(np.float32),
                          [(int(cu[b]), int(lens[b])) for b in some if lens[b]], q_next=qn[:, :hidden], s_out_next=s_next, next_bits=next_bits,
                          what=f"layer {hidden}/{heads}/{ffn}")
    # the output may take the input's place
    again = layer(x, ws, h_out=x, q_out_next=q_next)
    assert torch.equal(again, h_out)


def _small_layer(mkq, hidden, heads, ffn, seq, lens):
    """A 4-bit layer of small hidden size over a padding-free batch; its workspace after a run, tensors and output."""
    import torch
    from layer_checks import code_row_pitch
    p, _ = _layer_case(hidden + heads, 1, 8, hidden, heads, ffn)
    ln = {k: to_dev(p[k]) for k in ("ln1_gamma", "ln1_beta", "ln2_gamma", "ln2_beta")}
    packed = {}
    for nm in ("qkv", "ao", "up", "down"):
        pack = mkq.mkq_pack_weights_int4 if p["W_" + nm].shape[1] % 32 == 0 else mkq.mkq_pack_weights_int4_padded
        packed[nm] = pack(to_dev(p["W_" + nm])) + (to_dev(p["b_" + nm]),)
    M = sum(lens)
    cu = to_dev(np.concatenate([[0], np.cumsum(lens)]).astype(np.int32))
    layer = mkq.BertLayerInt4(len(lens), seq, hidden, heads, ffn, packed, {"qkv": 0.34, "ao": 0.05, "up": 0.34, "down": 0.05}, ln, p["ln_eps"], 0.4, 4,
                              cu_seqlens=cu, total_tokens=M)
    ws = torch.full((layer.workspace_bytes(),), 0x5A, dtype=torch.uint8, device="cuda")  # stale contents
    q_next = torch.full((M, code_row_pitch(hidden) // 2), 0x5A, dtype=torch.uint8, device="cuda")
    x = torch.randn((5000, hidden), generator=torch.Generator(device="cuda").manual_seed(hidden), device="cuda").half()[:M].contiguous()
    h_out = layer(x, ws, q_out_next=q_next)
    return dict(ws=ws, L=layer.layout, cu=cu, M=M, ln=ln, eps=p["ln_eps"], h_out=h_out, q_next=q_next, pitch=code_row_pitch(hidden),
                ffn_pitch=code_row_pitch(ffn))


def _f16_rows(r, at, cols):
    import torch
    return r["ws"][at: at + r["M"] * cols * 2].view(torch.float16).view(r["M"], cols)


# heads of 26 (words), 32, 16, 8, 4 (16-byte pieces and words), sequences of one, two and four tiles of tokens, whole and ragged
@pytest.mark.parametrize("hidden,heads,seq,lens", [(312, 12, 128, (128, 1, 16, 17, 32, 33, 64, 65, 127, 96)), (384, 12, 128, (128, 100, 64, 3) * 8),
                                                   (256, 16, 64, (64, 33, 32, 31) * 12), (128, 16, 32, (32, 1, 17) * 40), (104, 26, 128, (128, 77) * 9)])
def test_attention_of_small_layers_is_that_of_its_own_launch(mkq, hidden, heads, seq, lens):
    """Context codes of a layer that runs q, k, v and the attention in one launch: bit for bit those of the attention on the same q, k, v."""
    r = _small_layer(mkq, hidden, heads, 256, seq, lens)
    qkv = _f16_rows(r, r["L"].qkv, 3 * hidden).contiguous()
    _, want = mkq.mkq_attention_varlen(qkv, r["cu"], seq, hidden, heads, s_next=0.05, want_ctx=False, q_bits=4)
    got = r["ws"][r["L"].c1: r["L"].c1 + r["M"] * r["pitch"] // 2].view(r["M"], -1)
    assert np.array_equal(to_np(got[:, :hidden // 2]), to_np(want))
    assert not got[:, hidden // 2:].any()


# rows that a whole wave sums (a half-full second chunk of the half wave, one value of it, all of it) and rows that fit one chunk
@pytest.mark.parametrize("hidden,heads", [(312, 12), (264, 12), (384, 12), (344, 43), (256, 8)])
def test_layernorms_of_small_layers_are_those_of_their_own_launch(mkq, hidden, heads):
    """Both LayerNorms of a layer that runs them with the linears: bit for bit mkq_layernorm's, whose order of a row's sum the same
    sentence meets in a larger batch; the codes of the last one likewise."""
    r = _small_layer(mkq, hidden, heads, 256, 128, (128,) * 12 + (77,))
    L, ln = r["L"], r["ln"]
    for at, got, gamma, beta in ((L.u, _f16_rows(r, L.h1, hidden), "ln1_gamma", "ln1_beta"), (L.d, r["h_out"], "ln2_gamma", "ln2_beta")):
        y, q = mkq.mkq_layernorm(_f16_rows(r, at, hidden).contiguous(), ln[gamma], ln[beta], r["eps"], s_next=0.4, want_q=True)
        assert np.array_equal(to_np(got).view(np.uint16), to_np(y).view(np.uint16))
    assert np.array_equal(to_np(r["q_next"][:, :hidden // 2]), to_np(q))


# one chunk of FFN columns, ragged and whole, two and three of either size; last workgroups of 1, 2 and 15 rows
@pytest.mark.parametrize("hidden,heads,ffn,tokens", [(312, 12, 1200, 2610), (384, 12, 1280, 720), (312, 12, 8, 1), (264, 12, 768, 130), (376, 47, 1320, 999),
                                                     (104, 4, 1536, 1025), (384, 12, 2304, 1712), (256, 8, 2560, 2047), (128, 2, 3840, 3248),
                                                     (312, 12, 3080, 4095)])
def test_a_sentence_has_the_same_bits_in_a_larger_batch(mkq, hidden, heads, ffn, tokens):
    """The same sequences where one launch runs what follows the attention (launch_rules.h, small_layer_tail) and among so many that
    kernels of their own do."""
    lens = [128] * (tokens // 128) + ([tokens % 128] if tokens % 128 else [])
    few, more = (_small_layer(mkq, hidden, heads, ffn, 128, part) for part in (lens, lens + [128] * ((4096 - tokens) // 128 + 1)))
    assert few["M"] == tokens and more["M"] > 4096
    assert np.array_equal(to_np(few["h_out"]).view(np.uint16), to_np(more["h_out"][:tokens]).view(np.uint16))
    assert np.array_equal(to_np(few["q_next"]), to_np(more["q_next"][:tokens]))
    for at, bytes_ in (("u", 2 * hidden), ("h1", 2 * hidden), ("c2", few["pitch"] // 2), ("c3", few["ffn_pitch"] // 2), ("d", 2 * hidden)):
        a, b = (r["ws"][getattr(r["L"], at):][:tokens * bytes_] for r in (few, more))
        assert np.array_equal(to_np(a), to_np(b)), at


# Attention output and LayerNorm in one launch (launch_rules.h, output_norm): the fewest and the most tokens, last workgroups of 1 and 15 rows,
# rows of whole 256-code units and with a half one, with padding codes, the smallest FFN and the base one
@pytest.mark.parametrize("hidden,heads,ffn,tokens", [(768, 12, 64, 2048), (768, 12, 3072, 2049), (640, 10, 128, 4095), (640, 10, 96, 4096), (744, 12, 200, 2063),
                                                     (760, 19, 64, 3000)])
@pytest.mark.parametrize("bias", [True, False])
def test_attention_output_with_its_layernorm(mkq, hidden, heads, ffn, tokens, bias):
    """Bit for bit what the same sequences give among more of them, which take the linear and the LayerNorm one after the other."""
    import torch
    p, _ = _layer_case(hidden + ffn, 1, 8, hidden, heads, ffn)
    ln = {k: to_dev(p[k]) for k in ("ln1_gamma", "ln1_beta", "ln2_gamma", "ln2_beta")}
    packed = {}
    for nm in ("qkv", "ao", "up", "down"):
        pack = mkq.mkq_pack_weights_int4 if p["W_" + nm].shape[1] % 32 == 0 else mkq.mkq_pack_weights_int4_padded
        packed[nm] = pack(to_dev(p["W_" + nm])) + (to_dev(p["b_" + nm]),)
    sx = {"qkv": 0.34, "ao": 0.05, "up": 0.34, "down": 0.05}
    lens = [128] * (tokens // 128) + ([tokens % 128] if tokens % 128 else [])
    more = lens + [128] * 17 + [77] * (len(lens) % 2)
    while sum(more) <= 4096:
        more.append(128)
    x = torch.randn((sum(more), hidden), generator=torch.Generator(device="cuda").manual_seed(hidden), device="cuda").half()
    from layer_checks import code_row_pitch
    results = []
    for part in (lens, more):
        M = sum(part)
        cu = to_dev(np.concatenate([[0], np.cumsum(part)]).astype(np.int32))
        layer = mkq.BertLayerInt4(len(part), 128, hidden, heads, ffn, packed, sx, ln, p["ln_eps"], 0.4, 4, cu_seqlens=cu, total_tokens=M)
        if not bias:
            for nm in ("qkv", "ao", "up", "down"):
                setattr(layer.params, "b_" + nm, None)
        ws = torch.full((layer.workspace_bytes(),), 0x5A, dtype=torch.uint8, device="cuda")  # stale contents
        q_next = torch.full((M, code_row_pitch(hidden) // 2), 0x5A, dtype=torch.uint8, device="cuda")
        h_out = layer(x[:M].contiguous(), ws, q_out_next=q_next)
        results.append((h_out[:tokens], q_next[:tokens]))
    assert torch.equal(results[0][0], results[1][0]) and torch.equal(results[0][1], results[1][1])
