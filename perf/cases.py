"""What a user of this library has it do, as timed cases: single quantized linears from one token to 65536, the
few-token weight stream, encoder layers and whole encoders in 4, 8, mixed and 16 bits, uniform and padding-free
batches, and the calibration of activation steps.

A case is a dict of plain values.  ``listed()`` names the ones that are always measured, ``draw(rng)`` gives more of
the same ranges; ``prepare`` makes what a program holds before the call (weights packed once, workspaces, inputs),
``run`` is one pass through the package's public entry points.
"""
import math

import torch

import paper_2203_13483_amd as mkq
from paper_2203_13483_amd import workloads as wl

BASE = dict(hidden=768, heads=12, ffn=3072)
LARGE = dict(hidden=1024, heads=16, ffn=4096)
STUDENT = dict(hidden=312, heads=12, ffn=1200)

# (K, N) of the linears of the BERT-base and BERT-large layers, and the square the few-token sweep uses
LINEAR_SHAPES = [(768, 2304), (768, 768), (768, 3072), (3072, 768),
                 (1024, 3072), (1024, 1024), (1024, 4096), (4096, 1024), (4096, 4096)]
# (K, N) of weights worth keeping in the streaming layout
STREAM_SHAPES = [(4096, 4096), (8192, 8192), (8192, 28672), (28672, 8192), (16384, 16384)]
LINEAR_NAMES = ("qkv", "ao", "up", "down")
OUT = {"f32": mkq.MKQ_F32, "f16": mkq.MKQ_F16, "bf16": mkq.MKQ_BF16, "i4": mkq.MKQ_I4}
TORCH_OUT = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
BYTES = {"f32": 4.0, "f16": 2.0, "bf16": 2.0, "i4": 0.5}

STEP = wl.LEARNED_STEP_UNIT_GAUSSIAN


def listed():
    return [
        # one sentence of 128 tokens through one linear, float activations in: the smallest call, two launches
        dict(name="linear_one_sentence", kind="linear", M=128, K=768, N=768, a="f32", out="f32", epi="plain"),
        # a few rows against one square matrix, canonical packing (the last layer's pooler, a classifier, decoding)
        dict(name="linear_few_rows", kind="linear", M=16, K=4096, N=4096, a="i4", out="f16", epi="plain"),
        # serving a few tokens against weights of a hundred megabytes, kept in the streaming layout
        dict(name="linear_few_rows_streaming", kind="stream", M=16, K=8192, N=28672, out="f16"),
        # FFN-up of a BERT-large layer on 16 x 512 tokens: GELU, codes for the next linear out
        dict(name="linear_ffn_up_gelu_codes", kind="linear", M=8192, K=1024, N=4096, a="i4", out="i4", epi="gelu"),
        # offline scoring, the largest single linear
        dict(name="linear_large_m", kind="linear", M=65536, K=1024, N=4096, a="i4", out="bf16", epi="plain"),
        # one layer on a padding-free batch of 16 short sentences: latency, every kernel is small
        dict(name="layer_ragged_440_tokens", kind="encoder", bits="4", layers=1, batch=16, seq=128, tokens=440, **BASE),
        # two consecutive layers of the BERT-base encoder with the codes handed over between them.  (Twelve layers
        # cost six times as much and cannot be compared: one code that falls the other way at a tie changes the
        # codes of its sequence downstream, and two correct implementations are 9 % apart after twelve layers.)
        dict(name="layers_base", kind="encoder", bits="4", layers=2, batch=32, seq=128, tokens=0, **BASE),
        # one BERT-large layer on long documents
        dict(name="layer_large_512", kind="encoder", bits="4", layers=1, batch=16, seq=512, tokens=0, **LARGE),
        # the whole 4-layer student: hidden size 312, heads of 26
        dict(name="encoder_student", kind="encoder", bits="4", layers=4, batch=32, seq=128, tokens=0, **STUDENT),
        # the seam of a mixed model: an 8-bit layer feeding a 4-bit one, padding-free
        dict(name="layers_mixed_ragged", kind="encoder", bits="84", layers=2, batch=64, seq=128, tokens=2298, **BASE),
        # the binary16 layer that the quantized ones are compared with
        dict(name="layer_binary16", kind="encoder", bits="16", layers=1, batch=32, seq=128, tokens=0, **BASE),
        # calibrating one activation step on captured activations, and the gradients that train it further
        dict(name="calibrate_step", kind="calibrate", M=16384, K=4096, x="f16", ppm=100),
    ]


def _spread(rng, lo, hi):
    """An integer between lo and hi, uniform in its logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["linear", "linear", "stream", "encoder", "encoder", "encoder", "calibrate"])
    if kind == "linear":
        K, N = rng.choice(LINEAR_SHAPES)
        epi, out = rng.choice([("plain", "f32"), ("plain", "f16"), ("plain", "bf16"), ("gelu", "i4"), ("plain", "i4"),
                               ("residual", "f16")])
        a = rng.choice(["i4", "i4", "f16", "f32"])
        if K * N > 1024 * 4096 or out == "f32" or a == "f32":
            most = 8192
        else:
            most = 65536 if epi == "plain" and a == "i4" else 32768
        return dict(kind="linear", M=_spread(rng, 1, most), K=K, N=N, a=a, out=out, epi=epi)
    if kind == "stream":
        K, N = rng.choice(STREAM_SHAPES)
        return dict(kind="stream", M=_spread(rng, 1, 128), K=K, N=N, out=rng.choice(["f16", "f32"]))
    if kind == "calibrate":
        x = rng.choice(["f16", "f32"])
        return dict(kind="calibrate", M=_spread(rng, 64, 16384 if x == "f16" else 8192),
                    K=rng.choice([768, 1024, 3072, 4096]), x=x, ppm=rng.choice([10, 100, 1000]))
    dims = rng.choice([BASE, BASE, LARGE, STUDENT])
    bits = "4" if dims is STUDENT else rng.choice(["4", "4", "8", "84", "48", "16"])
    seq = rng.choice([32, 64, 128, 128, 128, 200, 256, 384, 512])
    layers = 2 if bits in ("84", "48") else rng.randint(1, 2)
    most = (4096 if bits == "16" else 8192) // layers
    batch = _spread(rng, 1, most // seq)
    # half the batches padding-free, with any number of valid tokens that leaves at least one per sequence
    tokens = rng.randint(batch, batch * seq) if rng.random() < 0.5 else 0
    return dict(kind="encoder", bits=bits, layers=layers, batch=batch, seq=seq, tokens=tokens, **dims)


# ------------------------------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _randn(g, *shape, std=1.0, mean=0.0):
    return torch.randn(*shape, generator=g, device="cuda") * std + mean


def _activations(g, M, K):
    """Unit Gaussian activations, one in a hundred eight times as large (they clip)."""
    x = _randn(g, M, K)
    return torch.where(torch.rand(M, K, generator=g, device="cuda") < 0.01, x * 8.0, x)


def _prepare_linear(c, g):
    M, K, N = c["M"], c["K"], c["N"]
    stream = c["kind"] == "stream"
    st = dict(case=c)
    if stream:  # weights of this size: codes drawn directly
        codes = torch.randint(0, 256, (N, K // 2), generator=g, device="cuda", dtype=torch.uint8)
        st["W"] = mkq.mkq_repack_weights_int4_stream(codes, N, K)
        st["s_w"] = torch.rand(N, generator=g, device="cuda") * 0.01 + 0.001
        st["scratch"] = mkq.mkq_splitk_scratch_init()
        a = "i4"
    else:
        st["W"], st["s_w"] = mkq.mkq_pack_weights_int4(_randn(g, N, K, std=0.02))
        a = c["a"]
    st["b"] = _randn(g, N, std=0.01)
    x = _activations(g, M, K)
    if a == "i4":
        st["a"] = mkq.mkq_quantize(x, STEP)
    else:
        st["a"] = x.half() if a == "f16" else x
        st["ws"] = torch.empty(mkq.mkq_linear_int4_workspace_bytes(M, N, K, OUT["f16"]), dtype=torch.uint8, device="cuda")
    st["out"] = (torch.empty((M, N // 2), dtype=torch.uint8, device="cuda") if c["out"] == "i4"
                 else torch.empty((M, N), dtype=TORCH_OUT[c["out"]], device="cuda"))
    if c.get("epi") == "residual":
        st["res"] = _randn(g, M, N).half()
    return st


def _run_linear(st):
    c = st["case"]
    if c["kind"] == "stream":
        return mkq.mkq_linear_int4_stream(st["a"], STEP, st["W"], st["s_w"], st["b"], c["N"], c["K"], OUT[c["out"]],
                                          out=st["out"], splitk_scratch=st["scratch"])["out"]
    return mkq.mkq_linear_int4(st["a"], STEP, st["W"], st["s_w"], st["b"], c["N"], c["K"], OUT[c["out"]],
                               act=mkq.MKQ_ACT_GELU if c["epi"] == "gelu" else mkq.MKQ_ACT_NONE,
                               residual=st.get("res"), s_next=0.05 if c["out"] == "i4" else 0.0, out=st["out"],
                               workspace=st.get("ws"))["out"]


def _layer_bits(c):
    """Width of every layer: one width for all, or two digits for the first and the second half of the layers."""
    if c["bits"] in ("4", "8", "16"):
        return [int(c["bits"])] * c["layers"]
    half = c["layers"] // 2
    return [int(c["bits"][0])] * half + [int(c["bits"][1])] * (c["layers"] - half)


def _tokens(c):
    return c["tokens"] or c["batch"] * c["seq"]


def _prepare_encoder(c, g, seed):
    H, F, heads = c["hidden"], c["ffn"], c["heads"]
    bits, M = _layer_bits(c), _tokens(c)
    cu = None
    if c["tokens"]:
        lens = wl.ragged_lengths(c["tokens"], c["batch"], c["seq"], seed)
        cu = torch.zeros(c["batch"] + 1, dtype=torch.int32, device="cuda")
        cu[1:] = torch.cumsum(torch.from_numpy(lens).cuda(), 0)
    st = dict(case=c, h=_randn(g, M, H).half(), layers=[])
    ws_bytes = 0
    for i, nb in enumerate(bits):
        ln = {k: _randn(g, H, std=0.1, mean=1.0 if k.endswith("gamma") else 0.0)
              for k in ("ln1_gamma", "ln1_beta", "ln2_gamma", "ln2_beta")}
        weights = {}
        for nm, (_, K, N) in zip(LINEAR_NAMES, wl.layer_gemm_shapes(H, F)):
            W, b = _randn(g, N, K, std=0.02), _randn(g, N, std=0.01)
            if nb == 16:
                weights[nm] = (W.half(), b)
            elif nb == 8:
                weights[nm] = mkq.mkq_pack_weights_int8(W) + (b,)
            elif K % 32 == 0:
                weights[nm] = mkq.mkq_pack_weights_int4(W) + (b,)
            else:
                weights[nm] = mkq.mkq_pack_weights_int4_padded(W) + (b,)
        if nb == 16:
            layer = mkq.BertLayerFp16(c["batch"], c["seq"], H, heads, F, weights, ln, 1e-12, cu_seqlens=cu,
                                      total_tokens=M if cu is not None else 0)
            q_next = None
        else:
            # learned steps: unit-variance LayerNorm outputs, small attention contexts and GELU outputs
            fine = 1.0 if nb == 4 else 7.0 / 127.0
            sx = {"qkv": STEP * fine, "ao": 0.05 * fine, "up": STEP * fine, "down": 0.05 * fine}
            nxt = bits[i + 1] if i + 1 < len(bits) else 0
            cls = mkq.BertLayerInt4 if nb == 4 else mkq.BertLayerInt8
            layer = cls(c["batch"], c["seq"], H, heads, F, weights, sx, ln, 1e-12,
                        s_out_next=STEP * (1.0 if nxt == 4 else 7.0 / 127.0) if nxt else 0.0, next_bits=nxt,
                        cu_seqlens=cu, total_tokens=M if cu is not None else 0)
            if nxt == 8:
                q_next = torch.empty((M, H), dtype=torch.int8, device="cuda")
            elif nxt == 4:
                pitch = H if H % 32 == 0 else mkq.mkq_padded_k(H)
                q_next = torch.empty((M, pitch // 2), dtype=torch.uint8, device="cuda")
            else:
                q_next = None
        ws_bytes = max(ws_bytes, layer.workspace_bytes())
        st["layers"].append((layer, nb, torch.empty((M, H), dtype=torch.float16, device="cuda"), q_next))
    st["ws"] = torch.empty(ws_bytes, dtype=torch.uint8, device="cuda")
    return st


def _run_encoder(st):
    h, q, ws = st["h"], None, st["ws"]
    for layer, nb, h_out, q_next in st["layers"]:
        if nb == 16:
            layer(h, ws, h_out=h_out)
        else:
            layer(h, ws, h_out=h_out, q_in=q, q_out_next=q_next)
        h, q = h_out, q_next
    return h


def _prepare_calibrate(c, g):
    x = _activations(g, c["M"], c["K"])
    return dict(case=c, x=x.half() if c["x"] == "f16" else x,
                ws=torch.empty(mkq.mkq_percentile_scale_workspace_bytes(), dtype=torch.uint8, device="cuda"),
                s=torch.empty(1, dtype=torch.float32, device="cuda"),
                s_abs=torch.empty(1, dtype=torch.float32, device="cuda"),
                g=torch.empty(2, dtype=torch.float64, device="cuda"))


def _run_calibrate(st):
    """The two initial steps of section 3.1 and both scale gradients of section 4.1 under the current step."""
    c = st["case"]
    return [mkq.mkq_absmax_scale(st["x"], s_out=st["s_abs"]),
            mkq.mkq_percentile_scale(st["x"], c["ppm"], 4, s_out=st["s"], workspace=st["ws"]),
            mkq.mkq_scale_gradients(st["x"], STEP, 4, g_out=st["g"])]


def prepare(case, seed):
    g = _gen(seed)
    if case["kind"] == "encoder":
        return _prepare_encoder(case, g, seed)
    if case["kind"] == "calibrate":
        return _prepare_calibrate(case, g)
    return _prepare_linear(case, g)


def run(state):
    kind = state["case"]["kind"]
    if kind == "encoder":
        return _run_encoder(state)
    if kind == "calibrate":
        return _run_calibrate(state)
    return _run_linear(state)


# ------------------------------------------------------------------------------------------------
# The same results in binary64, from the same draws, in plain torch.  Steps and codes of the inputs are decided in
# binary32, as Eq. 1 defines them; everything after that is binary64, without the 16-bit storage between the kernels.
def _codes(x, s, bits=4):
    q = 2 ** (bits - 1)
    return torch.round(torch.clamp(x / s, -q, q - 1))


def _exact_weights(W, bits):
    """W as the quantized linear sees it."""
    if bits == 16:
        return W.half().double()
    top = W.abs().amax(dim=1, keepdim=True)
    s = torch.where(top > 0, top / (7.0 if bits == 4 else 127.0), torch.ones_like(top))
    return _codes(W, s, bits).double() * s.double()


def _f32(v):
    return torch.tensor(v, dtype=torch.float32, device="cuda")


def _exact_linear(c, g):
    M, K, N = c["M"], c["K"], c["N"]
    if c["kind"] == "stream":
        b = torch.randint(0, 256, (N, K // 2), generator=g, device="cuda", dtype=torch.uint8).int()
        w = torch.stack(((b & 15) ^ 8, (b >> 4) ^ 8), dim=2).reshape(N, K).sub_(8).float()
        s_w = torch.rand(N, generator=g, device="cuda") * 0.01 + 0.001
    else:
        w, s_w = _exact_weights(_randn(g, N, K, std=0.02), 4), None
    b = _randn(g, N, std=0.01)
    x = _activations(g, M, K)
    x = _codes(x.half().float() if c.get("a") == "f16" else x, _f32(STEP))
    if s_w is not None:
        # products of codes summed by binary32 are exact in parts of 2^18 codes and fewer
        y = (x @ w.t()).double() * s_w.double()
    else:
        y = x.double() @ w.t()
    y = y * _f32(STEP).double() + b.double()
    if c.get("epi") == "residual":
        y += _randn(g, M, N).half().double()
    return None if c["out"] == "i4" else y


def _exact_attention(qkv, lens, heads):
    ctx = torch.empty_like(qkv[:, :qkv.shape[1] // 3])
    at = 0
    for n in lens:
        q, k, v = (t.reshape(n, heads, -1).transpose(0, 1).contiguous() for t in qkv[at:at + n].chunk(3, dim=1))
        p = torch.softmax(q @ k.transpose(1, 2).contiguous() / math.sqrt(q.shape[2]), dim=2)
        ctx[at:at + n] = (p @ v).transpose(0, 1).reshape(n, -1)
        at += n
    return ctx


def _exact_encoder(c, g, seed):
    H, F, heads, M = c["hidden"], c["ffn"], c["heads"], _tokens(c)
    lens = [int(n) for n in wl.ragged_lengths(M, c["batch"], c["seq"], seed)] if c["tokens"] else [c["seq"]] * c["batch"]
    h = _randn(g, M, H).half().double()
    norm = torch.nn.functional.layer_norm
    for nb in _layer_bits(c):
        ln = [_randn(g, H, std=0.1, mean=m).double() for m in (1.0, 0.0, 1.0, 0.0)]
        step = {"qkv": STEP, "ao": 0.05, "up": STEP, "down": 0.05}
        lin = {}
        for nm, (_, K, N) in zip(LINEAR_NAMES, wl.layer_gemm_shapes(H, F)):
            W, b = _exact_weights(_randn(g, N, K, std=0.02), nb), _randn(g, N, std=0.01).double()
            s = _f32(step[nm] * (1.0 if nb == 4 else 7.0 / 127.0)).double()

            def linear(x, W=W, b=b, s=s):
                return (x if nb == 16 else _codes(x, s, nb) * s) @ W.t() + b

            lin[nm] = linear
        u = lin["ao"](_exact_attention(lin["qkv"](h), lens, heads)) + h
        h1 = norm(u, (H,), ln[0], ln[1], 1e-12)
        d = lin["down"](torch.nn.functional.gelu(lin["up"](h1))) + h1
        h = norm(d, (H,), ln[2], ln[3], 1e-12)
    return h


def _exact_calibrate(c, g):
    x = _activations(g, c["M"], c["K"])
    x = (x.half().float() if c["x"] == "f16" else x).reshape(-1)
    k = max(1, x.numel() * c["ppm"] // 1000000)
    kth = torch.topk(x.abs(), k, sorted=True).values[-1]
    r = _codes(x, _f32(STEP)).double()
    xd, s = x.double(), _f32(STEP).double()
    grads = torch.stack(((r - xd / s).sum(), 2.0 * ((r * s - xd) * r).sum()))
    return [(x.abs().max().double() / 7.0).reshape(1), (kth.double() / 7.0).reshape(1), grads]


def exact(case, seed):
    g = _gen(seed)
    if case["kind"] == "encoder":
        return _exact_encoder(case, g, seed)
    if case["kind"] == "calibrate":
        return _exact_calibrate(case, g)
    return _exact_linear(case, g)


# ------------------------------------------------------------------------------------------------
def work(case):
    c = case
    if c["kind"] == "calibrate":
        # one read of the activations for all three results
        n = c["M"] * c["K"]
        return dict(bytes=n * (2.0 if c["x"] == "f16" else 4.0), flops=20.0 * n)
    if c["kind"] == "encoder":
        H, F, M = c["hidden"], c["ffn"], _tokens(c)
        # the mean length stands for all: sum of squares of the lengths at least tokens^2 / batch
        length = M / c["batch"]
        weights = 4.0 * H * H + 2.0 * H * F
        flops = byts = 0.0
        for nb in _layer_bits(c):
            flops += 2.0 * M * weights + 4.0 * M * length * H
            byts += weights * nb / 8.0 + 8.0 * (5 * H + F)
        return dict(bytes=byts + 4.0 * M * H, flops=flops)
    M, K, N = c["M"], c["K"], c["N"]
    a = BYTES[c.get("a", "i4")]
    byts = M * K * a + N * K * 0.5 + 8.0 * N + M * N * BYTES[c["out"]]
    if c.get("epi") == "residual":
        byts += 2.0 * M * N
    return dict(bytes=byts, flops=2.0 * M * K * N)


def tolerance(case):
    """About four times what the path differs by from the same path with its float parts in binary64 (sums, softmax,
    LayerNorm and GELU; the integer contraction is exact either way)."""
    c = case
    if c["kind"] == "calibrate":
        return dict(rel=1e-10, max=1e-9)  # binary64 sums in any order; the two steps are exact
    if c["kind"] == "encoder":
        if c["bits"] == "16":  # seen 1.4e-4 after one layer: binary16 storage between the kernels
            return dict(rel=6e-4 * c["layers"], max=1e-2 * c["layers"])
        # seen 1e-5 to 7e-4 after one layer, 4e-3 to 7e-3 after two to four: codes at a tie
        return dict(rel=3e-3, max=0.3) if c["layers"] == 1 else dict(rel=2.8e-2, max=0.4)
    if c["out"] == "i4":  # seen 1e-6 of the bytes, through GELU at a tie
        return dict(rel=4e-3, max=0.99, differ=4e-6)
    # one binary32 rounding (seen 4e-8), and a 16-bit result that rounds the other way because of it (seen 1.5e-6)
    return {"f32": dict(rel=2e-7, max=5e-7), "f16": dict(rel=6e-6, max=1.5e-3), "bf16": dict(rel=5e-5, max=1.2e-2)}[c["out"]]
