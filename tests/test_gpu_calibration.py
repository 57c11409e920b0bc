"""GPU parity of the scale machinery (sections 3.1 and 4.1) against the oracle: the
percentile step is an exact order statistic (bit-exact); the scale-gradient sums are
binary64 sums whose order differs, compared to 1e-10 of the sum of the terms' magnitudes."""
import numpy as np
import pytest

import oracle
from helpers import to_dev, to_np

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mkq():
    import torch
    assert torch.cuda.is_available()
    import paper_2203_13483_amd as m
    m.load()
    return m


def _activations(M, K, seed, dtype):
    rng = np.random.default_rng(seed)
    x = rng.standard_normal((M, K)).astype(np.float32)
    x.flat[:: 101] *= 8  # outliers beyond the clamp
    return x.astype(dtype)


@pytest.mark.parametrize("dtype", [np.float32, np.float16])
@pytest.mark.parametrize("M,K,bits,s", [(1, 8, 4, 0.5), (37, 200, 4, 0.34), (1024, 768, 4, 0.34),
                                         (1024, 768, 8, 0.02), (4096, 3072, 4, 0.21),
                                         (128, 1024, 8, 0.02), (129, 1024, 8, 0.02)])  # small and large workgroups
def test_scale_gradients(mkq, M, K, bits, s, dtype):
    x = _activations(M, K, M + K + bits, dtype)
    g = to_np(mkq.mkq_scale_gradients(to_dev(x), s, bits))
    qmin, qmax = (-8, 7) if bits == 4 else (-128, 127)
    xf = x.astype(np.float32)
    ste, mse = oracle.scale_gradients(xf, s, qmin, qmax)
    c = oracle.quantize(xf, np.float32(s), qmin, qmax).astype(np.float64)
    xd, sd = xf.astype(np.float64), float(np.float32(s))
    mag_ste = np.abs(-xd / sd + c).sum()
    mag_mse = np.abs(2 * (sd * c - xd) * c).sum()
    assert abs(g[0] - ste) <= 1e-10 * mag_ste + 1e-12
    assert abs(g[1] - mse) <= 1e-10 * mag_mse + 1e-12


def test_scale_gradients_worked_example_and_strided_rows(mkq):
    # section 4.1: x = (0.2, 0.9), s = 1 -> -0.1 and +0.2 (padded with on-grid zeros, which add nothing)
    x = np.zeros((1, 8), np.float32)
    x[0, :2] = (0.2, 0.9)
    g = to_np(mkq.mkq_scale_gradients(to_dev(x), 1.0))
    assert g[0] == pytest.approx(-0.1, abs=1e-6) and g[1] == pytest.approx(0.2, abs=1e-6)
    big = _activations(64, 512, 5, np.float32)
    view = to_dev(big)[:, 128:384]
    g = to_np(mkq.mkq_scale_gradients(view, 0.3))
    ste, mse = oracle.scale_gradients(np.ascontiguousarray(big[:, 128:384]), 0.3)
    assert g[0] == pytest.approx(ste, rel=1e-9) and g[1] == pytest.approx(mse, rel=1e-9)


@pytest.mark.parametrize("dtype", [np.float32, np.float16])
@pytest.mark.parametrize("M,K", [(1, 8), (13, 72), (1024, 768), (4096, 3072)])
def test_percentile_scale_bit_exact(mkq, M, K, dtype):
    x = _activations(M, K, 3 * M + K, dtype)
    if M * K > 100:
        x.flat[7] = np.nan
    for ppm, bits in ((100, 8), (100, 4), (20000, 4), (0, 4), (1000000, 8), (500000, 4)):
        s = float(to_np(mkq.mkq_percentile_scale(to_dev(x), ppm, bits))[0])
        ref, _ = oracle.percentile_scale(x.astype(np.float32), ppm, 7 if bits == 4 else 127)
        assert s == ref, (ppm, bits)


def test_percentile_scale_ties_zeros_and_absmax(mkq):
    ties = np.array([[3, -3, 3, 1, 0, -3, 0, 0]], np.float32)
    for ppm in (0, 250000, 375000, 500000, 625000, 1000000):
        s = float(to_np(mkq.mkq_percentile_scale(to_dev(ties), ppm))[0])
        assert s == oracle.percentile_scale(ties, ppm)[0]
    z = np.zeros((4, 16), np.float32)
    assert float(to_np(mkq.mkq_percentile_scale(to_dev(z)))[0]) == 1.0
    x = _activations(128, 768, 9, np.float16)
    s0 = float(to_np(mkq.mkq_percentile_scale(to_dev(x), 0))[0])
    assert s0 == float(to_np(mkq.mkq_absmax_scale(to_dev(x)))[0])


def test_percentile_step_feeds_the_quantizer(mkq):
    """Calibrate, then quantize with the calibrated step: about top_ppm of the codes clip."""
    x = _activations(2048, 768, 11, np.float16)
    s = float(to_np(mkq.mkq_percentile_scale(to_dev(x), 20000))[0])  # top 2 %
    codes = oracle.unpack_nibbles(to_np(mkq.mkq_quantize(to_dev(x), s)), 768)
    ref = oracle.quantize(x.astype(np.float32), np.float32(s))
    assert np.array_equal(codes, ref)
    clipped = (np.abs(x.astype(np.float32)) >= 7 * s).mean()
    assert 0.015 < clipped < 0.025


@pytest.mark.parametrize("dtype", [np.float32, np.float16])
@pytest.mark.parametrize("order", ["random", "sorted", "outliers first", "constant"])
def test_percentile_in_any_order(mkq, order, dtype):
    """A little more than one group of eight per thread of the largest grid, so that most threads fetch past the end.  Any
    arrangement of the values and any stride of the rows gives the same order statistic."""
    M, K = 2049, 2056
    x = _activations(M, K, 17, dtype)
    if order == "sorted":
        x = np.sort(x, axis=None).reshape(M, K)
    elif order == "outliers first":
        x.flat[:8192] = 0.0
        x.flat[8192:8192 + 4096] = 60.0
    elif order == "constant":
        x[:] = 1.5
    wide = np.full((M, K + 24), 1000, dtype)
    wide[:, 8:8 + K] = x
    for ppm, bits in ((0, 4), (10, 8), (1000, 4), (3900, 4), (3910, 4)):
        ref, _ = oracle.percentile_scale(x.astype(np.float32), ppm, 7 if bits == 4 else 127)
        assert float(to_np(mkq.mkq_percentile_scale(to_dev(x), ppm, bits))[0]) == ref, ppm
        assert float(to_np(mkq.mkq_percentile_scale(to_dev(wide)[:, 8:8 + K], ppm, bits))[0]) == ref, ppm
    assert float(to_np(mkq.mkq_absmax_scale(to_dev(wide)[:, 8:8 + K]))[0]) == np.float32(np.abs(x.astype(np.float32)).max()) / np.float32(7)


@pytest.mark.parametrize("bits,s", [(4, 1.0 / 3), (8, 0.0173), (4, 2.0 ** -120)])
def test_scale_gradients_next_to_rounding_boundaries(mkq, bits, s):
    """Values at, and an ulp beside, every boundary k + 1/2 (and far beyond the clamp range), where the product with
    1/s could round the other way: the codes are the division's, so the sums are the oracle's."""
    s = np.float32(s)
    q = 1 << (bits - 1)
    at = ((np.arange(-q - 2, q + 2, dtype=np.float64) + 0.5) * float(s)).astype(np.float32)
    x = np.concatenate([at, np.nextafter(at, np.float32(np.inf)), np.nextafter(at, np.float32(-np.inf)), at * np.float32(1e4)])
    x = np.concatenate([x, np.zeros(-len(x) % 8, np.float32)]).reshape(1, -1)
    g = to_np(mkq.mkq_scale_gradients(to_dev(x), float(s), bits))
    ste, mse = oracle.scale_gradients(x, s, -q, q - 1)
    # either side rounds every one of its n partial sums once, by 2^-53 of at most the sum of the terms' magnitudes; a
    # code that fell the other way would show as a whole unit (the sums hold 1e4 steps per code at most)
    c = oracle.quantize(x, s, -q, q - 1).astype(np.float64)
    xd, sd = x.astype(np.float64), float(s)
    bound = 2 * x.size * 2.0 ** -53
    assert abs(g[0] - ste) <= bound * np.abs(c - xd / sd).sum() < 0.5
    assert abs(g[1] - mse) <= bound * np.abs(2 * (sd * c - xd) * c).sum()


def test_rows_with_gaps_over_several_batches(mkq):
    """Rows with gaps take whole batches of groups without checks and a last one with them: a tensor of four groups per
    thread and a little more, for the percentile, the abs-max and the gradient sums."""
    M, K = 4100, 4104
    x = _activations(M, K, 23, np.float16)
    wide = np.full((M, K + 8), 1000, np.float16)
    wide[:, :K] = x
    view = to_dev(wide)[:, :K]
    xf = x.astype(np.float32)
    for ppm in (10, 200000):
        assert float(to_np(mkq.mkq_percentile_scale(view, ppm))[0]) == oracle.percentile_scale(xf, ppm, 7)[0]
    assert float(to_np(mkq.mkq_absmax_scale(view))[0]) == np.abs(xf).max() / np.float32(7)
    g = to_np(mkq.mkq_scale_gradients(view, 0.34))
    ste, mse = oracle.scale_gradients(xf, 0.34, -8, 7)
    c = oracle.quantize(xf, np.float32(0.34)).astype(np.float64)
    xd, sd = xf.astype(np.float64), float(np.float32(0.34))
    assert abs(g[0] - ste) <= 1e-10 * np.abs(c - xd / sd).sum()
    assert abs(g[1] - mse) <= 1e-10 * np.abs(2 * (sd * c - xd) * c).sum()


@pytest.mark.parametrize("M,K", [(1, 131072), (1, 131080), (8, 16392), (2048, 8192), (2049, 8200), (8200, 4104)])
def test_contiguous_tensors_around_the_batches(mkq, M, K):
    """One group more or less than what 64 small workgroups, one batch of the whole grid and whole windows of it cover; the
    largest value in the last and in the first place.  Order statistics and maxima: exact."""
    import torch
    for dtype in (torch.float16, torch.float32):
        g = torch.Generator(device="cuda").manual_seed(M + K)
        x = torch.randn(M, K, generator=g, device="cuda").to(dtype)
        for at in (-1, 0):
            x.view(-1)[at] = -70.0
            assert float(mkq.mkq_absmax_scale(x)) == np.float32(70.0) / np.float32(7)
            for ppm in (0, 200):
                k = max(1, M * K * ppm // 10 ** 6)
                kth = torch.topk(x.view(-1).abs().float(), k).values[-1]
                assert float(mkq.mkq_percentile_scale(x, ppm)) == np.float32(float(kth)) / np.float32(7), (dtype, at, ppm)
            x.view(-1)[at] = 0.5


@pytest.mark.parametrize("dtype", ["float16", "float32"])
def test_absmax_reads_every_place_of_its_windows(mkq, dtype):
    """Contiguous tensors of two windows of the grid (256 workgroups of 1024 threads, eight groups of eight values each) and a
    remainder: the largest value in every one of the eight steps, in the first, a middle and the last workgroup, in its first and
    last thread, of both windows, at the seams and in the remainder."""
    import torch
    M, K = 4100, 8208
    step, share = 1024 * 8, 8 * 1024 * 8          # values of a step, and of a workgroup's part of a window
    window = 256 * share
    assert 2 * window + 8 < M * K < 3 * window
    g = torch.Generator(device="cuda").manual_seed(7)
    x = torch.rand(M, K, generator=g, device="cuda").to(getattr(torch, dtype))
    places = [w * window + wg * share + a * step + t * 8 + (3 * a + wg + w) % 8
              for w in (0, 1) for wg in (0, 131, 255) for a in range(8) for t in (0, 1023)]
    places += [window - 1, window, 2 * window - 1, 2 * window, 2 * window + 7, M * K - 8, M * K - 1]
    flat, got = x.view(-1), []
    for i in places:
        old = flat[i].clone()
        flat[i] = -70.0
        got.append(mkq.mkq_absmax_scale(x))
        flat[i] = old
    got = to_np(torch.cat(got))
    assert np.all(got == np.float32(70.0) / np.float32(7)), [p for p, s in zip(places, got) if s != got.max()]


@pytest.mark.parametrize("larger", [2.0, 1.0 + 2.0 ** -10])
def test_percentile_counts_every_value_of_its_windows_once(mkq, larger):
    """A contiguous binary16 tensor of two windows of the grid (512 workgroups of 1024 threads, eight groups of eight values each)
    and a remainder, of two values in random places, the rank being the number of the larger ones, or one more: one less of
    them, or one counted twice, is another result.  The first pass tells 1 from 2, the second 1 from 1 + 2^-10."""
    import torch
    M, K = 8193, 8200
    n, window = M * K, 512 * 1024 * 8 * 8
    assert 2 * window + 8 < n < 3 * window and n % 2 == 0
    k = n // 2
    g = torch.Generator(device="cuda").manual_seed(11)
    is_larger = torch.rand(n, generator=g, device="cuda") < 0.5
    surplus = int(is_larger.sum()) - k
    from_these = (is_larger if surplus > 0 else ~is_larger).nonzero()[:, 0]
    is_larger[from_these[torch.randperm(len(from_these), generator=g, device="cuda")[:abs(surplus)]]] = surplus < 0
    assert int(is_larger.sum()) == k
    x = torch.where(is_larger, larger, 1.0).half().view(M, K)
    assert float(mkq.mkq_percentile_scale(x, 500000)) == np.float32(larger) / np.float32(7)
    x.view(-1)[is_larger.nonzero()[k // 3, 0]] = 1.0
    assert float(mkq.mkq_percentile_scale(x, 500000)) == np.float32(1) / np.float32(7)


def test_percentile_of_every_binary16_value(mkq):
    """All 65536 bit patterns, subnormals, infinities and NaN (which rank as 0) among them, at every rank."""
    import torch
    x = np.arange(65536, dtype=np.uint16).view(np.float16).reshape(64, 1024)
    order = np.sort(np.where(np.isnan(x), 0, np.abs(x)).astype(np.float32), axis=None)[::-1]
    d = to_dev(x)
    for ppm in (0, 16, 31, 1000, 30000, 31250, 40000, 250000, 499000, 900000, 968000, 999990, 1000000):
        t = order[max(1, 65536 * ppm // 10 ** 6) - 1]
        want = np.float32(t) / np.float32(7) if t > 0 else np.float32(1)
        assert to_np(mkq.mkq_percentile_scale(d, ppm))[0] == want, ppm
