"""The rules of launches (csrc/launch_rules.h, plain arithmetic) at their edges, compiled for the host."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ONE_BLOCK, HELD, BLOCKS = range(3)
SRC = """
#include "launch_rules.h"
using namespace mkq;
extern "C" int route(int64_t batch, int64_t seq, int64_t hidden, int64_t heads, int64_t q_pitch)
{
    return attention_route(batch, seq, hidden, heads, q_pitch);
}
extern "C" int held_blocks(int64_t sequence_heads, int q_blocks, int64_t resident)
{
    return attention_held_blocks(sequence_heads, q_blocks, resident);
}
extern "C" int run_index(unsigned wg, int64_t sequence_heads, int64_t heads)
{
    return xcd_run_index(wg, attention_runs(sequence_heads, heads));
}
extern "C" int piece_index(unsigned wg, unsigned total) { return xcd_index(wg, total); }
extern "C" int first_half(int64_t sequence_heads, int q_blocks, int per_wg)
{
    return attention_held_first_half(sequence_heads, q_blocks, per_wg);
}
extern "C" int fetch_ahead(bool full, int groups) { return held_fetch_ahead(full, groups); }
extern "C" bool half_waves(int64_t M, int64_t D) { return layernorm_half_waves(M, D); }
extern "C" bool small_attention(int64_t batch, int64_t seq, int64_t hidden, int64_t heads, int64_t row)
{
    return small_layer_attention(batch, seq, hidden, heads, row);
}
extern "C" bool small_attention_taken(int64_t batch, int64_t seq, int64_t hidden, int64_t heads, int64_t row, bool padding_free)
{
    return small_layer_attention_choice(batch, seq, hidden, heads, row, padding_free);
}
extern "C" int few(int64_t M, int64_t N, int64_t row_bytes, int bits) { return few_tile(M, N, row_bytes, bits); }
extern "C" int i8_tiles_of_three(int64_t M, int64_t N, int64_t K, bool gelu, bool residual)
{
    return i8_128x96(M, N, K, gelu) + 2 * i8_256x192(M, N, K, gelu, residual);
}
extern "C" int f16_tiles_of_three(int64_t M, int64_t N, int64_t K, bool gelu, bool residual)
{
    return f16_128x96(M, N, K, gelu, residual) + 2 * f16_256x192_suits(N, K, residual);
}
extern "C" int few_taken(int64_t M, int64_t N, int64_t row_bytes, int bits) { return few_choice(M, N, row_bytes, bits); }
extern "C" int few_asked(int64_t M, int64_t N, int64_t row_bytes, int bits) { return few_tile_or_largest(M, N, row_bytes, bits); }
extern "C" int few_at(unsigned wg, int64_t M, int64_t N, int64_t row_bytes, int channels, int tokens)
{
    const FewOrder o = few_order(M, N, row_bytes, channels, tokens);
    const int64_t ct = (N + channels - 1) / channels, tt = (M + tokens - 1) / tokens;
    if (!o.inner) return (int)wg;
    const FewPlace at = few_place(wg, (unsigned)(ct * tt), o);
    return (int)(at.tokens * ct + at.channels);
}
extern "C" bool small_tail(int64_t tokens, int64_t row, int64_t ffn_row) { return small_layer_tail(tokens, row, ffn_row); }
extern "C" bool output_with_norm(int64_t tokens, int64_t hidden, int64_t row) { return output_norm(tokens, hidden, row); }
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    (d / "rules.cpp").write_text(SRC)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC",
                    "-I", os.path.join(ROOT, "paper_2203_13483_amd", "csrc"), "-o", str(d / "rules.so"), str(d / "rules.cpp")],
                   check=True)
    lib = C.CDLL(str(d / "rules.so"))
    lib.route.argtypes = [C.c_int64] * 5
    lib.held_blocks.argtypes = [C.c_int64, C.c_int, C.c_int64]
    lib.run_index.argtypes = [C.c_uint, C.c_int64, C.c_int64]
    lib.piece_index.argtypes = [C.c_uint, C.c_uint]
    lib.first_half.argtypes = [C.c_int64, C.c_int, C.c_int]
    lib.fetch_ahead.argtypes = [C.c_bool, C.c_int]
    lib.half_waves.argtypes, lib.half_waves.restype = [C.c_int64] * 2, C.c_bool
    lib.small_attention_taken.argtypes, lib.small_attention_taken.restype = [C.c_int64] * 5 + [C.c_bool], C.c_bool
    lib.small_attention.argtypes, lib.small_attention.restype = [C.c_int64] * 5, C.c_bool
    lib.output_with_norm.argtypes, lib.output_with_norm.restype = [C.c_int64] * 3, C.c_bool
    lib.i8_tiles_of_three.argtypes = [C.c_int64] * 3 + [C.c_bool] * 2
    lib.f16_tiles_of_three.argtypes = [C.c_int64] * 3 + [C.c_bool] * 2
    lib.few_at.argtypes = [C.c_uint, C.c_int64, C.c_int64, C.c_int64, C.c_int, C.c_int]
    lib.small_tail.argtypes, lib.small_tail.restype = [C.c_int64] * 3, C.c_bool
    return lib


def test_attention_of_ordinary_sizes(rules):
    assert rules.route(4, 128, 768, 12, 768) == ONE_BLOCK
    assert rules.route(4, 128, 768, 12, 896) == HELD
    assert rules.route(4, 129, 768, 12, 768) == HELD
    assert rules.route(4, 512, 1024, 16, 1024) == HELD
    assert rules.route(4, 513, 1024, 16, 1024) == BLOCKS
    assert rules.route(4, 128, 312, 12, 384) == HELD   # heads of 26
    assert rules.route(4, 128, 320, 8, 320) == HELD    # of 40
    assert rules.route(4, 128, 336, 8, 336) == BLOCKS  # of 42


def test_rows_beyond_32_bit_offsets_keep_the_kernel_with_64_bit_ones(rules):
    """A sequence's rows of q, k and v are 6 hidden bytes each."""
    for dk in (8, 32, 64):
        for seq in (129, 384, 511, 512):
            most = 2 ** 32 // (seq * 6)                  # hidden sizes up to here fit
            heads = most // dk
            assert rules.route(4, seq, heads * dk, heads, heads * dk) == HELD
            assert rules.route(4, seq, (heads + 1) * dk, heads + 1, (heads + 1) * dk) == BLOCKS
    assert rules.route(1, 512, 1400896, 21889, 1400896) == BLOCKS
    assert rules.route(4, 128, 64 * 10 ** 6, 10 ** 6, 64 * 10 ** 6) == ONE_BLOCK


def test_launches_stay_within_the_work_items_of_a_dimension(rules):
    """Fewer than 2^32: 8388607 workgroups of 512 threads, of 256 twice as many and one."""
    limit = (2 ** 32 - 1) // 512
    for heads, dk in ((8, 8), (12, 26), (1, 48)):
        H = heads * dk
        assert rules.route(limit // heads, 1, H, heads, H) == HELD
        assert rules.route(limit // heads + 1, 1, H, heads, H) == BLOCKS
        assert rules.route(limit // heads, 512, H, heads, H) == HELD
    for sequence_heads in (1, 12, 255, 256, 257, 1000, 65536, limit // 4, limit // 4 + 1, limit // 2 + 1, limit):
        for q_blocks in (1, 2, 3, 4):
            for resident in (256, 512, 1024):
                c = rules.held_blocks(sequence_heads, q_blocks, resident)
                assert 1 <= c <= q_blocks
                assert sequence_heads * -(-q_blocks // c) <= limit
    # as many workgroups as the device holds at a time, where blocks can be spread
    assert [rules.held_blocks(n, 4, 256) for n in (1, 64, 65, 128, 256, 10 ** 6)] == [1, 1, 2, 2, 4, 4]


def test_layernorm_of_more_rows_than_fit_a_launch_four_to_a_workgroup(rules):
    most = 4 * ((2 ** 32 - 1) // 256)
    for D in (264, 312, 512, 776, 1024):
        assert not rules.half_waves(2048, D) and not rules.half_waves(most, D)
        assert rules.half_waves(most + 1, D) and rules.half_waves(2 * most, D)
    for D in (8, 256, 520, 768):
        assert not rules.half_waves(2047, D)
        assert rules.half_waves(2048, D) and rules.half_waves(most + 1, D)
    assert not rules.half_waves(most + 1, 1032)  # no half-wave kernel of this size


@pytest.mark.parametrize("batch,heads", [(1, 1), (3, 5), (5, 12), (8, 8), (16, 12), (21, 16), (64, 12), (67, 12), (300, 3)])
def test_every_sequence_and_head_is_dealt_once(rules, batch, heads):
    n = batch * heads
    assert sorted(rules.run_index(w, n, heads) for w in range(n)) == list(range(n))
    assert sorted(rules.piece_index(w, n) for w in range(n)) == list(range(n))


@pytest.mark.parametrize("batch,longest", [(16, 512), (64, 128), (32, 256), (8, 512)])
@pytest.mark.parametrize("order", ["rising", "falling", "shuffled"])
def test_sequences_of_different_lengths_are_dealt_evenly(rules, batch, longest, order):
    """Work of a sequence and head: its keys times its queries and the staging (half a block of queries).  The XCD with most of it
    has at most half as much again as the mean; an eighth of the sequences in one piece has twice the mean and more."""
    lens = np.linspace(longest // 16, longest, batch).astype(int)
    lens = {"rising": lens, "falling": lens[::-1], "shuffled": np.random.default_rng(batch).permutation(lens)}[order]
    heads = 12
    n = batch * heads

    def busiest(index):
        load = np.zeros(8)
        for w in range(n):
            length = int(lens[index(w) // heads])
            load[w % 8] += length * (length + 64)
        return load.max() / load.mean()
    assert busiest(lambda w: rules.run_index(w, n, heads)) < 1.5
    if order != "shuffled":
        assert busiest(lambda w: rules.piece_index(w, n)) > 2.0


def test_only_sequences_that_one_workgroup_would_have_are_shared(rules):
    limit = (2 ** 32 - 1) // 512
    assert [rules.first_half(256, q, q) for q in (1, 2, 3, 4)] == [0, 1, 2, 2]
    assert rules.first_half(256, 4, 2) == 0 and rules.first_half(256, 3, 1) == 0
    assert rules.first_half(limit // 2, 4, 4) == 2 and rules.first_half(limit // 2 + 1, 4, 4) == 0


def test_only_groups_of_keys_that_exist_are_fetched_ahead(rules):
    assert [rules.fetch_ahead(full, g) for full in (False, True) for g in (2, 4, 6, 8, 10, 12, 14, 16)] == [0] * 12 + [1] * 4


def test_small_layers(rules):
    assert rules.small_attention(32, 128, 312, 12, 384) and rules.small_attention(1, 1, 128, 4, 128)
    assert not rules.small_attention(32, 129, 312, 12, 384)   # longer than four tiles of 32 tokens
    assert not rules.small_attention(32, 128, 384, 6, 384)    # heads of 64
    assert not rules.small_attention(32, 128, 768, 24, 768) and not rules.small_attention(32, 128, 320, 10, 320)
    # one workgroup of 256 threads per sequence and head
    most = 0xFFFFFFFF // 256
    assert rules.small_attention(most // 12, 128, 312, 12, 384) and not rules.small_attention(most // 12 + 1, 128, 312, 12, 384)
    assert rules.small_tail(4096, 384, 1280) and rules.small_tail(1, 128, 128)
    assert not rules.small_tail(4097, 384, 1280)
    assert not rules.small_tail(4096, 512, 2048) and not rules.small_tail(4096, 352, 1280) and not rules.small_tail(4096, 384, 1312)


def test_small_layers_keep_the_kernel_that_their_attention_would_take(rules):
    """In one launch with q, k, v only where the launch of its own is the held kernel, whose bits it has: beyond, that is another kernel."""
    most = 0xFFFFFFFF // 512
    for hidden, heads, row in ((312, 12, 384), (128, 4, 128), (384, 12, 384)):
        for batch in (1, most // heads, most // heads + 1):
            assert rules.small_attention_taken(batch, 128, hidden, heads, row, False) == (rules.route(batch, 128, hidden, heads, row) == HELD)


def test_small_layers_of_many_small_heads_keep_kernels_of_their_own(rules):
    def taken(batch, seq, hidden, heads, padding_free=False):
        return rules.small_attention_taken(batch, seq, hidden, heads, -(-hidden // 128) * 128, padding_free)
    for ragged in (False, True):
        assert taken(16, 128, 256, 32, ragged) and not taken(17, 128, 256, 32, ragged)     # heads of 8
        assert taken(32, 64, 256, 32, ragged) and not taken(33, 64, 256, 32, ragged)
        assert taken(64, 32, 256, 32, ragged) and not taken(65, 32, 256, 32, ragged)
        assert taken(42, 128, 384, 24, ragged) and not taken(43, 128, 384, 24, ragged)     # of 16
        assert taken(78, 128, 312, 13, ragged) and not taken(79, 128, 312, 13, ragged)     # of 24
        assert taken(85, 128, 312, 12, ragged) and taken(86, 128, 312, 12, ragged) == (not ragged)  # of 26
        assert taken(315, 32, 312, 13, ragged) and taken(316, 32, 312, 13, ragged) == (not ragged)


def test_small_layers_in_one_launch(rules):
    """FFN columns in whole chunks: 768 always, beyond 600 more than there are tokens, 3840 at most."""
    assert rules.small_tail(16, 384, 768) and not rules.small_tail(16, 384, 896) and not rules.small_tail(16, 384, 8192)
    assert rules.small_tail(680, 384, 1280) and not rules.small_tail(679, 384, 1280) and not rules.small_tail(440, 384, 1280)
    assert rules.small_tail(936, 384, 1408) and not rules.small_tail(935, 384, 1408)  # two narrow chunks
    assert rules.small_tail(4096, 384, 3840) and rules.small_tail(3240, 384, 3840) and not rules.small_tail(3239, 384, 3840)
    assert not rules.small_tail(4096, 384, 3968) and not rules.small_tail(4096, 384, 16384)


def test_output_norm(rules):
    assert all(rules.output_with_norm(m, *hr) for m in (2048, 4096) for hr in ((768, 768), (640, 640), (744, 768)))
    assert not rules.output_with_norm(2047, 768, 768) and not rules.output_with_norm(4097, 768, 768)
    assert not rules.output_with_norm(4096, 1024, 1024) and not rules.output_with_norm(4096, 512, 512)
    assert not rules.output_with_norm(4096, 672, 672)  # no whole half units of 128 codes


def test_tiles_of_three_parts_leave_short_k_loops_to_smaller_ones(rules):
    """(M, N, K): neither, 1 128x96, 2 256x192; plain, with a residual, with GELU."""
    def kinds(*shape):
        return [rules.i8_tiles_of_three(*shape, gelu, res) for gelu, res in ((False, False), (False, True), (True, False))]
    assert kinds(8653, 256, 1536) == [1, 1, 0] and kinds(3815, 768, 2048) == [1, 1, 1] and kinds(3815, 768, 1472) == [0, 0, 0]
    assert kinds(10942, 768, 128) == [0, 0, 0] and kinds(10942, 768, 320) == [0, 0, 0] and kinds(10942, 768, 384) == [0, 0, 2]
    assert kinds(10942, 768, 512) == [0, 2, 2] and kinds(10942, 768, 1536) == [2, 2, 2]
    assert kinds(11546, 936, 512) == [0, 0, 2] and kinds(11546, 936, 960) == [0, 0, 2] and kinds(11546, 936, 1024) == [0, 2, 2]
    assert kinds(16384, 768, 1024) == [0, 2, 2] and kinds(16385, 768, 1024) == [0, 0, 0]  # one round


def test_binary16_tiles_of_three_parts_leave_short_k_loops_to_smaller_ones(rules):
    """(M, N, K): 1 128x96 is taken, 2 256x192 may be; plain, with a residual, with GELU."""
    def kinds(*shape):
        return [rules.f16_tiles_of_three(*shape, gelu, res) for gelu, res in ((False, False), (False, True), (True, False))]
    assert kinds(5204, 512, 128) == [3, 2, 2] and kinds(5204, 512, 384) == [3, 3, 2] and kinds(5204, 512, 640) == [3, 3, 3]
    assert kinds(11647, 936, 384) == [2, 0, 2] and kinds(11428, 936, 768) == [2, 2, 2] and kinds(11647, 960, 384) == [2, 2, 2]


def test_few_tokens_leaves_short_and_uneven_rows_to_the_persistent_kernels(rules):
    few = lambda *s, bits=4: rules.few_taken(*map(C.c_int64, s), bits)  # noqa: E731
    assert few(1024, 512, 64) == 2 and few(1024, 513, 64) == -1 and few(41, 12288, 64) == -1  # one piece: a second 32x64 per CU
    assert few(1024, 512, 128) == 2 and few(1024, 544, 128) == -1 and few(59, 12288, 128) == 3 and few(65, 8192, 128) == -1
    assert few(1024, 544, 192) == 3
    # 18 and 20 pieces of 64 bytes among eight waves, 24 and 16, 20 of 128 bytes
    assert few(1040, 768, 1152) == 4 and few(1041, 768, 1152) == 4 and few(1664, 512, 1152) == 4 and few(1665, 512, 1152) == -1
    assert few(1152, 512, 1280) == 4 and few(1153, 512, 1280) == -1
    assert few(2048, 512, 1536) == 4 and few(2048, 512, 1024) == 4 and few(2048, 512, 2560) == 9
    assert few(2049, 512, 1536) == -1


@pytest.mark.parametrize("M,N,row_bytes,channels,tokens", [(1024, 512, 256, 32, 64), (2048, 256, 1024, 32, 64), (16384, 64, 64, 64, 64), (33, 8, 64, 32, 32),
                                                           (440, 768, 384, 32, 32), (444, 768, 5120, 32, 64), (700, 940, 4096, 64, 64), (500, 936, 64, 32, 32), (900, 2000, 4096, 64, 64), (128, 1 << 17, 1024, 64, 64),
                                                           (128, 30000, 4096, 64, 64), (7379, 64, 4096, 32, 64)])
def test_tiles_of_few_tokens_by_xcd(rules, M, N, row_bytes, channels, tokens):
    """Every tile has its workgroup, and each XCD an eighth of the tokens with all channels, or of the channels with all tokens, unless both
    fit its L2 anyway."""
    ct, tt = -(-N // channels), -(-M // tokens)
    at = np.array([rules.few_at(w, M, N, row_bytes, channels, tokens) for w in range(ct * tt)])
    assert np.array_equal(np.sort(at), np.arange(ct * tt))
    if M > N or (2 * M > N and N * row_bytes <= 3 << 19):
        if M * row_bytes < 1 << 16:
            return  # little to read
        for x in range(8):
            assert len(set(at[x::8] // ct)) <= -(-tt // 8) + 1
    elif (M + N) * row_bytes > 1 << 22 and tt > 2:
        for x in range(8):
            assert len(set(at[x::8] % ct)) <= -(-ct // 8) + 1


def test_few_tokens(rules):
    """The tile of the kernels of few tokens, and the shapes that their GPU test means to take each with."""
    from test_gpu_few import SHAPES
    few = lambda *s, bits=4: rules.few(*map(C.c_int64, s), bits)  # noqa: E731
    assert [few(*s) for s in SHAPES] == [0] * 3 + [1] * 2 + [2] * 3 + [3] * 2 + [4] * 2 + [5, 6, 7, 8, 9, 9]
    assert [few(*s, bits=8) for s in SHAPES] == [0] * 3 + [1] * 2 + [2] * 3 + [-1] * 4 + [5, 6, 7, 8, -1, 9]
    assert few(16, 1 << 20, 64) == 0 and few(17, 8192, 64) == 1 and few(17, 8193, 64) == 2
    assert few(640, 768, 384) == 2 and few(704, 768, 384) == 3 and few(641, 768, 1024) == 4 and few(512, 512, 768, bits=8) == 2
    assert few(256, 1024, 1024, bits=8) == 2 and few(257, 1024, 1024, bits=8) == 3
    assert few(4096, 768, 384) == -1 and few(64, 30522, 384) == -1   # persistent kernels
    assert few(1, 8, 32) == -1 and few(1, 8, 96) == -1               # pieces of 64 bytes
    assert few(8, 8, 2112) == 0                                      # long, but not in pieces of 128
    assert few(16, 0xFFFFFFFF // 512 * 16, 64) == 0 and few(16, 0xFFFFFFFF // 512 * 16 + 1, 64) == -1  # what a launch takes
    # asked for by number, up to 128 tokens: some tile, whatever the size
    assert all(rules.few_asked(C.c_int64(M), C.c_int64(N), C.c_int64(r), b) >= 0
               for M in (1, 65, 128) for N in (8, 30522, 1 << 20) for r in (128, 1024, 4096) for b in (4, 8))
