"""The rules of launches (csrc/launch_rules.h, plain arithmetic) at their edges, compiled for the host."""
import ctypes as C
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ONE_BLOCK, HELD, BLOCKS = range(3)
SRC = """
#include "launch_rules.h"
using namespace mkq;
extern "C" int route(int64_t seq, int64_t hidden, int64_t heads, int64_t q_pitch)
{
    return attention_route(seq, hidden, heads, q_pitch);
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    (d / "rules.cpp").write_text(SRC)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC",
                    "-I", os.path.join(ROOT, "paper_2203_13483_amd", "csrc"), "-o", str(d / "rules.so"), str(d / "rules.cpp")],
                   check=True)
    lib = C.CDLL(str(d / "rules.so"))
    lib.route.argtypes = [C.c_int64] * 4
    return lib


def test_attention_of_ordinary_sizes(rules):
    assert rules.route(128, 768, 12, 768) == ONE_BLOCK
    assert rules.route(128, 768, 12, 896) == HELD
    assert rules.route(129, 768, 12, 768) == HELD
    assert rules.route(512, 1024, 16, 1024) == HELD
    assert rules.route(513, 1024, 16, 1024) == BLOCKS
    assert rules.route(128, 312, 12, 384) == HELD   # heads of 26
    assert rules.route(128, 320, 8, 320) == HELD    # of 40
    assert rules.route(128, 336, 8, 336) == BLOCKS  # of 42


def test_rows_beyond_32_bit_offsets_keep_the_kernel_with_64_bit_ones(rules):
    """A sequence's rows of q, k and v are 6 hidden bytes each."""
    for dk in (8, 32, 64):
        for seq in (129, 384, 511, 512):
            most = 2 ** 32 // (seq * 6)                  # hidden sizes up to here fit
            heads = most // dk
            assert rules.route(seq, heads * dk, heads, heads * dk) == HELD
            assert rules.route(seq, (heads + 1) * dk, heads + 1, (heads + 1) * dk) == BLOCKS
    assert rules.route(512, 1400896, 21889, 1400896) == BLOCKS
    assert rules.route(128, 64 * 10 ** 6, 10 ** 6, 64 * 10 ** 6) == ONE_BLOCK
