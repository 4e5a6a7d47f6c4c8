"""Host arithmetic of the few-frames path's first launch (CPU only)."""
import ctypes
import os
import subprocess

import pytest

import paper_1812_06545_amd as L

SOURCE = """
#include "few_layout.h"
extern "C" void few(int32_t n, int32_t W, int32_t max_iter, int32_t es, int64_t *out)
{
    const ldpc::FewInit s = ldpc::few_init(n, W, max_iter, es != 0);
    out[0] = s.unsat_words;
    out[1] = s.words;
    out[2] = s.blocks;
}
"""


@pytest.fixture(scope="module")
def few(tmp_path_factory):
    folder = tmp_path_factory.mktemp("few")
    (folder / "few.cpp").write_text(SOURCE)
    include = os.path.join(os.path.dirname(L.__file__), "csrc")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I", include, str(folder / "few.cpp"), "-o",
                    str(folder / "few.so")], check=True)
    lib = ctypes.CDLL(str(folder / "few.so"))

    def call(n, W, max_iter, es):
        out = (ctypes.c_int64 * 3)()
        lib.few(n, W, max_iter, int(es), out)
        return tuple(out)
    return call


@pytest.mark.parametrize("max_iter", [0, 1, 50, (1 << 26) - 1, 1 << 26, (1 << 31) - 1])
@pytest.mark.parametrize("W", [2, 8, 32])
def test_every_mark_is_set(few, W, max_iter):
    """Whatever the iteration cap, every unsatisfied mark and every channel value
    is among the words that the launch sets, and its grid's threads stay below
    2^32 (the limit of one launch)."""
    for n in (1, 16200, 400000):
        for es in (False, True):
            unsat, words, blocks = few(n, W, max_iter, es)
            assert unsat == (max_iter * W if es else 0)
            assert words == max(n * W, unsat)
            assert 1 <= blocks and blocks * 256 < 1 << 32
            assert blocks * 256 >= words or blocks == 1 << 20
