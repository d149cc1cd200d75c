"""The index arithmetic of csrc/qgx_plan.h, built with the host compiler: what the kernels rest their bounds on."""
import ctypes as C
import itertools
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

WRAPPER = r"""
#include "qgx_plan.h"
extern "C" int half_words(uint32_t off, uint32_t start, uint32_t end, uint32_t max_words, uint64_t cap, uint64_t* out)
{
    const qgx::HalfWords h = qgx::half_words(off, start, end, max_words, cap);
    out[0] = h.at; out[1] = h.w0; out[2] = h.words;
    return h.ok;
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "w.cpp").write_text(WRAPPER)
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-shared", "-fPIC", "-I",
                           os.path.join(ROOT, "paper_2308_09187_amd", "csrc"), "-o", str(d / "w.so"), str(d / "w.cpp")])
    return C.CDLL(str(d / "w.so"))


def test_half_words_stay_inside_the_payload(plan):
    """Whatever the tables say, max(words, 4) words from `at` lie inside the payload (that is what a decoder reads),
    and every extent of a valid stream passes."""
    plan.half_words.argtypes = [C.c_uint32, C.c_uint32, C.c_uint32, C.c_uint32, C.c_uint64, C.c_void_p]
    out = (C.c_uint64 * 3)()
    max_words = 64 * 14 + 8                                  # half a chunk of 14-bit symbols
    bits = [0, 1, 31, 32, 33, 127, 128, 129, 255, 256, 2048, 28672, 28800, 57344, 65535]
    for cap in (4, 8, 1792, 4096, (1 << 32) - 4):
        offs = {0, 1, 4, 1788, 4092, 4096, (1 << 32) - 4, (1 << 32) - 1, *(cap - 4 * j for j in range(0, 6) if cap >= 4 * j)}
        for off, start, end in itertools.product(sorted(offs), bits, bits):
            ok = plan.half_words(off & 0xFFFFFFFF, start, end, max_words, cap, out)
            at, w0, words = out
            assert at + max(words, 4) <= cap and at % 4 == 0 and words % 4 == 0 and words <= max_words, (cap, off, start, end)
            last = (end + 127) // 128 * 4                    # one past the words that hold bits start .. end - 1
            valid = off % 4 == 0 and start < end and last - start // 128 * 4 <= max_words and off + last <= cap
            assert not valid or (ok and at == off + w0 and w0 == start // 128 * 4 and words == last - w0), (cap, off, start, end)
