"""The index arithmetic of csrc/qgx_plan.h, built with the host compiler: what the kernels rest their bounds on."""
import ctypes as C
import itertools
import os
import subprocess

import numpy as np
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
// out[i] = k * units + unit, or -1; lg < 0: block_by_unit
extern "C" void blocks(uint32_t grid, uint32_t K, uint32_t units, int lg, int64_t* out)
{
    for (uint32_t i = 0; i < grid; ++i) {
        const qgx::BlockWork b = lg < 0 ? qgx::block_by_unit(i, K, units) : qgx::block_by_worker(i, K, units, (uint32_t)lg);
        out[i] = b.there ? (int64_t)b.k * units + b.unit : -1;
    }
}
extern "C" uint32_t grid_by_worker(uint32_t K, uint32_t units, uint32_t lg) { return qgx::grid_by_worker(K, units, lg); }
extern "C" uint32_t worker_groups_log2(uint32_t K, uint32_t parts, uint32_t held) { return qgx::worker_groups_log2(K, parts, held); }
extern "C" uint32_t held_per_xcd(uint32_t waves, size_t lds, uint32_t n_cu) { return qgx::held_per_xcd(waves, lds, n_cu); }
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


def _blocks(plan, K, units, lg):
    grid = K * units if lg < 0 else plan.grid_by_worker(K, units, lg)
    out = np.empty(grid, np.int64)
    plan.blocks(C.c_uint32(grid), C.c_uint32(K), C.c_uint32(units), C.c_int(lg), out.ctypes.data_as(C.c_void_p))
    return out


@pytest.mark.parametrize("lg", [-1, 0, 1, 2, 3])
def test_every_worker_has_every_unit_once(plan, lg):
    for K, units in itertools.product([1, 2, 3, 5, 7, 8, 9, 16, 31, 33, 63, 64], [1, 2, 7, 8, 9, 15, 16, 17, 40, 67]):
        got = _blocks(plan, K, units, lg)
        np.testing.assert_array_equal(np.sort(got[got >= 0]), np.arange(K * units), err_msg="K %d units %d" % (K, units))
        if lg < 0:                                           # a unit's workgroups in whole rounds: one XCD, one after the other
            for unit in range(units // 8 * 8):
                np.testing.assert_array_equal(got[unit // 8 * 8 * K + unit % 8 + 8 * np.arange(K)], np.arange(K) * units + unit)
        if lg == 0 or K % 8 == 0 and lg > 0:
            i = np.arange(K * units)
            np.testing.assert_array_equal(got, i % K * units + i // K)
        if lg > 0:
            there = np.flatnonzero(got >= 0)
            np.testing.assert_array_equal(there % (1 << lg), got[there] // units % (1 << lg))


def _stalls(work, K, units, parts, held, late):
    """XCD `late` starts its workgroups after all the others have started theirs: does it come to hold nothing but
    workgroups that wait for partners in its own queue?  A bucket goes on when all its parts have started."""
    k = np.where(work >= 0, work // units, -1)
    mine = np.arange(len(work)) % 8 == late
    started = np.bincount(k[~mine & (k >= 0)], minlength=K)  # tickets taken, worker by worker
    waiting = np.zeros(K, np.int64)                          # of those, on the late XCD, in the worker's newest bucket
    for w in k[mine & (k >= 0)]:
        if waiting.sum() >= held:
            return True
        started[w] += 1
        waiting[w] = 0 if started[w] % parts == 0 else waiting[w] + 1
    return False


def test_no_xcd_fills_up_with_workgroups_that_wait(plan):
    """Buckets of four parts, an XCD that is behind: the map that a launch takes always leaves it a place (with 160, 128
    or 96 workgroups to an XCD; the game's form takes block_by_unit when one group is enough)."""
    assert [plan.held_per_xcd(C.c_uint32(5), C.c_size_t(n), C.c_uint32(256)) for n in (30000, 40000, 53000)] == [160, 128, 96]
    parts, units, seen = 4, 64, 0
    for K, held, late in itertools.product([1, 8, 31, 32, 33, 42, 43, 47, 48, 53, 54, 57, 63, 64], [96, 128, 160], [0, 3, 7]):
        lg = plan.worker_groups_log2(K, parts, held)
        assert not (lg == 0 and 3 * K >= held) and 3 * -(-K // (1 << lg)) < held
        for m in (lg,) if lg else (-1, 0):
            assert not _stalls(_blocks(plan, K, units, m), K, units, parts, held, late), (K, held, late, m)
        seen += _stalls(_blocks(plan, K, units, -1), K, units, parts, held, late)
    assert seen                                              # the model knows a stall: many workers, all on every XCD
