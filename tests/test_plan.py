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
extern "C" void blocks_by_unit(uint32_t K, uint32_t units, int64_t* out)
{
    for (uint32_t i = 0; i < K * units; ++i) {
        const qgx::BlockWork b = qgx::block_by_unit(i, K, units);
        out[i] = (int64_t)b.k * units + b.unit;
    }
}
extern "C" uint32_t worker_span(uint32_t K, uint32_t parts, uint32_t held) { return qgx::worker_span(K, parts, held); }
extern "C" uint32_t waves_per_task(uint32_t n, uint32_t K, uint32_t simds, uint32_t streams) { return qgx::waves_per_task(n, K, simds, streams); }
extern "C" uint32_t worker_spread(uint32_t k, uint32_t unit, uint32_t span) { return qgx::worker_spread(k, unit, span); }
extern "C" int spread_workers(uint32_t K, uint32_t units) { return qgx::spread_workers(K, units); }
extern "C" uint32_t buckets_per_group(uint32_t waves, uint64_t chunks, int ordered) { return qgx::buckets_per_group(waves, chunks, ordered != 0); }
extern "C" uint32_t waves_with_a_bucket(uint32_t unit, uint32_t group, uint32_t waves, uint32_t NB) { return qgx::waves_with_a_bucket(unit, group, waves, NB); }
extern "C" int use_staged(uint64_t chunks, uint32_t n_simd) { return qgx::use_staged(chunks, n_simd); }
extern "C" int use_columns(uint64_t chunks, uint32_t per_bucket, int shared, int ordered, uint32_t n_simd) { return qgx::use_columns(chunks, per_bucket, shared != 0, ordered != 0, n_simd); }
extern "C" int columns_pay(uint64_t chunks, uint32_t per_bucket, uint32_t rows, int shared, int ordered, int powers, int crowded, uint32_t n_sym, uint32_t n_simd) { return qgx::columns_pay(chunks, per_bucket, rows, shared != 0, ordered != 0, powers != 0, crowded != 0, n_sym, n_simd); }
extern "C" int levels_crowded(const float* levels, uint32_t n_sym, int mant) { return qgx::levels_crowded(levels, n_sym, mant, 24); }
extern "C" int eight_waves_first(uint32_t n, uint32_t K, uint32_t simds) { return qgx::eight_waves(n, K, simds, 1, false); }
extern "C" int eight_waves(uint32_t n, uint32_t K, uint32_t simds, uint32_t streams) { return qgx::eight_waves(n, K, simds, streams); }
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


def _blocks(plan, K, units, span):
    """worker * units + unit of every block, -1 where there is none; span 0: block_by_unit"""
    if span:
        i = np.arange(span * units)
        return np.where(i % span < K, i % span * units + i // span, -1)
    out = np.empty(K * units, np.int64)
    plan.blocks_by_unit(C.c_uint32(K), C.c_uint32(units), out.ctypes.data_as(C.c_void_p))
    return out


def test_a_units_workgroups_on_one_xcd(plan):
    for K, units in itertools.product([1, 2, 3, 5, 7, 8, 9, 16, 31, 33, 63, 64], [1, 2, 7, 8, 9, 15, 16, 17, 40, 67]):
        got = _blocks(plan, K, units, 0)
        np.testing.assert_array_equal(np.sort(got), np.arange(K * units), err_msg="K %d units %d" % (K, units))
        for unit in range(units // 8 * 8):                   # in whole rounds: one XCD, one after the other
            np.testing.assert_array_equal(got[unit // 8 * 8 * K + unit % 8 + 8 * np.arange(K)], np.arange(K) * units + unit)


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
    or 96 workgroups to an XCD; the game's form takes block_by_unit while 3 K is below that)."""
    assert [plan.held_per_xcd(C.c_uint32(5), C.c_size_t(n), C.c_uint32(256)) for n in (30000, 40000, 53000)] == [160, 128, 96]
    parts, units, seen = 4, 64, 0
    for K, held, late in itertools.product([1, 8, 31, 32, 33, 42, 43, 47, 48, 53, 54, 57, 63, 64], [96, 128, 160], [0, 3, 7]):
        span = plan.worker_span(K, parts, held)
        assert K <= span < K + 8 and (span == K or 3 * K >= held)
        assert not _stalls(_blocks(plan, K, units, span), K, units, parts, held, late), (K, held, late, span)
        by_unit = _stalls(_blocks(plan, K, units, 0), K, units, parts, held, late)
        assert not (by_unit and 3 * K < held), (K, held, late)
        seen += by_unit
    assert seen                                              # the model knows a stall: many workers, all on every XCD


# tasks, workers, {waves: us} of the first and of the second half-step on 1024 SIMDs, where one choice is clearly better
MEASURED = [
    (512, 3, {1: 12.7, 2: 10.6}, {1: 21.5, 2: 19.2}), (1024, 3, {1: 13.4, 2: 12.3}, None), (3072, 3, {1: 21.1, 2: 22.9}, {1: 40.2, 2: 49.6}),
    (256, 4, {1: 14.6, 2: 10.3, 4: 8.7}, {1: 23.8, 2: 17.9, 4: 14.6}), (512, 4, None, {1: 24.6, 2: 19.1, 4: 17.1}),
    (1024, 4, {1: 15.5, 2: 12.6, 4: 14.1}, {1: 28.5, 2: 25.5, 4: 26.0}), (4096, 4, {1: 27.8, 2: 31.3, 4: 41.4}, {1: 54.8, 2: 62.3, 4: 69.1}),
    (512, 5, {1: 17.0, 2: 12.7, 4: 12.2}, {1: 27.8, 2: 22.4, 4: 20.2}), (1024, 5, {1: 17.8, 2: 14.8, 4: 16.3}, {1: 31.8, 2: 28.4, 4: 29.2}),
    (3072, 5, {1: 26.4, 2: 28.1, 4: 38.9}, {1: 50.7, 2: 59.6, 4: 66.2}), (4096, 5, {1: 31.0, 2: 35.5, 4: 48.3}, {1: 62.0, 2: 72.4, 4: 86.3}),
    (512, 8, {1: 23.3, 2: 15.1, 4: 12.6}, {1: 37.3, 2: 26.0, 4: 22.0}), (2048, 8, {1: 30.2, 2: 26.2, 4: 30.7}, None),
    (4096, 8, {1: 40.8, 2: 45.7, 4: 53.2}, {1: 81.8, 2: 87.9, 4: 97.1}), (4816, 8, {1: 48.2, 2: 61.1, 4: 64.7}, {1: 113.3, 2: 105.1, 4: 111.8}),
    (1024, 12, {1: 34.2, 2: 22.6, 4: 21.5}, {1: 54.8, 2: 41.7, 4: 40.5}), (2048, 12, {1: 39.7, 2: 33.1, 4: 37.6}, {1: 67.1, 2: 64.2, 4: 70.8}),
    (2048, 16, {1: 49.3, 2: 39.9, 4: 44.8}, {1: 82.3, 2: 77.3, 4: 83.5}),
    (9216, 16, {1: 175.5, 2: 158.6, 4: 161.8}, None), (2048, 32, {1: 87.8, 2: 67.8, 4: 72.3}, {1: 143.8, 2: 131.8, 4: 135.8}),
    (4096, 32, {1: 123.7, 2: 128.0, 4: 129.8}, None), (3072, 32, {1: 100.2, 2: 94.5, 4: 96.8}, None),
]


def test_waves_per_task_follow_the_measurements(plan):
    for tasks, K, first, second in MEASURED:
        for streams, us in ((1, first), (2, second)):
            if us:
                got = plan.waves_per_task(C.c_uint32(tasks), C.c_uint32(K), C.c_uint32(1024), C.c_uint32(streams))
                assert us[got] <= 1.025 * min(us.values()), (tasks, K, streams, got)
    for tasks, K in itertools.product([1, 2, 100000, (1 << 32) - 1], [1, 2, 3, 4, 65535]):
        assert 1 <= plan.waves_per_task(C.c_uint32(tasks), C.c_uint32(K), C.c_uint32(1024), C.c_uint32(1)) <= min(K, 4)


def test_turned_rows_give_every_worker_every_unit_on_four_xcds(plan):
    for K in (8, 16, 24, 64):
        assert plan.spread_workers(K, 16 * K) and not plan.spread_workers(K, 16 * K - 1) and not plan.spread_workers(K + 1, 1 << 20)
        xcds = [set() for _ in range(K)]
        for unit in range(33):
            row = [plan.worker_spread(k, unit, K) for k in range(K)]
            assert sorted(row) == list(range(K))
            for k, worker in enumerate(row):
                xcds[worker].add((unit * K + k) % 8)
        assert all(len(x) == 4 for x in xcds)


def test_buckets_per_group_fills_four_waves(plan):
    plan.buckets_per_group.argtypes = [C.c_uint32, C.c_uint64, C.c_int]
    for waves, chunks, ordered in itertools.product(range(1, 17), (1, 255, 256, 4095, 4096, 1 << 40), (0, 1)):
        n = plan.buckets_per_group(waves, chunks, ordered)
        assert n == (4 // waves if waves <= 2 and chunks >= (256 if ordered else 4096) else 1), (waves, chunks, ordered)


def test_use_staged_up_to_two_rounds_of_four_waves(plan):
    plan.use_staged.argtypes = [C.c_uint64, C.c_uint32]
    for simds, chunks in itertools.product((4, 1024), (1, 32, 33, 8192, 8193, (1 << 32) + 1)):
        assert plan.use_staged(chunks, simds) == (chunks <= 8 * simds), (simds, chunks)


def test_waves_without_a_bucket_are_a_workers_last(plan):
    """The waves whose sums a workgroup of several buckets looks at: those whose bucket is one of the worker's."""
    for waves, NB in itertools.product((1, 2), (1, 2, 3, 4, 5, 127, 128, 350)):
        group = 4 // waves
        for unit in range((NB + group - 1) // group):
            want = sum(unit * group + w // waves < NB for w in range(4))
            assert plan.waves_with_a_bucket(unit, group, waves, NB) == want, (waves, NB, unit)


def test_four_waves_to_a_chunk_fit_a_workgroup(plan):
    """Whatever the rule sends to that form has at most two chunks to a workgroup (four where shared chunks keep an order), and where
    it keeps an order its units are those of the other form, a bucket each: tickets of both come from one counter."""
    plan.use_columns.argtypes = [C.c_uint64, C.c_uint32, C.c_int, C.c_int, C.c_uint32]
    plan.buckets_per_group.argtypes = [C.c_uint32, C.c_uint64, C.c_int]
    for chunks in (1, 15, 255, 256, 257, 1023, 1024, 1025, 4096, 4097, 1 << 20):
        for per_bucket in range(1, 17):
            for ordered in (0, 1):
                if plan.use_columns(chunks, per_bucket, 0, ordered, 1024):
                    assert per_bucket <= 2 and chunks <= 1024
                    assert not ordered or plan.buckets_per_group(per_bucket, chunks, 1) == 1
        assert plan.use_columns(chunks, 1, 1, 1, 1024) == (chunks <= 1024)
        assert plan.use_columns(chunks, 1, 1, 0, 1024) == (chunks <= 4096)


def test_eight_waves_to_a_task_have_a_worker_each_and_a_place(plan):
    for tasks, K, streams in itertools.product((1, 256, 257, 384, 385, (1 << 32) - 1), (1, 7, 8, 65535), (1, 2)):
        got = plan.eight_waves(C.c_uint32(tasks), C.c_uint32(K), C.c_uint32(1024), C.c_uint32(streams))
        assert bool(got) == (K >= 8 and tasks <= (256 if streams == 2 else 384))


@pytest.mark.parametrize("what,yes,no", [
    # (chunks to a bucket, rows, shared, ordered, powers, crowded, levels): chunks where four waves to one are no slower, and where they are
    ((1, 1, 0, 0, 0, 0, 17), (1, 256), (320, 1024)),
    ((1, 1, 0, 0, 1, 0, 17), (), (1, 1024)),
    ((1, 1, 0, 0, 0, 0, 33), (), (1, 1024)),
    ((1, 1, 0, 0, 0, 1, 41), (), (1, 1024)),
    ((1, 1, 0, 0, 0, 0, 127), (512,), (1024,)),
    ((1, 1, 0, 0, 1, 0, 127), (1, 512), (640,)),
    ((1, 1, 0, 0, 0, 0, 65), (256,), (512,)),
    ((1, 2, 0, 0, 0, 0, 127), (1024,), ()),
    ((1, 3, 0, 0, 0, 0, 65), (1024,), ()),
    ((1, 9, 0, 0, 0, 0, 127), (256,), (384,)),
    ((1, 10, 0, 0, 0, 0, 127), (512,), (640,)),
    ((1, 16, 0, 0, 0, 0, 127), (1024,), ()),
    ((1, 1, 0, 1, 1, 0, 17), (), (1, 248)),
    ((1, 1, 0, 1, 0, 0, 17), (1, 248), ()),
    ((1, 2, 0, 0, 0, 0, 17), (512,), (640, 1024)),
    ((1, 2, 0, 0, 1, 0, 17), (256,), (384,)),
    ((1, 5, 0, 0, 0, 0, 17), (512,), (640,)),
    ((1, 9, 0, 0, 0, 0, 17), (), (192, 1024)),
    ((1, 9, 0, 1, 0, 0, 17), (), (192,)),
    ((1, 9, 0, 0, 0, 0, 33), (256,), (384,)),
    ((1, 10, 0, 0, 0, 0, 17), (), (384, 1024)),
    ((1, 10, 0, 0, 1, 0, 17), (1024,), ()),
    ((1, 10, 0, 0, 0, 1, 33), (1024,), ()),
    ((1, 12, 0, 0, 0, 0, 17), (512,), (640, 1024)),
    ((1, 16, 0, 0, 1, 0, 17), (1024,), ()),
    ((2, 16, 0, 0, 0, 0, 17), (1024,), ()),
    ((2, 9, 0, 0, 0, 0, 17), (512,), (640, 1024)),
    ((2, 9, 0, 0, 1, 0, 17), (1024,), ()),
    ((2, 2, 0, 0, 0, 0, 17), (1024,), ()),
    ((1, 4, 1, 0, 0, 0, 17), (1, 4096), ()),
    ((1, 4, 1, 0, 0, 0, 127), (1536,), (2048, 4096)),
    ((1, 8, 1, 0, 0, 0, 17), (1536,), (2048, 4096)),
    ((1, 8, 1, 0, 1, 0, 17), (1536,), (2048, 4096)),
    ((1, 8, 1, 0, 0, 0, 127), (1280,), (1536, 4096)),
    ((1, 8, 1, 0, 0, 1, 33), (4096,), ()),
    ((1, 4, 1, 0, 0, 1, 127), (4096,), ()),
    ((1, 8, 1, 0, 1, 1, 33), (2560,), (4096,)),
    ((1, 8, 1, 1, 1, 0, 127), (1, 1024), ()),
])
def test_four_waves_to_a_chunk_where_they_are_no_slower(plan, what, yes, no):
    per_bucket, rows, shared, ordered, powers, crowded, n_sym = what
    for chunks, want in [(c, 1) for c in yes] + [(c, 0) for c in no]:
        got = plan.columns_pay(C.c_uint64(chunks), *(C.c_uint32(x) for x in (per_bucket, rows)), shared, ordered, powers, crowded, C.c_uint32(n_sym), C.c_uint32(1024))
        assert got == want, (what, chunks)


def test_crowded_levels_by_the_cells_themselves(plan):
    """Cell edges of 1/16, 1/32 and 1/64 octave, written out in binary64: two interior levels strictly between two of them."""
    plan.levels_crowded.argtypes = [C.c_void_p, C.c_uint32, C.c_int]
    rng = np.random.default_rng(3)
    seen = set()
    for n_sym in (2, 3, 4, 17, 33, 34, 65, 66, 127):
        mant = 4 if n_sym <= 33 else 5 if n_sym <= 65 else 6
        edges = np.concatenate([[0.0], np.outer(2.0 ** np.arange(-24, 0), 1.0 + np.arange(1 << mant) / (1 << mant)).ravel()[1:], [1.0, np.inf]])
        tables = [np.arange(n_sym) / (n_sym - 1), np.concatenate([[0.0], 2.0 ** np.arange(-(n_sym - 2.0), 1.0)])]
        for _ in range(60):
            t = np.sort(rng.uniform(size=n_sym) ** rng.integers(1, 9))
            if n_sym > 3:                                        # levels on edges, and between them
                t[rng.integers(1, n_sym - 1, size=n_sym // 2)] = rng.choice(edges[1:-2], size=n_sym // 2)
            t[0], t[-1] = 0.0, 1.0
            tables.append(np.sort(t))
        for t in tables:
            t = t.astype(np.float32)
            if (np.diff(t) <= 0).any():
                continue
            inner = t[1:-1].astype(np.float64)
            cell = np.searchsorted(edges, inner, side="right") - 1
            inside = inner > edges[cell]
            want = bool((np.bincount(cell[inside], minlength=1) > 1).any()) if len(inner) else False
            assert bool(plan.levels_crowded(t.ctypes.data, n_sym, mant)) == want, (n_sym, t)
            seen.add(want)
    assert seen == {False, True}


def test_means_and_first_half_steps_have_eight_waves_where_they_gain(plan):
    for tasks, K in itertools.product((1, 256, 257, 320, 384, 385), (1, 7, 8, 12, 15, 16, 32, 65535)):
        got = plan.eight_waves_first(C.c_uint32(tasks), C.c_uint32(K), C.c_uint32(1024))
        assert bool(got) == (K >= 8 and tasks <= (384 if K >= 16 else 256))
