"""The coding kernel with four waves to a chunk, against the one with a wave per chunk: the same vectors coded by a few workers
(few chunks; with some tables and norms the rule has short chunks coded by the latter all the same) and by the first of many (more chunks
than the former takes).  Every bit of the streams and every norm are the same."""
import numpy as np
import pytest
import torch

import oracle
from paper_2308_09187_amd import synth
from test_gpu_parity import dev, make_ctx, qgx  # noqa: F401

pytestmark = pytest.mark.gpu


def coded(qgx, V, bucket, norm, levels, slotted, norms_in=None):
    K, d = V.shape
    ctx, lay = make_ctx(qgx, d, K, bucket, norm, levels, seed=77)
    s = ctx.new_stream(slotted=slotted)
    out = []
    for call in (3, 4):                                      # (a second launch takes the next tickets)
        ctx.quantize_encode(V, call, s, norms_in=norms_in)
        h = s.to_host()
        chunks = []
        for k in range(4):
            for c in range(lay.NC):
                at, words = int(h["chunk_off"][k, c]), (int(h["sub_end"][k, c, -1]) + 127) // 128 * 4
                chunks.append(h["payload"][k, at: at + words].copy())
        out.append((h["norms"][:4].copy(), h["sub_end"][:4].copy(), h["chunk_off"][:4].copy(), np.concatenate(chunks)))
    err = ctx.poll_error()
    ctx.close()
    return out, err


@pytest.mark.parametrize("norm", [oracle.NORM_L2, oracle.NORM_LINF, 3])
@pytest.mark.parametrize("bucket,d", [(128, 300), (256, 255), (256, 4097), (512, 1024), (512, 2305), (1024, 1024), (1024, 1500), (1024, 3073),
                                      (1024, 9001), (2048, 1027), (2048, 2048), (2048, 6145), (3000, 8999), (4096, 4096), (4096, 8191),
                                      (6000, 6001), (8192, 2049), (8192, 8192), (16384, 5000)])
def test_same_as_a_wave_per_chunk(qgx, bucket, d, norm):
    levels = synth.levels_exponential(16)
    rng = np.random.default_rng(d + bucket)
    few = rng.standard_normal((4, d), dtype=np.float32)
    few[1, : d // 2] *= np.float32(1e25)                     # squares beyond binary32
    few[1, d // 2:] *= np.float32(1e-30)
    few[2, : min(bucket, d - 1)] = 0.0                       # a bucket of zeros
    few[3, d // 3] = np.nan
    few[3, -1] = np.inf
    chunks = oracle.layout(d, bucket).NC
    K = 4096 // chunks + 1
    assert K * chunks > 4096
    many = dev(few).repeat((K + 3) // 4, 1)[:K].contiguous()
    for slotted in (False, True):
        (a, ea), (b, eb) = (coded(qgx, x, bucket, norm, levels, slotted) for x in (dev(few), many))
        assert ea == eb == qgx.EBIT_NONFINITE
        for call in range(2):
            for x, y in zip(a[call], b[call]):
                np.testing.assert_array_equal(x, y)


@pytest.mark.parametrize("n_sym", [3, 65, 127])
def test_table_sizes_and_given_norms(qgx, n_sym):
    """Each cell size, a table too fine for the cells, and norms given by the caller, one of them below its bucket's own."""
    d, bucket = 7001, 1024
    rng = np.random.default_rng(n_sym)
    few = rng.standard_normal((4, d), dtype=np.float32)
    lay = oracle.layout(d, bucket)
    K = 4096 // lay.NC + 1
    many = dev(few).repeat((K + 3) // 4, 1)[:K].contiguous()
    for levels in (synth.levels_uniform(n_sym - 1), synth.levels_exponential(min(n_sym - 1, 40))):
        for given in (False, True):
            norms = None
            if given:
                norms = np.full((4, lay.NB), 40.0, np.float32)
                norms[2, 1] = 0.5
            parts = []
            for V in (dev(few), many):
                n = None if norms is None else dev(norms).repeat((V.shape[0] + 3) // 4, 1)[: V.shape[0]].contiguous()
                parts.append(coded(qgx, V, bucket, oracle.NORM_L2, levels, True, n))
            (a, ea), (b, eb) = parts
            assert ea == eb == 0
            for call in range(2):
                for x, y in zip(a[call], b[call]):
                    np.testing.assert_array_equal(x, y)


@pytest.mark.parametrize("norm,scale", [(1, 1.0), (oracle.NORM_L2, 2.0 ** 60), (oracle.NORM_L2, 2.0 ** -40)])
@pytest.mark.parametrize("bucket,d,first", [(4096, 4096, 0), (4096, 3000, 0), (8192, 8192, 0), (8192, 8192, 4096), (6000, 12000, 6000)])
def test_norms_summed_from_memory_have_one_order(qgx, bucket, d, first, norm, scale):
    """The sums that are formed from memory in binary64 (q norms; squares beyond binary32): terms below half a unit in the last place
    of a sum that lies between two binary32 norms.  One at a time they are lost, added to each other first they turn the norm up."""
    V = np.zeros((2, d), np.float32)
    at = first + 64 * np.arange(4)                           # (all in the coordinates of one lane)
    V[:, at] = [1.0, 2.0 ** -24, 0.0, 0.0] if norm == 1 else [1.0, 2.0 ** -12, 2.0 ** -12, 2.0 ** -24]
    small = 2.0 ** -54 if norm == 1 else 2.0 ** -27
    V[0, first + 1024 + 64 * np.arange(16)] = small
    V[1, first + 1 + 64 * np.arange(16)] = 64 * small        # (in another lane: they count)
    V *= np.float32(scale)
    levels = synth.levels_exponential(16)
    ctx, lay = make_ctx(qgx, d, 2, bucket, norm, levels, seed=77)
    norms, sym = ctx.quantize(dev(V), 3)
    want = norms.cpu().numpy()
    b = first // bucket
    np.testing.assert_array_equal(want[:, b], np.float32(scale) * np.float32([1.0, 1.0 + 2.0 ** -23]))
    for slotted in (False, True):
        s = ctx.new_stream(slotted=slotted)
        ctx.quantize_encode(dev(V), 3, s)
        np.testing.assert_array_equal(s.norms.cpu().numpy(), want)
    assert ctx.poll_error() == 0
    ctx.close()


@pytest.mark.parametrize("norm", [oracle.NORM_L2, 3])
@pytest.mark.parametrize("slotted", [False, True])
@pytest.mark.parametrize("bucket,d", [(128, 2051), (300, 3001), (2304, 9000)])
def test_forms_change_with_the_table(qgx, bucket, d, slotted, norm):
    """Calls of one context take one form or the other by the table in use (order and tickets go on from call to call): each stream is
    that of the symbols quantised and coded on their own."""
    V = dev(np.random.default_rng(d).standard_normal((4, d), dtype=np.float32))
    ctx, lay = make_ctx(qgx, d, 4, bucket, norm, synth.levels_exponential(16), seed=7)
    for call, levels in enumerate((synth.levels_uniform(126), synth.levels_exponential(32), synth.levels_uniform(32), synth.levels_exponential(16),
                                   synth.levels_exponential(40), synth.levels_uniform(64))):
        ctx.set_levels(levels)
        one, two = ctx.new_stream(slotted=slotted), ctx.new_stream(slotted=slotted)
        for _ in range(2):
            ctx.quantize_encode(V, call, one)
        norms, sym = ctx.quantize(V, call)
        ctx.encode(norms, sym, two)
        a, b = one.to_host(), two.to_host()
        for name in ("norms", "sub_end", "chunk_off"):
            np.testing.assert_array_equal(a[name], b[name])
        for k in range(4):
            for c in range(lay.NC):
                at, words = int(a["chunk_off"][k, c]), (int(a["sub_end"][k, c, -1]) + 31) // 32
                np.testing.assert_array_equal(a["payload"][k, at: at + words], b["payload"][k, at: at + words])
    assert ctx.poll_error() == 0
    ctx.close()
