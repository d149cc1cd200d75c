"""The coding kernel's rows at their edges: chunks with 0 .. 15 whole rows and a short one, workers whose vectors start
at odd addresses, buckets of one chunk, of several, and sharing chunks.  Streams and symbols bit for bit."""
import numpy as np
import pytest
import torch

import oracle
from paper_2308_09187_amd import synth
from test_gpu_parity import assert_slotted_equal, assert_stream_equal, dev, make_ctx, oracle_stream, qgx  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bucket", [1000, 1024, 4096, 20000])
@pytest.mark.parametrize("d", [255, 257, 511, 3839, 3841, 4095, 4097, 24577, 25001])
def test_rows(qgx, d, bucket):
    K, seed = 3, 17
    levels = synth.levels_exponential(16)
    ctx, lay = make_ctx(qgx, d, K, bucket, oracle.NORM_L2, levels, seed=seed)
    V = synth.student_t3(K, d, seed=d + bucket)
    V[1, : d // 3] = 0.0                                     # buckets that are all zero, and one that is in part
    s = ctx.new_stream()
    ctx.quantize_encode(dev(V), 5, s)
    h = s.to_host()
    _, idx, neg, so = oracle_stream(V, lay, oracle.NORM_L2, levels, seed, 5, h["norms"], ctx.worst_words)
    assert_stream_equal(h, so, lay)
    norms, sym = ctx.quantize(dev(V), 5)
    np.testing.assert_array_equal(norms.cpu().numpy(), h["norms"])
    np.testing.assert_array_equal(sym.cpu().numpy(), (idx | (neg << 7)).astype(np.uint8))
    again = ctx.new_stream()
    ctx.encode(norms, sym, again)
    assert_stream_equal(again.to_host(), so, lay)
    assert ctx.poll_error() == 0
    ctx.close()


@pytest.mark.parametrize("norm", [oracle.NORM_L2, oracle.NORM_LINF, 3])
@pytest.mark.parametrize("bucket,d", [(4096, 32 * 4096 + 1), (4096, 34 * 4096), (8192, 65 * 4096 + 77), (3000, 400001), (6000, 400004)])
def test_buckets_side_by_side(qgx, bucket, d, norm):
    """Several buckets to a workgroup (256 chunks in order, 4096 in slots): neighbours whose squares overflow or vanish in
    binary32, zeros, a non-finite coordinate, and a worker's last workgroup without buckets for all its waves."""
    K, seed = 128 if d < 200000 else 32, 23
    levels = synth.levels_exponential(16)
    ctx, lay = make_ctx(qgx, d, K, bucket, norm, levels, seed=seed)
    rng = np.random.default_rng(d + bucket)
    V = rng.standard_normal((K, d), dtype=np.float32)
    V[1, :bucket] *= np.float32(1e25)
    V[1, 3 * bucket: 4 * bucket] *= np.float32(1e-30)
    V[2, 2 * bucket: 3 * bucket] = 0.0
    V[3, -1] *= np.float32(1e24)
    V[4, bucket + 5] = np.inf
    V[5, 0] = np.nan
    V[6, -1] = np.nan
    for slotted in (False, True):
        s = ctx.new_stream(slotted=slotted)
        ctx.quantize_encode(dev(V), 9, s)
        assert ctx.poll_error() == qgx.EBIT_NONFINITE
        h = s.to_host()
        assert h["norms"][4, 1] == 0 and h["norms"][5, 0] == 0 and h["norms"][6, -1] == 0 and np.isfinite(h["norms"]).all()
        assert (h["norms"][1, [0, 3]] > 0).all() and h["norms"][2, 2] == 0 and h["norms"][2, 1] > 0
        clean = np.nan_to_num(V, nan=0.0, posinf=0.0)
        clean[4, bucket: 2 * bucket] = 0.0
        clean[5, :bucket] = 0.0
        clean[6, (lay.NB - 1) * bucket:] = 0.0
        norms_o = oracle.quantize(clean, lay, norm, levels, seed, 9)[0]
        np.testing.assert_allclose(h["norms"], norms_o, rtol=1e-6, atol=0)
        _, idx, neg, so = oracle_stream(clean, lay, norm, levels, seed, 9, h["norms"], ctx.worst_words)
        if slotted:
            assert_slotted_equal(h, so, lay, s.slot_words)
        else:
            assert_stream_equal(h, so, lay)
    ctx.close()


@pytest.mark.parametrize("slotted", [False, True])
@pytest.mark.parametrize("n_sym", [33, 65, 127])
@pytest.mark.parametrize("bucket,d", [(516, 1024 * 516), (516, 1024 * 516 + 259), (4096, 1024 * 4096), (4096, 1024 * 4096 + 257),
                                      (16384, 1025 * 4096 + 513)])
def test_both_sides_of_the_look_ups_ahead(qgx, bucket, d, n_sym, slotted):
    """8192 and 8200 chunks, where the kernel's form changes on 1024 SIMDs, with whole rows in every chunk (rows that are not
    whole take a path of their own, the same in both forms), and tables of each cell size; no cell of a uniform one holds two levels, so
    the rows are coded by the straight path."""
    K, seed = 8, 29
    levels = np.linspace(0, 1, n_sym).astype(np.float32)
    ctx, lay = make_ctx(qgx, d, K, bucket, oracle.NORM_LINF, levels, seed=seed)
    assert K * lay.NC in (8192, 8200, 8208)
    g = torch.Generator(device="cuda")
    g.manual_seed(d)
    V = torch.randn((K, d), generator=g, device="cuda")
    s = ctx.new_stream(slotted=slotted)
    ctx.quantize_encode(V, 3, s)
    h = s.to_host()
    _, _, _, so = oracle_stream(V.cpu().numpy(), lay, oracle.NORM_LINF, levels, seed, 3, h["norms"], ctx.worst_words)
    if slotted:
        assert_slotted_equal(h, so, lay, s.slot_words)
    else:
        assert_stream_equal(h, so, lay)
    assert ctx.poll_error() == 0
    ctx.close()


@pytest.mark.parametrize("slotted", [False, True])
@pytest.mark.parametrize("d", [1023 * 100 + 1, 1024 * 100 + 1, 4096 * 100])
def test_many_chunks_without_a_whole_row(qgx, d, slotted):
    """8192, 8200 and 32768 chunks of 100 coordinates, four buckets to a workgroup."""
    K, seed, bucket = 8, 29, 100
    levels = synth.levels_exponential(16)
    ctx, lay = make_ctx(qgx, d, K, bucket, oracle.NORM_L2, levels, seed=seed)
    V = synth.student_t3(K, d, seed=d)
    s = ctx.new_stream(slotted=slotted)
    ctx.quantize_encode(dev(V), 3, s)
    h = s.to_host()
    _, _, _, so = oracle_stream(V, lay, oracle.NORM_L2, levels, seed, 3, h["norms"], ctx.worst_words)
    if slotted:
        assert_slotted_equal(h, so, lay, s.slot_words)
    else:
        assert_stream_equal(h, so, lay)
    assert ctx.poll_error() == 0
    ctx.close()


@pytest.mark.parametrize("slotted", [False, True])
@pytest.mark.parametrize("norm", [oracle.NORM_L2, oracle.NORM_LINF, 3])
@pytest.mark.parametrize("bucket,d,K,n_sym", [(8192, 5 * 8192 + 700, 2, 17), (1024, 3 * 4096 + 1500, 3, 17), (4096, 4 * 4096, 2, 65),
                                              (16384, 3 * 16384, 2, 127), (32768, 3 * 32768, 2, 33), (516, 1030 * 516, 8, 17)])
def test_norms_without_a_finite_reciprocal(qgx, bucket, d, K, n_sym, norm, slotted):
    """Buckets of subnormal coordinates between ordinary ones: up to a norm of 2^-128 the reciprocal is infinite.  Their
    coordinates go to the top level as the oracle's, and their neighbours are bit for bit what they are without them."""
    seed = 31
    levels = synth.levels_exponential(16) if n_sym == 17 else np.linspace(0, 1, n_sym).astype(np.float32)
    ctx, lay = make_ctx(qgx, d, K, bucket, norm, levels, seed=seed)
    V = synth.student_t3(K, d, seed=d)
    for k, b, top in ((0, 1, 1e-41), (1, 0, 2.0 ** -128), (1, 2, 2.0 ** -128 + 2.0 ** -149), (K - 1, lay.NB - 1, 2.0 ** -149)):
        at = slice(b * bucket, min(d, (b + 1) * bucket))
        V[k, at] = (V[k, at].astype(np.float64) * (top / np.abs(V[k, at]).max())).astype(np.float32)
        assert V[k, at].any() and np.abs(V[k, at]).max() < 2.0 ** -126
    s = ctx.new_stream(slotted=slotted)
    ctx.quantize_encode(dev(V), 2, s)
    h = s.to_host()
    norms_o = oracle.quantize(V, lay, norm, levels, seed, 2)[0]
    np.testing.assert_allclose(h["norms"], norms_o, rtol=1e-6, atol=2.0 ** -149)     # (a subnormal's spacing)
    with np.errstate(over="ignore"):
        assert 2 <= np.isinf(np.float32(1) / h["norms"]).sum() <= 4
    _, idx, neg, so = oracle_stream(V, lay, norm, levels, seed, 2, h["norms"], ctx.worst_words)
    if slotted:
        assert_slotted_equal(h, so, lay, s.slot_words)
    else:
        assert_stream_equal(h, so, lay)
    norms, sym = ctx.quantize(dev(V), 2)
    np.testing.assert_array_equal(norms.cpu().numpy(), h["norms"])
    np.testing.assert_array_equal(sym.cpu().numpy(), (idx | (neg << 7)).astype(np.uint8))
    assert ctx.poll_error() == 0
    ctx.close()
