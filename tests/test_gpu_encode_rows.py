"""The coding kernel's rows at their edges: chunks with 0 .. 15 whole rows and a short one, workers whose vectors start
at odd addresses, buckets of one chunk, of several, and sharing chunks.  Streams and symbols bit for bit."""
import numpy as np
import pytest
import torch

import oracle
from paper_2308_09187_amd import synth
from test_gpu_parity import assert_stream_equal, dev, make_ctx, oracle_stream, qgx  # noqa: F401

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
