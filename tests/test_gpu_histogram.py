"""The level fit's histogram where a workgroup walks over unlike buckets: whole and short chunks, rows that end inside a lane's four
coordinates, a vector's odd end, more buckets than workgroups, dead and rejected buckets between live ones."""
import numpy as np
import pytest
import torch

import oracle
from paper_2308_09187_amd import synth
from test_gpu_parity import dev, make_ctx, qgx  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("norm", [oracle.NORM_L2, oracle.NORM_LINF, 3])
@pytest.mark.parametrize("bucket,d,K", [(4096, 4096, 1), (3000, 300001, 9), (6000, 700002, 9), (16384, 1 << 21, 7), (20000, 2000003, 5),
                                        (65536, 65536 * 70 + 4099, 4)])
def test_histogram(qgx, bucket, d, K, norm):
    levels = synth.levels_exponential(8)
    ctx, lay = make_ctx(qgx, d, K, bucket, norm, levels, seed=5)
    V = np.random.default_rng(bucket + d).standard_normal((K, d), dtype=np.float32)
    V[0, : min(bucket, d) // 2] *= np.float32(1e-3)
    bad = 0
    if lay.NB > 3:
        V[K - 1, bucket: 2 * bucket] = 0.0
        V[0, 2 * bucket + 1] = np.nan
        V[K - 1, -1] = -np.inf
        bad = qgx.EBIT_NONFINITE
    hist = torch.empty(4096, dtype=torch.float64, device="cuda")
    again = torch.empty_like(hist)
    ctx.fit_levels(dev(V), 9, 4096, sweeps=0, hist_out=hist)
    ctx.fit_levels(dev(V), 9, 4096, sweeps=0, hist_out=again)
    assert ctx.poll_error() == bad
    assert torch.equal(hist, again)
    clean = V.copy()
    if bad:
        clean[0, 2 * bucket: 3 * bucket] = 0.0
        clean[K - 1, (lay.NB - 1) * bucket:] = 0.0
    want = oracle.histogram(clean, lay, norm, 4096)
    got = hist.cpu().numpy()
    # the two sides' norms may differ in the last bit, which moves coordinates on a bin's edge into the next bin
    assert abs(got.sum() - want.sum()) <= 1e-6 * want.sum()
    assert np.abs(np.cumsum(got) - np.cumsum(want)).max() <= 1e-5 * want.sum()
    ctx.close()
