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


@pytest.mark.parametrize("seed", [153, 299, 0, 1])
def test_level_where_the_mass_ends(qgx, seed):
    """All mass below the second level lies under 2^-63, so the update's share of it is the whole mass up to a rounding: the
    level goes to where that mass ends, whatever the order its sums are rounded in (seeds 153 and 299: a bin without mass is the
    first whose prefix sum reaches the share)."""
    rng = np.random.default_rng(seed)
    K, bucket, NB = 3, 64, 40
    edges = oracle.bin_edges(4096)
    m = rng.integers(2, 12)
    bins = 1 + rng.choice(63, m, replace=False)
    mids = (0.5 * (edges[bins] + edges[bins + 1])).astype(np.float32)
    norms = (1 + rng.random((K, NB, 1))).astype(np.float32)
    u = mids[rng.integers(0, m, (K, NB, bucket))]
    u[:, :, 0] = 1
    V = (u * norms).astype(np.float32).reshape(K, -1)
    start = np.array([0, 0.25, 0.5, 1], np.float32)
    ctx, lay = make_ctx(qgx, V.shape[1], K, bucket, oracle.NORM_LINF, start, seed=0)
    hist = torch.empty(4096, dtype=torch.float64, device="cuda")
    ctx.fit_levels(dev(V), 4, 4096, sweeps=1, hist_out=hist)
    want = oracle.histogram(V, lay, oracle.NORM_LINF, 4096)
    np.testing.assert_allclose(hist.cpu().numpy(), want, rtol=1e-12, atol=0)
    # the second level rests on the smallest gap, 2^-24; the third differs by the histogram's roundings only
    np.testing.assert_allclose(ctx.get_levels(), oracle.fit_levels(want, start, sweeps=1), rtol=1e-6, atol=1e-9)
    assert ctx.poll_error() == 0
    ctx.close()


@pytest.mark.parametrize("n_bins", [64, 192, 4096])
def test_where_the_histogram_goes(qgx, n_bins):
    """The caller's buffer: device memory, device memory at an odd word, pinned host memory, none; all the same values, and a buffer's end
    stays as it was."""
    d, K = 70001, 3
    V = dev(synth.student_t3(K, d, seed=4))
    ctx, _ = make_ctx(qgx, d, K, 4096, oracle.NORM_L2, synth.levels_exponential(8), seed=1)
    room = torch.full((2 * (n_bins + 4),), -1.0, dtype=torch.float32, device="cuda")
    buffers = [torch.full((n_bins + 2,), -1.0, dtype=torch.float64, device="cuda"), room[1:],
               torch.full((n_bins + 2,), -1.0, dtype=torch.float64, pin_memory=True), None]
    got = []
    for b in buffers:
        ctx.fit_levels(V, 9, n_bins, sweeps=0, hist_out=b)
        torch.cuda.synchronize()
        if b is not None:
            h = b.cpu().numpy()
            got.append(h[: 2 * n_bins].copy().view(np.float64) if h.dtype == np.float32 else h[:n_bins])
            assert (h[2 * n_bins:] == -1.0).all() if h.dtype == np.float32 else (h[n_bins:] == -1.0).all()
    assert got[0].sum() > 0
    for h in got[1:]:
        np.testing.assert_array_equal(h, got[0])
    assert ctx.poll_error() == 0
    ctx.close()
