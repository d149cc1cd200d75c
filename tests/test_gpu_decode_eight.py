"""The fused decoders with eight waves to a task (eight workers and more, few tasks): means, iterates and S against the plain
decoder's vectors in binary64 and against one wave to a task; whole, short and missing halves, equal and unequal runs of workers, also
with more tasks than eight waves are taken for; a level table for each half (by the library's rule, on a device of 256 compute units)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2308_09187_amd import synth
from test_gpu_parity import dev, make_ctx, qgx  # noqa: F401

pytestmark = pytest.mark.gpu


def one_table(qgx, K, d, bucket, levels):
    V = [np.random.default_rng(s + d).standard_normal((K, d), dtype=np.float32) for s in (1, 2)]
    x1 = synth.gaussian_vector(d, seed=3)
    out = []
    for waves in (0, 1):
        ctx, lay = make_ctx(qgx, d, K, bucket, oracle.NORM_L2, levels, seed=5)
        ctx.debug_set_waves_per_position(waves)
        ctx.state_init(dev(x1))
        ctx.average_reset(True)
        a, b = ctx.new_stream(slotted=True), ctx.new_stream()
        xh, xn, mean = (torch.empty(d, device="cuda") for _ in range(3))
        ctx.quantize_encode(dev(V[0]), 0, a)
        ctx.quantize_encode(dev(V[1]), 1, b)
        v = [ctx.decode(s).cpu().numpy().astype(np.float64) for s in (a, b)]
        ctx.decode_average(a, mean)
        ctx.eg_step(0, a, None, xh)
        ctx.eg_step(1, b, a, xn)
        first = ctx.scalars()
        ctx.eg_step(1, b, None, xn)                          # (no previous stream)
        assert ctx.poll_error() == 0
        out.append([t.cpu().numpy().astype(np.float64) for t in (mean, xh, xn)] + [ctx.average_export()[0].cpu().numpy().astype(np.float64), first["S"], ctx.scalars()["S"]])
        ctx.close()
    S = ((v[1] - v[0]) ** 2).sum()
    for mean, xh, xn, avg, s1, s2 in out:
        # K - 1 binary32 additions and a product, each within 6e-8 of the partial sums, which the magnitudes bound
        assert (np.abs(mean - v[0].mean(0)) <= K * 6e-8 * np.abs(v[0]).mean(0) + 1e-30).all()
        assert np.linalg.norm(avg - xh) <= 1e-6 * np.linalg.norm(xh)
        assert abs(s1 - S) <= 1e-6 * S and abs(s2 - S - (v[1] ** 2).sum()) <= 1e-6 * s2
    for x, y in zip(out[0][1:3], out[1][1:3]):
        assert np.linalg.norm(x - y) <= 1e-6 * np.linalg.norm(y)


@pytest.mark.parametrize("bucket", [1024, 6000])
@pytest.mark.parametrize("K,d", [(8, 255), (8, 2048), (9, 2049), (13, 4100), (16, 12289), (17, 30001), (33, 4096), (8, 500002), (8, 800000)])
def test_eight_waves(qgx, K, d, bucket):
    one_table(qgx, K, d, bucket, synth.levels_exponential(16))


@pytest.mark.parametrize("K,d", [(8, 255), (9, 6145), (17, 30001)])
def test_eight_waves_without_the_8_byte_table(qgx, K, d):
    one_table(qgx, K, d, 6000, synth.levels_uniform(64))


@pytest.mark.parametrize("n0,n1", [(17, 9), (17, 65), (65, 17), (66, 127)])
@pytest.mark.parametrize("K,d,bucket", [(8, 2048, 1024), (9, 6145, 6000), (8, 255, 1024), (13, 4100, 4096), (17, 30001, 6000), (8, 500002, 8192)])
def test_eight_waves_and_two_tables(qgx, K, d, bucket, n0, n1):
    """The second half-step whose streams have tables of their own: both with the decoders' 8-byte table (up to 63 levels), one of them, neither."""
    tables = [synth.levels_exponential(n - 1) if n < 20 else synth.levels_uniform(n - 1) for n in (n0, n1)]
    V = [np.random.default_rng(s + d).standard_normal((K, d), dtype=np.float32) for s in (1, 2)]
    x1 = synth.gaussian_vector(d, seed=3)
    out = []
    for waves in (0, 1):
        ctx, lay = make_ctx(qgx, d, K, bucket, oracle.NORM_L2, tables[0], seed=5)
        assert 2 * lay.NC <= 256                             # (eight waves by the rule)
        ctx.debug_set_waves_per_position(waves)
        ctx.select_table(1)
        ctx.set_levels(tables[1])
        ctx.state_init(dev(x1))
        a, v = [], []
        for t in (0, 1):
            ctx.select_table(t)
            a.append(ctx.new_stream(slotted=t == 0))
            ctx.quantize_encode(dev(V[t]), t, a[t])
            v.append(ctx.decode(a[t]).cpu().numpy().astype(np.float64))
        xn = torch.empty(d, device="cuda")
        ctx.select_table(1, 0)
        ctx.eg_step(1, a[1], a[0], xn)
        sc = ctx.scalars()
        Y = ctx.state_export()[0].cpu().numpy().astype(np.float64)
        assert ctx.poll_error() == 0
        out.append((xn.cpu().numpy().astype(np.float64), Y, sc["S"]))
        ctx.close()
    S = ((v[1] - v[0]) ** 2).sum()
    mean = v[1].mean(0)
    for xn, Y, s in out:
        assert abs(s - S) <= 1e-6 * S
        # K - 1 binary32 additions and a product, each within 6e-8 of the partial sums, which the magnitudes bound
        assert (np.abs(Y + mean) <= K * 6e-8 * np.abs(v[1]).mean(0) + 1e-30).all()
        assert np.linalg.norm(xn - (x1 + K / np.sqrt(1.0 + S) * Y)) <= 1e-6 * np.linalg.norm(xn)
    assert np.linalg.norm(out[0][0] - out[1][0]) <= 1e-6 * np.linalg.norm(out[1][0])
