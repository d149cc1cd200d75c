"""The fused decoders with eight waves to a task (eight workers and more, few tasks): means, iterates and S against the plain
decoder's vectors in binary64 and against one wave to a task; whole, short and missing halves, equal and unequal runs of workers."""
import numpy as np
import pytest
import torch

import oracle
from paper_2308_09187_amd import synth
from test_gpu_parity import dev, make_ctx, qgx  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bucket", [1024, 6000])
@pytest.mark.parametrize("K,d", [(8, 255), (8, 2048), (9, 2049), (13, 4100), (16, 12289), (17, 30001), (33, 4096), (8, 500002), (8, 800000)])
def test_eight_waves(qgx, K, d, bucket):
    levels = synth.levels_exponential(16)
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
