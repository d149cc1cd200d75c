"""The scalar end of the second half-step by the launch's size: one workgroup (X_{t+1} in the same launch), a few (the scalars in it), many."""
import numpy as np
import pytest
import torch

import oracle
from paper_2308_09187_amd import synth
from test_gpu_parity import dev, make_ctx, qgx  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("anchor", [False, True])
@pytest.mark.parametrize("K,d", [(1, 255), (2, 2047), (3, 4099), (4, 1024), (4, 8191), (4, 8193), (1, 32769), (8, 130001), (2, 600002), (1, 1200002), (5, 9000001)])
def test_end_of_an_iteration(qgx, K, d, anchor):
    """X_{t+1} with and without being asked for it, S and gamma against the oracle; the static entry point the same bit for bit."""
    levels = synth.levels_exponential(16)
    V = [synth.student_t3(K, d, seed=s) for s in (1, 2)]
    x1 = synth.gaussian_vector(d, seed=3) if anchor else None
    got = []
    for static, asked in ((False, True), (True, True), (False, False)):
        ctx, lay = make_ctx(qgx, d, K, 1024, oracle.NORM_L2, levels, seed=5)
        ctx.state_init(None if x1 is None else dev(x1))
        a, b = ctx.new_stream(slotted=True), ctx.new_stream(slotted=True)
        x = torch.full((d,), 7.0, device="cuda")
        ctx.quantize_encode(dev(V[0]), 0, a)
        ctx.quantize_encode(dev(V[1]), 1, b)
        for _ in range(2):                                   # (the second step starts from the first one's S, t and Y)
            ctx.eg_step(1, b, a, x if asked else None, static=static)
        torch.cuda.synchronize()
        assert ctx.poll_error() == 0
        sc = ctx.scalars()
        assert sc["t"] == 3
        got.append((x.cpu().numpy(), sc["S"], sc["gamma"]))
        v = [ctx.decode(s).cpu().numpy().astype(np.float64) for s in (a, b)]
        ctx.close()
    st = oracle.EGState(d, K, X1=x1)
    for _ in range(2):
        x_o = st.half1(v[1], v[0])
    np.testing.assert_array_equal(got[0][0], got[1][0])
    assert got[0][1:] == got[1][1:] == got[2][1:] and (got[2][0] == 7.0).all()
    assert abs(got[0][2] - st.gamma) <= 1e-6 * st.gamma
    # sums of K <= 8 binary32 terms, then gamma and one more sum: a few roundings of 6e-8 each
    assert np.linalg.norm(got[0][0] - x_o) <= 1e-6 * np.linalg.norm(x_o)
