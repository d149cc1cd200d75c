"""The decoder's tasks at their edges: half chunk positions of 1 .. 2047 coordinates beside full ones, halves whose
words do not fit the pieces that travel ahead, odd numbers of workers, vectors at odd addresses.  Decoded vectors bit
for bit against the oracle (one binary32 product each); mean, iterates and S within the bounds the parity tests derive."""
import math

import numpy as np
import pytest
import torch

import oracle
from paper_2308_09187_amd import synth
from test_gpu_parity import REL, WAVES_PER_POSITION, _vectors_of_very_different_density, assert_elementwise, dev, make_ctx, mean_abs, oracle_stream, qgx, rel_err  # noqa: F401

pytestmark = pytest.mark.gpu

ENDS = [1, 31, 32, 33, 2016, 2047, 2048, 2049, 2081, 4095]     # coordinates of the last position


@pytest.mark.parametrize("waves", [1, 4])
@pytest.mark.parametrize("n_levels", [16, 64])                  # with 64, half a chunk of dense vectors takes 830 words
@pytest.mark.parametrize("end", ENDS)
def test_short_halves(qgx, monkeypatch, end, n_levels, waves):
    monkeypatch.setitem(WAVES_PER_POSITION, "waves", waves)
    K = 5 if waves == 4 else 3
    d = 4096 + end
    levels = synth.levels_uniform(n_levels)
    ctx, lay = make_ctx(qgx, d, K, 4096, oracle.NORM_LINF, levels, seed=11)
    kinds = ["dense", "t3", "sparse", "dense", "zero"][:K]
    V = [_vectors_of_very_different_density(d, kinds), _vectors_of_very_different_density(d, kinds[::-1])]
    ctx.state_init(None)
    st = oracle.EGState(d, K)
    A, B = ctx.new_stream(slotted=True), ctx.new_stream(slotted=True)
    X = torch.empty(d, device="cuda")
    Vhat = []
    for call, s in ((0, A), (1, B)):
        ctx.quantize_encode(dev(V[call]), call, s)
        norms = s.norms.cpu().numpy()
        so = oracle_stream(V[call], lay, oracle.NORM_LINF, levels, 11, call, norms, ctx.worst_words)[3]
        Vhat.append(oracle.decode(so, norms, lay, levels)[0])
        flat = torch.full((K * d + 2,), -7.0, device="cuda")    # at an address that is a multiple of 4 bytes and no more
        ctx.decode(s, flat[1:-1].view(K, d))
        flat = flat.cpu().numpy()
        np.testing.assert_array_equal(flat[1:-1].reshape(K, d), Vhat[call])
        assert flat[0] == -7.0 and flat[-1] == -7.0
        assert_elementwise(ctx.decode_average(s).cpu().numpy(), oracle.mean(Vhat[call]), mean_abs(Vhat[call]), "mean")
    ctx.eg_step(0, A, None, X)
    assert rel_err(X.cpu().numpy(), st.half0(Vhat[0])) <= REL
    ctx.eg_step(1, B, A, X)
    assert rel_err(X.cpu().numpy(), st.half1(Vhat[1], Vhat[0])) <= REL
    assert abs(ctx.scalars()["S"] - st.S) <= REL * st.S
    assert ctx.poll_error() == 0
    ctx.close()


def test_tables_that_point_at_the_payloads_end(qgx):
    """Extents without words at the very end of the payload, and ends before their starts: refused by every decoder, for
    both streams of the second half-step, and the context goes on."""
    d, K = 4096 + 700, 2
    levels = synth.levels_exponential(16)
    ctx, lay = make_ctx(qgx, d, K, 4096, oracle.NORM_L2, levels, seed=3)
    ctx.state_init(None)
    good, bad = ctx.new_stream(), ctx.new_stream()
    X = torch.empty(d, device="cuda")
    for s in (good, bad):
        ctx.quantize_encode(dev(synth.student_t3(K, d, seed=8)), 0, s)
    Vhat = ctx.decode(good).cpu().numpy()
    cap = bad.payload.shape[1]
    ends, offs = bad.sub_end.clone(), bad.chunk_off.clone()
    for at, end in ((cap, 0), (cap - 4, 128), (cap - 4, 100)):
        bad.sub_end.fill_(end)                               # every run ends where it starts
        bad.chunk_off.fill_(at)
        for call in (lambda: ctx.decode(bad), lambda: ctx.decode_average(bad), lambda: ctx.eg_step(0, bad, None, X),
                     lambda: ctx.eg_step(1, bad, good, X), lambda: ctx.eg_step(1, good, bad, X), lambda: ctx.eg_step(1, bad, None, X)):
            call()
            assert ctx.poll_error() & qgx.EBIT_STREAM, (at, end)
    bad.sub_end.copy_(ends)
    bad.chunk_off.copy_(offs)
    np.testing.assert_array_equal(ctx.decode(bad).cpu().numpy(), Vhat)
    assert ctx.poll_error() == 0
    ctx.close()


@pytest.mark.parametrize("d,bucket", [(9000, 3000), (2 * 4095, 4092), (2048, 4096), (3072, 1024), (2500 + 700, 2500)])
def test_step_size_sum_of_short_positions(qgx, d, bucket):
    """S of layouts without a whole position: every squared difference formed and added in binary64, the first half of a
    position that is more than half full included.  A lane adds 32 K terms one after the other, what follows is fewer
    than 128 additions, none of a negative number: a relative error of at most (32 K + 128) 2^-53."""
    K, levels = 3, synth.levels_exponential(16)
    ctx, lay = make_ctx(qgx, d, K, bucket, oracle.NORM_L2, levels, seed=21)
    ctx.state_init(None)
    A, B = ctx.new_stream(slotted=True), ctx.new_stream(slotted=True)
    ctx.quantize_encode(dev(synth.student_t3(K, d, seed=5)), 0, A)
    ctx.quantize_encode(dev(synth.student_t3(K, d, seed=6)), 1, B)
    diff = ctx.decode(A).double() - ctx.decode(B).double()
    S = math.fsum((diff * diff).flatten().cpu().tolist())
    ctx.eg_step(1, B, A, None)
    assert abs(ctx.scalars()["S"] - S) <= (32 * K + 128) * 2.0 ** -53 * S
    assert ctx.poll_error() == 0
    ctx.close()


@pytest.mark.parametrize("waves", [1, 4])
def test_two_tables_in_workgroups_of_sixteen_waves(qgx, monkeypatch, waves):
    """The second half-step with a table for either stream and more waves than workgroups of eight can hold at once."""
    monkeypatch.setitem(WAVES_PER_POSITION, "waves", waves)
    K, d = 4, 2300 * 2048 + 700
    ctx, lay = make_ctx(qgx, d, K, 8192, oracle.NORM_L2, synth.levels_exponential(16), seed=9)
    ctx.select_table(1)
    ctx.set_levels(synth.levels_uniform(40))
    A, B = ctx.new_stream(slotted=True), ctx.new_stream(slotted=True)
    ctx.quantize_encode(dev(synth.student_t3(K, d, seed=1)), 0, A)
    Va = ctx.decode(A).cpu().numpy()
    ctx.select_table(0, 1)
    ctx.quantize_encode(dev(synth.student_t3(K, d, seed=2)), 1, B)
    Vb = ctx.decode(B).cpu().numpy()
    ctx.state_init(None)
    st = oracle.EGState(d, K)
    st.half0(Va)
    X = torch.empty(d, device="cuda")
    ctx.eg_step(1, B, A, X)
    assert rel_err(X.cpu().numpy(), st.half1(Vb, Va)) <= REL
    assert abs(ctx.scalars()["S"] - st.S) <= REL * st.S
    assert ctx.poll_error() == 0
    ctx.close()


@pytest.mark.parametrize("waves", [1, 4])
@pytest.mark.parametrize("groups", [1, 2, 63, 64, 65, 130])
def test_scalar_end_on_both_sides_of_its_line(qgx, monkeypatch, groups, waves):
    """The second half-step of up to 64 workgroups leaves S, gamma and t itself, larger ones have a kernel for that: several
    in a row without a wait between them, with and without a previous stream, a short last task, waves without one.  S is a sum of
    non-negative terms from groups of six in binary32, Y and X of K + 1 and 2 roundings a step: within REL, as the parity tests."""
    monkeypatch.setitem(WAVES_PER_POSITION, "waves", waves)
    K, tasks = 4, groups if waves == 4 else 4 * groups - 1       # (four waves to a workgroup: a task each, or all on one)
    d = 2048 * tasks - 300
    levels = synth.levels_exponential(16)
    ctx, lay = make_ctx(qgx, d, K, 4096, oracle.NORM_L2, levels, seed=13)
    ctx.state_init(None)
    A, B = ctx.new_stream(slotted=True), ctx.new_stream(slotted=True)
    X = torch.empty(d, device="cuda")
    for call, s in ((0, A), (1, B)):
        ctx.quantize_encode(dev(synth.student_t3(K, d, seed=40 + call)), call, s)
    a, b = ctx.decode(A).double(), ctx.decode(B).double()
    S, Y, t0 = 0.0, torch.zeros(d, dtype=torch.float64, device="cuda"), ctx.scalars()["t"]
    for cur, prev, vc, vp in ((B, A, b, a), (A, B, a, b), (B, None, b, 0 * b), (B, A, b, a), (A, None, a, 0 * a)):
        ctx.eg_step(1, cur, prev, X)
        S += float(((vc - vp) ** 2).sum())
        Y -= vc.mean(0)
        X_o = K / math.sqrt(1.0 + S) * Y
    assert rel_err(X.cpu().numpy(), X_o.cpu().numpy()) <= REL
    sc = ctx.scalars()
    assert sc["t"] == t0 + 5 and abs(sc["S"] - S) <= REL * S
    assert abs(sc["gamma"] - K / math.sqrt(1.0 + S)) <= REL * sc["gamma"]
    assert ctx.poll_error() == 0
    ctx.close()
