"""The work that a program built on this library has it do, as cases whose time and outputs can be compared.

A case is one pass of a training loop's exchange through the public binding (`paper_2308_09187_amd.qgx`):

  iteration   an iteration of Algorithm 1: CODE o Q of the K dual vectors, first half-step, CODE o Q of the K dual
              vectors at X_{t+1/2}, second half-step with the step size.  `optimistic`: the variant that codes once an
              iteration and takes the stream of the iteration before as its first one.  `average`: with the
              ergodic average kept alongside.  `tables` = 2: a level table for each half.
  step        CODE o Q of the K vectors and the first half-step (what an iteration does between two operator calls)
  refit       the same at an update step: levels (and, with a fitted code, Psi) refitted first
  roundtrip   CODE o Q, then every worker's vector decoded on its own
  exchange    CODE o Q into the gap-free placement that goes over a wire, then the mean of the decoded vectors
  game        an iteration of the large quadratic game with operator and noise on the device
  game_refit  that game's update step: dual vectors written out, levels refitted and read

Sizes are the repository's five workloads, its benchmark's options and its parity tests' layouts; `draw` spreads over
the same kinds, layouts, norms, tables and codes.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2308_09187_amd import qgx, synth

GAN_D = int(np.sum(synth.GAN_SEGMENTS))
FIXED_SLOT_SYMBOL_BITS = 12          # longest word of a fitted code and its sign: the slot of a stream that outlives refits

_BASE = dict(K=4, d=1024, bucket=1024, tensors=False, norm=qgx.NORM_L2, n_sym=9, levels="exponential", code="omega",
             placement="slotted", dist="operator", anchor=False, optimistic=False, average=False, tables=1, sweeps=10)


def _case(name, kind, **kw):
    c = dict(_BASE, kind=kind, **kw)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # Stochastic bilinear game, four workers, one bucket: the smallest call, all launch and latency.
        _case("bilinear_iteration", "iteration", anchor=True),
        # The quantiser on its own: one vector of 2^20, coded for the wire and decoded again.
        _case("vector_roundtrip", "roundtrip", K=1, d=1 << 20, bucket=8192, n_sym=17, placement="compact", dist="normal"),
        # The benchmark's default: eight heavy-tailed vectors of 2^24, fitted levels, coded and taken through a half-step.
        _case("batch_step", "step", K=8, d=1 << 24, bucket=16384, n_sym=33, levels="fitted", dist="student"),
        # Whole iterations of a quarter of that batch with Psi fitted to the symbol probabilities.
        _case("batch_iteration_fitted_code", "iteration", K=8, d=1 << 22, bucket=16384, n_sym=33, levels="fitted",
              code="fitted", dist="student"),
        # An update step of Algorithm 1 on vectors of 2^20: levels and code refitted, then a step with them.
        _case("batch_refit", "refit", K=8, d=1 << 20, bucket=16384, n_sym=33, levels="fitted", code="fitted", dist="student"),
        # Data-parallel training of a network: 14 tensors with ends that are no whole chunks, L-infinity norm.
        _case("gan_iteration", "iteration", K=8, d=GAN_D, bucket=8192, tensors=True, norm=qgx.NORM_LINF, n_sym=17,
              dist="tensors", anchor=True),
        # The same tensors in the experiment's four-bit setting: buckets of 1024, uniform levels, words of one width.
        _case("gan_fixed4_iteration", "iteration", K=8, d=GAN_D, bucket=1024, tensors=True, norm=qgx.NORM_LINF, n_sym=8,
              levels="uniform", code="fixed", dist="tensors", anchor=True),
        # Its eight-bit setting, the optimistic variant (one coded stream an iteration) with the ergodic average.
        _case("gan_fixed8_optimistic", "iteration", K=8, d=GAN_D, bucket=1024, tensors=True, norm=qgx.NORM_LINF, n_sym=127,
              levels="uniform", code="fixed", dist="tensors", anchor=True, optimistic=True, average=True),
        # A vector length that is odd, buckets that are no whole chunks, five workers.
        _case("odd_iteration", "iteration", K=5, d=3000001, bucket=6000, n_sym=17, dist="operator"),
        # What goes over the network: streams without gaps, and the mean that a receiver forms from them.
        _case("wire_exchange", "exchange", K=8, d=1 << 22, bucket=16384, n_sym=33, levels="fitted", placement="compact",
              dist="student"),
        # The large quadratic game on the device: 16 workers, 2^26 coordinates.
        _case("game_iteration", "game", K=16, d=1 << 26, bucket=65536, n_sym=65, levels="fitted", sweeps=8),
        # Its update step (every tenth iteration).
        _case("game_refit", "game_refit", K=16, d=1 << 26, bucket=65536, n_sym=65, levels="fitted", sweeps=8),
    ]


def draw(rng):
    kind = rng.choice(["iteration", "iteration", "iteration", "step", "refit", "roundtrip", "exchange", "game"])
    K = rng.choice([1, 2, 3, 4, 5, 8, 8, 16, 32])
    total = 2.0 ** rng.uniform(12.0, 27.0)                      # coordinates over all workers
    d = max(256, int(total / K))
    tensors = kind != "game" and d >= 1 << 16 and rng.random() < 0.35
    if kind == "game" or rng.random() < 0.35:
        d = d // 8 * 8
    elif rng.random() < 0.3:
        d = 1 << int(math.log2(d))
    bucket = rng.choice([128, 512, 1000, 1024, 1024, 2048, 3000, 4096, 6000, 8192, 8192, 16384, 16384, 20000, 32768, 65536])
    if kind == "game" and bucket <= 2048:
        bucket *= 4096 // 128
    if bucket == 128:                                            # a chunk to every bucket: for small tensors
        d = min(d, max(256, (1 << 20) // K))
        tensors = tensors and d >= 1 << 16
    code = rng.choice(["omega", "omega", "omega", "fitted", "fixed"]) if kind not in ("game",) else "omega"
    n_sym = rng.choice([3, 8, 9, 15, 17, 17, 33, 33, 65, 127])
    levels = "uniform" if code == "fixed" else rng.choice(["exponential", "fitted"]) if n_sym <= 17 else "fitted"
    if kind == "refit" or code == "fitted":
        levels = "fitted"
    c = _case(None, kind, K=K, d=d, bucket=bucket, tensors=tensors, norm=rng.choice([qgx.NORM_L2, qgx.NORM_L2, qgx.NORM_LINF, 3]),
              n_sym=n_sym, levels=levels, code=code, placement="compact" if kind == "exchange" or rng.random() < 0.25 else "slotted",
              dist="tensors" if tensors else rng.choice(["operator", "normal", "student"]), anchor=rng.random() < 0.5)
    if kind == "game":
        c["norm"] = rng.choice([qgx.NORM_L2, qgx.NORM_LINF])
    if kind == "iteration":
        c["optimistic"] = rng.random() < 0.25
        c["average"] = rng.random() < 0.25
        c["tables"] = 2 if not c["optimistic"] and code == "omega" and rng.random() < 0.2 else 1
    return c


# ---- inputs --------------------------------------------------------------------------------------------------------


def _segments(c):
    """The 14 tensors' lengths, scaled to the vector's length."""
    if not c["tensors"]:
        return None
    f = c["d"] / GAN_D
    seg = [max(4, int(round(int(n) * f / 4)) * 4) for n in synth.GAN_SEGMENTS[:-1]]
    return seg + [c["d"] - sum(seg)]


def _vectors(c, seed, call):
    """[K][d] dual vectors, drawn on the device."""
    K, d = c["K"], c["d"]
    if c["dist"] == "student":                                   # heavy tails, as stochastic gradients have them
        return synth.student_t3_device(K, d, seed=(seed * 2 + call) % 1000003)
    g = torch.Generator(device="cuda")
    g.manual_seed(seed * 2 + call)
    V = torch.randn((K, d), generator=g, device="cuda")
    if c["dist"] == "operator":                                  # the operator's value, plus noise of each worker's own
        V.mul_(0.1).add_(torch.randn(d, generator=g, device="cuda"))
    elif c["dist"] == "tensors":                                 # a scale for each tensor
        at = 0
        for n, sigma in zip(_segments(c), synth.gan_sigmas()):
            V[:, at:at + n] *= float(sigma)
            at += n
    return V


def _width(n_sym):
    return max(1, (n_sym - 1).bit_length())


def _set_tables(ctx, c, V):
    exponential = synth.levels_exponential(c["n_sym"] - 1)
    ctx.set_levels(synth.levels_uniform(c["n_sym"] - 1) if c["levels"] == "uniform" else exponential)
    if c["levels"] == "fitted":
        ctx.fit_levels(V, c["n_sym"], 4096, sweeps=c["sweeps"])
    if c["code"] == "fitted":
        ctx.fit_code()
    elif c["code"] == "fixed":
        ctx.set_code_table(np.full(c["n_sym"], _width(c["n_sym"]), np.uint8), np.arange(c["n_sym"], dtype=np.uint32))


def _new_stream(ctx, c):
    if c["placement"] == "compact":
        return ctx.new_stream()
    if c["kind"] == "refit" and c["code"] == "fitted":           # the code, and with it the longest word, changes under the stream
        words = qgx.CHUNK * FIXED_SLOT_SYMBOL_BITS // 32
        return qgx.Stream(ctx.K, ctx.NB, ctx.NC, words * ctx.NC, ctx.device, slot_words=words)
    return ctx.new_stream(slotted=True)


def prepare(case, seed):
    c = dict(case)
    K, d = c["K"], c["d"]
    ctx = qgx.Context(d, K, c["bucket"], norm=c["norm"], seed=1000 + seed, segment_len=_segments(c),
                      code=qgx.CODE_ELIAS_OMEGA if c["code"] == "omega" else qgx.CODE_TABLE)
    s = dict(case=c, ctx=ctx, call=2 * (seed % 1000))
    g = torch.Generator(device="cuda")
    g.manual_seed(seed + 77)
    if c["kind"] in ("game", "game_refit"):
        s["a"] = torch.rand(d // 2, generator=g, device="cuda").mul_(2).sub_(1)
        s["b"] = torch.randn(d, generator=g, device="cuda")
        s["X"] = torch.randn(d, generator=g, device="cuda")
        s["mu"], s["sigma"], s["noise_seed"] = 0.1, 0.05, seed + 42
        V = torch.empty((K, d), device="cuda")
        ctx.set_levels(synth.levels_exponential(c["n_sym"] - 1))
        if c["kind"] == "game":
            ctx.game_dual_vectors(s["X"], s["a"], s["b"], s["mu"], s["sigma"], s["noise_seed"], 1 << 20, out=V)
            ctx.fit_levels(V, c["n_sym"], 4096, sweeps=c["sweeps"])
            del V
            ctx.state_init(s["X"])
            s["A"], s["B"] = ctx.new_stream(slotted=True), ctx.new_stream(slotted=True)
            s["Xh"], s["Xn"] = torch.empty(d, device="cuda"), torch.empty(d, device="cuda")
        else:
            s["V"], s["hist"] = V, torch.empty(4096, dtype=torch.float64, device="cuda")
        return s
    V = s["V"] = _vectors(c, seed, 0)
    if c["tables"] == 2:
        ctx.select_table(1)
        _set_tables(ctx, c, V)
        ctx.select_table(0)
    _set_tables(ctx, c, V)
    s["A"] = _new_stream(ctx, c)
    if c["kind"] in ("iteration", "step", "refit"):
        ctx.state_init(torch.randn(d, generator=g, device="cuda") if c["anchor"] else None)
        s["Xh"], s["Xn"] = torch.empty(d, device="cuda"), torch.empty(d, device="cuda")
    if c["kind"] == "iteration":
        s["V1"] = _vectors(c, seed, 1)
        s["B"] = _new_stream(ctx, c)
        if c["average"]:
            ctx.average_reset(True)
        if c["optimistic"]:                                      # the iteration before left its second stream
            ctx.quantize_encode(V, 1 << 20, s["A"])
    elif c["kind"] == "refit":
        s["hist"] = torch.empty(4096, dtype=torch.float64, device="cuda")
    elif c["kind"] == "roundtrip":
        s["Vhat"] = torch.empty((K, d), device="cuda")
    elif c["kind"] == "exchange":
        s["mean"] = torch.empty(d, device="cuda")
    return s


# ---- one pass ------------------------------------------------------------------------------------------------------


def _coded(st):
    return dict(norms=st.norms, sub_end=st.sub_end)


def run(s):
    c, ctx = s["case"], s["ctx"]
    kind = c["kind"]
    if kind == "iteration":
        A, B = s["A"], s["B"]
        two = c["tables"] == 2
        if not c["optimistic"]:
            ctx.quantize_encode(s["V"], qgx.CALL_FIRST_HALF, A)
        ctx.eg_step(0, A, None, s["Xh"])
        if two:
            ctx.select_table(1, 0)
        ctx.quantize_encode(s["V1"], qgx.CALL_SECOND_HALF, B)
        ctx.eg_step(1, B, A, s["Xn"])
        if two:
            ctx.select_table(0)
        if c["optimistic"]:
            s["A"], s["B"] = B, A
        return dict(Xh=s["Xh"], Xn=s["Xn"], first=_coded(A), second=_coded(B))
    if kind == "step":
        ctx.quantize_encode(s["V"], s["call"], s["A"])
        ctx.eg_step(0, s["A"], None, s["Xh"])
        return dict(Xh=s["Xh"], first=_coded(s["A"]))
    if kind == "refit":
        ctx.fit_levels(s["V"], c["n_sym"], 4096, sweeps=c["sweeps"], hist_out=s["hist"])
        out = {}
        if c["code"] == "fitted":
            out["p"], out["len"], out["bits"] = ctx.fit_code()
        ctx.quantize_encode(s["V"], s["call"], s["A"])
        ctx.eg_step(0, s["A"], None, s["Xh"])
        return dict(out, hist=s["hist"], Xh=s["Xh"], first=_coded(s["A"]))
    if kind == "roundtrip":
        ctx.quantize_encode(s["V"], s["call"], s["A"])
        ctx.decode(s["A"], s["Vhat"])
        return dict(Vhat=s["Vhat"], first=_coded(s["A"]))
    if kind == "exchange":
        ctx.quantize_encode(s["V"], s["call"], s["A"])
        ctx.decode_average(s["A"], s["mean"])
        return dict(mean=s["mean"], payload=s["A"].payload, chunk_off=s["A"].chunk_off, first=_coded(s["A"]))
    if kind == "game":
        game = (s["a"], s["b"], s["mu"], s["sigma"], s["noise_seed"])
        ctx.quantize_encode_game(s["X"], *game, qgx.CALL_FIRST_HALF, s["A"])
        ctx.eg_step(0, s["A"], None, s["Xh"])
        ctx.quantize_encode_game(s["Xh"], *game, qgx.CALL_SECOND_HALF, s["B"])
        ctx.eg_step(1, s["B"], s["A"], s["Xn"])
        s["X"], s["Xn"] = s["Xn"], s["X"]
        return dict(Xh=s["Xh"], Xn=s["X"], norms=s["A"].norms, norms_second=s["B"].norms)
    ctx.game_dual_vectors(s["X"], s["a"], s["b"], s["mu"], s["sigma"], s["noise_seed"], s["call"], out=s["V"])
    ctx.fit_levels(s["V"], c["n_sym"], 4096, sweeps=c["sweeps"], hist_out=s["hist"])
    return dict(V=s["V"], hist=s["hist"], levels=ctx.get_levels())


# ---- what a pass cannot do without, and how close another correct one comes ----------------------------------------


def _stream_bytes(c):
    """One coded stream of the K vectors: code words and signs, 16-bit ends of runs of 32, norms.

    Bits of a coordinate by the code: the width and the sign; about the entropy of a fitted table's symbols and the
    sign; the length that Elias' code takes on average over the table's upper half (fitted and exponential tables put
    most of the weight there)."""
    if c["code"] == "fixed":
        bits = _width(c["n_sym"]) + 1.0
    elif c["code"] == "fitted":
        bits = max(1.5, math.log2(c["n_sym"]) - 0.5)
    else:
        bits = {3: 3.0, 8: 6.0, 9: 6.5, 15: 8.0, 17: 8.0, 33: 11.9, 65: 13.0, 127: 14.0}[c["n_sym"]]
    return c["K"] * c["d"] * (bits / 8.0 + 2.0 / 32.0 + 4.0 / c["bucket"])


def work(case):
    c = dict(case)
    K, d, st = c["K"], c["d"], _stream_bytes(c)
    start = 4 * d if c["anchor"] or c["kind"] == "game" else 0
    code = 4 * K * d + st                                        # V read, stream written
    half0 = st + 4 * d + start + 4 * d + (16 * d if c["average"] else 0)     # stream, Y, X_1 read; X_{t+1/2} written
    half1 = 2 * st + 8 * d + start + 4 * d                       # both streams, Y read and written; X_1 read, X_{t+1} written
    if c["kind"] == "iteration":
        n, by = (1 if c["optimistic"] else 2), (1 if c["optimistic"] else 2) * code + half0 + half1
    elif c["kind"] == "step":
        n, by = 1, code + half0
    elif c["kind"] == "refit":
        n, by = 2, 4 * K * d + code + half0
    elif c["kind"] == "roundtrip":
        n, by = 1, code + st + 4 * K * d
    elif c["kind"] == "exchange":
        n, by = 1, code + st + 4 * d
    elif c["kind"] == "game":
        n, by = 2, 2 * (10 * d + st) + half0 + half1
    else:
        n, by = 1, 10 * d + 4 * K * d + 4 * K * d
    return {"bytes": by, "flops": 12.0 * n * K * d}


def tolerance(case):
    # Means and iterates are sums of K binary32 terms (against the same sums in binary64: up to 6e-8 in the 2-norm,
    # 7e-7 of the largest element); whole numbers stay the same.
    if case["kind"] == "game":
        # The second call codes vectors that depend on X_{t+1/2}: an iterate off by one unit in the last place here and
        # there flips a rounding decision now and then (measured at 2^22 coordinates: 6e-8 in the 2-norm, 4e-5 of the
        # root mean square at one coordinate; a flip weighs more in a shorter vector and with fewer workers).
        return {"rel": 3e-6, "max": 2e-3}
    return {"rel": 1e-6, "max": 1e-5}
