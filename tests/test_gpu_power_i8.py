"""The int8-MFMA power products of fp32-gradient layers (k_gemm_i8.hip) at the
edges of their tiles, stages, K slices and digit planes: sync steps against the float64 oracle, teacher-forced, within the bounds of
gpu_util.check_errors (fp64-accurate products behind fp32 state)."""
import os
import sys

import numpy as np
import pytest
import torch

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))

import oracle as O  # noqa: E402
import paper_2512_13728_amd as cdl  # noqa: E402
import synthetic as S  # noqa: E402
from gpu_util import (buffer_f32, check_errors, device_to_numpy, f32, f64, group_step_and_compare,  # noqa: E402
                      step_and_compare, sync_errors)

pytestmark = pytest.mark.gpu


class Beside:
    """A layer that steps in one group with a layer of another shape: units side
    by side take the digits at any size, where a small layer alone stays on the
    fp64 MFMA.  Steps and answers as the layer itself."""

    def __init__(self, m, n, r, **kw):
        self.layers = [cdl.Layer(m, n, r, **kw), cdl.Layer(m, n + 4, r, **kw)]
        self.group = cdl.Group(self.layers)
        g = torch.Generator("cuda").manual_seed(1)
        self.other = [torch.randn(*s, device="cuda", generator=g) for s in [(m, n + 4)] * 3 + [(n + 4, r)]]

    def step(self, G, M, X, Q, mu, eta, r):
        _, flag, per, status = self.group.step(*([a, b] for a, b in zip((G, M, X, Q), self.other)), mu, eta, r)
        return per[0], flag, status

    def __getattr__(self, name):
        return getattr(self.layers[0], name)


# the narrowest rank of the path and the one below it; column blocks of 32,
# tiles of 64 and 128 columns whole and partial; K of one stage and one past
# it, several slices, slices with a partial last chunk; rows not a multiple of
# four (unaligned loads); tall and wide; every width of the tiles that find B's
# row and column maxima; more rows of P or of R than the launch that cuts them
# has waves
@pytest.mark.parametrize("m,n,r", [
    (260, 257, 32), (260, 257, 33), (129, 64, 64), (64, 129, 64), (65, 66, 65), (127, 1030, 96),
    (1030, 127, 97), (200, 2051, 128), (2051, 200, 129), (150, 5000, 34), (5000, 150, 34), (600, 700, 320),
    (64, 9001, 33), (40, 33000, 33), (40, 40001, 33), (20000, 64, 40),
    (20000, 135, 130), (135, 20000, 130),
])
def test_power_product_edges(m, n, r):
    w = S.small_workload(m, n, r, k=min(24, r - 1), stream_id=700 + r)
    M, X, Q = (t.cuda().contiguous() for t in S.initial_state(w, 0, device="cpu"))
    L = Beside(m, n, r, policy=cdl.POLICY_ALWAYS_SYNC)
    stream = S.GradientStream(w, 0, device="cpu")
    for t in range(2):
        d = step_and_compare(L, stream.next().cuda(), M, X, Q, 0.95, 0.01, r, 0.5, O.POLICY_ALWAYS_SYNC)
        print(f"{m}x{n} r={r} t={t + 1}", {k: v for k, v in d.items() if k.startswith("err") or k == "kappa"}, flush=True)
        check_errors(d, False)


# the digits are relative to the largest |B| and to each column's largest |Q|:
# magnitudes near both ends of fp32, and a few entries far above the others
@pytest.mark.parametrize("kind", ["large", "small", "outlier", "spike", "column scales"])
def test_power_product_scales(kind):
    m, n, r = 192, 320, 48
    w = S.small_workload(m, n, r, k=24, stream_id=760)
    M, X, Q = (t.cuda().contiguous() for t in S.initial_state(w, 0, device="cpu"))
    G = S.GradientStream(w, 0, device="cpu").next().cuda()
    if kind in ("large", "small"):
        f = 2.0 ** (60 if kind == "large" else -60)
        M, G = M * f, G * f
    elif kind in ("outlier", "spike"):
        G[3, 5] += 1e3 if kind == "outlier" else 1e5
        G[100, 200] -= 1e3
    else:
        # a range of 2^12: kappa(P~) stays below the 3e6 at which pivots are floored
        Q *= torch.logspace(-6, 6, r, base=2.0, device="cuda")[None, :]
    L = Beside(m, n, r, policy=cdl.POLICY_ALWAYS_SYNC)
    d = step_and_compare(L, G, M, X, Q.contiguous(), 0.95, 0.01, r, 0.5, O.POLICY_ALWAYS_SYNC)
    print(kind, {k: v for k, v in d.items() if k.startswith("err") or k == "kappa"}, flush=True)
    check_errors(d, False)


# a NaN or an Inf in G reaches its row of B^T P only: its column of M is NaN and
# the others stay finite (the pivots of the NaN Gram matrix are floored and
# their columns completed); a NaN row of R makes every normalised column NaN,
# an infinite one leaves zeros beside it
@pytest.mark.parametrize("bad", [float("nan"), float("inf"), -float("inf")])
@pytest.mark.parametrize("m,n,r", [(300, 200, 48), (130, 515, 64), (300, 200, 97), (420, 515, 400)])
def test_power_product_nonfinite(m, n, r, bad):
    w = S.small_workload(m, n, r, k=24, stream_id=770)
    M, X, Q = (t.cuda().contiguous() for t in S.initial_state(w, 0, device="cpu"))
    G = S.GradientStream(w, 0, device="cpu").next().cuda()
    G[7, 11] = bad
    L = Beside(m, n, r, policy=cdl.POLICY_ALWAYS_SYNC)
    _, flag, status = L.step(G, M, X, Q, 0.95, 0.01, r)
    torch.cuda.synchronize()
    assert flag and status != 0
    want = torch.zeros(m, n, dtype=torch.bool)
    want[:, 11] = True
    assert torch.equal(torch.isnan(M).cpu(), want)
    Qc = Q.cpu()
    assert torch.isnan(Qc[11]).all()
    rest = torch.cat([Qc[:11], Qc[12:]])
    assert torch.isfinite(rest).all()
    if bad == bad:
        assert (rest == 0).all()


# the fp32-accurate update around the rank where it goes from three bf16 pieces
# to two scaled fp16 ones, with column padding and rows of R far apart in size;
# X starts from zero, so that its error is the correction's own: r fp32
# additions of products exact to about 2^-23, within the same 1e-5 as every
# other fp32 quantity
@pytest.mark.parametrize("r", [128, 129, 160, 191])
@pytest.mark.parametrize("m,n", [(300, 260), (257, 333)])
def test_update_pieces(m, n, r):
    w = S.small_workload(m, n, r, k=24, stream_id=780 + r)
    M, X, Q = (t.cuda().contiguous() for t in S.initial_state(w, 0, device="cpu"))
    G = S.GradientStream(w, 0, device="cpu").next().cuda()
    # a range of 2^8: kappa(P~) stays below the 3e6 at which pivots are floored
    G *= torch.logspace(-4, 4, n, base=2.0, device="cuda")[None, :]
    M *= torch.logspace(-4, 4, n, base=2.0, device="cuda")[None, :]
    X.zero_()
    L = cdl.Layer(m, n, r, policy=cdl.POLICY_ALWAYS_SYNC)
    d = step_and_compare(L, G.contiguous(), M.contiguous(), X, Q, 0.95, 0.01, r, 0.5, O.POLICY_ALWAYS_SYNC)
    print(f"{m}x{n} r={r}", {k: v for k, v in d.items() if k.startswith("err") or k == "kappa"}, flush=True)
    for k in ("err_M", "err_X", "err_dM", "err_dX"):
        assert d[k] < 1e-5, (k, d[k])


def _dominant(m, n, r, f, seed):
    """G, M, X, Q of a layer whose buffer has one row f times the others."""
    g = torch.Generator().manual_seed(seed)
    randn = lambda *s: torch.randn(s, generator=g)  # noqa: E731
    G = 4 * randn(m, 48) @ randn(48, n) + 0.4 * randn(m, n)
    G[7] *= f
    Q = torch.linalg.qr(randn(n, r).double())[0].float()
    return tuple(t.cuda().contiguous() for t in (G, torch.zeros(m, n), 0.02 * randn(m, n), Q))


# the smallest pivots of the digit Gram matrix are 5 to 80 times the floor of 1e-13
# of its largest diagonal entry (kappa(P~) up to 6e6), in K slices of 256, 450 and
# 500 (units side by side) and of all 2050 rows (13 layers fill the chip)
@pytest.mark.parametrize("shapes,r,f", [([(2048, 512), (2048, 516)], 400, 1e5), ([(1000, 1024), (900, 1024)], 96, 2e5), ([(2050, 770)] * 13, 512, 6e4)])
def test_gram_dominant_row(shapes, r, f):
    Ls = [cdl.Layer(m, n, r, policy=cdl.POLICY_ALWAYS_SYNC) for m, n in shapes]
    G, M, X, Q = (list(t) for t in zip(*[_dominant(m, n, r, f, 791 + i) for i, (m, n) in enumerate(shapes)]))
    grp = cdl.Group(Ls)
    check = range(min(2, len(shapes)))
    _, errs = group_step_and_compare(grp, Ls, G, M, X, Q, 0.95, 0.01, r, 0.5, O.POLICY_ALWAYS_SYNC, check=check)
    for i, d in errs.items():
        print(shapes[i], r, {k: v for k, v in d.items() if k.startswith("err") or k in ("kappa", "orth_P")}, flush=True)
    assert not any(L.rank_deficient() for L in Ls)
    for d in errs.values():
        check_errors(d, False)


# digit Gram matrices at the edges of their 64- and 128-column tiles and 32-column
# blocks, in two units side by side; ragged K slices
@pytest.mark.parametrize("r", [64, 65, 96, 97, 128, 129, 192, 193, 383, 384, 417, 513])
def test_gram_edges(r):
    shapes = [(701, 600), (650, 731)]
    w = [S.small_workload(m, n, r, k=24, stream_id=870 + r + i) for i, (m, n) in enumerate(shapes)]
    M, X, Q = (list(t) for t in zip(*[[t.cuda().contiguous() for t in S.initial_state(v, 0, device="cpu")] for v in w]))
    streams = [S.GradientStream(v, 0, device="cpu") for v in w]
    Ls = [cdl.Layer(m, n, r, policy=cdl.POLICY_ALWAYS_SYNC) for m, n in shapes]
    grp = cdl.Group(Ls)
    for t in range(2):
        G = [s.next().cuda() for s in streams]
        _, errs = group_step_and_compare(grp, Ls, G, M, X, Q, 0.95, 0.01, r, 0.5, O.POLICY_ALWAYS_SYNC)
        for i, d in errs.items():
            print(shapes[i], r, t + 1, {k: v for k, v in d.items() if k.startswith("err") or k == "kappa"}, flush=True)
            check_errors(d, False)


def _row_err(a, b):
    return (np.linalg.norm(a - b, axis=1) / np.linalg.norm(b, axis=1)).max()


# every row and every column of B has a scale of its own: with half of them
# 2^-40 of the others (a layer-wide scale would leave them 7 bits), each row of
# P, R, Q, dM and dX and each column of dM and dX is still as accurate as fp32
# state allows.  r = 32 takes the fp64 MFMA, r = 160 the update from fp16
# pieces.  The reference applies the inverse
# factor to the rows of P~, as a Householder QR is not accurate row by row.
@pytest.mark.parametrize("r", [32, 48, 97, 160])
@pytest.mark.parametrize("kind", ["rows", "columns", "both"])
@pytest.mark.parametrize("m,n", [(512, 640), (509, 643)])
def test_small_rows_and_columns(m, n, kind, r):
    w = S.small_workload(m, n, r, k=24, stream_id=810 + r)
    _, X, Q = (t.cuda().contiguous() for t in S.initial_state(w, 0, device="cpu"))
    G = S.GradientStream(w, 0, device="cpu").next().cuda()
    if kind != "columns":
        G[m // 2:] *= 2.0 ** -40
    if kind != "rows":
        G[:, ::2] *= 2.0 ** -40
    M = torch.zeros_like(G)
    X.zero_()
    B, Q0 = f64(G), f64(Q)
    L = Beside(m, n, r, policy=cdl.POLICY_ALWAYS_SYNC)
    L.step(G, M, X, Q, 0.95, 0.01, r)
    torch.cuda.synchronize()
    Pa, Ra = L.last_factors()
    P, R = device_to_numpy(Pa, (m, r)).astype(np.float64), device_to_numpy(Ra, (n, r)).astype(np.float64)
    Pt = B @ Q0
    T = np.linalg.qr(Pt)[1]
    Pw = Pt @ np.linalg.inv(T * np.sign(np.diagonal(T))[:, None])
    Rw = B.T @ Pw
    Qw = Rw / np.linalg.norm(Rw, axis=0)
    dM, dMw = B - f64(M), (1 - f32(0.95)) * Pw @ Rw.T
    dXw = -f32(0.01) * np.sqrt(m / n) * Pw @ Qw.T
    e = {"P": _row_err(P, Pw), "R": _row_err(R, Rw), "Q": _row_err(f64(Q), Qw), "dM": _row_err(dM, dMw),
         "dM'": _row_err(dM.T, dMw.T), "dX": _row_err(f64(X), dXw), "dX'": _row_err(f64(X).T, dXw.T)}
    print(f"{m}x{n} r={r} {kind}", {k: f"{v:.1e}" for k, v in e.items()}, "kappa %.1e" % np.linalg.cond(Pt), flush=True)
    # dM = B - M cancels all but (1 - mu) of B, which M rounds to fp32
    assert all(v < (2e-5 if k.startswith("dM") else 1e-5) for k, v in e.items()), e


# 32 layers fill the chip, so that every product is one K slice of more than
# 1024 rows and the digits take two launches; sizes that no tile, chunk or
# column block divides; a NaN in one layer, whose column of M it fills
def test_long_slices():
    m, n, r, layers, sick = 1050, 1101, 97, 32, 5
    w = S.small_workload(m, n, r, k=24, stream_id=830)
    M, X, Q = ([t.cuda().contiguous().clone() for _ in range(layers)] for t in S.initial_state(w, 0, device="cpu"))
    stream = S.GradientStream(w, 0, device="cpu")
    G = [stream.next().cuda() for _ in range(layers)]
    G[sick][17, 1100] = float("nan")
    Ls = [cdl.Layer(m, n, r, policy=cdl.POLICY_ALWAYS_SYNC) for _ in range(layers)]
    check = [0, layers - 1]
    snap = {i: (f64(M[i]), f64(X[i]), f64(Q[i])) for i in check}
    _, flag, _, status = cdl.Group(Ls).step(G, M, X, Q, 0.95, 0.01, r)
    torch.cuda.synchronize()
    assert flag and status != 0
    for i in check:
        M0, X0, Q0 = snap[i]
        B = buffer_f32(M0, f64(G[i]))
        ref = O.sync_update(B, X0, Q0, f32(0.95), f32(0.01), 1.0)
        P = device_to_numpy(Ls[i].last_factors()[0], (m, r)).astype(np.float64)
        d = sync_errors(ref, M0, X0, B, f64(M[i]), f64(X[i]), f64(Q[i]), P)
        print(i, {k: v for k, v in d.items() if k.startswith("err")}, flush=True)
        check_errors(dict(d, flag_oracle=True), False)
    want = torch.zeros(m, n, dtype=torch.bool)
    want[:, 1100] = True
    assert torch.equal(torch.isnan(M[sick]).cpu(), want)
    assert all(torch.isfinite(M[i]).all() and torch.isfinite(Q[i]).all() for i in range(layers) if i != sick)


# a grid that is full without a split, and K past the 16384 rows that int32 sums
# hold exactly: two slices all the same
def test_slices_past_the_exact_sums():
    m, n, r, layers = 2048, 16450, 512, 4
    g = torch.Generator("cuda").manual_seed(840)
    randn = lambda *s: torch.randn(*s, device="cuda", generator=g)  # noqa: E731
    G = [randn(m, 24) @ randn(24, n) + 0.1 * randn(m, n) for _ in range(layers)]
    M, X = ([0.02 * randn(m, n) for _ in range(layers)] for _ in range(2))
    Q = [torch.linalg.qr(randn(n, r))[0].contiguous() for _ in range(layers)]
    Ls = [cdl.Layer(m, n, r, policy=cdl.POLICY_ALWAYS_SYNC) for _ in range(layers)]
    _, errs = group_step_and_compare(cdl.Group(Ls), Ls, G, M, X, Q, 0.95, 0.01, r, 0.5, O.POLICY_ALWAYS_SYNC, check=[3])
    print({k: v for k, v in errs[3].items() if k.startswith("err") or k == "kappa"}, flush=True)
    check_errors(errs[3], False)


# blocks with a NaN or an Inf are formed again on the fp64 MFMA, not entry by
# entry: at 4096 x 16384, r = 1024 a step with a NaN takes 1.55 times one
# without (entry by entry 3.1, 16.4 ms of 5.3)
def test_nonfinite_step_time():
    m, n, r = 4096, 16384, 1024
    g = torch.Generator("cuda").manual_seed(850)
    L = cdl.Layer(m, n, r, policy=cdl.POLICY_ALWAYS_SYNC)
    Q0 = torch.linalg.qr(torch.randn(n, r, device="cuda", generator=g))[0].contiguous()
    X = torch.zeros(m, n, device="cuda")
    times = {}
    for bad in (False, True):
        G = torch.randn(m, n, device="cuda", generator=g)
        if bad:
            G[5, 7] = float("nan")
        for _ in range(4):
            M, Q = torch.zeros(m, n, device="cuda"), Q0.clone()
            torch.cuda.synchronize()
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            L.step(G, M, X, Q, 0.95, 0.01, r)
            b.record()
            torch.cuda.synchronize()
            times[bad] = min(times.get(bad, 1e9), a.elapsed_time(b))
    print(times, flush=True)
    assert times[True] < 2.2 * times[False], times


# where a layer alone goes from the fp64 MFMA to the digits: 1.3e9 multiplications,
# m n times r rounded up to 64
@pytest.mark.parametrize("r,digits", [(256, False), (320, True)])
def test_small_layers_alone_stay_on_fp64(r, digits):
    m = n = 2048
    w = S.small_workload(m, n, r, k=24, stream_id=890)
    M, X, Q = (t.cuda().contiguous() for t in S.initial_state(w, 0, device="cpu"))
    L = cdl.Layer(m, n, r, policy=cdl.POLICY_ALWAYS_SYNC)
    grp = cdl.Group([L])
    grp.set_timing(True)
    _, errs = group_step_and_compare(grp, [L], [S.GradientStream(w, 0, device="cpu").next().cuda()], [M], [X], [Q], 0.95, 0.01,
                                     r, 0.5, O.POLICY_ALWAYS_SYNC)
    kinds = set(grp.kernel_times())
    grp.set_timing(False)
    check_errors(errs[0], False)
    assert ("power_bq_i8x21" in kinds) == ("power_btp_i8x21" in kinds) == digits, kinds
    assert ("power_bq_f64" in kinds) == ("power_btp_f64" in kinds) != digits, kinds
    # the Gram matrices, m r^2, are far from it at either rank
    assert "gram_f64" in kinds and "gram_i8x26" not in kinds


# the allocation-free step carves the digits, the maxima and the partials from its
# fixed array: bit-identical to the layer's own step, above and below the size from
# which a layer alone takes the digits, after each other in the same array
def test_static_step_takes_the_same_products():
    for m, n, r in [(4096, 16384, 64), (700, 901, 97), (4096, 16384, 64)]:
        g = torch.Generator("cuda").manual_seed(860 + r)
        randn = lambda *s: torch.randn(*s, device="cuda", generator=g)  # noqa: E731
        a = [0.02 * randn(m, n), 0.02 * randn(m, n), torch.linalg.qr(randn(n, r))[0].contiguous()]
        b = [t.clone() for t in a]
        L = cdl.Layer(m, n, r, policy=cdl.POLICY_ALWAYS_SYNC)
        prev, step = torch.zeros(1, dtype=torch.float64, device="cuda"), 0
        for _ in range(2):
            G = randn(m, 16) @ randn(16, n) + 0.1 * randn(m, n)
            one = L.step(G, *a, 0.95, 0.01, r)
            rm, flag, status, step = cdl.step_static(m, n, r, prev, step, G, *b, 0.95, 0.01, r, policy=cdl.POLICY_ALWAYS_SYNC)
            torch.cuda.synchronize()
            assert one == (rm, flag, status)
            assert all(torch.equal(x, y) for x, y in zip(a, b)), (m, n, r, step)


# asynchronous steps enqueue both branches on the gate's decision: the digit
# products, their maxima and the fp16 pieces run on the steps that sync and
# leave everything alone on those that do not
@pytest.mark.parametrize("r", [48, 160])
def test_async_steps_bit_identical_to_blocking(r):
    shapes, steps, spikes = [(256, 384), (384, 257), (256, 384)], 8, (4, 6)
    g = torch.Generator("cuda").manual_seed(880 + r)
    randn = lambda *s: torch.randn(*s, device="cuda", generator=g)  # noqa: E731
    G = [[(40.0 if t in spikes else 1.0) * (randn(m, 24) @ randn(24, n) + 0.1 * randn(m, n)) for m, n in shapes] for t in range(steps)]
    start = [[0.02 * randn(m, n) for m, n in shapes], [0.02 * randn(m, n) for m, n in shapes],
             [torch.linalg.qr(randn(n, r))[0].contiguous() for _, n in shapes]]
    runs = []
    for wait in (True, False):
        Ls = [cdl.Layer(m, n, r, tau=0.5, weight_decay=0.05) for m, n in shapes]
        grp = cdl.Group(Ls)
        state = [[t.clone() for t in v] for v in start]
        flags = []
        for t in range(steps):
            got = grp.step(G[t], *state, 0.95, 0.01, r, wait=wait)
            flags.append((got if wait else grp.last_result())[1])
        torch.cuda.synchronize()
        runs.append((flags, state))
    assert runs[0][0] == runs[1][0] and runs[0][0][0] and True in runs[0][0][1:] and False in runs[0][0]
    for a, b in zip(*(sum(s, []) for _, s in runs)):
        assert torch.equal(a, b)
