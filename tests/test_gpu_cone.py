"""Torus walks held as the square of their live sites, against the kernels of the
whole lattice (asked for with stream_kernel) and the oracle.

Every live amplitude is the same expression whichever kernel computes it, so
states agree bit for bit (in complex64 below the smallest normal number too, where it
matters at which steps the levels' powers of two are multiplied back: a difference
there climbs, one rounding at a time).  The Fourier coin's complex128 butterflies and the inverse walk (which drops the rounding noise outside the
shrinking cone) agree to the sum of their roundings: T steps of at most 8 epsilon.
"""
import numpy as np
import pytest

import oracle
from paper_1003_3779_amd import inputs, qwalk

pytestmark = pytest.mark.gpu

EPS = {qwalk.QW_C128: 2.0 ** -53, qwalk.QW_C64: 2.0 ** -24}


@pytest.fixture(scope="module", autouse=True)
def gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    qwalk.load()
    yield


def _run(ext, table, kind, psi0, x0, plan, prec, dense=None, **opts):
    w = qwalk.Walk(ext, getattr(inputs, table), kind, psi0, x0, prec=prec, dense=dense)
    w.set_options(renorm_every=0, **opts)
    for n in plan:
        (w.step if n >= 0 else w.step_inverse)(abs(n))
    out = w.probabilities(), w.get_state(), w.norm(), w.time()
    w.destroy()
    return out


@pytest.mark.parametrize("prec", [qwalk.QW_C128, qwalk.QW_C64])
@pytest.mark.parametrize("table", ["PAIR", "EQ8", "DIAG"])
@pytest.mark.parametrize("kind", [qwalk.GROVER, qwalk.HADAMARD2, qwalk.FOURIER, qwalk.DENSE])
@pytest.mark.parametrize("ext,plans", [
    # the smallest torus; the last step before the seam, on it and past it; every remainder of 16
    ((32, 33), ([0], [1], [15], [16], [17], [3, 5, 20])),
    ((130, 97), ([47], [48], [49], [31, 9, 7, 1], [40, -13, 6], [20, -20], [9, -12])),
    # squares past what the small-square kernel takes, strips and segments with remainders
    ((905, 870), ([433], [417, -30])),
])
def test_cone_equals_whole_lattice(prec, table, kind, ext, plans):
    rng = np.random.default_rng([ext[0], kind, prec, len(table)])
    dense = inputs.haar_unitary(rng, 4) if kind == qwalk.DENSE else None
    psi0 = inputs.haar_state(rng, 4)
    x0 = (int(rng.integers(0, ext[0])), int(rng.integers(0, ext[1])))
    for plan in plans:
        P, psi, n, t = _run(ext, table, kind, psi0, x0, plan, prec, dense)
        Pr, ref, nr, tr = _run(ext, table, kind, psi0, x0, plan, prec, dense, stream_kernel=1)
        assert t == tr == sum(plan)
        steps = sum(abs(k) for k in plan)
        same = not (kind == qwalk.FOURIER and prec == qwalk.QW_C128) and min(plan) >= 0
        tol = 0.0 if same else 8 * steps * EPS[prec]
        assert np.max(np.abs(psi - ref)) <= tol, plan
        assert np.max(np.abs(P - Pr)) <= max(2 * tol, 4 * EPS[qwalk.QW_C128]), plan
        assert abs(n - nr) <= max(2 * tol, 64 * EPS[qwalk.QW_C128]), plan


@pytest.mark.parametrize("table", ["PAIR", "EQ8", "DIAG"])
def test_cone_against_oracle_on_the_seam(table):
    """Both axes' outermost points meet at t = L / 2 (where P sums them)."""
    L, T = 64, 32
    psi0 = inputs.haar_state(np.random.default_rng(5), 4)
    C = oracle.coin(oracle.GROVER, 4)
    P, psi, n, _ = _run((L, L), table, qwalk.GROVER, psi0, (60, 3), [T], qwalk.QW_C128)
    ref = oracle.walk(L, L, getattr(inputs, table), C, (60, 3), psi0, T)
    assert np.max(np.abs(P - oracle.prob(ref))) <= 1e-12
    assert np.max(np.abs(psi - np.transpose(ref, (2, 0, 1)))) <= 1e-12


def test_leaving_the_cone():
    """What the square cannot hold takes the walk to the whole lattice, unchanged:
    other kernels asked for, links that break, a state set by the caller."""
    ext, x0 = (80, 70), (11, 60)
    psi0 = inputs.haar_state(np.random.default_rng(6), 4)
    ref = _run(ext, "PAIR", qwalk.GROVER, psi0, x0, [30], qwalk.QW_C128, stream_kernel=1)[1]
    w = qwalk.Walk(ext, inputs.PAIR, qwalk.GROVER, psi0, x0)
    w.step(20)
    before = w.get_state()
    w.set_options(block_depth=1)
    assert np.array_equal(w.get_state(), before)
    w.step(10)
    assert np.array_equal(w.get_state(), ref)
    w.set_options(block_depth=0)
    w.reset(psi0, x0)
    w.step(20)
    state = w.get_state()
    assert np.array_equal(state, before)
    w.set_state(state)
    w.step(10)
    assert np.array_equal(w.get_state(), ref)
    w.reset(psi0, x0)
    w.set_broken_links(1.0, seed=3)
    w.step(6)
    P = w.probabilities()
    assert abs(P[x0[1], x0[0]] - 1.0) <= 1e-14      # every link broken: the walker stays
    w.set_options()
    w.reset(psi0, x0)
    w.set_broken_links(0.0)
    w.step(30)
    assert np.array_equal(w.get_state(), ref)
    w.destroy()


def test_cone_norm_checks_complex64():
    """The rescales of complex64 walks: a check every 64 steps, as on the whole lattice."""
    psi0 = inputs.haar_state(np.random.default_rng(7), 4)
    res = []
    for opts in ({}, {"stream_kernel": 1}):
        w = qwalk.Walk((600, 610), inputs.PAIR, qwalk.HADAMARD2, psi0, (3, 4), prec=qwalk.QW_C64)
        w.set_options(**opts)
        w.step(290)
        st = w.stats()
        res.append((w.probabilities(), w.norm(), st.renorm_checks, st.renorms))
        w.destroy()
    assert res[0][2] == res[1][2] == 290 // 64 and res[0][3] == res[1][3]
    assert np.max(np.abs(res[0][0] - res[1][0])) <= 2 * EPS[qwalk.QW_C64] * np.max(res[1][0])
    assert abs(res[0][1] - 1.0) <= 1e-6


def test_narrow_torus_of_many_rows():
    """More than 65535 rows of 64 x 64 tiles: past what a grid's second dimension takes."""
    import torch
    ext, x0 = (32, 65536 * 64 + 1), (30, 4194200)
    psi0 = inputs.haar_state(np.random.default_rng(9), 4)
    P = torch.empty(ext[1], ext[0], dtype=torch.float64, device="cuda")
    w = qwalk.Walk(ext, inputs.PAIR, qwalk.GROVER, psi0, x0, prec=qwalk.QW_C64)
    v = qwalk.Walk((32, 64), inputs.PAIR, qwalk.GROVER, psi0, (30, 40), prec=qwalk.QW_C64)   # the same cone on a torus that holds it
    for T in (12, 8):     # on the square of live sites, and past it (the seam is at 16)
        w.step(T)
        v.step(T)
        w.probabilities(out=P)
        ref = v.probabilities()
        rows = (np.arange(64) - 40 + x0[1]) % ext[1]
        got = P[torch.as_tensor(rows, device="cuda")].cpu().numpy()
        assert np.array_equal(got, ref)
        assert float(P.sum()) == pytest.approx(float(ref.sum()), abs=1e-12)
    w.destroy()
    v.destroy()


@pytest.mark.parametrize("prec", [qwalk.QW_C128, qwalk.QW_C64])
@pytest.mark.parametrize("table", ["PAIR", "DIAG"])
@pytest.mark.parametrize("ext", [(64, 64), (50, 83), (2048, 2048), (2049, 2049), (64, 70001)])
def test_cone_probabilities_on_both_kernels(prec, table, ext):
    """P by sites (up to 2^22 of them) and by tiles (more, narrow tori among them), at the last steps
    before the seam and on it: the squares of the state's amplitudes."""
    L = min(ext)
    psi0, x0 = inputs.haar_state(np.random.default_rng(8), 4), (L - 3, 5)
    w = qwalk.Walk(ext, getattr(inputs, table), qwalk.GROVER, psi0, x0, prec=prec)
    for T in (L // 2 - 1, 1):
        w.step(T)
        P, psi = w.probabilities(), w.get_state()
        # sums of eight squares, in another order
        assert np.max(np.abs(P - np.sum(psi.real ** 2 + psi.imag ** 2, axis=0))) <= 8 * EPS[qwalk.QW_C128]
        assert abs(P.sum() - 1.0) <= (1e-12 if prec == qwalk.QW_C128 else 1e-5)
    w.destroy()


def test_small_lattices_are_not_slower_than_the_whole_lattice():
    """P of a 512^2 walk, again and again: on the square it lasts no longer than on the whole
    lattice (a fill and a kernel; by tiles it was 1.9 times that)."""
    import time
    import torch
    psi0 = inputs.haar_state(np.random.default_rng(7), 4)
    P = torch.empty(512, 512, dtype=torch.float64, device="cuda")
    ws, best = [], [1e9, 1e9]
    for opts in ({}, {"stream_kernel": 1}):
        ws.append(qwalk.Walk((512, 512), inputs.PAIR, qwalk.GROVER, psi0, (256, 256)))
        ws[-1].set_options(**opts)
        ws[-1].step(128)
    for _ in range(8):
        for i, w in enumerate(ws):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            for _ in range(200):
                w.probabilities(out=P)
            torch.cuda.synchronize()
            best[i] = min(best[i], time.perf_counter() - t0)
    for w in ws:
        w.destroy()
    assert best[0] <= 1.2 * best[1]


# from side 700 on a launch takes up to 32 steps in four stages.  Whole launches, and ones of 17 to
# 31 steps (later stages pass rows through); complex64 groups of 12 steps end inside a stage;
# strips and segments with remainders on both axes.
DEEP = (2300, 2111)


def _deep(table, kind, prec, plan, **opts):
    import torch
    w = qwalk.Walk(DEEP, getattr(inputs, table), kind, inputs.haar_state(np.random.default_rng([12, kind]), 4), (2290, 1000),
                   prec=prec)
    w.set_options(renorm_every=0, **opts)
    for n in plan:
        w.step(n)
    psi = torch.empty(4, DEEP[1], DEEP[0], dtype=torch.complex128, device="cuda")
    w.get_state(out=psi)
    n = w.norm()
    w.destroy()
    return psi, n


@pytest.mark.parametrize("table", ["PAIR", "EQ8", "DIAG"])
@pytest.mark.parametrize("kind", [qwalk.GROVER, qwalk.HADAMARD2])
@pytest.mark.parametrize("prec,opts", [(qwalk.QW_C128, {}), (qwalk.QW_C64, {}), (qwalk.QW_C64, {"block_depth": 12})])
def test_four_stage_launches_bitwise(table, kind, prec, opts):
    """complex64: bit for bit, subnormal numbers too.  complex128 multiplies the levels' powers of two back
    at the end of a launch, wherever the whole lattice's launches end: numbers below 2^-1022 (the fronts from t = 1022
    on) round at other steps, each launch by 2^-1075 a value or sqrt(2300 2111 8) 2^-1075 in the 2-norm, which
    the steps keep, so 66 launches by less than 2^-1055; every value above 2^-1002 agrees bit for bit."""
    import torch
    for plan in ([1055], [701, 32, 17, 1], [1000, 31, 24]):
        psi, n = _deep(table, kind, prec, plan, **opts)
        ref, nr = _deep(table, kind, prec, plan, stream_kernel=1, **opts)
        assert float((torch.view_as_real(psi) - torch.view_as_real(ref)).abs().max()) <= (2.0 ** -1055 if prec == qwalk.QW_C128 else 0.0), plan
        assert abs(n - nr) <= 1e-12


@pytest.mark.parametrize("kind", [qwalk.GROVER, qwalk.HADAMARD2])
def test_four_stage_norm_checks(kind):
    """Norm sums left by launches of 32 steps: complex64 checks every 64 steps up to t = 1050.  A rescale whose
    norm was summed in another order rounds within 2^-24 of the state, so P differs by at most
    2 sqrt(max P) 2^-24 for each of the 16 checks."""
    res = []
    for opts in ({}, {"stream_kernel": 1}):
        w = qwalk.Walk(DEEP, inputs.PAIR, kind, inputs.haar_state(np.random.default_rng(13), 4), (3, 4), prec=qwalk.QW_C64)
        w.set_options(**opts)
        w.step(1050)
        st = w.stats()
        res.append((w.probabilities(), st.renorm_checks, st.renorms, st.last_norm))
        w.destroy()
    assert res[0][1] == res[1][1] == 16 and res[0][2] == res[1][2]
    assert abs(res[0][3] - res[1][3]) <= 16 * 2.0 ** -23
    assert np.max(np.abs(res[0][0] - res[1][0])) <= 16 * 2 * np.sqrt(np.max(res[1][0])) * EPS[qwalk.QW_C64]
