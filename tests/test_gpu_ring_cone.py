"""One-walk rings on the points they reach (k_ring_cone) against one step per launch:
the same expressions per point, so bit for bit the same amplitudes."""
import numpy as np
import pytest

from paper_1003_3779_amd import inputs, qwalk

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    qwalk.load()
    yield


# points per lane 1 to 9 (the windows of a quarter of the points and 32 more), the round
# of 32 steps and its neighbours, and the last steps before the points
# meet
@pytest.mark.parametrize("prec", [qwalk.QW_C128, qwalk.QW_C64])
@pytest.mark.parametrize("real", [True, False])
@pytest.mark.parametrize("N,pieces", [(3, (1,)), (5, (2,)), (66, (31, 1)), (67, (33,)), (260, (96, 31)),
                                      (2001, (1000,)), (4096, (1100, 640, 200)), (4096, (2040,))])
def test_ring_cone_bitwise(prec, real, N, pieces):
    rng = np.random.default_rng(N + sum(pieces))
    th = 0.83
    U = (np.array([[np.cos(th), np.sin(th)], [-np.sin(th), np.cos(th)]], dtype=np.complex128) if real
         else inputs.haar_unitary(rng, 2))
    psi0, x0 = inputs.haar_state(rng, 2), (int(rng.integers(0, N)), 0)
    got = []
    for depth in (1, 0):
        w = qwalk.Walk((N,), inputs.RING, qwalk.DENSE, psi0, x0, prec=prec, dense=U)
        w.set_options(block_depth=depth, renorm_every=0)
        for n in pieces:
            w.step(n)
        got.append((w.get_state(), w.probabilities(), w.norm()))
        if depth == 0:   # points 0 .. t at time t, two components each
            T = sum(pieces)
            whole = real or prec == qwalk.QW_C64 or T < 2048
            if whole:
                assert w.stats().updates == T * (T + 1)
        w.destroy()
    assert np.array_equal(got[0][0], got[1][0])
    # P is the same sum of squares of each site; outside the box it is zero
    assert np.array_equal(got[0][1], got[1][1])
    assert abs(got[0][2] - got[1][2]) <= 1e-12
