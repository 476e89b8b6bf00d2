"""The surrogate's products on both tile sizes and on turned operands, and its
prediction head by rows."""
import numpy as np
import pytest

from oracle import surrogate as S
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


def _walk_params(seed, n):
    rng = np.random.default_rng(seed)
    N = np.full(n, 4097, dtype=np.int64)
    T = rng.integers(256, 2049, n)
    return N, T, inputs.su2_angles(rng, n), np.stack([inputs.haar_state(rng, 2) for _ in range(n)])


def test_forward_rows_do_not_depend_on_the_call():
    """Tiles of 64 (few rows) and of 128 (many), whole and partial blocks of four head
    rows: K runs in the same order in both, so each row has the same bits."""
    N, T, ang, psi0 = _walk_params(5, 4099)
    s = qwalk.Surrogate(seed=9)
    X = s.features(N, T, ang, psi0)
    q = s.forward(X, T)
    for n in (1, 5, 128, 515):
        assert np.array_equal(s.forward(X[:n], T[:n]), q[:n]), n
    s.destroy()


@pytest.mark.parametrize("n", [128, 384, 1152])  # 2, 6 and 18 K tiles of dW, four in flight
def test_gradients_of_turned_operands(n):
    """dW = dZ^T H and dZ W against the fp64 oracle on the same bf16 operands.  An
    activation that rounds the other way is 2^-9 off, and few do: the bound is 1e-2
    of the gradient's norm."""
    N, T, ang, psi0 = _walk_params(n, n)
    b = qwalk.Batch(N, T, ang, psi0, prec=qwalk.QW_C64, nbins=512)  # (targets with no mass out of the walk's reach:
    b.run()                                                         # the loss is infinite there)
    y = b.binned().astype(np.float64)
    b.destroy()
    y /= y.sum(axis=1, keepdims=True)
    s = qwalk.Surrogate(seed=n)
    X = s.features(N, T, ang, psi0)
    _, g = s.loss_grad(X, y.astype(np.float32), T)
    p = S.unflatten(s.params(bf16_rounded=True).astype(np.float64))
    s.destroy()
    gr = S.backward(p, S.bf16_round(X), y, T, bf16=True)
    gg = S.unflatten(g.astype(np.float64))
    for k in S.ORDER:
        if k == "cb":
            continue
        assert np.linalg.norm(gg[k] - gr[k]) <= 1e-2 * np.linalg.norm(gr[k]), k
