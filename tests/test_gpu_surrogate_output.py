"""What surr_predict does with the caller's memory."""
import numpy as np
import pytest

from paper_1003_3779_amd import inputs, qwalk

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bad", ["angles", "psi0"])
def test_a_failed_prediction_leaves_its_output_alone(bad):
    """Every walk is re-checked, and the plain walk refuses one of them (a coin angle that is
    not finite, a start state of norm 2): the device output keeps what it held."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    rng = np.random.default_rng(1)
    n = 300
    ang, psi0 = inputs.su2_angles(rng, n), np.stack([inputs.haar_state(rng, 2) for _ in range(n)])
    if bad == "angles":
        ang[77, 1] = np.inf
    else:
        psi0[77] *= 2.0
    out = torch.full((n, 512), -3.0, dtype=torch.float32, device="cuda")
    s = qwalk.Surrogate(seed=2)
    with pytest.raises(qwalk.QWError):
        s.predict(np.full(n, 4097), rng.integers(256, 2049, n), ang, psi0, recheck_frac=1.0, out=out)
    torch.cuda.synchronize()
    assert bool((out == -3.0).all())
    # the same handle answers the next call
    ang[77], psi0[77] = ang[76], psi0[76]
    got, _, _ = s.predict(np.full(n, 4097), rng.integers(256, 2049, n), ang, psi0, recheck_frac=0.01, tvd_tol=1.0, out=out)
    torch.cuda.synchronize()
    assert bool((out >= 0.0).all()) and float(out.sum()) > 0.0
    s.destroy()
