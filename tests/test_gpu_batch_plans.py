"""Batches whose plan changes after create, or that are larger than one launch or the
card's memory takes: the same results, and what was accepted stays accepted."""
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


def _walks(seed, N, T):
    rng = np.random.default_rng(seed)
    N, T = np.array(N, dtype=np.int64), np.array(T, dtype=np.int64)
    return N, T, inputs.su2_angles(rng, N.size), np.stack([inputs.haar_state(rng, 2) for _ in range(N.size)])


@pytest.mark.parametrize("prec", [qwalk.QW_C64, qwalk.QW_C128])
@pytest.mark.parametrize("variant", [1, 3, 6])
def test_tuning_a_forced_variant(prec, variant, tmp_path, monkeypatch):
    """A batch created with tiles the slim kernel does not run may be tuned into those
    it does (128 slots): its slot buffers are there by the next run."""
    monkeypatch.setenv("QWALK_TUNE_CACHE", str(tmp_path / "tune.txt"))
    walks = _walks(variant, [2049, 4097, 4097, 5001, 9999, 9999, 12001], [1000, 2048, 300, 0, 4000, 17, 2500])
    b = qwalk.Batch(*walks, prec=prec, nbins=64, tiled_variant=variant, renorm_every=-1)
    b.run()
    before = b.binned(), b.moments()
    b.tune(samples=7, save=False)
    b.run()
    assert np.array_equal(b.binned(), before[0])
    assert np.array_equal(b.moments(), before[1])
    b.destroy()
