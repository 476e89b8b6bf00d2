"""Batched rings on their live points (in registers, or a block of steps per launch
for all long walks together) against the queue's tiled kernels (a forced variant) and
the oracle.

The amplitudes are the same expressions, so P and the bins (exact integer sums of P
rounded once) agree bit for bit; moments sum the same P in another order, at most T + 1
terms of one sign: T 2^-53 relative to the sum of |terms|.
"""
import numpy as np
import pytest

import oracle
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


def _walks(seed, T, N):
    rng = np.random.default_rng(seed)
    T = np.array(T, dtype=np.int64)
    N = np.maximum(N, 2 * T + 1).astype(np.int64)
    ang = inputs.su2_angles(rng, T.size)
    ang[:2, 0] = (0.3, 1.3)     # both factorings of the rotation
    psi0 = np.stack([inputs.haar_state(rng, 2) for _ in range(T.size)])
    x0 = rng.integers(0, N)
    return N, T, ang, psi0, x0


def _compare(walks, prec, variant, nbins, keep, **opts):
    N, T, ang, psi0, x0 = walks
    res = []
    for v in (0, variant):
        b = qwalk.Batch(N, T, ang, psi0, x0, prec=prec, nbins=nbins, keep_probabilities=keep, tiled_variant=v, **opts)
        b.run()
        b.run()
        res.append((b.moments(), b.binned() if nbins else None, b.probabilities() if keep else None))
        b.destroy()
    if nbins:
        assert np.array_equal(res[0][1], res[1][1])
    if keep:
        for p, q in zip(res[0][2], res[1][2]):
            assert np.array_equal(p, q)
    size = np.stack([np.ones(T.size), np.maximum(T, 1.0), np.maximum(T, 1.0) ** 2], 1)
    assert np.all(np.abs(res[0][0] - res[1][0]) <= (T[:, None] + 1) * 2.0 ** -52 * size)
    return res[0]


# steps around the block depths and where a lane takes more points, up to the most held in registers
EDGES = [1, 2, 15, 16, 17, 31, 32, 33, 64, 127, 128, 129, 255, 256, 383, 384, 511, 512, 703, 704, 895, 896, 1087, 1088, 1343,
         1344, 1599, 1600, 1855, 1856, 2048, 2110, 2111]


@pytest.mark.parametrize("prec", [qwalk.QW_C64, qwalk.QW_C128])
@pytest.mark.parametrize("nmin,variant", [(4097, 8), (10001, 4)])
@pytest.mark.parametrize("opts", [{}, {"renorm_every": 1}, {"renorm_every": -1}])
def test_short_walks_in_registers(prec, nmin, variant, opts):
    for nbins in (512, 6):
        _compare(_walks(nmin + prec, EDGES, nmin), prec, variant, nbins, False, **opts)


@pytest.mark.parametrize("prec", [qwalk.QW_C64, qwalk.QW_C128])
@pytest.mark.parametrize("nmin,variant,T", [
    (4226, 8, [2112, 2113, 2144, 2500, 4000, 4999]),
    (10001, 4, [2112, 2175, 2176, 2177, 3000, 5001, 12345, 30000]),
])
@pytest.mark.parametrize("keep", [False, True])
def test_long_walks_together(prec, nmin, variant, T, keep):
    _compare(_walks(nmin + prec, T, nmin), prec, variant, 512, keep, renorm_every=1 if prec == qwalk.QW_C128 else 0)


def test_many_long_walks_use_every_tile_size():
    """Enough walks that a block's tiles are large early, fewer and smaller late; short
    walks, wrapping ones and every P kept share the batch."""
    rng = np.random.default_rng(3)
    T = np.concatenate([rng.integers(2112, 4000, 400), [9000, 20000], rng.integers(1, 2112, 40)])
    N, T, ang, psi0, x0 = _walks(11, T, 10001)
    N[-3:] = 2 * T[-3:] - 1     # cones that wrap: the queue's kernel
    _compare((N, T, ang, psi0, x0), qwalk.QW_C64, 4, 512, False)


def test_against_oracle():
    N, T, ang, psi0, x0 = _walks(5, [700, 2050, 3000], 6101)
    for prec, tol in ((qwalk.QW_C128, 1e-12), (qwalk.QW_C64, 2e-5)):
        b = qwalk.Batch(N, T, ang, psi0, x0, prec=prec, nbins=64)
        b.run()
        bins = b.binned()
        b.destroy()
        for i in range(3):
            C = oracle.coin(oracle.SU2, 2, *ang[i])
            ref = oracle.prob(oracle.walk(int(N[i]), 1, inputs.RING, C, (int(x0[i]), 0), psi0[i], int(T[i])))[0]
            assert np.max(np.abs(bins[i] - oracle.bin_ring(ref, x0[i], 64))) <= tol + 1e-6


@pytest.mark.parametrize("prec", [qwalk.QW_C128, qwalk.QW_C64])
@pytest.mark.parametrize("N", [1, 2, 513, 1024, 1025, 2047, 2048])
@pytest.mark.parametrize("p,walls", [(0.3, True), (0.3, False), (1.0, False), (0.0, True)])
def test_links_of_a_batch_are_the_single_walks(prec, N, p, walls):
    """A batched walk with broken links against the single walk of the same realization
    (another kernel, the same draws and expressions): the same P to the rounding of its
    two-term sum."""
    T = min(90, 2 * N)
    psi0 = inputs.haar_state(np.random.default_rng(N), 2)
    x0 = N // 3
    b = qwalk.Batch([N, N], [T, T], [[0.7, 0.4, 1.1]] * 2, [psi0] * 2, [x0] * 2, prec=prec, keep_probabilities=True,
                    renorm_every=-1, walls=walls, link_p=p, link_seed=9 << 33, realization0=5)
    b.run()
    P = b.probabilities()[1]
    b.destroy()
    w = qwalk.Walk((N,), inputs.RING, qwalk.SU2, psi0, (x0, 0), prec=prec, theta=0.7, phi=0.4, chi=1.1)
    w.set_options(renorm_every=0)
    w.set_broken_links(p, seed=9 << 33, realization=6)
    w.set_reflecting_walls(walls)
    w.step(T)
    ref = w.probabilities()[0]
    w.destroy()
    # complex64: the single walk's coin is rounded once from the same fp64 entries
    assert np.max(np.abs(P - ref)) <= (4 * 2.0 ** -53 if prec == qwalk.QW_C128 else 4 * T * 2.0 ** -24)
