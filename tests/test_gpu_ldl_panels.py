"""The Hessian factorisation's panels: one, two and an odd number of look-ahead
launches, badly scaled Hessians, and which pivot is reported when several fail
(the last one of the matrix: factorisation runs from the last pivot)."""
import numpy as np
import pytest

import oracle
from test_gpu_ldl import EPS, block_diag, factor, hessian, lib  # noqa: F401  (lib: fixture that loads the library)

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [128, 256, 640])
@pytest.mark.parametrize("spread", [0, 12])
def test_panels(K, spread):
    """Rows and columns scaled by powers of two up to 2^spread (exact, so that
    the factor's error scales with them): U = S U' S^-1, D = S D' S."""
    rng = np.random.default_rng(K + spread)
    H = hessian(rng, K)
    s = np.exp2(np.repeat(rng.integers(0, spread + 1, K // 4), 4)) if spread else np.ones(K)
    U, D, info = factor(H * s[:, None] * s[None, :])
    assert info == 0
    Uo, Do = oracle.ldl_blocks(H)
    ev = np.linalg.eigvalsh(H)
    tol = 100 * (ev[-1] / ev[0]) * EPS  # 100 cond(H) eps, as for the unscaled factor
    U, D = U * s[None, :] / s[:, None], D / (s[::4, None, None] ** 2)
    assert np.abs(U - Uo).max() <= tol * max(1.0, np.abs(Uo).max())
    assert np.abs(D - Do).max() <= tol * np.abs(Do).max()
    R = U @ block_diag(D) @ U.T
    assert np.abs(R - H).max() <= 1e-12 * np.abs(H).max()


@pytest.mark.parametrize("bad", [[2, 5], [0, 15], [3, 20], [16, 17, 31], [15, 16]])
@pytest.mark.parametrize("value", [-1.0, 0.0, float("nan")])
def test_several_bad_pivots(bad, value):
    K = 128
    H = np.eye(K)
    for j in bad:
        H[4 * j + 2, 4 * j + 2] = value
    _, D, info = factor(H)
    assert info == max(bad) + 1
    good = [j for j in range(K // 4) if j not in bad]
    if value < 0:  # block diagonal: the other pivots are untouched (a singular one spreads NaN upwards)
        assert np.array_equal(D[good], np.broadcast_to(np.eye(4), (len(good), 4, 4)))
