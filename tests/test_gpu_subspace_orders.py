"""The dense solver of the Rayleigh-Ritz step at the edges of its register,
LDS and workgroup shares: orders around 32, 48, 64, 80, 96, 112, 128 and 256 (where
the kernels change), one eigenpair and all of them, multiplets longer than a workgroup's
share of 16, off-diagonal elements whose squares underflow, and a matrix that
stops being positive definite at a given pivot.

Tolerance.  Cholesky, the reduction and the Sturm counts are backward stable:
eigenvalues to a few n 2^-53 ||H||, below 2e-13 at n = 257 with S of condition
two; vectors of separate eigenvalues are orthogonal to a few 2^-53 ||T|| over
their gap (above 1e-5 ||T||, closer ones being orthogonalised): 1e-10.
"""

import numpy as np
import pytest
import scipy.linalg as sla

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

ORDERS = [1, 2, 3, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64, 65, 66, 79, 80, 81, 96, 97, 112, 113,
          127, 128, 129, 130, 255, 256, 257]


def _random(rng, n):
    x = rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n))
    return x, x + x.conj().T


def _solve(h, s, nb):
    import paper_2104_10502_amd as q
    e, y = q.subspace_eigh(torch.from_numpy(h).cuda(), torch.from_numpy(s).cuda(), nb)
    return e.cpu().numpy(), y.cpu().numpy()


def _check(h, s, nb, label):
    print(label, len(h), nb, flush=True)
    e, y = _solve(h, s, nb)
    ref = sla.eigh(h, s, eigvals_only=True)
    norm = np.abs(ref).max()
    assert np.abs(e - ref[:nb]).max() < 1e-12 * norm
    assert np.linalg.norm(h @ y - s @ y * e, axis=0).max() < 1e-11 * norm
    assert np.abs(y.conj().T @ s @ y - np.eye(nb)).max() < 1e-10


@pytest.mark.parametrize("n", ORDERS)
def test_random_pencils(n):
    rng = np.random.default_rng(n)
    x, h = _random(rng, n)
    s = np.eye(n) + 0.2 * (x @ x.conj().T) / n
    for nb in sorted({1, (n + 1) // 2, n}):
        _check(h, s, nb, "random")


@pytest.mark.parametrize("n", [33, 64, 65, 128, 129, 256])
def test_long_multiplets(n):
    rng = np.random.default_rng(1000 + n)
    u = np.linalg.qr(_random(rng, n)[0])[0]
    w = np.repeat(np.arange(n // 20 + 1, dtype=float), 20)[:n] - 1.5
    h = (u * w) @ u.conj().T
    _check((h + h.conj().T) / 2, np.eye(n, dtype=np.complex128), n, "multiplets")


@pytest.mark.parametrize("n", [30, 64, 100, 128, 150])
def test_elements_whose_squares_underflow(n):
    rng = np.random.default_rng(2000 + n)
    _, h = _random(rng, n)
    h *= 1e-160
    h[np.diag_indices(n)] = np.sort(rng.standard_normal(n))
    _check(h, np.eye(n, dtype=np.complex128), n, "tiny off-diagonals")


@pytest.mark.parametrize("n,at", [(16, 0), (32, 31), (64, 33), (65, 64), (128, 64), (128, 127),
                                  (200, 70), (200, 199)])
def test_not_positive_definite(n, at):
    import paper_2104_10502_amd as q
    rng = np.random.default_rng(3000 + n)
    _, h = _random(rng, n)
    s = np.eye(n, dtype=np.complex128)
    s[at, at] = -1.0
    with pytest.raises(q.QehError):
        _solve(h, s, 1)
