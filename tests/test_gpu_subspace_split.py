"""The dense solver where its tridiagonal matrix falls into blocks: diagonal
matrices with exactly representable entries (trial points of the eigenvalue
search meet them), in orders that mix small and large, multiplets spread over
blocks, and matrices scaled until their squares leave the exponent range.

Tolerance.  With S = 1 a diagonal H passes the Cholesky factorisation, the
solves and the reduction unchanged, and the eigenvalue of a 1 x 1 block is its
entry, so eigenvalues are equal and vectors are unit vectors.  In general an
eigenvalue is the middle of a bracket at most eps ||T|| / 2 wide and the
reduction is backward stable to a few n 2^-53 ||H||: 1e-12 at these orders.
"""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _solve(h, nb):
    import paper_2104_10502_amd as q
    s = np.eye(len(h), dtype=np.complex128)
    e, y = q.subspace_eigh(torch.from_numpy(np.ascontiguousarray(h)).cuda(),
                           torch.from_numpy(s).cuda(), nb)
    return e.cpu().numpy(), y.cpu().numpy()


def _check_diagonal(d, nb):
    print(len(d), nb, flush=True)
    e, y = _solve(np.diag(d).astype(np.complex128), nb)
    ref = np.sort(d)[:nb]
    assert np.array_equal(e, ref)
    assert np.abs(d[:, None] * y - y * ref).max() == 0.0
    assert np.abs(y.conj().T @ y - np.eye(nb)).max() < 1e-15


@pytest.mark.parametrize("m,n,nb", [(61, 258, 122), (65, 258, 122), (67, 258, 122), (127, 258, 122),
                                    (121, 515, 242), (122, 515, 242), (123, 515, 242),
                                    (124, 515, 242)])
def test_diagonal_progressions(m, n, nb):
    _check_diagonal((m * np.arange(n)) % n * 1.0, nb)


@pytest.mark.parametrize("n", [130, 200, 257, 258, 320, 400, 515])
def test_shuffled_integers(n):
    rng = np.random.default_rng(n)
    for nb in (1, n // 3, n // 2, n):
        _check_diagonal(rng.permutation(n) * 1.0, nb)


@pytest.mark.parametrize("n", [20, 128, 300])
def test_repeated_entries(n):
    rng = np.random.default_rng(n)
    d = rng.integers(-3, 4, size=n) * 0.5
    _check_diagonal(d, n)
    # the wanted ones end inside a multiplet; entries far below the largest
    _check_diagonal(np.where(rng.random(n) < 0.5, d, d * 2.0 ** -960), n // 2)


@pytest.mark.parametrize("n", [1, 16, 100, 200])
def test_zero_matrix(n):
    _check_diagonal(np.zeros(n), n)


@pytest.mark.parametrize("n", [24, 100, 128, 200])
@pytest.mark.parametrize("scale", [-520, -700, 500])
def test_scaled_matrices(n, scale):
    # H of about 2^scale: the squares of T's elements under- or overflow
    rng = np.random.default_rng(n)
    x = rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n))
    h = x + x.conj().T
    print(n, scale, flush=True)
    e, y = _solve(h * 2.0 ** scale, n // 2)
    e = np.ldexp(e, -scale)
    ref = np.linalg.eigvalsh(h)
    norm = np.abs(ref).max()
    assert np.abs(e - ref[:n // 2]).max() < 1e-12 * norm
    assert np.linalg.norm(h @ y - y * e, axis=0).max() < 1e-11 * norm
    assert np.abs(y.conj().T @ y - np.eye(n // 2)).max() < 1e-10


@pytest.mark.parametrize("n,size", [(96, 3), (200, 5), (513, 27)])
def test_equal_blocks(n, size):
    # blocks of the same eigenvalues: multiplets whose members lie in different blocks
    rng = np.random.default_rng(n)
    x = rng.standard_normal((size, size)) + 1j * rng.standard_normal((size, size))
    b = x + x.conj().T
    h = np.zeros((n, n), dtype=np.complex128)
    for i in range(0, n, size):
        m = min(size, n - i)
        h[i:i + m, i:i + m] = b[:m, :m]
    print(n, size, flush=True)
    for nb in (n // 2, n):
        e, y = _solve(h, nb)
        ref = np.linalg.eigvalsh(h)
        norm = np.abs(ref).max()
        assert np.abs(e - ref[:nb]).max() < 1e-12 * norm
        assert np.linalg.norm(h @ y - y * e, axis=0).max() < 1e-11 * norm
        assert np.abs(y.conj().T @ y - np.eye(nb)).max() < 1e-10
