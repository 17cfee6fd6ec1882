"""Two-factor plane pass against the oracle at compiled box sizes: the smallest
(both factors 2 to 4), odd and prime-power ones, unequal factors (14 = 7 x 2,
125 = 25 x 5), sizes with one and with several row chunks, one workgroup per CU
and more; spheres that fill half of a line or less (first passes over half of
the inputs) and boxes they almost fill (all inputs), k points whose stick ranges
are not centred, and Gamma band pairs with a lone last band.

Tolerance: a 3D transform pair of N^3 points in FP64 keeps about
2 log2(N^3) eps ~ 1e-14, in single precision 2 log2(N^3) 2^-24 ~ 2.5e-6 of the
local term; the whole H is larger than it.
"""

import numpy as np
import pytest

import cellgen
import oracle
from oracle import gamma

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _err(a, b):
    return (np.linalg.norm(a - b, axis=1) / np.linalg.norm(b, axis=1)).max()


def _run(cell, psi, prec, block):
    import paper_2104_10502_amd as q
    ctx = q.Context.from_cell(cell, precision=prec, block=block)
    out = ctx.apply_h(torch.from_numpy(psi).cuda(), part=0).cpu().numpy()
    info = ctx.info()
    ctx.close()
    return out, info


# (N, N3, extent of the sphere in h and k relative to N)
@pytest.mark.parametrize("n,n3,fill", [
    (12, 15, 0.5), (14, 12, 0.45), (15, 18, 0.5), (18, 27, 0.9), (21, 20, 0.5), (25, 24, 0.5),
    (27, 32, 0.95), (35, 24, 0.5), (45, 30, 0.5), (45, 30, 0.8), (54, 16, 0.5), (63, 12, 0.5),
    (75, 12, 0.5), (81, 12, 0.6), (84, 15, 0.5), (100, 12, 0.5), (125, 12, 0.5), (128, 12, 0.5),
    (135, 12, 0.5), (160, 12, 0.45),
])
@pytest.mark.parametrize("prec", [0, 1])
def test_plane_sizes_vs_oracle(n, n3, fill, prec):
    a, az = 0.5 * n, 0.5 * n3
    r = min((fill * n - 1) / 2, 0.95 * (n3 - 1) / 2 * a / az) - 0.3
    ecut = (2 * np.pi / a * r) ** 2
    c = cellgen.make_cell("t", seed=3, lattice=np.diag([a, a, az]),
                          frac=np.array([[0.1, 0.2, 0.3], [0.6, 0.5, 0.9]]),
                          kpt=np.array([0.9, -0.6, 0.2]) * np.pi / a * 0.5, ecutwfc=ecut,
                          ecutrho=4 * ecut, fft=(n, n, n3), proj="sp", nobeta=True, nbnd=3)
    psi = cellgen.make_psi0(c.npw, 3, seed=n)
    got, info = _run(c, psi, prec, 2)
    print(n, n3, prec, info, flush=True)
    ref = oracle.kinetic(c)[None] * psi + oracle.vloc_psi(c, psi)
    assert _err(got, ref) < (1e-13 if prec == 0 else 2.5e-6)


@pytest.mark.parametrize("n,n3", [(27, 25), (45, 24)])
@pytest.mark.parametrize("prec", [0, 1])
def test_plane_gamma_pairs_vs_oracle(n, n3, prec):
    a, az = 0.5 * n, 0.5 * n3
    ecut = (2 * np.pi / a * (min(n / 2, n3 / 2 * a / az) / 2 - 1)) ** 2
    c = cellgen.make_cell("t", seed=4, lattice=np.diag([a, a, az]),
                          frac=np.array([[0.1, 0.2, 0.3]]), kpt=(0.0, 0.0, 0.0), ecutwfc=ecut,
                          ecutrho=4 * ecut, fft=(n, n, n3), proj="sp", nobeta=True, nbnd=5)
    h = cellgen.gamma_half(c)
    psi = cellgen.make_psi0(h.npw, 5, seed=n)
    psi[:, 0] = psi[:, 0].real
    got, _ = _run(h, psi, prec, 5)
    full = gamma.expand(psi)
    ref = gamma.restrict(oracle.kinetic(c)[None] * full + oracle.vloc_psi(c, full))
    assert _err(got, ref) < (1e-13 if prec == 0 else 2.5e-6)


def test_two_factor_matches_lds_passes(monkeypatch):
    # the same bands through the LDS-pass kernel of the generic path
    for n in (36, 90, 120):
        a = 0.45 * n
        ecut = (2 * np.pi / a * (n / 4 - 1)) ** 2
        c = cellgen.make_cell("t", seed=5, lattice=np.diag([a, a, 6.0]),
                              frac=np.array([[0.4, 0.2, 0.7]]), kpt=(0.0, 0.0, 0.0), ecutwfc=ecut,
                              ecutrho=4 * ecut, fft=(n, n, 32), proj="sp", nobeta=True, nbnd=2)
        psi = cellgen.make_psi0(c.npw, 2, seed=n)
        monkeypatch.delenv("QEH_PLANE_KERNEL", raising=False)
        x = [_run(c, psi, p, 2)[0] for p in (0, 1)]
        monkeypatch.setenv("QEH_PLANE_KERNEL", "generic")
        y = [_run(c, psi, p, 2)[0] for p in (0, 1)]
        assert _err(x[0], y[0]) < 1e-13 and _err(x[1], y[1]) < 2.5e-6
