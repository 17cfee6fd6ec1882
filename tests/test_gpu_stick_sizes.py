"""Two-factor z transforms (K1, K3) against the oracle at compiled N3: the
smallest, odd and prime-power ones, unequal factors (125 = 25 x 5), the largest;
spheres that fill a quarter of a line at either end or less (half of the inputs),
and nearly all of it; fewer sticks than a workgroup takes and counts that leave
a partial one; k points whose l range is not centred; Gamma band pairs, whose
sticks go with their mirror images, with a lone last band; and the same bands
through the LDS passes.

Tolerance: a 3D transform pair of N points in FP64 keeps about 2 log2(N) eps
~ 1e-14, in single precision 2 log2(N) 2^-24 ~ 2.5e-6 of the local term; the
whole H is larger than it.
"""

import numpy as np
import pytest

import cellgen
import oracle
from oracle import gamma

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

SIZES = [(12, 15, 0.5), (15, 12, 0.5), (16, 24, 0.5), (21, 20, 0.9), (25, 12, 0.5), (27, 30, 0.5),
         (45, 12, 0.45), (50, 16, 0.95), (63, 12, 0.5), (72, 18, 0.5), (81, 12, 0.5),
         (105, 12, 0.5), (125, 12, 0.55), (128, 12, 0.9), (135, 12, 0.5), (168, 15, 0.5),
         (192, 12, 0.5)]
N2 = {12: 15, 15: 18, 16: 18, 18: 20, 20: 21, 24: 27, 30: 32}


def _err(a, b):
    return (np.linalg.norm(a - b, axis=1) / np.linalg.norm(b, axis=1)).max()


def _cell(n3, n, fill, gam, nbnd):
    # l fills the given part of N3, h and k about half of their box
    az = 0.5 * n3
    rz = (fill * n3 - 1) / 2 - 0.3
    a = az * (n / 4 - 0.6) / rz
    ecut = (2 * np.pi / az * rz) ** 2
    kpt = (0.0, 0.0, 0.0) if gam else np.array([0.3 / a, -0.2 / a, 0.45 / az]) * np.pi
    return cellgen.make_cell("t", seed=3, lattice=np.diag([a, a, az]),
                             frac=np.array([[0.1, 0.2, 0.3], [0.6, 0.5, 0.9]]), kpt=kpt,
                             ecutwfc=ecut, ecutrho=4 * ecut, fft=(n, N2[n], n3), proj="sp",
                             nobeta=True, nbnd=nbnd)


def _run(cell, psi, prec, block):
    import paper_2104_10502_amd as q
    ctx = q.Context.from_cell(cell, precision=prec, block=block)
    out = ctx.apply_h(torch.from_numpy(psi).cuda(), part=0).cpu().numpy()
    print(ctx.info(), flush=True)
    ctx.close()
    return out


def _case(n3, n, fill, gam, prec):
    c = _cell(n3, n, fill, gam, 3)
    cell = cellgen.gamma_half(c) if gam else c
    psi = cellgen.make_psi0(cell.npw, 3, seed=n3)
    if gam:
        psi[:, 0] = psi[:, 0].real
    return c, cell, psi


@pytest.mark.parametrize("n3,n,fill", SIZES)
@pytest.mark.parametrize("gam", [False, True])
@pytest.mark.parametrize("prec", [0, 1])
def test_stick_sizes_vs_oracle(n3, n, fill, gam, prec):
    c, cell, psi = _case(n3, n, fill, gam, prec)
    got = _run(cell, psi, prec, 3)
    full = gamma.expand(psi) if gam else psi
    ref = oracle.kinetic(c)[None] * full + oracle.vloc_psi(c, full)
    assert _err(got, gamma.restrict(ref) if gam else ref) < (1e-13 if prec == 0 else 2.5e-6)


@pytest.mark.parametrize("gam", [False, True])
def test_two_factor_matches_lds_passes(gam, monkeypatch):
    for n3, n, fill in ((20, 12, 0.5), (90, 18, 0.5), (120, 15, 0.9)):
        _, cell, psi = _case(n3, n, fill, gam, 0)
        monkeypatch.delenv("QEH_STICK_KERNEL", raising=False)
        x = [_run(cell, psi, p, 2) for p in (0, 1)]
        monkeypatch.setenv("QEH_STICK_KERNEL", "generic")
        y = [_run(cell, psi, p, 2) for p in (0, 1)]
        assert _err(x[0], y[0]) < 1e-13 and _err(x[1], y[1]) < 2.5e-6
