"""The fused charge density pass against the oracle at plane sizes with one, two,
three and four row chunks, odd and prime-power ones and unequal factors, one and
two workgroups' worth of LDS; spheres that fill half of a line (half of the
inputs) and most of it; band counts that leave a ragged subgroup; Gamma bands
paired by occupation; and the unfused rows of the same bands.

Tolerance: relative to the largest density value, FP64 sums of a few dozen
bands 1e-12; single-precision transforms keep 2 log2(N^3) 2^-24 per amplitude,
twice that per square, 5e-6.
"""

import numpy as np
import pytest

import cellgen
import oracle
from oracle import gamma

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# (N, N3, extent relative to N)
SIZES = [(12, 15, 0.5), (15, 12, 0.5), (14, 12, 0.9), (27, 24, 0.9), (35, 12, 0.5), (45, 16, 0.5),
         (64, 12, 0.5), (72, 12, 0.5), (75, 12, 0.5), (80, 12, 0.5), (96, 12, 0.5), (100, 12, 0.5),
         (112, 12, 0.5), (120, 12, 0.5), (128, 12, 0.5), (150, 12, 0.45), (160, 12, 0.45)]


def _cell(n, n3, fill, gam):
    a, az = 0.5 * n, 0.5 * n3
    r = min((fill * n - 1) / 2, 0.95 * (n3 - 1) / 2 * a / az) - 0.3
    ecut = (2 * np.pi / a * r) ** 2
    kpt = (0.0, 0.0, 0.0) if gam else np.array([0.9, -0.6, 0.2]) * np.pi / a * 0.5
    return cellgen.make_cell("t", seed=3, lattice=np.diag([a, a, az]),
                             frac=np.array([[0.1, 0.2, 0.3]]), kpt=kpt, ecutwfc=ecut,
                             ecutrho=4 * ecut, fft=(n, n, n3), proj="sp", nobeta=True, nbnd=7)


def _rho(cell, psi, occ, prec, block):
    import paper_2104_10502_amd as q
    ctx = q.Context.from_cell(cell, precision=prec, block=block)
    out = ctx.density(torch.from_numpy(psi).cuda(), occ).cpu().numpy()
    print(ctx.info(), flush=True)
    ctx.close()
    return out


def _close(got, ref, prec):
    err = np.abs(got - ref).max() / np.abs(ref).max()
    assert err < (1e-12 if prec == 0 else 5e-6), err


@pytest.mark.parametrize("n,n3,fill", SIZES)
@pytest.mark.parametrize("prec", [0, 1])
def test_density_sizes_vs_oracle(n, n3, fill, prec, monkeypatch):
    c = _cell(n, n3, fill, False)
    psi = cellgen.make_psi0(c.npw, 7, seed=n)
    occ = np.linspace(2.0, 0.3, 7)
    ref = oracle.density(c, psi, occ)
    _close(_rho(c, psi, occ, prec, 7), ref, prec)
    monkeypatch.setenv("QEH_DENSITY_KERNEL", "generic")
    _close(_rho(c, psi, occ, prec, 7), ref, prec)


@pytest.mark.parametrize("n,n3", [(18, 20), (45, 12), (81, 12)])
@pytest.mark.parametrize("prec", [0, 1])
def test_density_sizes_gamma(n, n3, prec):
    c = _cell(n, n3, 0.5, True)
    h = cellgen.gamma_half(c)
    psi = cellgen.make_psi0(h.npw, 21, seed=n)
    psi[:, 0] = psi[:, 0].real
    occ = np.repeat([2.0, 1.0, 0.5], 7)   # pairs inside, lone bands at the steps
    _close(_rho(h, psi, occ, prec, 8), oracle.density(c, gamma.expand(psi), occ), prec)
