"""The plane pass of spheres that fill a box beyond half of a line, on either side
of the extents at which the columns' LDS leaves room for few rows: which kernel
runs (2 two-factor, 3 with unpadded columns, 0 and 1 the LDS passes and the split
kernels), its result against the oracle, and the density of such a context.

Tolerance: as for all sizes of the plane pass, 2 log2(N^3) roundings: 1e-13 in FP64,
2.5e-6 in single precision; densities twice the latter.
"""

import numpy as np
import pytest

import cellgen
import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _cell(n, ext, n3=12):
    # ext columns: the sphere's radius in units of the x reciprocal step, centred or half off
    odd = ext % 2
    r = (ext - 1) / 2 + 0.3 if odd else ext / 2 - 0.2
    a = 0.5 * n
    az = a * (n3 / 2 - 1.2) / r
    ecut = (2 * np.pi / a * r) ** 2
    kpt = np.array([0.0 if odd else np.pi / a, 0.0, 0.0])
    c = cellgen.make_cell("t", seed=3, lattice=np.diag([a, a, az]),
                          frac=np.array([[0.1, 0.2, 0.3], [0.6, 0.5, 0.9]]), kpt=kpt, ecutwfc=ecut,
                          ecutrho=4 * ecut, fft=(n, n, n3), proj="sp", nobeta=True, nbnd=3)
    assert c.miller[:, 0].max() - c.miller[:, 0].min() + 1 == ext
    return c


# (precision, N, columns, kernel; None: either of the others)
CASES = [(1, 140, 130, 2), (1, 140, 131, 3), (1, 140, 140, 3), (1, 144, 128, 2), (1, 144, 129, 3),
         (1, 144, 136, 3), (1, 144, 140, 3), (1, 144, 141, None), (1, 150, 134, 3),
         (1, 150, 135, None), (1, 160, 110, 2), (1, 160, 111, 3), (1, 160, 116, 3),
         (1, 160, 123, 3), (1, 160, 124, 3), (1, 160, 125, None), (1, 168, 117, 3),
         (1, 168, 118, None), (1, 180, 99, 3), (1, 180, 109, 3), (1, 180, 110, None), (1, 192, 90, 2), (1, 192, 91, 3),
         (1, 192, 97, 3), (1, 192, 102, 3), (1, 192, 103, None),
         (0, 112, 79, 2), (0, 112, 80, None), (0, 125, 78, 2), (0, 125, 79, None), (0, 128, 68, 2),
         (0, 128, 69, None), (0, 135, 73, 2), (0, 135, 74, None), (0, 144, 63, 2),
         (0, 144, 64, None), (0, 160, 55, 2), (0, 160, 56, None), (0, 192, 46, 2),
         (0, 192, 47, None)]


@pytest.mark.parametrize("prec,n,ext,kernel", CASES)
def test_wide_spheres(prec, n, ext, kernel):
    import paper_2104_10502_amd as q
    c = _cell(n, ext)
    psi = cellgen.make_psi0(c.npw, 3, seed=n)
    ctx = q.Context.from_cell(c, precision=prec, block=2)
    info = ctx.info()
    print(prec, n, ext, info["plane_kernel"], flush=True)
    assert info["ext"] == ext
    assert info["plane_kernel"] == kernel if kernel else info["plane_kernel"] in (0, 1)
    got = ctx.apply_h(torch.from_numpy(psi).cuda(), part=0).cpu().numpy()
    ctx.close()
    ref = oracle.kinetic(c)[None] * psi + oracle.vloc_psi(c, psi)
    err = (np.linalg.norm(got - ref, axis=1) / np.linalg.norm(ref, axis=1)).max()
    assert err < (1e-13 if prec == 0 else 2.5e-6)


@pytest.mark.parametrize("n,ext", [(144, 133), (160, 119)])
def test_density_of_unpadded_columns(n, ext):
    import paper_2104_10502_amd as q
    c = _cell(n, ext)
    psi = cellgen.make_psi0(c.npw, 5, seed=n)
    occ = np.linspace(2.0, 0.5, 5)
    ctx = q.Context.from_cell(c, precision=1, block=4)
    info = ctx.info()
    assert info["plane_kernel"] == 3 and info["density_kernel"] != 2
    got = ctx.density(torch.from_numpy(psi).cuda(), occ).cpu().numpy()
    ctx.close()
    ref = oracle.density(c, psi, occ)
    assert np.abs(got - ref).max() < 5e-6 * np.abs(ref).max()
