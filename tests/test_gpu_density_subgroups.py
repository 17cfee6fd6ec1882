"""The reduction of the charge density over many subgroups of bands: whole groups of
eight, remainders and fewer than eight, against the oracle; the same bands in one
block and in several.

Tolerance: FP64 sums of some hundred bands 1e-12 of the largest value; single
precision as for the fused pass, 5e-6.
"""

import numpy as np
import pytest

import cellgen
import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("nb,block", [(5, 5), (29, 29), (32, 32), (66, 66), (131, 131), (131, 37)])
@pytest.mark.parametrize("prec", [0, 1])
def test_many_subgroups(nb, block, prec):
    import paper_2104_10502_amd as q
    n, n3 = 16, 12
    a = 0.5 * n
    ecut = (2 * np.pi / a * 3.4) ** 2
    c = cellgen.make_cell("t", seed=3, lattice=np.diag([a, a, 0.5 * n3]),
                          frac=np.array([[0.1, 0.2, 0.3]]), kpt=(0.1, 0.0, 0.05), ecutwfc=ecut,
                          ecutrho=4 * ecut, fft=(n, n, n3), proj="sp", nobeta=True, nbnd=nb)
    psi = cellgen.make_psi0(c.npw, nb, seed=nb)
    occ = np.linspace(2.0, 0.1, nb)
    ctx = q.Context.from_cell(c, precision=prec, block=block)
    i = ctx.info()
    print(nb, block, prec, -(-block // i["density_bands"]), flush=True)
    assert i["density_kernel"] == 2
    got = ctx.density(torch.from_numpy(psi).cuda(), occ).cpu().numpy()
    ctx.close()
    ref = oracle.density(c, psi, occ)
    assert np.abs(got - ref).max() < (1e-12 if prec == 0 else 5e-6) * np.abs(ref).max()
