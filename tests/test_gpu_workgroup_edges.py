"""Local part of H where the workgroups of the two-factor passes end raggedly: band
counts on both sides of the eight-way remapping of (plane, band) to workgroups, with
odd numbers of planes; planes in one and in several row chunks; sphere sticks that
fill the last stick group to one stick, to all but one and exactly.

A band's result is the oracle's (tolerance of the transforms: 1e-13 in FP64, 2.5e-6 in
single precision) and the same bits whatever the number of bands.
"""

import numpy as np
import pytest

import cellgen
import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _cell(n, n3, r):
    a = 0.5 * n
    az = a * (n3 / 2 - 1.2) / r
    ecut = (2 * np.pi / a * r) ** 2
    return cellgen.make_cell("t", seed=3, lattice=np.diag([a, a, az]),
                             frac=np.array([[0.1, 0.2, 0.3], [0.6, 0.5, 0.9]]),
                             kpt=np.array([0.3, -0.2, 0.1]) * np.pi / a, ecutwfc=ecut,
                             ecutrho=4 * ecut, fft=(n, n, n3), proj="sp", nobeta=True, nbnd=3)


# box, and radii of the sphere in units of the x reciprocal step
@pytest.mark.parametrize("n,n3,radii", [(36, 15, (3.15, 3.2)), (90, 21, (4.0, 4.4)),
                                        (120, 15, (3.15, 3.2))])
@pytest.mark.parametrize("prec", [0, 1])
def test_band_counts_and_stick_groups(n, n3, radii, prec):
    import paper_2104_10502_amd as q
    group = 16 if prec == 0 else 32
    left = set()
    for r in radii:
        c = _cell(n, n3, r)
        psi = cellgen.make_psi0(c.npw, 17, seed=n)
        ref = oracle.kinetic(c)[None] * psi + oracle.vloc_psi(c, psi)
        ctx = q.Context.from_cell(c, precision=prec, block=17)
        info = ctx.info()
        left.add(info["nst"] % group)
        print(n, n3, prec, info["nst"], info["ext"], flush=True)
        assert info["plane_kernel"] == 2 and info["stick_kernel"] == 1
        p = torch.from_numpy(psi).cuda()
        full = ctx.apply_h(p, part=0)
        err = np.linalg.norm(full.cpu().numpy() - ref, axis=1) / np.linalg.norm(ref, axis=1)
        assert err.max() < (1e-13 if prec == 0 else 2.5e-6)
        for nb in (1, 3, 7, 8, 9, 16):
            assert torch.equal(ctx.apply_h(p[:nb], part=0), full[:nb]), (r, nb)
        ctx.close()
    assert len(left) == len(radii)
