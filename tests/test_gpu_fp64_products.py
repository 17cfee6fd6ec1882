"""Double-precision products at the edges of their tiles (16 x 64 and 64 x 64)
and of the rule between them: one band, bands around 16 and 64, projector counts
that are no multiple of 64, plane-wave counts that end inside a K slice, blocks
smaller than the band count, complex and Gamma.

Tolerance.  Every output is at most three nested sums over the plane waves and
the projectors (6 000 terms at most) of products rounded to 2^-53; the worst
case of such sums, (terms) 2^-53 relative to the sum of magnitudes, is below
1e-12 here.
"""

import numpy as np
import pytest

import cellgen
import oracle
from oracle import gamma, overlap

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

TOL = 1e-12


def _cell(nat, proj, ecut, k_zero):
    a = (25.0 * nat) ** (1.0 / 3.0)
    frac = np.random.default_rng(99 + nat).uniform(0.0, 1.0, size=(nat, 3))
    return cellgen.make_cell("t", seed=7, lattice=np.diag([a, a, 1.1 * a]), frac=frac,
                             kfrac=(0.0, 0.0, 0.0) if k_zero else (0.25, 0.25, 0.25),
                             ecutwfc=ecut, ecutrho=4 * ecut, fft=None, proj=proj, dfixed=False,
                             nbnd=8, block=8, overlap=True)


@pytest.mark.parametrize("gamma_path", [False, True])
@pytest.mark.parametrize("nat,proj,ecut,nb,block", [
    (1, "sp", 8.0, 1, 1),            # 4 projectors, one band: flat tiles, one chunk
    (5, "s2pd", 9.0, 17, 17),        # one band past a flat tile, 60 projectors
    (17, "2s2p", 10.0, 64, 40),      # blocks of 40 (flat by padding) and 24
    (33, "2s2p", 8.0, 130, 65),      # a band past the 64-row tile
    (64, "2s2p", 36.0, 449, 449),    # 512 projectors: 64 x 64 tiles in both products
])
def test_nonlocal_and_overlap_vs_oracle(gamma_path, nat, proj, ecut, nb, block):
    import paper_2104_10502_amd as q
    c = _cell(nat, proj, ecut, gamma_path)
    cell = cellgen.gamma_half(c) if gamma_path else c
    psi = cellgen.make_psi0(cell.npw, nb, seed=5)
    if gamma_path:
        psi[:, 0] = psi[:, 0].real
        full = gamma.expand(psi)
        ref_nl, ref_h, ref_s = (gamma.restrict(f(c, full)) for f in
                                (oracle.vnl_psi, oracle.apply_h, overlap.apply_s))
    else:
        ref_nl, ref_h, ref_s = (f(c, psi) for f in
                                (oracle.vnl_psi, oracle.apply_h, overlap.apply_s))
    ctx = q.Context.from_cell(cell, precision=q.QEH_FP64, block=block)
    d = torch.from_numpy(psi).cuda()
    print(c.name, cell.npw, c.nkb, gamma_path, nb, block, flush=True)
    for got, ref in ((ctx.apply_h(d, part=1), ref_nl), (ctx.apply_h(d), ref_h),
                     (ctx.apply_s(d), ref_s)):
        g = got.cpu().numpy()
        err = np.linalg.norm(g - ref, axis=1) / np.linalg.norm(ref, axis=1)
        assert err.max() < TOL, err.max()
    ctx.close()


@pytest.mark.parametrize("nb,nvecx", [(2, 8), (9, 40)])
def test_subspace_products_of_a_few_bands(nb, nvecx):
    """Reductions and rotations of the iterative solver with few bands, the whole
    basis against itself included (the double-precision finish): their split sums
    stay inside their scratch and the eigenvalues are the dense matrix's."""
    import paper_2104_10502_amd as q
    cell = cellgen.make_cell("c1")
    want = np.linalg.eigvalsh(oracle.dense_h(cell))[:nb]
    ctx = q.Context.from_cell(cell, precision=q.QEH_MIXED, block=nb)
    c64 = q.Context.from_cell(cell, precision=q.QEH_FP64, block=nb)
    psi = torch.from_numpy(cellgen.make_psi0(cell.npw, nb, seed=5)).cuda()
    print(cell.npw, nb, nvecx, flush=True)
    eig, info = ctx.davidson(psi, nvecx=nvecx, rtol=1e-8, maxiter=400, refine=c64)
    assert info["refine_iters"] >= 1
    assert np.abs(eig - want).max() < 1e-6   # residuals <= 1e-5: errors are their squares / gaps
    ctx.close()
    c64.close()
