"""Single-precision projector products on split operands (three bf16 parts per
value) at the edges of their tiles: bands around 64 and 128, projector counts
that are no multiple of a tile, plane-wave counts that end inside a K slice of
16 or leave a chunk of its own, blocks smaller than the band count, and psi
read in double (the nonlocal part alone and the overlap) or from its
single-precision copy (the whole H).

Tolerance.  The parts carry every bit of the single-precision operands and the
products left out are below 2^-24 of the largest, so the error is the rounding
of the operands (2^-24 each) and of single-precision sums of at most a few
hundred steps per chunk: relative L2 below 40 * 2^-24 = 2.4e-6 per band.
"""

import numpy as np
import pytest

import cellgen
import oracle
from oracle import gamma, overlap

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

TOL = 40 * 2.0 ** -24


def _cell(nat, proj, ecut, k_zero):
    a = (25.0 * nat) ** (1.0 / 3.0)
    frac = np.random.default_rng(99 + nat).uniform(0.0, 1.0, size=(nat, 3))
    return cellgen.make_cell("t", seed=7, lattice=np.diag([a, a, 1.1 * a]), frac=frac,
                             kfrac=(0.0, 0.0, 0.0) if k_zero else (0.25, 0.25, 0.25),
                             ecutwfc=ecut, ecutrho=4 * ecut, fft=None, proj=proj, dfixed=False,
                             nbnd=8, block=8, overlap=True)


@pytest.mark.parametrize("gamma_path", [False, True])
@pytest.mark.parametrize("nat,proj,ecut,nb,block", [
    (1, "sp", 8.0, 1, 1),          # 4 projectors, one band, fewer plane waves than a chunk
    (5, "s2pd", 9.0, 65, 65),      # 60 projectors: under one tile; a band past the 64-row tile
    (17, "2s2p", 10.0, 64, 40),    # 136 projectors: past 128; blocks of 40 and 24
    (33, "2s2p", 8.0, 130, 129),   # 264 projectors; blocks of 129 and 1
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
    ctx = q.Context.from_cell(cell, precision=q.QEH_MIXED, block=block)
    d = torch.from_numpy(psi).cuda()
    print(c.name, cell.npw, c.nkb, gamma_path, nb, block, flush=True)
    for got, ref in ((ctx.apply_h(d, part=1), ref_nl), (ctx.apply_h(d), ref_h),
                     (ctx.apply_s(d), ref_s)):
        g = got.cpu().numpy()
        err = np.linalg.norm(g - ref, axis=1) / np.linalg.norm(ref, axis=1)
        assert err.max() < TOL, err.max()
    ctx.close()
