"""H psi and S psi do not depend on how the bands are grouped into calls, bit for
bit, on contexts whose whole block and whose single bands differ in the size class
of the FP64 products (64 atoms: 128 x 512 x 23 976 against 1 x 512 x 23 976), with
blocks that leave a ragged tail, and where the whole block is small.  On Gamma
contexts bands share a transform in consecutive pairs: groups of whole pairs.
A Davidson served by reverse communication a few bands at a time is qeh_davidson's.
"""

import numpy as np
import pytest

import cellgen

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _ctx(cell, prec, block):
    import paper_2104_10502_amd as q
    return q.Context.from_cell(cell, precision=prec, block=block,
                               projgen=cellgen.projgen_tables(cell))


def _groups(ctx, psi, sizes, what):
    out = torch.empty_like(psi)
    b = 0
    while b < psi.shape[0]:
        for n in sizes:
            n = min(n, psi.shape[0] - b)
            if n > 0:
                out[b:b + n] = getattr(ctx, what)(psi[b:b + n].contiguous())
            b += n
    return out


def _cell(nat, edge, ecut, gamma=False):
    rng = np.random.default_rng(nat)
    k = (0.0, 0.0, 0.0) if gamma else np.array([.25, .25, .25]) * 2 * np.pi / edge
    c = cellgen.make_cell("t", seed=5, lattice=np.eye(3) * edge, frac=rng.random((nat, 3)), kpt=k,
                          ecutwfc=ecut, proj="2s2p", nbnd=4, with_beta=False, overlap=True)
    return cellgen.gamma_half(c) if gamma else c


# (atoms, edge, cutoff, block, bands): products in three-product 64 x 64 tiles for the
# block; a block of one flat tile row past 64; all flat
@pytest.mark.parametrize("nat,edge,ecut,block,nb", [(64, 20.52, 30.0, 128, 150),
                                                    (48, 18.0, 25.0, 77, 90),
                                                    (8, 10.0, 20.0, 16, 21)])
@pytest.mark.parametrize("prec", [0, 1])
def test_groups_of_bands_bitwise(nat, edge, ecut, block, nb, prec):
    c = _cell(nat, edge, ecut)
    ctx = _ctx(c, prec, block)
    print(nat, block, nb, prec, ctx.info(), flush=True)
    psi = torch.from_numpy(cellgen.make_psi0(c.npw, nb, seed=nat)).cuda()
    for what in ("apply_h", "apply_s"):
        ref = getattr(ctx, what)(psi)
        for sizes in ((1,), (block // 2, 3), (17, 64, 16)):
            assert torch.equal(_groups(ctx, psi, sizes, what), ref), (what, sizes)
    ctx.close()


@pytest.mark.parametrize("prec", [0, 1])
def test_groups_of_gamma_pairs_bitwise(prec):
    c = _cell(64, 20.52, 30.0, gamma=True)
    ctx = _ctx(c, prec, 128)
    psi = torch.from_numpy(cellgen.make_psi0(c.npw, 130, seed=2)).cuda()
    for what in ("apply_h", "apply_s"):
        ref = getattr(ctx, what)(psi)
        for sizes in ((2,), (64, 6)):
            assert torch.equal(_groups(ctx, psi, sizes, what), ref), (what, sizes)
    ctx.close()


def test_reverse_communication_in_groups_is_davidson():
    c = _cell(64, 20.52, 30.0)
    c.qmat = None
    ctx = _ctx(c, 0, 128)
    p = torch.from_numpy(cellgen.make_psi0(c.npw, 128, seed=3)).cuda()
    a, b = p.clone(), p.clone()
    eig, info = ctx.davidson(a, rtol=1e-6, maxiter=4, allow_notconv=True)

    def apply(x, y):
        for i in range(0, x.shape[0], 50):
            ctx.apply_h(x[i:i + 50], out=y[i:i + 50])

    eig_r, info_r = ctx.davidson_rci(b, apply, rtol=1e-6, maxiter=4, allow_notconv=True)
    print(info["iters"], info["status"], info_r["status"], flush=True)
    assert np.array_equal(eig, eig_r) and torch.equal(a, b)
    ctx.close()
