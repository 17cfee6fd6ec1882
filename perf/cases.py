"""Timed workloads of the plane-wave H|psi> library: what its users have it do.

A case is a dict of plain values (see ``listed``); ``prepare`` builds what a
program holds before the call (the cell, its context on the device, start
vectors, workspaces), ``run`` makes one pass through the public entry points of
``paper_2104_10502_amd``, ``exact`` computes the same in plain 64-bit torch, and
``work`` counts the bytes and operations a pass cannot do without.

Cells come from ``cellgen`` (the seeded generator shared by the tests and the
benchmark): its named cells with jittered sites, or random cells of any size,
cutoff, shape and projector set.  Start vectors have the spread of a plane-wave
code's starting wavefunctions: random amplitudes and phases damped as
1 / (1 + |k+G|^2), normalised band by band.

The mixed form works in single precision inside (transforms, local potential,
projector products) and returns H psi in the library's complex128 layout.  The
programs here that use it keep the result in complex64, which is all that form
computes; those that use the FP64 form keep complex128.
"""

from __future__ import annotations

import functools
import math
import time

import numpy as np
import torch

import cellgen
import cellgen.cells

#: sites of the named cells: (lattice edges, sites, box or None, k in 2 pi / a, cutoff, projectors)
_NAMED = {
    "two_atoms": ((10.0, 10.0, 10.0), "bcc", (30, 30, 30), (0.0, 0.0, 0.0), 20.0, "sp"),
    "diamond64": ((20.52, 20.52, 20.52), "diamond2", (72, 72, 72), (.25, .25, .25), 30.0, "2s2p"),
    "fcc256": ((32.6, 32.6, 32.6), "fcc4", (135, 135, 135), (0.0, 0.0, 0.0), 40.0, "2s2p"),
    "diamond512": ((40.0, 40.0, 42.0), "diamond4", (160, 160, 168), (0.0, 0.0, 0.0), 30.0, "s2pd"),
}
_KFRAC = ((.25, .25, .25), (.25, .25, -.25), (.25, -.25, .25), (-.25, .25, .25))


def listed():
    return [
        # the smallest call: a two-atom cell's 16 bands, where latency and launches count
        dict(name="hpsi_2atom_fp64", kind="hpsi", cell="two_atoms", precision="fp64", nb=16,
             block=16),
        # one k-point of an ordinary request of the served stream (odd 45^3 box, ragged 202 bands)
        dict(name="hpsi_101atom_odd_mixed", kind="hpsi", cell="random", nat=101, vol=20.0,
             ecut=30.0, aspect=1.0, proj="sp", k=1, precision="mixed", nb=202, block=202),
        # the 64-atom supercell at a general k, both precisions: the ordinary SCF cell
        dict(name="hpsi_64atom_mixed", kind="hpsi", cell="diamond64", precision="mixed", nb=128,
             block=128),
        dict(name="hpsi_64atom_fp64", kind="hpsi", cell="diamond64", precision="fp64", nb=128,
             block=128),
        # the 256-atom cell at Gamma on its odd 135^3 box, in launches of 64 bands
        dict(name="hpsi_256atom_gamma_mixed", kind="hpsi", cell="fcc256", gamma=True,
             precision="mixed", nb=256, block=64),
        dict(name="hpsi_256atom_gamma_fp64", kind="hpsi", cell="fcc256", gamma=True,
             precision="fp64", nb=64, block=64),
        # the largest: all bands of the 512-atom cell at Gamma, the benchmark's workload
        dict(name="hpsi_512atom_gamma_mixed", kind="hpsi", cell="diamond512", gamma=True,
             precision="mixed", nb=1024, block=128),
        # the overlap of the generalized problem on a ragged block of a tetragonal cell
        dict(name="overlap_48atom_fp64", kind="overlap", cell="random", nat=48, vol=90.0,
             ecut=25.0, aspect=1.3, proj="2s2p", k=2, precision="fp64", nb=77, block=77),
        # the charge density that follows a diagonalisation
        dict(name="density_64atom_fp64", kind="density", cell="diamond64", precision="fp64",
             nb=128, block=128),
        # projectors of a new k-point or of moved atoms
        dict(name="projectors_64atom_mixed", kind="projectors", cell="diamond64",
             precision="mixed", nb=1, block=1),
        # one diagonalisation from start vectors and its density: a step of an SCF cycle
        dict(name="scf_step_32atom_fp64", kind="scf", cell="random", nat=32, vol=20.0, ecut=30.0,
             aspect=1.0, proj="sp", k=0, precision="fp64", nb=64, block=64),
        # a few requests at once to the request server (1-2 k-points each, mixed form)
        dict(name="serve_burst", kind="serve", nat=12, requests=4, ecut=25.0),
    ]


def draw(rng):
    """One more case of the same ranges; odd sizes and non-cubic boxes among them."""
    kind = rng.choice(["hpsi"] * 6 + ["overlap", "density", "density", "projectors", "scf", "serve"])
    if kind == "serve":
        return dict(kind=kind, nat=rng.randint(8, 16), requests=rng.randint(2, 5),
                    ecut=rng.choice([20.0, 25.0, 30.0]))
    precision = rng.choice(["fp64", "mixed"])
    c = dict(kind=kind, cell="random", ecut=rng.choice([20.0, 25.0, 30.0]), vol=20.0, aspect=1.0,
             proj="sp", k=rng.randrange(4), precision=precision)
    if kind == "scf":
        c.update(nat=rng.randint(8, 32), precision="fp64")
        c.update(nb=2 * c["nat"], block=2 * c["nat"])
        return c
    c["nat"] = int(round(math.exp(rng.uniform(math.log(4), math.log(256)))))
    c["proj"] = rng.choice(["sp", "2s2p", "s2pd"])
    # 20 (the served cells) to 135 bohr^3 an atom (the 64-atom supercell), dense when there are many
    c["vol"] = round(math.exp(rng.uniform(math.log(20), math.log(135 if c["nat"] <= 100 else 40))), 2)
    c["aspect"] = rng.choice([1.0, 1.0, 1.05, 1.3])
    c["nb"] = int(round(math.exp(rng.uniform(math.log(8), math.log(300)))))
    c["block"] = c["nb"] if rng.random() < 0.6 else rng.randint(max(1, c["nb"] // 4), c["nb"])
    if kind in ("hpsi", "density") and rng.random() < 0.35:
        c.update(gamma=True, k=-1)
    if kind == "projectors":
        c.update(nb=1, block=1)
    return c


# ---------------------------------------------------------------------------- cells


def _sites(kind):
    fcc = np.array([[0, 0, 0], [0, .5, .5], [.5, 0, .5], [.5, .5, 0]])
    if kind == "bcc":
        return np.array([[0, 0, 0], [.5, .5, .5]])
    n = int(kind[-1])
    grid = np.array([[i, j, k] for i in range(n) for j in range(n) for k in range(n)])
    f = (grid[:, None, :] + fcc[None, :, :]).reshape(-1, 3) / n
    return f if kind.startswith("fcc") else np.concatenate([f, f + 0.25 / n]) % 1.0


def _shape(case):
    """(lattice, box, k in cartesian 1/bohr, cutoff, projector set, number of atoms)."""
    if case["cell"] in _NAMED:
        edges, sites, box, kf, ecut, proj = _NAMED[case["cell"]]
        nat = len(_sites(sites))
    else:
        nat, ecut, proj = case["nat"], case["ecut"], case["proj"]
        a = (case["vol"] * nat / case["aspect"]) ** (1.0 / 3.0)
        edges, box = (a, a, a * case["aspect"]), None
        kf = (0.0, 0.0, 0.0) if case["k"] < 0 else _KFRAC[case["k"]]
    lattice = np.diag(edges)
    kpt = np.asarray(kf) * (2.0 * math.pi / edges[0])
    return lattice, box or cellgen.fft_box_min(lattice, 4.0 * ecut), kpt, ecut, proj, nat


def _potential(lattice, box, positions):
    """cellgen's model potential on the grid, its Fourier series summed on the device."""
    n1, n2, n3 = box
    b = 2.0 * math.pi * np.linalg.inv(lattice).T
    freq = [np.rint(np.fft.fftfreq(n) * n) for n in box]
    e = [torch.from_numpy(np.exp(-1j * np.outer(positions @ b[i], freq[i]))).cuda() for i in range(3)]
    s = (e[2].t() @ (e[1][:, :, None] * e[0][:, None, :]).reshape(len(positions), -1))
    f = [torch.from_numpy(v).cuda() for v in freq]
    # every lattice here is orthorhombic: |G|^2 is a sum over the axes
    g2 = ((f[2] * b[2, 2]) ** 2)[:, None, None] + ((f[1] * b[1, 1]) ** 2)[None, :, None] \
        + ((f[0] * b[0, 0]) ** 2)[None, None, :]
    w2 = cellgen.cells.VLOC_WIDTH ** 2
    vt = cellgen.cells.VLOC_AMP * (2.0 * math.pi * w2) ** 1.5 * torch.exp(-0.5 * w2 * g2)
    c = vt * s.reshape(n3, n2, n1) / abs(np.linalg.det(lattice))
    return (torch.fft.ifftn(c) * float(n1 * n2 * n3)).real.contiguous().cpu().numpy()


def _cell(case, seed):
    lattice, box, kpt, ecut, proj, nat = _shape(case)
    rng = np.random.default_rng(seed)
    if case["cell"] in _NAMED:
        pos = _sites(_NAMED[case["cell"]][1]) @ lattice + rng.normal(0.0, 0.1, size=(nat, 3))
    else:
        pos = rng.uniform(0.0, 1.0, size=(nat, 3)) @ lattice
    cell = cellgen.make_cell(
        "case", seed=seed, lattice=lattice, frac=pos @ np.linalg.inv(lattice), kpt=kpt, fft=box,
        ecutwfc=ecut, proj=proj, dfixed=False, nbnd=case["nb"], block=case["block"],
        with_beta=False, vloc=_potential(lattice, box, pos), overlap=case["kind"] == "overlap")
    return cellgen.gamma_half(cell) if case.get("gamma") else cell


def _start_vectors(cell, nb, seed):
    """(nb, npw) complex128 on the device; each band's norm over the full sphere is 1."""
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    q = cell.miller @ (2.0 * math.pi * np.linalg.inv(cell.lattice).T) + np.asarray(cell.kpt)
    damp = 1.0 / (1.0 + torch.from_numpy((q * q).sum(axis=1)).cuda())
    psi = torch.randn(nb, cell.npw, 2, generator=g, device="cuda", dtype=torch.float64)
    psi = torch.view_as_complex(psi) * damp
    if cell.gamma:
        psi[:, 0].imag.zero_()
        n2 = 2.0 * psi.abs().square().sum(1, keepdim=True) - psi[:, :1].abs().square()
    else:
        n2 = psi.abs().square().sum(1, keepdim=True)
    return (psi / n2.sqrt()).contiguous()


def _occupations(nb):
    """Closed shells with a few partly filled levels at the top, as a smeared SCF step has them."""
    f = 2.0 * np.ones(nb)
    top = max(1, nb // 8)
    f[nb - top:] = 2.0 / (1.0 + np.exp(np.linspace(-4.0, 4.0, top)))
    return f


# ---------------------------------------------------------------------------- the calls


def _serve_requests(case, seed):
    reqs = []
    for i in range(case["requests"]):
        nat = case["nat"] + 3 * i
        cells = [cellgen.random_served_cell(nat, case["ecut"], k, seed * 101 + i, with_beta=False)
                 for k in range(1 + i % 2)]
        for c in cells:
            c.projgen = cellgen.projgen_tables(c)
        psi = [cellgen.make_psi0(c.npw, c.nbnd, seed=seed * 7 + k) for k, c in enumerate(cells)]
        reqs.append((cells, psi))
    return reqs


def prepare(case, seed):
    import paper_2104_10502_amd as qeh
    if case["kind"] == "serve":
        return dict(kind="serve", qeh=qeh, requests=_serve_requests(case, seed),
                    server=qeh.Server(2 << 30, max_slots=8))
    cell = _cell(case, seed)
    prec = qeh.QEH_MIXED if case["precision"] == "mixed" else qeh.QEH_FP64
    tables = cellgen.projgen_tables(cell)
    st = dict(kind=case["kind"], qeh=qeh, precision=prec)
    if case["kind"] == "projectors":
        st.update(cell=cell, tables=tables)
        return st
    ctx = qeh.Context.from_cell(cell, precision=prec, block=case["block"], projgen=tables)
    psi = _start_vectors(cell, case["nb"], seed)
    st.update(ctx=ctx, psi=psi)
    if case["kind"] in ("hpsi", "overlap"):
        st["out"] = torch.empty_like(psi)
        if prec == qeh.QEH_MIXED:
            st["kept"] = torch.empty(psi.shape, dtype=torch.complex64, device=psi.device)
        return st
    n1, n2, n3 = cell.fft
    st.update(occ=_occupations(case["nb"]),
              rho=torch.empty((n3, n2, n1), dtype=torch.float64, device=psi.device),
              density_work=torch.empty(max(ctx.density_plan(), 256), dtype=torch.uint8,
                                       device=psi.device))
    if prec == qeh.QEH_MIXED:
        st["kept"] = torch.empty((n3, n2, n1), dtype=torch.float32, device=psi.device)
    if case["kind"] == "scf":
        st.update(bands=torch.empty_like(psi),
                  work=torch.empty(ctx.davidson_plan(case["nb"]), dtype=torch.uint8,
                                   device=psi.device))
    return st


def _keep(st, out):
    """The mixed form's result as a program keeps it: in single precision."""
    return st["kept"].copy_(out) if "kept" in st else out


def run(st):
    kind = st["kind"]
    if kind == "hpsi":
        return _keep(st, st["ctx"].apply_h(st["psi"], out=st["out"]))
    if kind == "overlap":
        return _keep(st, st["ctx"].apply_s(st["psi"], out=st["out"]))
    if kind == "density":
        return _keep(st, st["ctx"].density(st["psi"], st["occ"], out=st["rho"],
                                           work=st["density_work"]))
    if kind == "projectors":
        c = st["cell"]
        return st["qeh"].generate_beta(c.lattice, c.kpt, c.miller, c.nproj, st["tables"],
                                       precision=st["precision"])
    if kind == "scf":
        # the Ritz vectors themselves are defined up to phases and rotations among equal
        # eigenvalues; the eigenvalues and the density carry them
        st["bands"].copy_(st["psi"])
        eig, _ = st["ctx"].davidson(st["bands"], work=st["work"])
        rho = st["ctx"].density(st["bands"], 2.0 * np.ones(len(eig)), out=st["rho"],
                                work=st["density_work"])
        return dict(eig=eig, rho=rho)
    srv, left, done = st["server"], {}, {}
    for i, (cells, psi) in enumerate(st["requests"]):
        left[srv.submit(cells, psi, cells[0].nbnd)] = i
    while left:
        for t in list(left):
            r = srv.poll(t)
            if r is not None:
                if r["status"] != 0:
                    raise RuntimeError("request failed: %s" % r["error"])
                done[left.pop(t)] = r["eig"]
        time.sleep(0.0005)
    return [done[i] for i in range(len(done))]


# ---------------------------------------------------------------------------- 64-bit values


def _beta64(cell):
    """Projectors on the sphere as the table form defines them: cubic Lagrange interpolation of
    F_c at |q|, real harmonics of q / |q|, structure phase; (nkb, npw) complex128."""
    tab = cellgen.projgen_tables(cell)
    q = torch.from_numpy(cell.miller @ (2.0 * math.pi * np.linalg.inv(cell.lattice).T)
                         + np.asarray(cell.kpt)).cuda()
    qn = q.norm(dim=1)
    x, y, z = (q / qn.clamp_min(1e-300)[:, None]).unbind(1)
    t = qn / tab["dq"]
    j = t.floor().clamp_min(1.0)
    t, j = t - j, j.long()
    lag = [-t * (t - 1) * (t - 2) / 6, (t + 1) * (t - 1) * (t - 2) / 2,
           -(t + 1) * t * (t - 2) / 2, (t + 1) * t * (t - 1) / 6]
    pi = math.pi
    ang = {0: [torch.full_like(x, 1 / math.sqrt(4 * pi))],
           1: [math.sqrt(3 / (4 * pi)) * v for v in (x, y, z)],
           2: [math.sqrt(15 / (4 * pi)) * v for v in (x * y, y * z, z * x)]
           + [math.sqrt(5 / (16 * pi)) * (3 * z * z - 1),
              math.sqrt(15 / (16 * pi)) * (x * x - y * y)]}
    rows = []
    for c, l in enumerate(tab["lchan"]):
        f = torch.from_numpy(tab["tab"][c]).cuda()
        f = sum(w * f[j + o] for w, o in zip(lag, (-1, 0, 1, 2)))
        rows += [f * a * (-1j) ** int(l) for a in ang[int(l)]]
    shape = torch.stack(rows) * (4.0 * pi / math.sqrt(cell.omega))
    tau = torch.from_numpy(tab["tau"]).cuda()
    out = torch.empty(len(tau), len(rows), cell.npw, dtype=torch.complex128, device="cuda")
    for a in range(len(tau)):
        arg = -(q @ tau[a])
        torch.mul(shape, torch.complex(arg.cos(), arg.sin()), out=out[a])
    return out.reshape(-1, cell.npw)


def _sphere(cell):
    """Flat box positions of the full sphere, and whether it is stored by half."""
    m = cell.miller if not cell.gamma else np.concatenate([-cell.miller[:0:-1], cell.miller])
    n1, n2, n3 = cell.fft
    i = ((m[:, 2] % n3).astype(np.int64) * n2 + m[:, 1] % n2) * n1 + m[:, 0] % n1
    return torch.from_numpy(i).cuda()


def _full(cell, psi):
    if not cell.gamma:
        return psi
    p = psi.clone()
    p[:, 0].imag.zero_()
    return torch.cat([p[:, 1:].flip(1).conj(), p], dim=1)


def _real_space(cell, psi, at):
    n1, n2, n3 = cell.fft
    box = torch.zeros(psi.shape[0], n1 * n2 * n3, dtype=torch.complex128, device="cuda")
    box[:, at] = _full(cell, psi)
    return torch.fft.ifftn(box.view(-1, n3, n2, n1), dim=(1, 2, 3), norm="forward")


def _batches(cell, nb):
    """Bands a transform of the 64-bit values takes at once (2 GiB of boxes)."""
    step = max(1, (1 << 27) // cell.nfft)
    return [slice(i, min(nb, i + step)) for i in range(0, nb, step)]


def _blocks(blocks, nproj):
    out, off = [], 0
    for n in nproj:
        out.append(torch.from_numpy(blocks[off:off + n * n].reshape(n, n)).cuda())
        off += n * n
    return torch.stack(out)


def _projected(cell, beta, blocks, psi):
    """beta D beta^H psi (all atoms have the same number of projectors)."""
    becp = psi @ beta.conj().t()
    if cell.gamma:
        becp = (2.0 * becp - psi[:, :1].real * beta[:, 0].conj()[None, :]).real.to(psi.dtype)
    d = _blocks(blocks, cell.nproj)
    nat, n = d.shape[:2]
    ps = torch.empty_like(becp).view(-1, nat, n)
    b = becp.view(-1, nat, n)
    for a in range(nat):
        ps[:, a] = b[:, a] @ d[a].t().contiguous()
    return ps.view(-1, nat * n) @ beta


def _hpsi64(cell, psi):
    at = _sphere(cell)
    v = torch.from_numpy(cell.vloc).cuda()
    out = torch.empty_like(psi)
    for s in _batches(cell, psi.shape[0]):
        r = _real_space(cell, psi[s], at) * v
        out[s] = torch.fft.fftn(r, dim=(1, 2, 3), norm="forward").view(r.shape[0], -1)[
            :, at[-cell.npw:]]
    q = torch.from_numpy(cell.miller @ (2.0 * math.pi * np.linalg.inv(cell.lattice).T)
                         + np.asarray(cell.kpt)).cuda()
    out += q.square().sum(1) * psi
    return out + _projected(cell, _beta64(cell), cell.dmat, psi)


def _density64(cell, psi, occ):
    at, rho = _sphere(cell), 0.0
    for s in _batches(cell, psi.shape[0]):
        w = torch.from_numpy(occ[s]).cuda()[:, None, None, None]
        rho = rho + (w * _real_space(cell, psi[s], at).abs().square()).sum(0)
    return rho / cell.omega


def _eigh64(cell, nb):
    """The nb lowest eigenpairs of H written out as a matrix."""
    n1, n2, n3 = cell.fft
    vt = torch.fft.fftn(torch.from_numpy(cell.vloc).cuda().to(torch.complex128), norm="forward")
    m = torch.from_numpy(cell.miller.astype(np.int64)).cuda()
    d = m[:, None, :] - m[None, :, :]
    h = vt[d[..., 2] % n3, d[..., 1] % n2, d[..., 0] % n1]
    beta = _beta64(cell)
    blocks = _blocks(cell.dmat, cell.nproj)
    nat, n = blocks.shape[:2]
    w = torch.empty_like(beta).view(nat, n, -1)
    for a in range(nat):
        w[a] = blocks[a].t().contiguous() @ beta.view(nat, n, -1)[a].conj()
    h = h + beta.t().contiguous() @ w.reshape(nat * n, -1)
    q = m.cpu().numpy() @ (2.0 * math.pi * np.linalg.inv(cell.lattice).T) + np.asarray(cell.kpt)
    h = h.cpu().numpy() + np.diag((q * q).sum(axis=1))
    import scipy.linalg
    return scipy.linalg.eigh(0.5 * (h + h.conj().T), subset_by_index=[0, nb - 1])


def exact(case, seed):
    if case["kind"] == "serve":
        return [np.stack([_eigh64(c, c.nbnd)[0] for c in cells])
                for cells, _ in _serve_requests(case, seed)]
    cell = _cell(case, seed)
    if case["kind"] == "projectors":
        return _beta64(cell)
    if case["kind"] == "scf":
        eig, y = _eigh64(cell, case["nb"])
        psi = torch.from_numpy(np.ascontiguousarray(y.T)).cuda()
        return dict(eig=eig, rho=_density64(cell, psi, 2.0 * np.ones(case["nb"])))
    psi = _start_vectors(cell, case["nb"], seed)
    if case["kind"] == "density":
        return _density64(cell, psi, _occupations(case["nb"]))
    if case["kind"] == "overlap":
        return psi + _projected(cell, _beta64(cell), cell.qmat, psi)
    return _hpsi64(cell, psi)


# ---------------------------------------------------------------------------- work


@functools.lru_cache(maxsize=64)
def _counts(items):
    """(stored plane waves, sticks, x-extent, projectors, box) of a case."""
    case = dict(items)
    lattice, box, kpt, ecut, proj, nat = _shape(case)
    m = cellgen.sphere_miller(lattice, kpt, ecut)
    nst = len(np.unique(m[:, :2], axis=0))
    ext = int(m[:, 0].max() - m[:, 0].min()) + 1
    nkb = nat * sum(2 * l + 1 for l, _ in cellgen.PROJ_SETS[proj])
    npw = (len(m) + 1) // 2 if case.get("gamma") else len(m)
    return npw, nst, ext, nkb, box


def _fft(n):
    return 5.0 * n * math.log2(n)


def work(case):
    """Each input read once and each output written once; transforms at 5 n log2 n operations
    over the sticks, columns and rows the sphere touches; 8 operations a complex multiply-add
    (4 where real wavefunctions need half)."""
    if case["kind"] == "serve":
        total = dict(bytes=0.0, flops=0.0)
        for i in range(case["requests"]):
            nat = case["nat"] + 3 * i
            w = work(dict(kind="scf", cell="random", nat=nat, vol=20.0, ecut=case["ecut"],
                          aspect=1.0, proj="sp", k=0, precision="mixed", nb=2 * nat,
                          block=2 * nat))
            for k in total:
                total[k] += w[k] * (1 + i % 2)
        return total
    npw, nst, ext, nkb, (n1, n2, n3) = _counts(tuple(sorted(case.items())))
    nb, real = case["nb"], 4 if case["precision"] == "mixed" else 8
    gam = bool(case.get("gamma"))
    if case["kind"] == "projectors":
        return dict(bytes=2.0 * real * nkb * npw, flops=10.0 * nkb * npw)
    one_way = nst * _fft(n3) + ext * n3 * _fft(n2) + n2 * n3 * _fft(n1)
    transforms = (nb + 1) // 2 if gam else nb
    projected = 2.0 * (4 if gam else 8) * nb * nkb * npw
    beta = 2.0 * real * nkb * npw
    if case["kind"] == "overlap":
        return dict(bytes=32.0 * nb * npw + beta, flops=projected)
    if case["kind"] == "density":
        return dict(bytes=16.0 * nb * npw + 8.0 * n1 * n2 * n3,
                    flops=transforms * (one_way + 4.0 * n1 * n2 * n3))
    h = dict(bytes=32.0 * nb * npw + beta + real * n1 * n2 * n3,
             flops=transforms * (2.0 * one_way + 2.0 * n1 * n2 * n3) + projected)
    if case["kind"] == "scf":
        # about a dozen block steps: H on the block, the two projected matrices and the rotation
        # of a basis of 2 nb vectors
        step = h["flops"] + 8.0 * npw * nb * 2 * nb * 4
        return dict(bytes=12.0 * (h["bytes"] + 16.0 * npw * nb * 8), flops=12.0 * step)
    return h
