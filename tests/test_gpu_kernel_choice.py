"""Which kernels run: qeh_ctx_info's plane, stick and density kernels on the boxes
that the tests of the two-factor passes use (a fallback to the LDS passes would
give the same numbers), on sizes without a compiled form, and under the test
hooks.  Nothing is computed here.
"""

import numpy as np
import pytest

import cellgen
from test_gpu_density_sizes import SIZES as DENSITY_SIZES, _cell as _density_cell
from test_gpu_stick_sizes import SIZES as STICK_SIZES, _cell as _stick_cell

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

LDS, SPLIT, TWO, TIGHT = 0, 1, 2, 3   # plane kernel
ROWS, PAIR_ROWS, FUSED = 0, 1, 2      # density kernel


def _info(cell, prec, block=7):
    import paper_2104_10502_amd as q
    ctx = q.Context.from_cell(cell, precision=prec, block=block)
    i = ctx.info()
    ctx.close()
    return i


def _plane_cell(n1, n2, fill=0.5, n3=12):
    a, b, c = 0.5 * n1, 0.5 * n2, 0.5 * n3
    r = min((fill * n1 - 1) / 2, 0.95 * (n3 - 1) / 2 * a / c) - 0.3
    ecut = (2 * np.pi / a * r) ** 2
    return cellgen.make_cell("t", seed=3, lattice=np.diag([a, b, c]), frac=np.array([[.1, .2, .3]]),
                             kpt=np.array([0.9, -0.6, 0.2]) * np.pi / a * 0.5, ecutwfc=ecut,
                             ecutrho=4 * ecut, fft=(n1, n2, n3), proj="sp", nobeta=True, nbnd=3)


@pytest.mark.parametrize("prec", [0, 1])
def test_two_factor_planes(prec):
    for n in (12, 14, 15, 18, 21, 25, 27, 35, 45, 54, 63, 72, 75, 81, 84, 90, 100, 120, 125, 128, 135):
        assert _info(_plane_cell(n, n), prec)["plane_kernel"] == TWO, n
    # single precision up to 192; in FP64 the columns of half a line fit up to 135
    for n in (140, 160, 180):
        assert (_info(_plane_cell(n, n), prec)["plane_kernel"] == TWO) == (prec == 1), n


@pytest.mark.parametrize("prec", [0, 1])
def test_planes_without_a_two_factor_form(prec, monkeypatch):
    # not square; 49 = 7 x 7 and 98 = 14 x 7 are not compiled
    for n1, n2 in ((24, 25), (40, 36), (49, 49), (98, 98)):
        assert _info(_plane_cell(n1, n2), prec)["plane_kernel"] == LDS, (n1, n2)
    c = _plane_cell(36, 36)
    monkeypatch.setenv("QEH_PLANE_KERNEL", "generic")
    assert _info(c, prec)["plane_kernel"] == LDS
    monkeypatch.delenv("QEH_PLANE_KERNEL")
    monkeypatch.setenv("QEH_FORCE_SPLIT_PLANE", "1")
    assert _info(c, prec)["plane_kernel"] == SPLIT


@pytest.mark.parametrize("prec", [0, 1])
def test_stick_kernels(prec, monkeypatch):
    for n3, n, fill in STICK_SIZES:
        for gam in (False, True):
            c = _stick_cell(n3, n, fill, gam, 3)
            assert _info(cellgen.gamma_half(c) if gam else c, prec)["stick_kernel"] == 1, n3
    monkeypatch.setenv("QEH_STICK_KERNEL", "generic")
    assert _info(c, prec)["stick_kernel"] == 0
    monkeypatch.delenv("QEH_STICK_KERNEL")
    assert _info(_plane_cell(24, 24, n3=49), prec)["stick_kernel"] == 0


@pytest.mark.parametrize("prec", [0, 1])
def test_density_kernels(prec, monkeypatch):
    c = None
    for n, n3, fill in DENSITY_SIZES:
        c = _density_cell(n, n3, fill, False)
        i = _info(c, prec)
        want = n <= (120 if prec == 0 else 160)
        assert (i["density_kernel"] == FUSED) == want, n
        assert 4 <= i["density_bands"] <= 16
    c = _density_cell(72, 12, 0.5, False)
    monkeypatch.setenv("QEH_DENSITY_KERNEL", "rows")
    i = _info(c, prec)
    assert i["density_kernel"] == (PAIR_ROWS if prec == 1 else ROWS) and i["density_bands"] == 16
    monkeypatch.setenv("QEH_DENSITY_KERNEL", "generic")
    assert _info(c, prec)["density_kernel"] == ROWS
