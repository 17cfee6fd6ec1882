"""The benchmark's byte models against the kernels that run: what one launch reads
and writes, counted from the shapes that a context reports."""

import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench  # noqa: E402

# 64 bands or Gamma band pairs of a 135^3 box
SHAPE = dict(npw=74047, nst=3289, nkb=2048, n1=135, n2=135, n3=135, ext=65, block=64,
             plane_kernel=2, stick_kernel=1, density_kernel=2, density_bands=4)


def test_gamma_k3_separates_its_pairs():
    # sticks of 32 pairs and the box map of the full sphere; psi, H psi and |G|^2 of the half
    sh = dict(SHAPE, gamma=True)
    sticks = 32 * (8 * 3289 * 135 + 4 * (2 * 74047 - 1))
    half = 64 * 2 * 16 * 74047 + 8 * 74047
    assert bench.algorithmic("k3_zfwd_gather", sh, 1, 64) == ("hbm", sticks + half)
    # behind the LDS passes the pairs go through a full-sphere buffer of complex doubles
    buffered = 32 * 2 * 16 * (2 * 74047 - 1)
    assert bench.algorithmic("k3_zfwd_gather", dict(sh, stick_kernel=0), 1, 64) == \
        ("hbm", sticks + half + buffered)


def test_k1_writes_the_single_precision_copy():
    for gam, nt, full in ((False, 64, 74047), (True, 32, 2 * 74047 - 1)):
        sh = dict(SHAPE, gamma=gam)
        sticks = nt * (4 * full + 8 * 3289 * 135)
        assert bench.algorithmic("k1_scatter_zinv", sh, 1, 64)[1] == 64 * 24 * 74047 + sticks
        f64 = bench.algorithmic("k1_scatter_zinv", sh, 0, 64)[1]
        assert f64 == 64 * 16 * 74047 + nt * (4 * full + 16 * 3289 * 135)


def test_density_follows_the_subgroups():
    nfft = 135 ** 3
    for bands, nsub in ((4, 16), (7, 10), (16, 4)):
        sh = dict(SHAPE, gamma=False, density_bands=bands)
        assert bench.algorithmic("density_reduce", sh, 1, 64)[1] == 8 * (nsub + 1) * nfft
        assert bench.algorithmic("density_rows", sh, 1, 64)[1] == \
            64 * 8 * 3289 * 135 + 8 * nsub * nfft
        rows = bench.algorithmic("density_rows", dict(sh, density_kernel=0), 1, 64)[1]
        assert rows == 64 * 8 * 65 * 135 * 135 + 8 * nsub * nfft


def test_stored_counters_cover_the_included_headers():
    # a change of any source or header of the H|psi> kernels retires the stored counters
    csrc = os.path.join(ROOT, "paper_2104_10502_amd", "csrc")
    for f in bench.HPSI_SOURCES:
        for line in open(os.path.join(csrc, f)):
            if line.startswith('#include "') and "/" not in line:
                assert line.split('"')[1] in bench.HPSI_SOURCES, (f, line)
