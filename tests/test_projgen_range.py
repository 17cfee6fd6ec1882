"""The range check of device-built projectors looks at the ends of each (h, k) run
of the Miller list only: a table that just covers the largest |k+G| of the whole
list is accepted and one that just does not is refused, also for lists in other
orders and with a far point in the middle of a run."""

import ctypes

import numpy as np
import pytest

import cellgen


def _plan(c, miller, qmax_steps, dq):
    import paper_2104_10502_amd as q
    pg = dict(cellgen.projgen_tables(c))
    pg.update(dq=dq, tab=np.zeros((len(pg["lchan"]), qmax_steps + 3)))
    keep = []
    s = q._cell_struct(c.lattice, (1, 1, 1), c.kpt, miller, np.zeros(1), c.nproj, None,
                       np.zeros(0, dtype=np.complex128), q.QEH_FP64, 1, keep, projgen=pg)
    n = ctypes.c_size_t()
    return q._lib.qeh_beta_plan(ctypes.byref(s), ctypes.byref(n)) == q.QEH_OK


@pytest.mark.parametrize("order", ["as built", "shuffled", "reversed", "middle"])
@pytest.mark.parametrize("kfrac", [(0.0, 0.0, 0.0), (0.25, -0.4, 0.1)])
def test_table_end(order, kfrac):
    c = cellgen.make_cell("c1", kfrac=kfrac)
    m = np.asarray(c.miller)
    rng = np.random.default_rng(1)
    if order == "shuffled":
        m = m[rng.permutation(len(m))]
    elif order == "reversed":
        m = m[::-1]
    elif order == "middle":   # the farthest point of a run in its middle
        m = m.copy()
        run = np.flatnonzero((m[:, 0] == 0) & (m[:, 1] == 0))
        m[run[len(run) // 2], 2] = -40
    b = 2 * np.pi * np.linalg.inv(np.asarray(c.lattice)).T
    qmax = np.linalg.norm(np.asarray(c.kpt) + m @ b, axis=1).max()
    for rel, ok in ((1e-9, True), (-1e-9, False)):
        assert _plan(c, m, 500, qmax * (1 + rel) / 500) == ok
