"""Tetrahedra in Kuhn cells: the block tiles take a cell's six tetrahedra in one lane where every
six elements in a row form one (whatever the cells' order), else one tetrahedron per lane.  Both
against the oracle's assembled matrix at the tolerances of the apply tests, on boxes of one cell,
of tiles with partial steps and of several tiles."""
import numpy as np
import pytest

import seeded_inputs as si
from helpers import TOL, rel_err
from test_gpu_family import apply, family_problem, make_family_op

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("order", ["cells", "cells shuffled", "elements shuffled", "one swapped"])
@pytest.mark.parametrize("physics", [1, 3])
@pytest.mark.parametrize("n", [(1, 1, 1), (5, 4, 3), (17, 9, 6)])
def test_tet_cells(orc, monkeypatch, n, physics, order, dtype):
    import paper_2308_09839_amd as q1
    print(f"\n[tet cells] n={n} physics={physics} order={order} dtype={dtype}", flush=True)
    monkeypatch.setenv("Q1_OWNER_TILE", "0")
    pr = family_problem(4, physics, n, 0.1, 2331, True)
    ne = pr["conn"].shape[1]
    rng = np.random.default_rng(2331)
    if order == "cells shuffled":
        perm = (6 * rng.permutation(ne // 6)[:, None] + np.arange(6)).ravel()
    elif order == "elements shuffled":
        perm = rng.permutation(ne)
    else:
        perm = np.arange(ne)
        if order == "one swapped":
            perm[[ne - 1, ne - 2]] = perm[[ne - 2, ne - 1]]
    pr["conn"] = np.ascontiguousarray(pr["conn"][:, perm])
    pr["coef"] = np.ascontiguousarray(np.atleast_2d(pr["coef"])[:, perm])
    A = orc.assemble(physics, pr["xyz"], pr["conn"], pr["coef"], pr["mask"])
    x = si.vec_uniform(A.n, 2331, si.STREAM_X)
    ref = A.matvec(x)
    y = apply(make_family_op(q1, pr, dtype), x, dtype)
    assert rel_err(y, ref) <= TOL[dtype]
    assert np.max(np.abs(y - ref)) <= 10 * TOL[dtype] * np.max(np.abs(ref))
