"""The line kernel of the triquadratic and tricubic hexahedra where its wavefronts end: 7 or 4
elements each, 28 or 16 to a workgroup.  The elements run along x, in a random order, and on
randomly numbered nodes, so that neighbouring lanes share a node, share none, or share it in
another position, and masked nodes fall on the joints.  Against the oracle's assembled matrix at
the tolerances of the family tests (1e-12 in FP64, 2e-5 in FP32)."""
import numpy as np
import pytest

import seeded_inputs as si
from helpers import TOL, rel_err
from test_gpu_family import apply, family_problem, make_family_op

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def q1():
    import paper_2308_09839_amd as q1
    return q1


@pytest.mark.parametrize("order", ["x", "shuffled"])
@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("elem,physics,n", [
    (27, 1, (6, 1, 1)), (27, 1, (7, 1, 1)), (27, 3, (29, 1, 1)), (27, 1, (8, 4, 2)),
    (64, 1, (3, 1, 1)), (64, 3, (4, 1, 1)), (64, 1, (17, 1, 1)), (64, 1, (5, 4, 2))])
def test_line_kernel_joints(q1, orc, elem, physics, n, dtype, order):
    print(f"\n[family lines] elem={elem} physics={physics} n={n} dtype={dtype} {order}", flush=True)
    pr = family_problem(elem, physics, n, 0.1, 71)
    nn, ne = pr["xyz"].shape[1], pr["conn"].shape[1]
    rng = np.random.default_rng(71)
    if order == "shuffled":
        e, p = rng.permutation(ne), rng.permutation(nn)
        pr["xyz"], pr["mask"] = pr["xyz"][:, np.argsort(p)], pr["mask"][np.argsort(p)]
        pr["conn"], pr["coef"] = p[pr["conn"][:, e]].astype(np.int32), pr["coef"][:, e]
    A = orc.assemble(physics, pr["xyz"], pr["conn"], pr["coef"], pr["mask"])
    x = si.vec_uniform(A.n, 71, si.STREAM_X)
    ref = A.matvec(x)
    y = apply(make_family_op(q1, pr, dtype), x, dtype)
    assert rel_err(y, ref) <= TOL[dtype]
    assert np.max(np.abs(y - ref)) <= 10 * TOL[dtype] * np.max(np.abs(ref))
