"""Triquadratic and tricubic applies far from the origin.  The operator does not change when the
mesh is moved.  All nodes lie on a grid of 1/512 and are moved by 2048 and 4096, which is exact, and
the apply works on differences of an element's coordinates, which are exact too.  So the results of
the two places differ by no more than the order of the atomic additions: 1e-13 leaves a factor of
some hundred.  Sums of the coordinates themselves would round at 4096 2^-53 = 5e-13 of an element
and more after differentiation."""
import numpy as np
import pytest

import seeded_inputs as si
from helpers import rel_err
from test_gpu_family import apply, family_problem, make_family_op

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("physics", [1, 3])
@pytest.mark.parametrize("elem", [27, 64])
def test_moved_mesh(elem, physics):
    import paper_2308_09839_amd as q1
    print(f"\n[family origin] elem={elem} physics={physics}", flush=True)
    pr = family_problem(elem, physics, (5, 3, 2), 0.1, 73)
    pr["xyz"] = np.round(pr["xyz"] * 512) / 512
    shift = np.array([[4096.0], [-4096.0], [2048.0]])
    moved = dict(pr, xyz=pr["xyz"] + shift)
    assert np.array_equal(moved["xyz"] - shift, pr["xyz"])
    x = si.vec_uniform(pr["xyz"].shape[1] * (1 if physics == 1 else 3), 73, si.STREAM_X)
    y, z = (apply(make_family_op(q1, p), x, 0) for p in (pr, moved))
    err = rel_err(z, y)
    print(f"  {err:.2e}", flush=True)
    assert err <= 1e-13
