"""The sums of tetrahedra in FP32 operators on block tiles: every tetrahedron's contribution to a
corner is added in FP64, also where a lane forms the six of a Kuhn cell.  One unit cell of corners
c = i + 2j + 4k, tetrahedra (0,1,3,7) (0,5,1,7) (0,3,2,7) (0,2,6,7) (0,6,4,7) (0,4,5,7): the row of
corner 0 is sum_t k_t (u_0 - u_s) / 6 with s = 1, 1, 2, 2, 4, 4 the first corner of each
tetrahedron's path.  With u_1 = 1, u_2 = -1 and k = K on one tetrahedron of each, K a power of two
far above 2^24, two exactly opposite contributions of K / 6 hide the others in FP32 sums; in FP64
sums they cancel and leave -(k_1 - k_3 + u_4 (k_4 + k_5)) / 6 in full.  Each contribution has at most
a few FP32 roundings, hence 1e-6."""
import numpy as np
import pytest

from test_gpu_family import apply, make_family_op

pytestmark = pytest.mark.gpu

TETS = ((0, 1, 3, 7), (0, 5, 1, 7), (0, 3, 2, 7), (0, 2, 6, 7), (0, 6, 4, 7), (0, 4, 5, 7))


@pytest.mark.parametrize("physics", [1, 3])
@pytest.mark.parametrize("order", ["cell", "one swapped"])
def test_hidden_contributions(physics, order):
    import paper_2308_09839_amd as q1
    print(f"\n[tet sums] physics={physics} order={order}", flush=True)
    xyz = np.array([[c & 1, c >> 1 & 1, c >> 2] for c in range(8)], dtype=np.float64).T.copy()
    conn = np.array(TETS, dtype=np.int32).T.copy()
    K = 2.0 ** 30
    k = np.array([K, 1.0, K, 1.0, 1.0, 1.0])
    if order == "one swapped":  # no Kuhn cell in a row: a lane per tetrahedron
        conn[:, [0, 1]], k[[0, 1]] = conn[:, [1, 0]], k[[1, 0]]
    u = np.zeros(8)
    u[[1, 2, 4]] = 1.0, -1.0, 1.0
    if physics == 1:
        coef, x, dpn = k[None], u, 1
    else:  # mu = k, lambda = 0, displacements along z
        # mu (grad u + grad u^T) adds to the z row of corner 0 what d u_z / d z makes, twice
        coef, x, dpn = np.stack([0 * k, k]), np.kron(u, (0.0, 0.0, 1.0)), 3
    op = make_family_op(q1, dict(elem=4, physics=physics, xyz=xyz, conn=conn, coef=coef,
                                 mask=None), 1)
    assert q1.q1_op_info(op)["variant"] == 5  # block tiles
    y = apply(op, x, 1)[dpn - 1]
    # Laplace: the K's cancel, 1 and 3 too, 4 and 5 leave -1/6 each; elasticity: each of these
    # two counts twice
    assert abs(y - (-2.0 if physics == 1 else -4.0) / 6) <= 1e-6, y
