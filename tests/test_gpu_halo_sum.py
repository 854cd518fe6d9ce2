"""The halo sum of a node on many tiles: its slots past the first two are read several at a
time, so counts that are no multiple of that, and more than a lattice node's six, are covered by
a ring of wedges (hexahedra whose inner face is collapsed onto the axis) in tiles of one element.
Against the oracle's assembled matrix at the tolerances of the apply tests (1e-12 in FP64, 2e-5
in FP32)."""
import numpy as np
import pytest

import seeded_inputs as si
from helpers import TOL, gpu_apply, make_op, rel_err

pytestmark = pytest.mark.gpu


def ring(m):
    """m wedges around the z axis, two layers; nodes: 3 on the axis, then m per plane."""
    t = 2 * np.pi * np.arange(m) / m
    xyz = np.zeros((3, 3 + 3 * m))
    xyz[2, :3] = np.arange(3)
    conn = []
    for k in range(3):
        s = 3 + m * k
        xyz[:, s:s + m] = np.stack([np.cos(t), np.sin(t), np.full(m, float(k))])
    for k in range(2):
        for j in range(m):
            lo, hi = 3 + m * k, 3 + m * (k + 1)
            n = (j + 1) % m
            conn.append([k, lo + j, k, lo + n, k + 1, hi + j, k + 1, hi + n])
    return xyz, np.array(conn, dtype=np.int32).T.copy()


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("physics", [1, 3])
@pytest.mark.parametrize("m", [7, 13, 24])
def test_node_on_many_tiles(orc, monkeypatch, m, physics, dtype):
    print(f"\n[halo sum] wedges={m} physics={physics} dtype={dtype}", flush=True)
    monkeypatch.setenv("Q1_BLOCK_SHAPE", "1,1,1")
    xyz, conn = ring(m)
    ne = conn.shape[1]
    if physics == 1:
        coef = si.field_lognormal(ne, 0.0, 1.0, 81)[None]
    else:
        coef = np.stack(si.lame_from_E_nu(*si.field_elastic(ne, 81)))
    mask = np.zeros(xyz.shape[1], dtype=np.uint8)
    mask[[0, 5]] = 1
    A = orc.assemble(physics, xyz, conn, coef, mask)
    x = si.vec_uniform(A.n, 81, si.STREAM_X)
    op = make_op(dict(physics=physics, xyz=xyz, conn=conn, coef=coef, mask=mask), dtype, 5)
    y, ref = gpu_apply(op, x, dtype), A.matvec(x)
    assert rel_err(y, ref) <= TOL[dtype]
    assert np.max(np.abs(y - ref)) <= 10 * TOL[dtype] * np.max(np.abs(ref))
