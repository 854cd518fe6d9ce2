"""The flag that ends a solve is raised by one workgroup of a launch whose other workgroups read
it: what they read must not change what is computed.  The mixed solver stops its recurrences at
every refresh and goes on with the direction it has, so solves with many refreshes, on more
workgroups than run at once, are repeated and compared bit for bit (the operators are
reproducible, and so is every sum)."""
import numpy as np
import pytest

import seeded_inputs as si
from helpers import dev, make_op, problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("physics,n", [
    (1, (64, 32, 32)),   # owner-computes tiles
    (1, (61, 45, 33)),   # tiles of several shapes
    (3, (33, 29, 31))])
def test_restarts_repeat(physics, n):
    import torch
    import paper_2308_09839_amd as q1
    print(f"\n[stop flag] physics={physics} n={n}", flush=True)
    pr = problem(physics, n, 0.0, 97, True)
    dpn = 1 if physics == 1 else 3
    b = si.vec_uniform(pr["xyz"].shape[1] * dpn, 97, si.STREAM_RHS)
    b[np.repeat(pr["mask"].astype(bool), dpn)] = 0.0
    bd = dev(b)
    op64, op32 = make_op(pr, 0), make_op(pr, 1)
    assert op64.reproducible and op32.reproducible
    first = None
    for _ in range(6):
        x = torch.full_like(bd, 2.0)
        st = q1.q1_mpcg(op64, op32, bd, x, 1e-8, 0.7, 20000)
        assert st["status"] == 0 and st["outer_iters"] >= 20
        got = (st["iters"], st["outer_iters"], x.cpu().numpy())
        first = first or got
        assert got[:2] == first[:2] and np.array_equal(got[2], first[2])
