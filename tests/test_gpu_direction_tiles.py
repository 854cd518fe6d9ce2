"""The direction step inside the apply on tiles that stage their nodes in several rounds (256 per
round and thread slot: three rounds' worth at once for scalar tiles, two for three unknowns, four
where a tile has more), at tile sizes on both sides of those limits, and on the owner-computes
tiles of tetrahedra.  q1_pcg, whose applies take the step within a batch of iterations, against
q1_pcg_noalloc, which keeps the separate kernel: equal bit for bit; the apply itself against the
oracle's assembled matrix at the tolerances of the apply tests."""
import numpy as np
import pytest

import seeded_inputs as si
from helpers import TOL, dev, gpu_apply, make_op, problem, rel_err, torch_dtype
from test_gpu_family import family_problem, make_family_op

pytestmark = pytest.mark.gpu


def same_solves(q1, op, b, dtype):
    import torch
    bd = dev(b, torch_dtype(dtype))
    for rtol, maxit in ((0.0, 3), (0.0, 12), (1e-4, 3000)):
        x, ref = torch.full_like(bd, 3.0), torch.full_like(bd, -5.0)
        st = q1.q1_pcg(op, 1, bd, x, rtol, maxit)
        st_ref = q1.q1_pcg_noalloc(op, 1, bd, ref, rtol, maxit)
        for key in ("status", "iters", "true_rel_res"):
            assert st[key] == st_ref[key], (maxit, key)
        assert np.array_equal(x.cpu().numpy(), ref.cpu().numpy()), maxit


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("jitter", [0.0, 0.1])
@pytest.mark.parametrize("physics,shape,n", [
    (1, "16,8,4", (37, 17, 9)),     # 765 nodes: three
    (1, "76,1,4", (77, 2, 5)),      # 770: four
    (1, "128,1,4", (130, 3, 4)),    # 1,290: two rounds of four
    (3, "16,4,4", (17, 9, 5)),      # 425: two
    (3, "51,1,4", (52, 2, 5)),      # 520: four
    (2, "64,1,4", (66, 3, 4))])     # 650
def test_staging_rounds(orc, monkeypatch, physics, shape, n, jitter, dtype):
    import paper_2308_09839_amd as q1
    print(f"\n[direction tiles] physics={physics} {shape} n={n} jitter={jitter} dtype={dtype}",
          flush=True)
    monkeypatch.setenv("Q1_BLOCK_SHAPE", shape)
    monkeypatch.setenv("Q1_OWNER_TILE", "0")
    pr = problem(physics, n, jitter, 98, True)
    dpn = 1 if physics == 1 else 3
    op = make_op(pr, dtype, 5)
    assert op.reproducible
    b = si.vec_uniform(pr["xyz"].shape[1] * dpn, 98, si.STREAM_RHS)
    b[np.repeat(pr["mask"].astype(bool), dpn)] = 0.0
    same_solves(q1, op, b, dtype)
    A = orc.assemble(physics, pr["xyz"], pr["conn"], pr["coef"], pr["mask"])
    x = si.vec_uniform(A.n, 98, si.STREAM_X)
    assert rel_err(gpu_apply(op, x, dtype), A.matvec(x)) <= TOL[dtype]


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("n", [(16, 8, 4), (32, 16, 8)])
def test_owner_tetrahedra(n, dtype):
    import paper_2308_09839_amd as q1
    print(f"\n[direction tiles, tetrahedra] n={n} dtype={dtype}", flush=True)
    pr = family_problem(4, 1, n, 0.1, 99, True)
    op = make_family_op(q1, pr, dtype)
    assert op.reproducible
    b = si.vec_uniform(pr["xyz"].shape[1], 99, si.STREAM_RHS)
    b[pr["mask"].astype(bool)] = 0.0
    same_solves(q1, op, b, dtype)
