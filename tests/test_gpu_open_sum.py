"""The halo sum inside the PCG update: iterates after a few iterations against the oracle's
PCG, on a ring of wedges in tiles of one element (nodes on 2 to 48 tiles, so every count of
slots past the first two) and on boxes, with Dirichlet nodes on several tiles whose right-hand
side is not zero, in block and partial-assembly form.  Each iterate is a few applies (within the
apply tests' bound: 1e-12 in FP64, 2e-5 in FP32) and quotients of positive sums of such values,
hence a hundred times that bound.  Without a preconditioner: the operator's diagonal leaves out
the coupling of a wedge's two corners on one node, which the assembled matrix has."""
import numpy as np
import pytest

import seeded_inputs as si
from helpers import TOL, dev, make_op, problem, rel_err, torch_dtype
from test_gpu_halo_sum import ring

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("variant", [5, 6])
@pytest.mark.parametrize("physics", [1, 3])
@pytest.mark.parametrize("mesh", [7, 13, 24, (1, 1, 2), (9, 8, 7), (17, 5, 11)])
def test_open_sum(orc, monkeypatch, mesh, physics, variant, dtype):
    import torch
    import paper_2308_09839_amd as q1
    print(f"\n[open sum] mesh={mesh} physics={physics} variant={variant} dtype={dtype}", flush=True)
    if isinstance(mesh, int):
        monkeypatch.setenv("Q1_BLOCK_SHAPE", "1,1,1")
        xyz, conn = ring(mesh)
        ne = conn.shape[1]
        coef = (si.field_lognormal(ne, 0.0, 1.0, 83)[None] if physics == 1 else
                np.stack(si.lame_from_E_nu(*si.field_elastic(ne, 83))))
        mask = np.zeros(xyz.shape[1], dtype=np.uint8)
        mask[[0, 5, 9]] = 1
        pr = dict(physics=physics, xyz=xyz, conn=conn, coef=coef, mask=mask)
    else:
        pr = problem(physics, mesh, 0.1, 83, True)
    A = orc.assemble(physics, pr["xyz"], pr["conn"], pr["coef"], pr["mask"])
    b = si.vec_uniform(A.n, 83, si.STREAM_RHS)  # Dirichlet rows included
    op = make_op(pr, dtype, variant)
    bd = dev(b, torch_dtype(dtype))
    for k in (1, 2, 4):
        xd = torch.full_like(bd, 3.0)
        st = q1.q1_pcg(op, 0, bd, xd, 0.0, k)
        ref = orc.pcg(A, b, rtol=0.0, maxit=k, jacobi=False)
        assert st["iters"] == k
        assert rel_err(xd.double().cpu().numpy(), ref.x) <= 100 * TOL[dtype], k
