"""The batched solver's workgroups: one to four right-hand sides (lanes take one side of a node,
three leave a lane of each wave idle), problems of one tile beside larger ones, four waves per
workgroup on parallelepiped tiles and one on general ones, Dirichlet rows with a right-hand
side, nodes on many tiles and nodes on none, and more problems than four-wave workgroups fit on
the device.  The iterates after a few iterations are compared with q1_pcg on the same operators:
each is a few applies (within 1e-12) and quotients of positive sums of them, hence 1e-10."""
import numpy as np
import pytest

import seeded_inputs as si
from helpers import dev, make_op, problem, rel_err
from test_gpu_halo_sum import ring

pytestmark = pytest.mark.gpu

V_LDS_TILE = 3


def meshes(kind):
    if kind == "ring":
        out = []
        for m in (7, 24):
            xyz, conn = ring(m)
            mask = np.zeros(xyz.shape[1], dtype=np.uint8)
            mask[[0, 5, 9]] = 1
            coef = si.field_lognormal(conn.shape[1], 0.0, 1.0, 85)[None]
            out.append(dict(physics=1, xyz=xyz, conn=conn, coef=coef, mask=mask))
        return out
    jitter = 0.1 if kind == "general" else 0.0
    out = [problem(1, n, jitter, 85, True) for n in ((1, 1, 1), (17, 9, 5), (6, 7, 8))]
    p = out[1]  # two nodes that no element references
    p["xyz"] = np.concatenate([p["xyz"], np.full((3, 2), 9.0)], axis=1)
    p["mask"] = np.concatenate([p["mask"], np.zeros(2, dtype=p["mask"].dtype)])
    return out


def rhs(pr, c):
    b = si.vec_uniform(pr["xyz"].shape[1], 85 + c, si.STREAM_RHS)  # Dirichlet rows included
    used = np.zeros(b.size, dtype=bool)
    used[np.unique(pr["conn"])] = True
    b[~used] = 0.0
    return b


@pytest.mark.parametrize("kind", ["box", "general", "ring"])
@pytest.mark.parametrize("nrhs", [1, 2, 3, 4])
def test_batched_groups(nrhs, kind):
    import torch
    import paper_2308_09839_amd as q1
    print(f"\n[batched groups] nrhs={nrhs} kind={kind}", flush=True)
    prs = meshes(kind)
    ops = [make_op(pr, 0, V_LDS_TILE) for pr in prs]
    bs = [[dev(rhs(pr, c)) for c in range(nrhs)] for pr in prs]
    for k in (1, 2, 5):
        xs = [[torch.full_like(b, 3.0) for b in row] for row in bs]
        st = q1.q1_batched_pcg(ops, bs, xs, 1e-30, k)
        for i, op in enumerate(ops):
            for c in range(nrhs):
                ref = torch.empty_like(bs[i][c])
                r = q1.q1_pcg(op, 1, bs[i][c], ref, 1e-30, k)
                assert st[i * nrhs + c]["iters"] <= k
                if prs[i]["conn"].shape[1] == 1 or r["status"] not in (0, -4):
                    continue  # solved to rounding: the last iterates are noise
                err = rel_err(xs[i][c].cpu().numpy(), ref.cpu().numpy())
                assert err <= 1e-10, (k, i, c, err)


def test_more_problems_than_four_wave_groups():
    import torch
    import paper_2308_09839_amd as q1
    print("\n[batched groups, 1000 problems]", flush=True)
    pr = problem(1, (3, 2, 2), 0.0, 86, True)
    op = make_op(pr, 0, V_LDS_TILE)
    n = 1000  # above three four-wave workgroups on each of 256 compute units
    bs = [[dev(rhs(pr, i))] for i in range(n)]
    xs = [[torch.full_like(b[0], 3.0)] for b in bs]
    st = q1.q1_batched_pcg([op] * n, bs, xs, 1e-10, 200)
    assert all(s["status"] == 0 for s in st)
    for i in (0, 1, 511, 999):
        ref = torch.empty_like(bs[i][0])
        assert q1.q1_pcg(op, 1, bs[i][0], ref, 1e-10, 200)["status"] == 0
        assert rel_err(xs[i][0].cpu().numpy(), ref.cpu().numpy()) <= 1e-8
