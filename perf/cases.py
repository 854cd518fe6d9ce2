"""The workloads this library's speed is measured on, as plain cases.

A case is a dict of plain values; ``prepare`` builds what a program holds before the call (mesh,
coefficients, operator handle, vectors, network), ``run`` makes one pass through the public entry
points and returns its outputs, ``work`` states the bytes and operations the pass cannot do
without, and ``exact`` recomputes the outputs in 64 bits with plain torch.  Kinds of case:

* ``apply``     y = A x with an operator that is kept: hexahedra of order 1 to 3 and tetrahedra,
                scalar and vector Laplace and elasticity, FP64 and FP32, undistorted and jittered
                box meshes, with and without a Dirichlet face;
* ``pcg``       one FP64 Jacobi-PCG solve;
* ``mpcg``      one mixed FP32/FP64 solve with reliable updates;
* ``batched``   many small problems with several right-hand sides in one launch;
* ``forward``   the learned preconditioner's network, inference on one residual or a few;
* ``gradient``  loss and parameter gradient of the network on a batch (weights kept by an
                optimiser outside the library).
"""
from __future__ import annotations

import math

import numpy as np
import torch
import torch.utils.checkpoint

import paper_2308_09839_amd as q1

_KUHN = ((0, 1, 3, 7), (0, 5, 1, 7), (0, 3, 2, 7), (0, 2, 6, 7), (0, 6, 4, 7), (0, 4, 5, 7))
_ORDER = {8: 1, 27: 2, 64: 3, 4: 1}
_DTYPE = {"f64": (torch.float64, 0, 8), "f32": (torch.float32, 1, 4)}


# ---- the cases ---------------------------------------------------------------------------

def _apply(name, elem, physics, dtype, nx, ny, nz, jitter, fixed, field="iid"):
    c = {"name": name, "kind": "apply", "elem": elem, "physics": physics, "dtype": dtype,
         "nx": nx, "ny": ny, "nz": nz, "jitter": jitter, "fixed": fixed, "field": field}
    if name is None:
        del c["name"]
    return c


def listed():
    return [
        # the smallest problem in use, inside small solves and tests: latency of one call
        _apply("hex8_laplace_16", 8, 1, "f64", 16, 16, 16, 0.1, True),
        # the benchmark's headline apply: undistorted grid, layered coefficient
        _apply("hex8_laplace_128", 8, 1, "f64", 128, 128, 128, 0.0, False, "layered"),
        # a distorted mesh of odd size in single precision: the general element
        _apply("hex8_laplace_jittered_f32", 8, 1, "f32", 117, 93, 71, 0.1, True),
        # the elasticity workload of the mixed-precision solver
        _apply("hex8_elasticity_96", 8, 3, "f64", 96, 96, 96, 0.0, True),
        # simplicial elasticity on a distorted mesh of odd size
        _apply("tet4_elasticity", 4, 3, "f64", 51, 47, 61, 0.1, True),
        # triquadratic and tricubic elements at about two million nodes
        _apply("hex27_laplace_64", 27, 1, "f64", 64, 64, 64, 0.0, True),
        _apply("hex64_laplace_42", 64, 1, "f64", 42, 42, 42, 0.1, True),
        # one scalar solve as a time step or a training-pair harvest makes it
        {"name": "pcg_laplace_64", "kind": "pcg", "physics": 1, "nx": 64, "ny": 64, "nz": 64,
         "jitter": 0.0, "rtol": 1e-10},
        # one elasticity solve in mixed precision
        {"name": "mpcg_elasticity_48", "kind": "mpcg", "physics": 3, "nx": 48, "ny": 48, "nz": 48,
         "jitter": 0.0, "rtol": 1e-10},
        # a batch of small independent problems, four right-hand sides each
        {"name": "batched_12x4", "kind": "batched", "nprob": 12, "nrhs": 4, "lo": 16, "hi": 40,
         "rtol": 1e-10},
        # one network evaluation inside a flexible CG iteration on a 64^3 mesh (65^3 nodes)
        {"name": "network_forward", "kind": "forward", "D": 68, "H": 68, "W": 68, "batch": 1},
        # one training pass on a mini-batch of that grid
        {"name": "network_gradient", "kind": "gradient", "D": 68, "H": 68, "W": 68, "batch": 4},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _edges(rng, lo, hi, cells):
    """Three edge lengths: a cube of a round size in a third of the draws, else unequal and
    mostly odd; at most `cells` elements."""
    if rng.random() < 1 / 3:
        n = max(4, 4 * (_log_int(rng, lo, hi) // 4))
        return (n, n, n) if n ** 3 <= cells else (hi // 2, hi // 2, hi // 2)
    n = _log_int(rng, lo, hi)
    e = [max(lo, min(hi, int(n * rng.uniform(0.7, 1.4)))) for _ in range(3)]
    while e[0] * e[1] * e[2] > cells:
        e = [max(lo, int(0.9 * v)) for v in e]
    return tuple(e)


def draw(rng):
    kind = rng.choices(("apply", "pcg", "mpcg", "batched", "forward", "gradient"),
                       (7, 1, 1, 1, 1, 1))[0]
    if kind == "apply":
        elem = rng.choices((8, 4, 27, 64), (4, 1, 1, 1))[0]
        physics = rng.choice((1, 2, 3) if elem == 8 else (1, 3))
        dtype = rng.choice(("f64", "f64", "f32"))
        jitter = rng.choice((0.0, 0.1))
        vec = physics != 1
        lo, hi, cells = {8: (8, 96 if vec else 128, 96 ** 3 if vec else 128 ** 3),
                         4: (6, 64 if vec else 96, 64 ** 3 if vec else 96 ** 3),
                         27: (4, 40 if vec else 64, 32 ** 3 if vec else 64 ** 3),
                         64: (3, 28 if vec else 42, 21 ** 3 if vec else 42 ** 3)}[elem]
        nx, ny, nz = _edges(rng, lo, hi, cells)
        return _apply(None, elem, physics, dtype, nx, ny, nz, jitter, rng.random() < 0.6)
    if kind in ("pcg", "mpcg"):
        physics = rng.choice((1, 2, 3)) if kind == "pcg" else rng.choice((1, 3))
        nx, ny, nz = _edges(rng, 10, 72 if physics == 1 else 48,
                            64 ** 3 if physics == 1 else 40 ** 3)
        return {"kind": kind, "physics": physics, "nx": nx, "ny": ny, "nz": nz,
                "jitter": rng.choice((0.0, 0.1)), "rtol": 1e-10}
    if kind == "batched":
        lo = rng.randint(9, 18)
        return {"kind": kind, "nprob": rng.randint(4, 14), "nrhs": rng.randint(1, 4), "lo": lo,
                "hi": lo + rng.randint(6, 20), "rtol": 1e-10}
    D, H, W = (4 * rng.randint(4, 17) for _ in range(3))
    return {"kind": kind, "D": D, "H": H, "W": W,
            "batch": 1 if kind == "forward" and rng.random() < 0.5 else rng.randint(1, 4)}


# ---- inputs ------------------------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _uniform(g, n, lo, hi):
    return lo + (hi - lo) * torch.rand(n, generator=g, device="cuda", dtype=torch.float64)


def _mesh(elem, nx, ny, nz, jitter, g):
    """Coordinates [3, nodes] FP64 and connectivity int32 [elem, n] of a box of unit cells whose
    interior vertices move by up to `jitter` per coordinate; the other nodes of higher-order
    elements sit at the trilinear interpolation of their vertices."""
    p = _ORDER[elem]
    ar = lambda n: torch.arange(n, device="cuda")  # noqa: E731
    k, j, i = torch.meshgrid(ar(nz + 1), ar(ny + 1), ar(nx + 1), indexing="ij")
    v = torch.stack([i, j, k]).to(torch.float64)
    if jitter:
        inside = ((i > 0) & (i < nx) & (j > 0) & (j < ny) & (k > 0) & (k < nz)).to(torch.float64)
        v = v + inside * _uniform(g, v.shape, -jitter, jitter)
    if p > 1:
        for axis, n in ((1, nz), (2, ny), (3, nx)):
            I = ar(p * n + 1)
            i0 = torch.clamp(I // p, max=n - 1)
            t = ((I - p * i0).to(torch.float64) / p).reshape([-1 if a == axis else 1 for a in range(4)])
            v = v.index_select(axis, i0) * (1 - t) + v.index_select(axis, i0 + 1) * t
    NX, NY = p * nx + 1, p * ny + 1
    ez, ey, ex = torch.meshgrid(ar(nz), ar(ny), ar(nx), indexing="ij")
    base = (p * ex + NX * (p * ey + NY * (p * ez))).reshape(-1)
    m = p + 1
    off = [(a % m) + NX * ((a // m) % m + NY * (a // (m * m))) for a in range(m ** 3)]
    if elem == 4:
        conn = torch.stack([torch.stack([base + off[c[a]] for c in _KUHN], 1).reshape(-1)
                            for a in range(4)])
    else:
        conn = torch.stack([base + o for o in off])
    return v.reshape(3, -1).contiguous(), conn.to(torch.int32).contiguous()


def _coefficients(physics, ne, cells, field, g):
    if physics == 3:
        E = torch.exp(math.log(10.0) + torch.randn(ne, generator=g, device="cuda", dtype=torch.float64))
        nu = _uniform(g, ne, 0.15, 0.35)
        return torch.stack([E * nu / ((1 + nu) * (1 - 2 * nu)), E / (2 * (1 + nu))])
    k = torch.randn(ne, generator=g, device="cuda", dtype=torch.float64)
    if field == "layered":  # one value per layer of four cells times a factor per cell
        nx, ny, nz = cells
        lay = torch.randn((nz + 3) // 4, generator=g, device="cuda", dtype=torch.float64)
        ez = torch.arange(ne, device="cuda") // ((ne // (nx * ny * nz)) * nx * ny)
        return torch.exp(1.5 * lay[ez // 4] + 0.5 * k)[None]
    return torch.exp(k)[None]


class _Problem:
    """Mesh, coefficients and mask of a box problem on the device, in the case's precision."""

    def __init__(self, c, seed, elem=None, dtype="f64"):
        g = _gen(seed)
        self.elem, self.physics = elem or 8, c["physics"]
        self.n = (c["nx"], c["ny"], c["nz"])
        xyz, self.conn = _mesh(self.elem, *self.n, c["jitter"], g)
        self.nn, self.ne = xyz.shape[1], self.conn.shape[1]
        self.dpn = 1 if self.physics == 1 else 3
        coef = _coefficients(self.physics, self.ne, self.n, c.get("field", "iid"), g)
        self.xyz = xyz.to(_DTYPE[dtype][0])
        self.coef = coef.to(_DTYPE[dtype][0]).contiguous()
        p = _ORDER[self.elem]
        self.mask = None
        if c.get("fixed", True):  # the z = 0 face
            self.mask = torch.zeros(self.nn, dtype=torch.uint8, device="cuda")
            self.mask[:(p * self.n[0] + 1) * (p * self.n[1] + 1)] = 1
        self.v = _uniform(g, self.nn * self.dpn, -1.0, 1.0).to(_DTYPE[dtype][0])
        if c["kind"] != "apply":
            self.v[self.dofs()] = 0

    def dofs(self):
        """Constrained degrees of freedom as a truth vector."""
        if self.mask is None:
            return torch.zeros(self.nn * self.dpn, dtype=torch.bool, device="cuda")
        return self.mask.bool().repeat_interleave(self.dpn)

    def op(self, dtype="f64", variant=0):
        t = _DTYPE[dtype][0]
        return q1.q1_op_create_elem(self.elem, self.physics, _DTYPE[dtype][1], variant,
                                    self.xyz.to(t), self.conn, self.coef.to(t), self.mask)


def _batch(c, seed):
    n = c["nprob"]
    edges = [c["lo"] + (c["hi"] - c["lo"]) * i // max(1, n - 1) for i in range(n)]
    probs = []
    for i, e in enumerate(edges):
        p = _Problem({"kind": "batched", "physics": 1, "nx": e, "ny": e, "nz": e, "jitter": 0.0},
                     seed * 1000 + i)
        g = _gen(seed * 1000 + 500 + i)
        p.b = _uniform(g, (c["nrhs"], p.nn), -1.0, 1.0)
        p.b[:, p.mask.bool()] = 0
        probs.append(p)
    return probs


# the network's layers: input channels, output channels (weights [27][in][out], then the bias)
_CONVS = ((2, 16), (16, 16), (16, 32), (32, 32), (32, 64), (64, 64), (96, 32), (32, 32), (48, 16),
          (16, 16))


def _network(c, seed):
    """He-normal parameters, one encoded residual per sample (unit RMS) beside a smooth
    coefficient channel, a target of unit RMS and its weights (zero on the z = 0 face and on
    the grid's last plane, which pads the nodes)."""
    g = _gen(seed)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda")  # noqa: E731
    theta = []
    for ci, co in _CONVS:
        theta += [rnd(27 * ci * co) * math.sqrt(2.0 / (27 * ci)), 0.05 * rnd(co)]
    theta += [rnd(16) * 0.25, 0.05 * rnd(1)]
    shape = (c["batch"], c["D"], c["H"], c["W"])
    inp = torch.zeros(shape + (8,), dtype=torch.bfloat16, device="cuda")
    weight = torch.ones(shape, device="cuda")
    weight[:, 0] = weight[:, -1] = weight[:, :, -1] = weight[:, :, :, -1] = 0
    inp[..., 0] = (rnd(*shape) * weight).to(torch.bfloat16)
    inp[..., 1] = (0.35 * rnd(*shape)).to(torch.bfloat16)
    return torch.cat(theta), inp, rnd(*shape) * weight, weight


def prepare(case, seed):
    c, kind = case, case["kind"]
    s = {"kind": kind, "case": dict(c)}
    if kind == "apply":
        p = _Problem(c, seed, c["elem"], c["dtype"])
        s.update(op=p.op(c["dtype"]), x=p.v, y=torch.empty_like(p.v))
    elif kind in ("pcg", "mpcg"):
        p = _Problem(c, seed)
        s.update(op=p.op(), b=p.v, x=torch.empty_like(p.v))
        if kind == "mpcg":
            s["op32"] = p.op("f32")
    elif kind == "batched":
        probs = _batch(c, seed)
        s["ops"] = [p.op(variant=q1.Q1_V_LDS_TILE) for p in probs]
        s["b"] = [list(p.b) for p in probs]
        s["x"] = [torch.empty_like(p.b) for p in probs]
        s["rows"] = [list(x) for x in s["x"]]
    else:
        theta, s["inp"], s["target"], s["weight"] = _network(c, seed)
        s["net"] = q1.q1_unet_create(c["D"], c["H"], c["W"], c["batch"], 0)
        s["net"].set_params(theta)
        s["theta"] = theta
        s["out"] = torch.empty_like(s["target"])
        s["dout"] = torch.empty_like(s["target"])
        s["loss"] = torch.zeros(1, device="cuda")
    return s


def run(s):
    kind, c = s["kind"], s["case"]
    if kind == "apply":
        s["op"].apply(s["x"], s["y"])
        return s["y"]
    if kind == "pcg":
        q1.q1_pcg(s["op"], q1.Q1_PC_JACOBI, s["b"], s["x"], c["rtol"], 20000)
        return s["x"]
    if kind == "mpcg":
        q1.q1_mpcg(s["op"], s["op32"], s["b"], s["x"], c["rtol"])
        return s["x"]
    if kind == "batched":
        q1.q1_batched_pcg(s["ops"], s["b"], s["rows"], c["rtol"], 20000)
        return s["x"]
    net = s["net"]
    if kind == "forward":
        net.forward(s["inp"], s["out"], c["batch"])
        return s["out"]
    net.set_params(s["theta"])
    net.forward(s["inp"], s["out"], c["batch"])
    net.mse(s["out"], s["target"], s["weight"], s["dout"], s["loss"])
    net.backward(s["dout"])
    return {"loss": s["loss"], "out": s["out"], "gradient": net.get(1)}


# ---- what a pass cannot do without -------------------------------------------------------

def _apply_work(elem, physics, real, n, jitter, fixed):
    """Each input read once and the result written once; operations of the sum-factorised
    element (a constant-Jacobian hexahedron needs only its closed form on the modes)."""
    p = _ORDER[elem]
    nn = math.prod(p * v + 1 for v in n)
    ne = math.prod(n) * (6 if elem == 4 else 1)
    dpn = 1 if physics == 1 else 3
    ncoef = 2 if physics == 3 else 1
    by = ne * (4 * elem + ncoef * real) + nn * (3 + 2 * dpn) * real + (nn if fixed else 0)
    if elem == 4:
        fl = {1: 80, 2: 140, 3: 170}[physics]
    elif elem == 8:
        fl = {1: 1070, 2: 1900, 3: 2070}[physics] if jitter else {1: 100, 2: 260, 3: 420}[physics]
    else:
        m = p + 1  # three 1-D passes per field, forward for coordinates and input, back once
        fl = 2 * 8 * m ** 4 * (3 + 2 * dpn) + m ** 3 * (70 + 40 * dpn)
    return float(by), float(ne * fl)


def _iterations(c):
    """About the Jacobi-PCG iterations to 1e-10 on these problems (they grow with the edge)."""
    if c["kind"] == "batched":
        return 7.5
    return {1: 7.5, 2: 7.5, 3: 28.0}[c["physics"]]


def work(case):
    c, kind = case, case["kind"]
    if kind == "apply":
        by, fl = _apply_work(c["elem"], c["physics"], _DTYPE[c["dtype"]][2],
                             (c["nx"], c["ny"], c["nz"]), c["jitter"], c["fixed"])
    elif kind in ("pcg", "mpcg"):
        n = (c["nx"], c["ny"], c["nz"])
        it = _iterations(c) * max(n)
        by, fl = _apply_work(8, c["physics"], 8 if kind == "pcg" else 4, n, c["jitter"], True)
        dof = math.prod(v + 1 for v in n) * (1 if c["physics"] == 1 else 3)
        # x, r updated, the inverse diagonal, p and q read, p written
        by, fl = it * (by + dof * (9 if kind == "pcg" else 7) * 8), it * (fl + 12 * dof)
    elif kind == "batched":
        by = fl = 0.0
        for i in range(c["nprob"]):
            e = c["lo"] + (c["hi"] - c["lo"]) * i // max(1, c["nprob"] - 1)
            b, f = _apply_work(8, 1, 8, (e, e, e), 0.0, True)
            nn = (e + 1) ** 3
            it = _iterations(c) * e
            by += it * (b + (c["nrhs"] - 1) * nn * 16 + c["nrhs"] * nn * 72)
            fl += it * c["nrhs"] * (f + 12 * nn)
    else:
        v = c["batch"] * c["D"] * c["H"] * c["W"]
        level = (1, 1, 8, 8, 64, 64, 8, 8, 1, 1)
        macs = sum(27 * ci * co * v / l for (ci, co), l in zip(_CONVS, level)) + 16 * v
        npar = sum(27 * ci * co + co for ci, co in _CONVS) + 17
        by, fl = 20.0 * v + 4 * npar, 2 * macs
        if kind == "gradient":  # backward in the data and in the weights
            fl = 3 * fl - 2 * 27 * 2 * 16 * v
            by += 12.0 * v + 4 * npar
    return {"bytes": by, "flops": fl}


# ---- the outputs in 64 bits --------------------------------------------------------------

def _shape(elem):
    """Weights [q] and shape gradients [q, node, 3] at the element's quadrature points."""
    if elem == 4:
        d = torch.tensor([[-1., -1, -1], [1, 0, 0], [0, 1, 0], [0, 0, 1]])
        return torch.tensor([1 / 6.], dtype=torch.float64, device="cuda"), d.double().cuda()[None]
    p = _ORDER[elem]
    m = p + 1
    gx, gw = np.polynomial.legendre.leggauss(m)
    t = np.linspace(-1, 1, m)
    N, D = np.zeros((m, m)), np.zeros((m, m))
    for a in range(m):
        e = np.poly1d([1.0])
        for b in range(m):
            if b != a:
                e = e * np.poly1d([1.0, -t[b]]) / (t[a] - t[b])
        N[:, a], D[:, a] = e(gx), e.deriv()(gx)
    q = [(i, j, k) for k in range(m) for j in range(m) for i in range(m)]
    w = np.array([gw[i] * gw[j] * gw[k] for i, j, k in q])
    d = np.array([[[D[i, a] * N[j, b] * N[k, c], N[i, a] * D[j, b] * N[k, c],
                    N[i, a] * N[j, b] * D[k, c]] for a, b, c in q] for i, j, k in q])
    return torch.from_numpy(w).cuda(), torch.from_numpy(d).cuda()


def _inverse(J):
    """Cofactor inverse and determinant of [..., 3, 3]."""
    a, b, c = J[..., 0, :], J[..., 1, :], J[..., 2, :]
    adj = torch.stack([torch.linalg.cross(b, c), torch.linalg.cross(c, a),
                       torch.linalg.cross(a, b)], -1)
    det = (a * adj[..., :, 0]).sum(-1)
    return adj / det[..., None, None], det


def _exact_apply(p, x):
    w, d = _shape(p.elem)
    nq, na = d.shape[:2]
    dm = d.permute(1, 0, 2).reshape(na, nq * 3).contiguous()  # [node, (q, ref axis)]
    free = x.masked_fill(p.dofs(), 0.0).reshape(p.nn, p.dpn)
    y = torch.zeros_like(free)
    step = max(1, 24_000_000 // (nq * 9 * 6))
    for e0 in range(0, p.ne, step):
        cn = p.conn[:, e0:e0 + step].long()
        X = p.xyz[:, cn].double().permute(2, 0, 1)  # [e, 3, node]
        ne = X.shape[0]
        J = (X.reshape(-1, na) @ dm).reshape(ne, 3, nq, 3).transpose(1, 2)  # [e, q, x_r, xi_c]
        inv, det = _inverse(J)
        u = free[cn].permute(1, 2, 0)  # [e, comp, node]
        G = (u.reshape(-1, na) @ dm).reshape(ne, p.dpn, nq, 3).transpose(1, 2)
        H = G @ inv  # physical gradients [e, q, comp, 3]
        cf = p.coef[:, e0:e0 + step].double()
        if p.physics == 3:
            tr = H.diagonal(dim1=-2, dim2=-1).sum(-1)
            S = cf[1][:, None, None, None] * (H + H.transpose(-1, -2))
            S = S + (cf[0][:, None] * tr)[..., None, None] * torch.eye(3, device="cuda", dtype=torch.float64)
        else:
            S = cf[0][:, None, None, None] * H
        F = (S @ inv.transpose(-1, -2)) * (det * w)[..., None, None]  # [e, q, comp, xi]
        r = F.transpose(1, 2).reshape(ne * p.dpn, nq * 3) @ dm.t().contiguous()
        y.index_add_(0, cn.t().reshape(-1), r.reshape(ne, p.dpn, na).transpose(1, 2).reshape(-1, p.dpn))
    y = y.reshape(-1)
    return torch.where(p.dofs(), x, y)


def _matrices(p):
    """Element matrices [e, na * dpn, na * dpn], node-major."""
    w, d = _shape(p.elem)
    na = d.shape[1]
    n = na * p.dpn
    K = torch.zeros((p.ne, n, n), dtype=torch.float64, device="cuda")
    X = p.xyz.double()[:, p.conn.long()].permute(2, 0, 1)
    cf = p.coef.double()
    eye = torch.eye(3, dtype=torch.float64, device="cuda")
    for q in range(len(w)):
        inv, det = _inverse(X @ d[q])
        B = d[q] @ inv  # [e, node, 3] physical gradients
        wd = (w[q] * det)[:, None, None]
        L = B @ B.transpose(1, 2)
        if p.physics == 1:
            K += cf[0][:, None, None] * wd * L
        elif p.physics == 2:
            K += ((cf[0][:, None, None] * wd * L)[:, :, None, :, None] * eye[None, None, :, None, :]).reshape(-1, n, n)
        else:
            f = B.reshape(-1, n)
            K += cf[0][:, None, None] * wd * (f[:, :, None] * f[:, None, :])
            m = (cf[1][:, None, None] * wd)[:, :, None, :, None]
            K += (m * (L[:, :, None, :, None] * eye[None, None, :, None, :]
                       + B[:, :, None, None, :] * B[:, None, :, :, None].transpose(2, 3))).reshape(-1, n, n)
    return K


def _exact_solve(p, b):
    """Jacobi-CG on the element matrices, to the rounding of 64 bits; b: [rhs, dof]."""
    K = _matrices(p)
    c = p.conn.t().long()
    idx = (c[:, :, None] * p.dpn + torch.arange(p.dpn, device="cuda")).reshape(p.ne, -1)
    flat, free = idx.reshape(-1), (~p.dofs()).double()
    xs = []
    diag = torch.zeros(p.nn * p.dpn, dtype=torch.float64, device="cuda")
    diag.index_add_(0, flat, K.diagonal(dim1=1, dim2=2).reshape(-1))
    inv = torch.where(diag != 0, 1 / diag, torch.zeros_like(diag)) * free
    for row in b:
        x, r = torch.zeros_like(row), row * free
        z = inv * r
        d, rz, stop = z.clone(), r @ z, 1e-14 * row.norm()
        for it in range(20000):
            q = torch.zeros_like(d)
            q.index_add_(0, flat, (K @ d[idx][:, :, None]).reshape(-1))
            q *= free
            a = rz / (d @ q)
            x += a * d
            r -= a * q
            z = inv * r
            new = r @ z
            d = z + (new / rz) * d
            rz = new
            if it % 64 == 63 and bool(r.norm() <= stop):
                break
        xs.append(x)
    return torch.stack(xs)


def _exact_network(c, seed, grad):
    theta, inp, target, weight = _network(c, seed)
    th = theta.double().requires_grad_(grad)
    W, o = [], 0
    for ci, co in _CONVS:
        n = 27 * ci * co
        W.append((th[o:o + n].reshape(27, ci, co), th[o + n:o + n + co]))
        o += n + co
    head, hb = th[o:o + 16], th[o + 16]
    taps = [(z, y, x) for z in range(3) for y in range(3) for x in range(3)]

    def conv(x, l):
        w, b = W[l]

        def f(x, w, b):
            D, H, V = x.shape[:3]
            xp = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1, 1, 1))
            y = b
            for t, (dz, dy, dx) in enumerate(taps):
                y = y + xp[dz:dz + D, dy:dy + H, dx:dx + V] @ w[t]
            return torch.relu(y)
        if not grad:
            return f(x, w, b)
        return torch.utils.checkpoint.checkpoint(f, x, w, b, use_reentrant=False)

    def pool(x):
        D, H, V, C = x.shape
        return x.reshape(D // 2, 2, H // 2, 2, V // 2, 2, C).mean((1, 3, 5))

    def up(x):
        for a in range(3):
            x = x.repeat_interleave(2, a)
        return x

    outs, loss, total = [], 0.0, weight.double().sum()
    for s in range(c["batch"]):
        s1 = conv(conv(inp[s, ..., :2].double(), 0), 1)
        s2 = conv(conv(pool(s1), 2), 3)
        b3 = conv(conv(pool(s2), 4), 5)
        t2 = conv(conv(torch.cat([up(b3), s2], -1), 6), 7)
        t1 = conv(conv(torch.cat([up(t2), s1], -1), 8), 9)
        out = t1 @ head + hb
        if grad:
            part = (weight[s].double() * (out - target[s].double()) ** 2).sum() / total
            part.backward()
            loss = loss + part.detach()
        outs.append(out.detach())
    out = torch.stack(outs)
    return {"loss": loss.reshape(1), "out": out, "gradient": th.grad} if grad else out


def exact(case, seed):
    c, kind = case, case["kind"]
    if kind == "apply":
        p = _Problem(c, seed, c["elem"], c["dtype"])
        return _exact_apply(p, p.v.double())
    if kind in ("pcg", "mpcg"):
        p = _Problem(c, seed)
        return _exact_solve(p, p.v[None])[0]
    if kind == "batched":
        return [_exact_solve(p, p.b) for p in _batch(c, seed)]
    return _exact_network(c, seed, kind == "gradient")
