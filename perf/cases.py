"""Performance cases of the monodomain solver: time steps, solves and adjoint steps.

A case is one call (or the few calls of one reverse step) of the Python binding on a synthetic mesh.
`prepare` makes what a simulation holds before it: the solver of the mesh, set up once and kept, and a
state with an excitation front whose place and radius the seed draws.  `run` is one pass, started from
that saved state (one copy), so that every pass does the same work.  `exact` computes the same step in
plain FP64 torch: quadrature sums of the bilinear form and conjugate gradients, no multigrid.
"""
import functools
import math

import numpy as np
import torch

from paper_2602_16312_amd import api

DEV = "cuda"
COLS = 8
BO = [6.0, 6.0, 43.0, 0.2, 2.8723, 0.11, 1.4506, 60.0, 1150.0, 70.0, 20.0, 2.7342, 3.0, 280.0, 0.07, 65.0,
      2.0994, 2.0, 0.94, 0.3, 0.015, 0.015, 0.03, 0.9087, 1.58, 0.006, 0.65, 0.0]
# model: (name, parameters, gates, chi, Cm, dt, conductivity along and across the fibres)
MODELS = {
    "fhn": ("fhn", [19.5, 0.13, 0.01, 0.5], 1, 1.0, 1.0, 1e-2, 1e-3, 1e-3),
    "fhn_si": ("fhn", [19.5, 0.013, 40.0, 0.1], 1, 1e5, 1e-2, 1e-4, 0.12, 0.12),
    "ap": ("ap", [8.0, 0.15, 0.002], 1, 1.0, 1.0, 1e-2, 1e-3, 1e-3),
    "bo": ("bo", BO, 3, 1.0, 1.0, 5e-2, 1.2e-3, 2.5e-4),
}
BASE = dict(what="step", mesh="square", n=0, h=0.0, jitter=0.0, p=1, model="ap", precision="mixed",
            jacobi="point", tol=1e-8, tol_mode="rel_r0")


def _case(**kw):
    return {**BASE, **kw}


def listed():
    return [
        # the smallest simulation: a 32x32 Q1 square in FP64, launches and latency only
        _case(name="square_q1_small", n=32, model="fhn", precision="fp64", tol=1e-10),
        # the 2D workload of the benchmark: a 256x256 jittered Q2 square, both precisions
        _case(name="square_q2_mixed", n=256, jitter=0.2, p=2),
        _case(name="square_q2_fp64", n=256, jitter=0.2, p=2, precision="fp64"),
        # higher degree, a size whose agglomerates are uneven
        _case(name="square_q3_ragged", n=150, jitter=0.1, p=3),
        # the paper's 2D test at its highest degree: boxes, SI units, an absolute tolerance
        _case(name="square_q4_boxes", n=128, p=4, model="fhn_si", precision="fp64", tol=1e-14, tol_mode="abs"),
        # the 3D workload on boxes: a 64^3 Q2 cube with rotating fibres
        _case(name="cube_q2_boxes", mesh="cube", n=64, p=2, model="bo"),
        # a distorted Q2 cube of odd size: stored blocks
        _case(name="cube_q2_jittered", mesh="cube", n=27, jitter=0.1, p=2, model="bo"),
        # one solve from a zero guess in FP64 at the highest 3D degree
        _case(name="cube_q3_solve", what="solve", mesh="cube", n=16, p=3, model="bo", precision="fp64"),
        # the ventricle-like shell of about a million hexahedra
        _case(name="shell_q1_mixed", mesh="shell", h=0.0147, jitter=0.15, model="bo"),
        # a smaller shell with the cell-block smoother, the faster option there
        _case(name="shell_q1_block", mesh="shell", h=0.03, jitter=0.15, model="bo", jacobi="cell_block"),
        # eight stimulus sites stepped together
        _case(name="shell_q1_8col", what="step_multi", mesh="shell", h=0.02, jitter=0.15, model="bo"),
        # one reverse step of the conductivity gradient, FP64 at the adjoint's tolerance
        _case(name="square_q2_adjoint", what="adjoint", n=256, jitter=0.2, p=2, precision="fp64", tol=1e-13),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    prec = rng.choice(["mixed", "mixed", "fp64"])
    k = rng.randrange(10)
    if k == 0:
        return _case(n=round(_log(rng, 16, 512)), model="fhn", precision=prec, tol=1e-10)
    if k == 1:
        return _case(n=round(_log(rng, 24, 400)), jitter=0.2, p=2, precision=prec)
    if k == 2:
        return _case(n=round(_log(rng, 24, 256)), jitter=0.1, p=3, precision=prec)
    if k == 3:
        return _case(n=round(_log(rng, 20, 160)), p=rng.choice([2, 3, 4]), model="fhn_si", precision="fp64", tol=1e-14,
                     tol_mode="abs")
    if k == 4:
        return _case(mesh="cube", n=round(_log(rng, 10, 64)), p=2, model="bo", precision=prec)
    if k == 5:
        return _case(mesh="cube", n=round(_log(rng, 8, 36)), jitter=0.1, p=2, model="bo", precision=prec)
    if k == 6:
        return _case(what="solve", mesh="cube", n=round(_log(rng, 5, 24)), p=3, model="bo", precision=prec)
    if k == 7:
        return _case(mesh="shell", h=round(_log(rng, 0.0148, 0.08), 4), jitter=0.15, model="bo", precision=prec,
                     jacobi=rng.choice(["point", "cell_block"]))
    if k == 8:
        return _case(what="step_multi", mesh="shell", h=round(_log(rng, 0.02, 0.08), 4), jitter=0.15, model="bo",
                     precision=prec)
    return _case(what="adjoint", n=round(_log(rng, 24, 256)), jitter=0.2, p=2, precision="fp64", tol=1e-13)


# ---------------------------------------------------------------- meshes

def _grid(dim, n, jitter):
    """n^dim cells of the unit box, x fastest; interior vertices displaced by up to jitter h."""
    ax = np.arange(n + 1) / n
    idx = np.stack([g.ravel() for g in np.meshgrid(*[np.arange(n + 1)] * dim, indexing="ij")][::-1], axis=1)
    xyz = ax[idx]
    if jitter:
        d = np.random.default_rng(2602).uniform(-jitter / n, jitter / n, xyz.shape)
        xyz = xyz + np.where((idx > 0) & (idx < n), d, 0.0)
    ijk = np.stack([g.ravel() for g in np.meshgrid(*[np.arange(n)] * dim, indexing="ij")][::-1], axis=1)
    stride = (n + 1) ** np.arange(dim)
    v0 = ijk @ stride
    cells = np.stack([v0 + sum(stride[k] for k in range(dim) if c >> k & 1) for c in range(2 ** dim)], axis=1)
    return xyz, cells.astype(np.int64)


OUTER, INNER = np.array([1.0, 1.0, 2.5]), np.array([0.7, 0.7, 2.0])


def _shell(h, jitter):
    """Voxels of spacing h between two half ellipsoids (z < 0); interior vertices displaced."""
    n = np.ceil(np.array([2.0, 2.0, 2.5]) / h).astype(int)
    lo = -OUTER
    c = [lo[k] + (np.arange(n[k]) + 0.5) * h for k in range(3)]
    X, Y, Z = c[0][None, None, :], c[1][None, :, None], c[2][:, None, None]
    level = lambda e: (X / e[0]) ** 2 + (Y / e[1]) ** 2 + (Z / e[2]) ** 2
    sel = (level(OUTER) <= 1.0) & (level(INNER) > 1.0) & (Z <= 0.0)
    ijk = np.stack(np.nonzero(sel)[::-1], axis=1)
    stride = np.array([1, n[0] + 1, (n[0] + 1) * (n[1] + 1)])
    corner = np.array([[c & 1, c >> 1 & 1, c >> 2] for c in range(8)])
    gid = ijk @ stride
    gid = gid[:, None] + (corner @ stride)[None]
    used, inv, count = np.unique(gid, return_inverse=True, return_counts=True)
    cells = inv.reshape(gid.shape).astype(np.int64)
    v = np.stack([used % stride[1], used // stride[1] % (n[1] + 1), used // stride[2]], axis=1)
    d = np.random.default_rng(2603).uniform(-jitter * h, jitter * h, v.shape)
    return lo + v * h + np.where((count == 8)[:, None], d, 0.0), cells


def _conductivity(case, cen):
    """Packed per-cell tensors st I + (sl - st) f f^T: fibres rotate from -60 to 60 degrees."""
    sl, st = MODELS[case["model"]][6:]
    n, d = cen.shape
    if d == 2:
        return np.tile([sl, 0.0, sl], (n, 1))
    if case["mesh"] == "cube":
        th = np.deg2rad(120.0 * cen[:, 2] - 60.0)
        f = np.stack([np.cos(th), np.sin(th), 0 * th], axis=1)
    else:
        mid = 0.5 * (OUTER + INNER)
        th = np.deg2rad(60.0 * np.clip(6.0 * (np.linalg.norm(cen / mid, axis=1) - 1.0), -1.0, 1.0))
        e = np.stack([-cen[:, 1], cen[:, 0], 0 * th], axis=1)
        e /= np.maximum(np.linalg.norm(e, axis=1), 1e-12)[:, None]
        nv = cen / mid ** 2
        nv /= np.linalg.norm(nv, axis=1)[:, None]
        f = np.cos(th)[:, None] * e + np.sin(th)[:, None] * np.cross(nv, e)
    D = st * np.eye(3) + (sl - st) * f[:, :, None] * f[:, None, :]
    return np.stack([D[:, a, b] for a in range(3) for b in range(a, 3)], axis=1)


def _bins(case, dim):
    """Bins per axis of the grid-grouped levels: factors of 4 in 2D and 2 in 3D from the coarsest level up."""
    f, most = (4, 16) if dim == 2 else (2, 4 if case["p"] == 3 else 8)
    c, k = case["n"], 0
    while c > most or (dim == 2 and c // f >= 8):
        c, k = c // f, k + 1
    if k == 0:
        c, k = max(1, case["n"] // f), 1
    return [[1, 1, 1]] + [[c * f ** (k - l)] * dim + [1] * (3 - dim) for l in range(1, k + 1)]


def _gauss(q):
    x, w = np.polynomial.legendre.leggauss(q)
    return 0.5 * (x + 1.0), 0.5 * w


def _lobatto(p):
    inner = np.polynomial.legendre.Legendre.basis(p).deriv().roots()
    return 0.5 * (np.concatenate([[-1.0], np.sort(np.real(inner)), [1.0]]) + 1.0)


def _lagrange(p, x):
    """Values and derivatives [len(x), p+1] of the Lagrange basis on the Gauss-Lobatto nodes."""
    t = _lobatto(p)
    v, d = np.ones((len(x), p + 1)), np.zeros((len(x), p + 1))
    for j in range(p + 1):
        others = [m for m in range(p + 1) if m != j]
        for m in others:
            v[:, j] *= (x - t[m]) / (t[j] - t[m])
            term = np.full(len(x), 1.0 / (t[j] - t[m]))
            for o in others:
                if o != m:
                    term *= (x - t[o]) / (t[j] - t[o])
            d[:, j] += term
    return v, d


def _tensor(tables):
    """Product of 1D tables [q_k, m_k], x fastest in both indices."""
    out = tables[0]
    for t in tables[1:]:
        out = np.einsum("ab,cd->cadb", out, t).reshape(t.shape[0] * out.shape[0], -1)
    return out


class _Program:
    """What a program keeps for one mesh: the solver and the nodes' positions."""

    def __init__(self, case, with_solver=True):
        dim = 2 if case["mesh"] == "square" else 3
        xyz, cells = _shell(case["h"], case["jitter"]) if case["mesh"] == "shell" else _grid(dim, case["n"], case["jitter"])
        name, par, self.S, self.chi, self.Cm, self.dt = MODELS[case["model"]][:6]
        self.dim, self.p, self.xyz, self.cells = dim, case["p"], xyz, cells
        self.D = _conductivity(case, xyz[cells].mean(axis=1))
        self.name, self.par = name, np.array(par)
        self.nc, self.b = len(cells), (self.p + 1) ** dim
        self.N = self.nc * self.b
        # boxes take the paper's penalty, distorted cells twice that
        self.penalty = ("fixed", 10.0 * case["n"]) if case["model"] == "fhn" else ("paper",) if not case["jitter"] else ("paper", 2.0)
        X = torch.from_numpy(xyz).to(DEV)[torch.from_numpy(cells).to(DEV)]
        t = _lobatto(self.p)
        corners = torch.from_numpy(_tensor([np.stack([1 - t, t], axis=1)] * dim)).to(DEV)
        self.nodes = torch.matmul(corners, X).reshape(self.N, dim)
        rng = np.random.default_rng(2605)
        self.sensor_cells = np.sort(rng.choice(self.nc, min(64, self.nc), replace=False)).astype(np.int64)
        self.sensor_ref = rng.uniform(0.0, 1.0, (len(self.sensor_cells), dim))
        if not with_solver:
            return
        if case["mesh"] == "shell":
            levels = 1
            while self.nc / 8.0 ** (levels - 1) > 300 and levels < 5:
                levels += 1
            hier = api.build_hierarchy(xyz, cells, levels, method="rtree_str", fanout=8)
        else:
            bins = _bins(case, dim)
            hier = api.build_hierarchy(xyz, cells, len(bins), method="grid", grid_bins=bins)
        multi, adj = case["what"] == "step_multi", case["what"] == "adjoint"
        self.solver = api.setup_levels(hier, self.p, self.D, self.chi, self.Cm, self.dt, name, self.par,
                                       penalty=self.penalty, precision=case["precision"], setup="device",
                                       allocator="torch", jacobi=case["jacobi"], max_rhs=COLS if multi else 1,
                                       mfma=multi, adjoint=adj)
        if adj:
            api.set_sensors(self.solver, self.sensor_cells, self.sensor_ref)


@functools.lru_cache(maxsize=12)
def _program(items):
    return _Program(dict(items))


def _key(case):
    """The part of a case that its solver depends on."""
    return tuple(sorted((k, v) for k, v in case.items() if k not in ("name", "tol", "tol_mode")))


def _inputs(case, P, seed):
    """The state before the call, from the seed: an excitation front around a drawn point."""
    g = np.random.default_rng(int(seed))
    cols = COLS if case["what"] == "step_multi" else 1
    dt_r = 0.002
    width = max(0.02, 0.6 * (case["h"] or 1.0 / case["n"]))
    parts = {k: [] for k in ("U", "Uprev", "W", "Wprev", "iapp")}
    for _ in range(cols):
        at = P.nodes[int(g.integers(P.N))]
        rho = float(g.uniform(0.12, 0.3))
        r = torch.linalg.norm(P.nodes - at, dim=1)
        front = lambda shift, w: torch.sigmoid((rho - shift - r) / w)
        parts["U"].append(front(0.0, width))
        parts["Uprev"].append(front(dt_r, width))
        for key, lag in (("W", 0.08), ("Wprev", 0.08 + dt_r)):
            s = front(lag, 0.03)
            gates = {"fhn": [0.2 * s], "ap": [0.5 * s], "bo": [1.0 - s, 1.0 - 0.4 * s, 0.7 * s]}[P.name]
            parts[key].append(torch.stack(gates))
        inside = (r.reshape(P.nc, P.b).mean(dim=1) < 0.5 * rho).double()   # a stimulus is per cell
        parts["iapp"].append(0.3 * inside.repeat_interleave(P.b))
    out = {k: torch.stack(v, dim=-1) for k, v in parts.items()}
    if cols == 1:
        out = {k: v.squeeze(-1) for k, v in out.items()}
    if P.name != "bo":
        out["iapp"] = None
    if case["what"] == "solve":
        gen = torch.Generator(device=DEV).manual_seed(int(seed))
        out = {"b": out["U"] + 0.1 * torch.randn(P.N, dtype=torch.float64, device=DEV, generator=gen)}
    if case["what"] == "adjoint":
        # the adjoints that later steps handed back are smooth fields of the front's size
        out["Unew"] = 2.0 * out["U"] - out["Uprev"]
        bars = torch.sin(9.0 * P.nodes @ torch.from_numpy(g.uniform(-1.0, 1.0, (2, 6))).to(DEV)) * out["U"][:, None]
        for k, name in enumerate(("Ub_new", "Wb_new", "Ub", "Ub_prev", "Wb", "Wb_prev")):
            out[name] = bars[:, k].contiguous()
        out["target"] = torch.from_numpy(g.uniform(0.0, 1.0, len(P.sensor_cells))).to(DEV)
    return {k: None if v is None else v.contiguous() for k, v in out.items()}


class _State:
    """Views of one flat buffer that a pass starts by restoring."""

    def __init__(self, tensors):
        sizes = [t.numel() for t in tensors]
        self.saved = torch.cat([t.reshape(-1) for t in tensors])
        self.flat = torch.empty_like(self.saved)
        self.views = [v.view(t.shape) for v, t in zip(self.flat.split(sizes), tensors)]

    def restore(self):
        self.flat.copy_(self.saved)
        return self.views


def prepare(case, seed):
    P = _program(_key(case))
    x = _inputs(case, P, seed)
    if case["what"] == "solve":
        work = [torch.zeros_like(x["b"])]
    elif case["what"] == "adjoint":
        z = torch.zeros_like
        work = [x["Ub_new"], x["Ub"], x["Ub_prev"], x["Wb"], x["Wb_prev"], z(x["U"]),
                torch.zeros(P.nc, dtype=torch.float64, device=DEV), torch.zeros(1, dtype=torch.float64, device=DEV)]
    else:
        work = [x["U"], x["Uprev"], x["W"].reshape(P.S, -1), x["Wprev"].reshape(P.S, -1)]
    st = _State(work)
    return dict(P=P, x=x, st=st, g=torch.empty_like(x.get("U", x.get("b"))), what=case["what"],
                opts=dict(tol=case["tol"], tol_mode=case["tol_mode"]))


def run(s):
    P, x, what, opts = s["P"], s["x"], s["what"], s["opts"]
    v = s["st"].restore()
    if what == "solve":
        api.pcg_solve(P.solver, x["b"], v[0], **opts)
        return {"x": v[0]}
    if what == "adjoint":
        ub_new, ub, ub_prev, wb, wb_prev, lam, grad, loss = v
        api.sensor_misfit(P.solver, x["Unew"], x["target"], ub_new, loss)
        api.pcg_solve(P.solver, ub_new, lam, **opts)
        api.grad_accumulate(P.solver, lam, x["Unew"], grad)
        api.adjoint_step(P.solver, x["U"], x["Uprev"], x["W"], x["Wprev"], lam, x["Wb_new"], ub, ub_prev, wb, wb_prev)
        return {"Ub_new": ub_new, "Ub": ub, "Ub_prev": ub_prev, "Wb": wb, "Wb_prev": wb_prev, "lam": lam, "grad": grad, "loss": loss}
    st = api.State(*v, s["g"])
    step = api.time_step_multi if what == "step_multi" else api.time_step
    step(P.solver, st, P.dt, iapp=x["iapp"], **opts)
    return {"U": st.U, "W": st.W}


def _sizes(case):
    dim = 2 if case["mesh"] == "square" else 3
    # the shell's volume is that of the two half ellipsoids' difference
    nc = case["n"] ** dim if case["mesh"] != "shell" else 2.0 / 3.0 * math.pi * (2.5 - 0.7 * 0.7 * 2.0) / case["h"] ** 3
    return dim, nc, (case["p"] + 1) ** dim


def work(case):
    """State in and out, mesh and conductivity once; the operations of about five PCG iterations
    of one V-cycle (18 smoothing products) and one outer product on the nonzeros of the operator."""
    dim, nc, b = _sizes(case)
    S, cols = MODELS[case["model"]][2], COLS if case["what"] == "step_multi" else 1
    N = nc * b
    vectors = {"solve": 2, "adjoint": 2 + 2 * S + 2 * (3 + 2 * S) + 3}.get(case["what"], 4 + 3 * S) * cols
    nf = b // (case["p"] + 1)
    nnz = nc * (b * b + 2 * dim * (2 * nf * b - nf * nf))
    return {"bytes": 8.0 * (N * vectors + nc * (dim + dim * (dim + 1) // 2)), "flops": 2.0 * 5 * 19 * nnz * cols}


# ---------------------------------------------------------------- plain FP64

class _Plain:
    """A_0 = cM M + A as quadrature sums (symmetric interior penalty, per-cell D), on [nc, b, cols]."""

    def __init__(self, P):
        d, p, nc = P.dim, P.p, P.nc
        q = p + 1
        T = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)
        X = T(P.xyz)[T(P.cells)]
        iu = [[(min(a, c), max(a, c)) for c in range(d)] for a in range(d)]
        pk = {ab: k for k, ab in enumerate((a, c) for a in range(d) for c in range(a, d))}
        D = torch.stack([torch.stack([T(P.D)[:, pk[iu[a][c]]] for c in range(d)], -1) for a in range(d)], -2)
        gx, gw = _gauss(q)
        lin = lambda x: (np.stack([1 - x, x], axis=1), np.tile([-1.0, 1.0], (len(x), 1)))

        def tables(points):
            """Basis and geometry tables at a tensor grid of 1D points."""
            B1, L1 = [_lagrange(p, x) for x in points], [lin(x) for x in points]
            grad = lambda t: T(np.stack([_tensor([t[k][1 if k == a else 0] for k in range(d)]) for a in range(d)]))
            return T(_tensor([t[0] for t in B1])), grad(B1), grad(L1)

        def jacobian(gl, cells):
            J = torch.stack([torch.matmul(gl[a], cells) for a in range(d)], dim=-1)   # [n, q, x, xi]
            return torch.linalg.inv(J).transpose(-1, -2).contiguous(), torch.linalg.det(J)

        self.cM = 3.0 * P.chi * P.Cm / (2.0 * P.dt)
        self.phi, self.gr, gl = tables([gx] * d)
        JiT, det = jacobian(gl, X)
        self.w = T(_tensor([gw[:, None]] * d)[:, 0]) * det
        # per point: J^-1 D J^-T w
        self.K = torch.matmul(torch.matmul(JiT.transpose(-1, -2).contiguous(), D[:, None]), JiT) * self.w[..., None, None]
        vol = self.w.sum(dim=1)
        fw = T(_tensor([gw[:, None]] * (d - 1))[:, 0])
        self.faces = []
        for a in range(d):
            lo_c = [c for c in range(2 ** d) if not c >> a & 1]
            key = lambda cs: np.ascontiguousarray(np.sort(P.cells[:, cs], axis=1))
            low, up = key(lo_c), key([c | 1 << a for c in lo_c])
            _, inv = np.unique(np.concatenate([up, low]), axis=0, return_inverse=True)
            inv = inv.ravel()
            at = np.full(inv.max() + 1, -1)
            at[inv[nc:]] = np.arange(nc)
            minus = at[inv[:nc]]
            plus, minus = T(np.flatnonzero(minus >= 0)), T(minus[minus >= 0])
            side = []
            for e, cells in ((1.0, plus), (0.0, minus)):
                phi, gr, gl = tables([np.array([e]) if k == a else gx for k in range(d)])
                JiT, det = jacobian(gl, X[cells])
                side.append((cells, phi, gr, JiT, det))
            # normal and area element of the plus side: det J J^-T e_a
            nu = side[0][3][..., a] * side[0][4][..., None]
            dA = torch.linalg.norm(nu, dim=-1)
            nrm, wA = nu / dA[..., None], fw * dA
            area = wA.sum(dim=1)
            Dn = [torch.einsum("nab,nqb->nqa", D[s[0]], nrm) for s in side]
            if P.penalty[0] == "fixed":
                eta = torch.full_like(area, P.penalty[1])
            else:
                c = P.penalty[1] if len(P.penalty) > 1 else 1.0
                eta = c * p * (p + 1) * 0.5 * (area / vol[plus] + area / vol[minus])
            sig = [0.5 * eta[:, None] * (v * nrm).sum(-1) for v in Dn]     # each side's share of the penalty
            # conormal derivative of a side as reference-gradient weights
            con = [torch.matmul(s[3].transpose(-1, -2).contiguous(), Dn[k][..., None])[..., 0] for k, s in enumerate(side)]
            self.faces.append((side, con, sig, wA))

    def mass(self, x):
        return torch.matmul(self.phi.t().contiguous(), self.w[..., None] * torch.matmul(self.phi, x))

    def cell_grad(self, x):
        return torch.stack([torch.matmul(g, x) for g in self.gr], dim=2)          # [n, q, d, cols]

    def apply(self, x, own=False):
        """A_0 x; with `own` the cells' diagonal blocks alone."""
        F = torch.matmul(self.K, self.cell_grad(x))
        y = self.cM * self.mass(x) + sum(torch.matmul(g.t().contiguous(), F[:, :, a]) for a, g in enumerate(self.gr))
        for side, con, sig, wA in self.faces:
            u = [torch.matmul(s[1], x[s[0]]) for s in side]
            f = [sum(c[..., a, None] * torch.matmul(g, x[s[0]]) for a, g in enumerate(s[2])) for s, c in zip(side, con)]
            for k, (s, c, sgn) in enumerate(zip(side, con, (1.0, -1.0))):
                other = 0.0 if own else 1.0
                uu = (u[0] - other * u[1]) if k == 0 else (other * u[0] - u[1])
                ff = f[k] + other * f[1 - k]
                val = wA[..., None] * (-0.5 * ff + (sig[0] + sig[1])[..., None] * uu) * sgn
                y[s[0]] += torch.matmul(s[1].t().contiguous(), val)
                jump = -0.5 * wA[..., None] * uu
                y[s[0]] += sum(torch.matmul(g.t().contiguous(), c[..., a, None] * jump) for a, g in enumerate(s[2]))
        return y

    def solve(self, b, x, rel):
        """Conjugate gradients with the inverse diagonal blocks, from x, to a residual of rel ||b - A x||."""
        n, m = b.shape[:2]
        blocks = torch.stack([self.apply(torch.eye(m, dtype=b.dtype, device=DEV)[k].expand(n, m)[..., None].contiguous(), own=True)[..., 0]
                              for k in range(m)], dim=-1)
        inv = torch.cat([torch.linalg.inv(c) for c in blocks.split(1 << 15)])
        dot = lambda u, v: (u * v).sum(dim=(0, 1))
        r = b - self.apply(x)
        r0 = dot(r, r).sqrt()
        z = torch.matmul(inv, r)
        p, rz = z, dot(r, z)
        for _ in range(600):
            q = self.apply(p)
            al = rz / dot(p, q)
            x, r = x + al * p, r - al * q
            if bool((dot(r, r).sqrt() <= rel * r0).all()):
                break
            z = torch.matmul(inv, r)
            new = dot(r, z)
            p, rz = z + new / rz * p, new
        return x

    def gradient(self, lam, u):
        """-lam^T (dA/ds_K) u per cell for D_K -> s_K D_K, faces sharing their penalty between both sides."""
        g = -torch.einsum("nqac,nqab,nqbc->n", self.cell_grad(lam), self.K, self.cell_grad(u))
        for side, con, sig, wA in self.faces:
            val = lambda x: [torch.matmul(s[1], x[s[0]])[..., 0] for s in side]
            flux = lambda x: [sum(c[..., a] * torch.matmul(gr, x[s[0]])[..., 0] for a, gr in enumerate(s[2])) for s, c in zip(side, con)]
            ul, uu, fl, fu = val(lam), val(u), flux(lam), flux(u)
            jl, ju = ul[0] - ul[1], uu[0] - uu[1]
            for k in (0, 1):
                g[side[k][0]] -= (wA * (-0.5 * (fu[k] * jl + fl[k] * ju) + sig[k] * jl * ju)).sum(dim=1)
        return g


def _gates(P, u):
    """Coefficients c1 w + c0 of dw/dt and their derivatives in u (FitzHugh-Nagumo and Aliev-Panfilov)."""
    p = P.par
    if P.name == "fhn":
        return [0 * u - p[2] * p[3]], [p[2] * u], [0 * u + p[2]]
    if P.name == "ap":
        return [0 * u - p[2]], [-p[2] * p[0] * u * (u - p[1] - 1.0)], [-p[2] * p[0] * (2.0 * u - p[1] - 1.0)]
    (to1, to2, tso1, tso2, tsi, tfi, t1p, t1m1, t1m2, t2m1, t2m2, t3m1, t3m2, t2p, t2inf, k2, k3, kso, winf, v1, v1m,
     v2, v2m, v3, vh, vo, vso, uo) = p
    H = lambda z: 0.5 * (1.0 + torch.sign(z))
    Hk = lambda z, k: 0.5 * (1.0 + torch.tanh(k * z))
    a0 = (1 - H(u - v1)) / (H(u - v1m) * (t1m2 - t1m1) + t1m1)
    a1 = (1 - H(u - v2)) / (Hk(u - v2m, k2) * (t2m2 - t2m1) + t2m1)
    a2 = 1.0 / (H(u - v2) * (t3m2 - t3m1) + t3m1)
    w1 = H(u - vo) * (winf - 1.0 + u / t2inf) + 1.0 - u / t2inf
    return [-H(u - v1) / t1p - a0, -H(u - v2) / t2p - a1, -a2], [a0 * (1 - H(u - v1m)), a1 * w1, a2 * Hk(u - v3, k3)], None


def _current(P, u, w):
    p = P.par
    if P.name != "bo":
        return p[0] * u * (u - p[1]) * (u - 1.0) + (w[0] if P.name == "fhn" else u * w[0])
    (to1, to2, tso1, tso2, tsi, tfi, t1p, t1m1, t1m2, t2m1, t2m2, t3m1, t3m2, t2p, t2inf, k2, k3, kso, winf, v1, v1m,
     v2, v2m, v3, vh, vo, vso, uo) = p
    H = lambda z: 0.5 * (1.0 + torch.sign(z))
    so = 0.5 * (1.0 + torch.tanh(kso * (u - vso)))
    return (-H(u - v1) * (u - v1) * (vh - u) * w[0] / tfi - H(u - v2) * w[1] * w[2] / tsi
            + (1 - H(u - v2)) * (u - uo) / (H(u - vo) * (to2 - to1) + to1) + H(u - v2) / (so * (tso2 - tso1) + tso1))


def exact(case, seed):
    if _sizes(case)[1] * _sizes(case)[2] > 3e6:
        return None   # over 20 seconds of plain conjugate gradients, or more memory than they are worth
    P = _Program(case, with_solver=False)
    x, A = _inputs(case, P, seed), _Plain(P)
    shape = (P.nc, P.b, -1)
    if case["what"] == "solve":
        b = x["b"].view(shape)
        return {"x": A.solve(b, torch.zeros_like(b), 1e-13).reshape(P.N)}
    us = 2.0 * x["U"] - x["Uprev"]
    c1, c0, dc0 = _gates(P, us)
    den = [3.0 - 2.0 * P.dt * c for c in c1]
    w = [(4.0 * x["W"][k] - x["Wprev"][k] + 2.0 * P.dt * c0[k]) / den[k] for k in range(P.S)]
    cU = P.chi * P.Cm / (2.0 * P.dt)
    if case["what"] == "adjoint":
        u = x["Unew"].view(P.nc, P.b)
        weights = torch.from_numpy(np.stack([_tensor([_lagrange(P.p, np.array([t]))[0] for t in ref])[0] for ref in P.sensor_ref])).to(DEV)
        at = torch.from_numpy(P.sensor_cells).to(DEV)
        miss = (weights * u[at]).sum(dim=1) - x["target"]
        ub_new = x["Ub_new"].view(P.nc, P.b).clone()
        ub_new[at] += 2.0 * miss[:, None] * weights
        lam = A.solve(ub_new[..., None], torch.zeros_like(ub_new)[..., None], 1e-14)
        fb = A.mass(lam).reshape(P.N)
        gb = -P.chi * fb
        p = P.par
        dI = p[0] * (3.0 * us * us - 2.0 * (p[1] + 1.0) * us + p[1]) + (w[0] if P.name == "ap" else 0.0)
        tot = x["Wb_new"] + (us if P.name == "ap" else 1.0) * gb
        usb = dI * gb + tot * 2.0 * P.dt * dc0[0] / den[0]
        return {"Ub_new": ub_new.reshape(P.N), "Ub": x["Ub"] + 4.0 * cU * fb + 2.0 * usb, "Ub_prev": x["Ub_prev"] - cU * fb - usb,
                "Wb": x["Wb"] + 4.0 * tot / den[0], "Wb_prev": x["Wb_prev"] - tot / den[0],
                "lam": lam.reshape(P.N), "grad": A.gradient(lam, u[..., None]), "loss": (miss ** 2).sum().reshape(1)}
    f = cU * (4.0 * x["U"] - x["Uprev"]) - P.chi * _current(P, us, w)
    if x["iapp"] is not None:
        f = f + x["iapp"]
    U = A.solve(A.mass(f.view(shape)), x["U"].view(shape), 1e-13)
    return {"U": U.reshape(x["U"].shape), "W": torch.stack(w).reshape(P.S, -1)}
