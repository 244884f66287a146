"""Workloads for timing the library through its Python entry points.

Each case is a plain dict: an element type with its mesh size, a material, a
precision and the call a program makes on it.  ``prepare`` builds what such a
program keeps (the mesh handle with its pattern, mass and output buffers) and
its inputs from a seed, ``run`` makes one call, ``work`` counts the bytes and
operations the call cannot do without, and ``exact`` evaluates the same result
in float64 with plain torch: shape functions, quadrature, stresses, tangents,
sums into the CSR pattern and the solver loop are written out here and use
nothing of the library but the seeded inputs of ``workloads``.
"""
import dataclasses
import functools
import math

import numpy as np
import torch

from paper_2604_10357_amd import workloads as W
from paper_2604_10357_amd.api import TLBatch, TLMesh
from paper_2604_10357_amd.autograd import internal_force

DT = 1e-3        # time step of the tangent h df/dq + df/dqdot and of the Newton pieces
DENSITY = 2700.0  # of the paper's benchmark bodies
ADAMW = dict(lr=1e-4, beta1=0.9, beta2=0.999, eps=1e-8, weight_decay=0.0)

MATERIALS = {
    "svk": W.Material(W.SVK, (1e7, 0.3, 0.0)),
    "svk_kv": W.Material(W.SVK, (1e7, 0.3, 0.0), 1e3, 1e3),
    "svk_stiff": W.Material(W.SVK, (7e8, 0.33, 0.0)),
    "mr": W.Material(W.MOONEY_RIVLIN, (2e5, 5e4, 1e8)),
    "mr_kv": W.Material(W.MOONEY_RIVLIN, (2e5, 5e4, 1e8), 1e3, 1e3),
}


# ----------------------------------------------------------------------------
# the cases
# ----------------------------------------------------------------------------
def _t10(name, cells, material, precision, call, **more):
    return dict(name=name, element="t10", nx=cells[0], ny=cells[1], nz=cells[2], material=material,
                precision=precision, call=call, **more)


def listed():
    return [
        # the smallest mesh of the tests: one body of 24 elements, bound by launches
        _t10("t10_24_fp64", (4, 1, 1), "svk", "fp64", "assemble"),
        # one Newton iteration's f and K of a mid-sized damped body
        _t10("t10_30720_mixed", (80, 8, 8), "mr_kv", "mixed", "assemble"),
        # the benchmark mesh: the largest body, mixed precision
        _t10("t10_480000_mixed", (200, 20, 20), "mr_kv", "mixed", "assemble"),
        # the same body all in float64
        _t10("t10_480000_fp64", (200, 20, 20), "mr_kv", "fp64", "assemble"),
        # explicit stepping of the largest body: the force alone
        _t10("t10_480000_force", (200, 20, 20), "mr_kv", "mixed", "force"),
        # reverse-mode differentiation of the force, odd cell counts: forward and
        # backward to positions, velocities and material constants
        _t10("t10_112398_grad", (131, 13, 11), "mr_kv", "fp64", "grad"),
        # a first-order step: 26 AdamW iterations, iterations replayed between checks
        _t10("t10_18000_adamw", (30, 10, 10), "mr_kv", "fp64", "adamw", iters=26, every=25),
        # the shell plate of the benchmark, undamped, mixed precision
        dict(name="plate_256_332", element="plate", n=256, rule="332", material="svk", precision="mixed",
             call="assemble"),
        # a Newton step of a shell for a Cholesky solver: H and its upper triangle, gradient; the paper's rule
        dict(name="plate_100_443_newton", element="plate", n=100, rule="443", material="svk", precision="fp64",
             call="newton_upper"),
        # the largest beam chain, one Newton step with damping off
        dict(name="beam_500000_newton", element="beam", n=500000, material="svk_stiff", precision="mixed",
             call="newton"),
        # explicit stepping of a small beam chain, odd count, damped
        dict(name="beam_2001_force", element="beam", n=2001, material="svk_kv", precision="fp64", call="force"),
        # many bodies of uneven size in one launch
        dict(name="cubes_64_batch", element="cubes", bodies=64, lo=2, hi=12, sizes=0, material="both",
             precision="mixed", call="batch"),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.49)))))))


def draw(rng):
    element = rng.choice(["t10", "t10", "t10", "plate", "beam", "cubes"])
    precision = rng.choice(["mixed", "mixed", "fp64"])
    if element == "cubes":
        lo = rng.randint(1, 4)
        return dict(element="cubes", bodies=_log_int(rng, 2, 64), lo=lo, hi=rng.randint(lo + 1, 12),
                    sizes=rng.randrange(1000), material="both", precision=precision, call="batch")
    damped = rng.random() < 0.5
    calls = ["assemble", "assemble", "tangent", "force", "grad", "newton", "adamw"]
    if not damped:
        calls += ["upper", "newton_upper"]
    call = rng.choice(calls)
    c = dict(element=element, precision="fp64" if call == "adamw" else precision, call=call)
    if call == "adamw":
        c.update(iters=rng.randint(5, 26), every=rng.randint(4, 25))
    big = call not in ("adamw", "grad")  # solves and differentiation stay at mid-sized meshes
    if element == "t10":
        c.update(nx=_log_int(rng, 1, 200 if big else 60), ny=_log_int(rng, 1, 20), nz=_log_int(rng, 1, 20),
                 material=rng.choice(["mr_kv", "svk_kv"]) if damped else rng.choice(["mr", "svk"]))
    elif element == "plate":
        rule = rng.choice(["332", "443"])
        c.update(n=_log_int(rng, 2, 256 if big and rule == "332" else 100), rule=rule,
                 material="svk_kv" if damped else rng.choice(["svk", "mr"]))
    else:
        c.update(n=_log_int(rng, 1, 500000 if big else 50000), material="mr_kv" if damped else "svk_stiff")
    return c


# ----------------------------------------------------------------------------
# inputs, handles, calls
# ----------------------------------------------------------------------------
@dataclasses.dataclass
class Body:
    mesh: W.Mesh
    material: W.Material
    q: np.ndarray
    qdot: np.ndarray
    w: np.ndarray


def _inputs(case, seed):
    """The bodies of a case, their states and cotangents, from the seed alone."""
    if case["element"] == "cubes":
        # sizes and materials belong to the case, the states to the seed
        rng, out = np.random.default_rng(1000 + seed), []
        for x in W.batched_bodies(case["bodies"], 1004 + case["sizes"], case["lo"], case["hi"]):
            edge = x.mesh.X.max() / round((x.mesh.n_elem / 6) ** (1 / 3))  # of a cell
            q = (x.mesh.X + rng.uniform(-0.02 * edge, 0.02 * edge, x.mesh.X.shape)).ravel()
            out.append(Body(x.mesh, x.material, q, rng.normal(0.0, 0.05, q.shape[0]), x.w))
        return out
    mat = MATERIALS[case["material"]]
    if case["element"] == "t10":
        nx, ny, nz = case["nx"], case["ny"], case["nz"]
        x = W.t10_beam(nx, ny, nz, 1000 + seed, "t10", lx=0.0125 * nx, ly=0.0125 * ny, lz=0.0125 * nz, material=mat)
    elif case["element"] == "plate":
        gl = (3, 3, 2) if case["rule"] == "332" else (4, 4, 3)
        x = W.shell_plate(case["n"], 1000 + seed, "plate", gl=gl)
        x.qdot = np.random.default_rng(7000 + seed).normal(0.0, 0.05, x.q.shape[0])
    else:
        x = W.beam_3243(case["n"], 1000 + seed, "beam")
    return [Body(x.mesh, mat, x.q, x.qdot, x.w)]


def _loads(case, seed, n):
    """Previous velocity and external force of a time step."""
    rng = np.random.default_rng(5000 + seed)
    return rng.normal(0.0, 0.05, n), rng.normal(0.0, 5.0, n)


@functools.lru_cache(maxsize=None)
def _side_stream():
    # batches and the first-order solver replay captured work, which the legacy stream cannot do
    return torch.cuda.Stream()


@dataclasses.dataclass
class State:
    call: str
    case: dict
    handles: list
    batch: object
    q: torch.Tensor
    qdot: torch.Tensor
    more: dict


def _cuda(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def prepare(case, seed):
    call = case["call"]
    bodies = _inputs(case, seed)
    handles = []
    for b in bodies:
        m = TLMesh(b.mesh, b.material, case["precision"])
        m.build_pattern()
        if call in ("newton", "newton_upper", "adamw"):
            m.build_mass(DENSITY)
        if call in ("upper", "newton_upper"):
            m.build_upper_pattern()
        handles.append(m)
    q = _cuda(np.concatenate([b.q for b in bodies]))
    qdot = _cuda(np.concatenate([b.qdot for b in bodies]))
    n, dev = q.numel(), q.device
    buf = functools.partial(torch.empty, dtype=torch.float64, device=dev)
    more, batch = {}, None
    if call == "batch":
        batch = TLBatch(handles)
        more = dict(f=buf(n), vals=buf(batch.nnz_off[-1]),
                    h=torch.full((len(bodies),), DT, dtype=torch.float64, device=dev))
    elif call in ("assemble", "newton"):
        more = dict(f=buf(n), vals=buf(handles[0].nnz))
    elif call == "tangent":
        more = dict(vals=buf(handles[0].nnz))
    elif call in ("upper", "newton_upper"):
        more = dict(f=buf(n), vals=buf(handles[0].nnz_upper))
    elif call == "force":
        more = dict(f=buf(n))
    elif call == "grad":
        mat = bodies[0].material
        params = torch.tensor([*mat.params, mat.kv_eta, mat.kv_lambda], dtype=torch.float64, device=dev)
        more = dict(w=_cuda(bodies[0].w), params=params.requires_grad_(True))
        q.requires_grad_(True)
        qdot.requires_grad_(True)
    if call in ("newton", "newton_upper", "adamw"):
        v_prev, f_ext = _loads(case, seed, n)
        more.update(v_prev=_cuda(v_prev), f_ext=_cuda(f_ext))
    if call in ("newton", "newton_upper"):
        more.update(g=buf(n))
    if call == "adamw":
        more.update(v=buf(n), q_out=buf(n), work=buf(4 * n))
    return State(call, case, handles, batch, q, qdot, more)


def run(s):
    m, b = s.handles[0], s.more
    if s.call == "assemble":
        return m.assemble(s.q, s.qdot, alpha=DT, beta=1.0, f=b["f"], vals=b["vals"])
    if s.call == "tangent":
        return m.tangent(s.q, s.qdot, h=DT, out=b["vals"])
    if s.call == "force":
        return m.internal_force(s.q, s.qdot, out=b["f"])
    if s.call == "upper":
        return m.assemble_upper(s.q, s.qdot, alpha=1.0, beta=0.0, f=b["f"], vals=b["vals"])
    if s.call in ("newton", "newton_upper"):
        if s.call == "newton":
            f, vals = m.assemble_newton(s.q, s.qdot, DT, f=b["f"], vals=b["vals"])
        else:
            f, vals = m.assemble_newton_upper(s.q, s.qdot, DT, f=b["f"], vals_upper=b["vals"])
        g = m.newton_gradient(s.qdot, b["v_prev"], f, b["f_ext"], DT, out=b["g"])
        return f, vals, g
    if s.call == "grad":
        f = internal_force(m, s.q, s.qdot, b["params"])
        gq, gqd, gp = torch.autograd.grad(f, [s.q, s.qdot, b["params"]], b["w"])
        return f.detach(), gq, gqd, gp
    with torch.cuda.stream(_side_stream()):
        if s.call == "batch":
            return s.batch.assemble(s.q, s.qdot, b["h"], f=b["f"], vals=b["vals"])
        b["v"].copy_(s.qdot)  # the step starts from the current velocity
        v, q, done, _, g = m.adamw_solve(s.q, b["v_prev"], b["v"], DT, f_ext=b["f_ext"],
                                         max_iters=s.case["iters"], check_every=s.case["every"], q=b["q_out"],
                                         work=b["work"], **ADAMW)
        return v, q, g, done


# ----------------------------------------------------------------------------
# work
# ----------------------------------------------------------------------------
@functools.lru_cache(maxsize=None)
def _t10_pairs(nx, ny, nz):
    """Ordered pairs of adjacent nodes of a Kuhn box: linear in each cell count
    (cells less what neighbouring cells share), fixed by the boxes of one and two cells."""
    if max(nx, ny, nz) <= 2:
        c = W.kuhn_t10_box(nx, ny, nz, 1.0, 1.0, 1.0).conn.astype(np.int64)
        return int(np.unique(c[:, :, None] * 100000 + c[:, None, :]).size)
    total = 0
    for i in (1, 2):
        for j in (1, 2):
            for k in (1, 2):
                wt = 1
                for n, x in ((nx, i), (ny, j), (nz, k)):
                    wt *= 2 - n if x == 1 else n - 1
                total += wt * _t10_pairs(i, j, k)
    return total


def _sizes(case):
    """(elements, coefficients, nnz of the full pattern, coefficients per element, connectivity ids, points)"""
    if case["element"] == "plate":
        n = case["n"]
        return n * n, 4 * (n + 1) ** 2, 144 * (3 * n + 1) ** 2, 16, 4, 18 if case["rule"] == "332" else 48
    if case["element"] == "beam":
        n = case["n"]
        return n, 4 * (n + 1), 144 * (3 * n + 1), 8, 2, 12
    if case["element"] == "t10":
        boxes = [(case["nx"], case["ny"], case["nz"])]
    else:  # cubes of random sizes: the mean of their range
        boxes = [(x, x, x) for x in range(case["lo"], case["hi"] + 1)]
    ne = sum(6 * x * y * z for x, y, z in boxes)
    nc = sum(W.t10_node_count(*x) for x in boxes)
    nnz = 9 * sum(_t10_pairs(*x) for x in boxes)
    k = case.get("bodies", 1) / len(boxes)
    return ne * k, nc * k, nnz * k, 10, 10, 5


def work(case):
    """q, qdot, X and the connectivity read once, every result written once; the
    kinematics, the stress and the sums over points (and the tangent contraction)."""
    ne, nc, nnz, nen, npn, nq = _sizes(case)
    dof, call = 3 * nc, case["call"]
    force_flops = ne * nq * (2 * 2 * 9 * nen + 2 * 9 * nen + 500)
    tangent_flops = ne * nq * 2 * (81 * nen + 27 * nen * nen)
    state = 24 * dof + 4 * npn * ne
    if call == "force":
        return {"bytes": state + 8 * dof, "flops": force_flops}
    if call == "grad":  # forward; then the cotangent read and two gradients written
        return {"bytes": 2 * state + 8 * dof + 24 * dof, "flops": 4 * force_flops}
    mass = nnz / 9.0  # one value per pair of coefficients
    if call == "adamw":  # per iteration: the force, the mass rows, moments, v and q
        it = case["iters"]
        return {"bytes": it * (state + 8 * mass + 96 * dof), "flops": it * (force_flops + 6 * mass + 20 * dof)}
    out = 8 * dof * (call != "tangent") + 8 * (nnz if "upper" not in call else (nnz + dof) / 2)
    more = 8 * mass + 32 * dof if call.startswith("newton") else 0
    return {"bytes": state + out + more, "flops": force_flops + tangent_flops}


# ----------------------------------------------------------------------------
# the same results in float64, plain torch
# ----------------------------------------------------------------------------
F64 = torch.float64


def _dev():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _gauss(n):
    x, w = np.polynomial.legendre.leggauss(n)
    return x.tolist(), w.tolist()


def _shape(element, p):
    """Unit-scaled shape functions at parent point p (a 3-vector), as a vector."""
    x, y, z = p[0], p[1], p[2]
    if element == "t10":
        L = [1 - x - y - z, x, y, z]
        v = [a * (2 * a - 1) for a in L] + [4 * L[a] * L[b] for a, b in ((0, 1), (1, 2), (0, 2), (0, 3), (1, 3), (2, 3))]
    elif element == "beam":
        t = (1 + x) / 2
        v = [1 - 3 * t**2 + 2 * t**3, t - 2 * t**2 + t**3, y * (1 - t), z * (1 - t),
             3 * t**2 - 2 * t**3, t**3 - t**2, y * t, z * t]
    else:
        v = []
        for sx, sy in ((-1, -1), (1, -1), (1, 1), (-1, 1)):
            a, b = 1 + sx * x, 1 + sy * y
            v += [a * b * (2 + sx * x + sy * y - x * x - y * y) / 8, sx * a * a * (sx * x - 1) * b / 8,
                  sy * b * b * (sy * y - 1) * a / 8, z * a * b / 4]
    return torch.stack(v)


def _points(element, rule):
    """Quadrature points and weights on the parent element."""
    if element == "t10":
        pts, wts = [(0.25, 0.25, 0.25)], [-4.0 / 30.0]
        for c in range(4):
            L = [0.5 if k == c else 1.0 / 6.0 for k in range(4)]
            pts.append(tuple(L[1:]))
            wts.append(9.0 / 120.0)
        return pts, wts
    nx, ny, nz = (3, 2, 2) if element == "beam" else (3, 3, 2) if rule == "332" else (4, 4, 3)
    (x, a), (y, b), (z, c) = _gauss(nx), _gauss(ny), _gauss(nz)
    pts = [(x[i], y[j], z[k]) for i in range(nx) for j in range(ny) for k in range(nz)]
    wts = [a[i] * b[j] * c[k] for i in range(nx) for j in range(ny) for k in range(nz)]
    return pts, wts


def _mass_points(element):
    """A rule that is exact for products of two shape functions."""
    x, w = _gauss(5)
    pts, wts = [], []
    for i in range(5):
        for j in range(5):
            for k in range(5):
                wt = w[i] * w[j] * w[k]
                if element != "t10":
                    pts.append((x[i], x[j], x[k]))
                    wts.append(wt)
                    continue
                u, v, t = (1 + x[i]) / 2, (1 + x[j]) / 2, (1 + x[k]) / 2  # the cube collapsed to the tetrahedron
                pts.append((u, v * (1 - u), t * (1 - u) * (1 - v)))
                wts.append(wt / 8 * (1 - u) ** 2 * (1 - v))
    return pts, wts


class _Exact:
    """One body's reference geometry and sums, in float64."""

    def __init__(self, case, body):
        dev = _dev()
        mesh, el = body.mesh, {"cubes": "t10"}.get(case["element"], case["element"])
        self.mc = 1 if el == "t10" else 4
        conn = torch.from_numpy(mesh.conn.astype(np.int64)).to(dev)
        self.nodes = conn
        self.coef = conn if self.mc == 1 else (4 * conn[:, :, None] + torch.arange(4, device=dev)).reshape(len(conn), -1)
        self.n_nodes, self.n_dof = mesh.n_coef // self.mc, mesh.n_dof
        X = torch.from_numpy(mesh.X).to(dev)
        self.X = X.reshape(-1)
        pts, wts = _points(el, case.get("rule"))
        jac = lambda p: torch.autograd.functional.jacobian(lambda t: _shape(el, t), torch.tensor(p, dtype=F64))  # noqa: E731
        dN = torch.stack([jac(p) for p in pts]).to(dev)  # (q, a, m)
        mp, mw = _mass_points(el)
        N = torch.stack([_shape(el, torch.tensor(p, dtype=F64)) for p in mp])
        self.mass_ref = (N.T @ (N * torch.tensor(mw, dtype=F64)[:, None])).to(dev)
        ne = len(conn)
        self.scale = torch.ones(ne, self.coef.shape[1], dtype=F64, device=dev)
        if self.mc == 4:
            r = X.reshape(-1, 4, 3)[:, 0]
            l1 = (r[conn[:, 1]] - r[conn[:, 0]]).norm(dim=1)
            l2 = (r[conn[:, 3]] - r[conn[:, 0]]).norm(dim=1) / 2 if el == "plate" else torch.full_like(l1, mesh.width / 2)
            self.scale[:, 1::4] = (l1 / 2 if el == "plate" else l1)[:, None]
            self.scale[:, 2::4] = l2[:, None]
            self.scale[:, 3::4] = mesh.thickness / 2
        self.dN, self.w = dN, torch.tensor(wts, dtype=F64, device=dev)
        self.mat = body.material

    def geometry(self, e):
        """Physical gradients g (e, q, a, 3) and volumes dV (e, q) of elements e."""
        d = self.dN[None] * self.scale[e][:, None, :, None]
        X = self._relative(self.X, e)
        J0 = (X[:, None, :, :, None] * d[:, :, :, None, :]).sum(2)
        g = d @ torch.linalg.inv(J0)
        return g, torch.linalg.det(J0) * self.w

    def _relative(self, u, e):
        """Nodal values (e, a, 3) with the first one taken out of every position coefficient."""
        x = u.reshape(-1, 3)[self.coef[e]]
        keep = torch.zeros(x.shape[1], dtype=F64, device=x.device)
        keep[:: self.mc] = 1.0
        return x - keep[None, :, None] * x[:, :1]

    def kinematics(self, q, qdot, e):
        g, dV = self.geometry(e)
        H = self._relative(q - self.X, e).transpose(1, 2).unsqueeze(1) @ g
        Fd = self._relative(qdot, e).transpose(1, 2).unsqueeze(1) @ g
        return g, dV, H, Fd

    def stress(self, H, Fd, p):
        I = torch.eye(3, dtype=F64, device=H.device)
        F = I + H
        E = 0.5 * (H + H.mT + H.mT @ H)
        tr = lambda M: M.diagonal(dim1=-2, dim2=-1).sum(-1)[..., None, None]  # noqa: E731
        if self.mat.kind == W.SVK:
            lam, mu = p[0] * p[1] / ((1 + p[1]) * (1 - 2 * p[1])), p[0] / (2 * (1 + p[1]))
            P = F @ (lam * tr(E) * I + 2 * mu * E)
        else:
            jm1 = self._jm1(H)
            J = 1 + jm1
            a, b = J ** (-2.0 / 3.0), J ** (-4.0 / 3.0)
            T = 4 * p[0] * a * (E - tr(E) / 3 * I) + p[2] * J * jm1 * I
            T = T + 2 * p[1] * b * (2 * E - 2 * tr(E) / 3 * I + 4 * tr(E) * E - 4 * E @ E
                                    + 4.0 / 3.0 * (tr(E @ E) - tr(E) ** 2) * I)
            P = torch.linalg.inv(F).mT @ T
        Ed = 0.5 * (Fd.mT @ F + F.mT @ Fd)
        return P + F @ (2 * p[3] * Ed + p[4] * tr(Ed) * I)

    @staticmethod
    def _jm1(H):
        t = H.diagonal(dim1=-2, dim2=-1).sum(-1)
        t2 = (H @ H).diagonal(dim1=-2, dim2=-1).sum(-1)
        return (t + 0.5 * (t * t - t2) + torch.linalg.det(H))[..., None, None]

    def params(self):
        m = self.mat
        return torch.tensor([*m.params, m.kv_eta, m.kv_lambda], dtype=F64, device=self.X.device)

    def chunks(self, per):
        ne = len(self.nodes)
        for a in range(0, ne, per):
            yield torch.arange(a, min(a + per, ne), device=self.X.device)

    def force(self, q, qdot, params=None):
        p = self.params() if params is None else params
        f = torch.zeros(self.n_dof // 3, 3, dtype=F64, device=self.X.device)
        for e in self.chunks(200000):
            g, dV, H, Fd = self.kinematics(q, qdot, e)
            P = self.stress(H, Fd, p) * dV[..., None, None]
            f = f.index_add(0, self.coef[e].reshape(-1), (g @ P.mT).sum(1).reshape(-1, 3))
        return f.reshape(-1)

    def tangent(self, H, Fd, alpha, beta):
        """A_iJkL = alpha dP_iJ/dF_kL + beta dP_iJ/dFdot_kL, from the textbook forms."""
        I = torch.eye(3, dtype=F64, device=H.device)
        F, C = I + H, (I + H).mT @ (I + H)
        B = F @ F.mT
        # products with entry (i, J, k, L): M_ik S_JL, M_iJ S_kL, M_iL S_kJ
        ik = lambda M, S: M[..., :, None, :, None] * S[..., None, :, None, :]  # noqa: E731
        iJkL = lambda M, S: M[..., :, :, None, None] * S[..., None, None, :, :]  # noqa: E731
        iLkJ = lambda M, S: M[..., :, None, None, :] * S.mT[..., None, :, :, None]  # noqa: E731
        Ib = I.expand_as(H)
        eta, lv = self.mat.kv_eta, self.mat.kv_lambda
        if self.mat.kind == W.SVK:
            E_, nu = self.mat.params[0], self.mat.params[1]
            lam, mu = E_ * nu / ((1 + nu) * (1 - 2 * nu)), E_ / (2 * (1 + nu))
            E = 0.5 * (H + H.mT + H.mT @ H)
            S = lam * E.diagonal(dim1=-2, dim2=-1).sum(-1)[..., None, None] * I + 2 * mu * E
            A = ik(Ib, S) + lam * iJkL(F, F) + mu * (ik(B, Ib) + iLkJ(F, F))
        else:
            m10, m01, kap = self.mat.params
            jm1 = self._jm1(H)[..., 0, 0]
            J = 1 + jm1
            a, b = J ** (-2.0 / 3.0), J ** (-4.0 / 3.0)
            x = lambda s: s[..., None, None, None, None]  # noqa: E731
            G = torch.linalg.inv(F).mT
            I1 = C.diagonal(dim1=-2, dim2=-1).sum(-1)
            I2 = 0.5 * (I1 * I1 - (C * C).sum((-1, -2)))
            D2 = I1[..., None, None] * F - F @ C  # dI2/dF / 2
            c_g = -2.0 / 3.0 * m10 * a * I1 - 4.0 / 3.0 * m01 * b * I2 + kap * J * jm1
            # P = 2 m10 a F + 2 m01 b D2 + c_g G
            A = x(2 * m10 * a) * (ik(Ib, Ib) - 2.0 / 3.0 * iJkL(F, G))
            A = A + x(2 * m01 * b) * (2 * iJkL(F, F) + x(I1) * ik(Ib, Ib) - ik(Ib, C) - iLkJ(F, F) - ik(B, Ib)
                                      - 4.0 / 3.0 * iJkL(D2, G))
            dc = (x(-4.0 / 3.0 * m10 * a) * iJkL(G, F) + x(-8.0 / 3.0 * m01 * b) * iJkL(G, D2)
                  + x(4.0 / 9.0 * m10 * a * I1 + 16.0 / 9.0 * m01 * b * I2 + kap * J * (2 * J - 1)) * iJkL(G, G))
            A = A + dc - x(c_g) * iLkJ(G, G)
        A = alpha * A
        if eta or lv:
            Ed = 0.5 * (Fd.mT @ F + F.mT @ Fd)
            Sv = 2 * eta * Ed + lv * Ed.diagonal(dim1=-2, dim2=-1).sum(-1)[..., None, None] * I
            A = A + alpha * (ik(Ib, Sv) + eta * (ik(F @ Fd.mT, Ib) + iLkJ(F, Fd)) + lv * iJkL(F, Fd))
            A = A + beta * (eta * (ik(B, Ib) + iLkJ(F, F)) + lv * iJkL(F, F))
        return A

    def pattern(self):
        """Sorted adjacent node pairs: rank of a pair in its row node's list, list lengths and starts."""
        n, npn = self.n_nodes, self.nodes.shape[1]
        keys = torch.unique(torch.cat([torch.unique((self.nodes[e][:, :, None] * n + self.nodes[e][:, None, :]).reshape(-1))
                                       for e in self.chunks(100000)]))
        rows = keys // n
        length = torch.bincount(rows, minlength=n)
        start = torch.cumsum(length, 0) - length
        return keys, length, start

    def assemble(self, q, qdot, alpha, beta, mass_over_h=0.0, upper=False):
        """CSR values of alpha df/dq + beta df/dqdot (+ mass_over_h M), rows of 3x3 blocks."""
        keys, length, start = self.pattern()
        mc, n, npn = self.mc, self.n_nodes, self.nodes.shape[1]
        nen, nq = self.coef.shape[1], len(self.w)
        vals = torch.zeros(9 * mc * mc * len(keys), dtype=F64, device=self.X.device)
        ar = lambda k: torch.arange(k, device=self.X.device)  # noqa: E731
        for e in self.chunks(max(256, 1500000 // (nq * nen))):
            g, dV, H, Fd = self.kinematics(q, qdot, e)
            A = self.tangent(H, Fd, alpha, beta) * dV[..., None, None, None, None]
            k = len(e)
            T = A.reshape(k * nq, 27, 3) @ g.reshape(k * nq, nen, 3).transpose(1, 2).contiguous()  # (.., iJk, b)
            T = T.reshape(k, nq, 3, 3, 3 * nen).permute(0, 2, 1, 3, 4).reshape(k, 3, nq * 3, 3 * nen)
            G = g.permute(0, 2, 1, 3).reshape(k, 1, nen, nq * 3).expand(k, 3, nen, nq * 3).contiguous()
            K = (G @ T).reshape(k, 3, nen, 3, nen)  # (e, i, a, k, b)
            if mass_over_h:
                det = (dV / self.w).mean(1)
                M = DENSITY * mass_over_h * det[:, None, None] * self.mass_ref * self.scale[e][:, :, None] * self.scale[e][:, None, :]
                for d in range(3):
                    K[:, d, :, d, :] += M
            nd = self.nodes[e]
            rank = torch.searchsorted(keys, nd[:, :, None] * n + nd[:, None, :]) - start[nd][:, :, None]
            # row (I, c, i), column (J, c', k): 9 mc^2 start_I + (3 c + i) 3 mc len_I + 3 mc rank + 3 c' + k
            pa, ca = ar(nen) // mc, ar(nen) % mc
            base = 9 * mc * mc * start[nd][:, pa]  # (e, a)
            wid = 3 * mc * length[nd][:, pa]
            row = base[:, None, :] + (3 * ca[None, None, :] + ar(3)[None, :, None]) * wid[:, None, :]  # (e, i, a)
            col = 3 * mc * rank[:, pa][:, :, pa] + 3 * ca[None, None, :]  # (e, a, b)
            idx = row[:, :, :, None, None] + col[:, None, :, None, :] + ar(3)[None, None, None, :, None]
            vals.index_add_(0, idx.reshape(-1), K.reshape(-1))
        if not upper:
            return vals
        r = 3 * mc * torch.repeat_interleave(keys // n, 9 * mc * mc)  # first row of each value's node
        pos = torch.arange(len(vals), device=vals.device) - 9 * mc * mc * start[r // (3 * mc)]
        wid = 3 * mc * length[r // (3 * mc)]
        sub, c = pos // wid, pos % wid
        col = 3 * mc * (keys[start[r // (3 * mc)] + c // (3 * mc)] % n) + c % (3 * mc)
        return vals[col >= r + sub]

    def mass_times(self, dv):
        out = torch.zeros(self.n_dof // 3, 3, dtype=F64, device=dv.device)
        for e in self.chunks(200000):
            g, dV = self.geometry(e)
            M = DENSITY * (dV / self.w).mean(1)[:, None, None] * self.mass_ref * self.scale[e][:, :, None] * self.scale[e][:, None, :]
            out.index_add_(0, self.coef[e].reshape(-1), (M @ dv.reshape(-1, 3)[self.coef[e]]).reshape(-1, 3))
        return out.reshape(-1)

    def gradient(self, v, v_prev, f, f_ext):
        return self.mass_times(v - v_prev) / DT + f - f_ext


def exact(case, seed):
    dev = _dev()
    bodies = _inputs(case, seed)
    to = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)  # noqa: E731
    call = case["call"]
    if call == "batch":
        f, vals = [], []
        for b in bodies:
            x = _Exact(case, b)
            q, qd = to(b.q), to(b.qdot)
            f.append(x.force(q, qd))
            vals.append(x.assemble(q, qd, DT, 1.0))
        return torch.cat(f), torch.cat(vals)
    b = bodies[0]
    x, q, qd = _Exact(case, b), to(b.q), to(b.qdot)
    if call == "grad":
        q.requires_grad_(True)
        qd.requires_grad_(True)
        p = x.params().requires_grad_(True)
        f = x.force(q, qd, p)
        gq, gqd, gp = torch.autograd.grad(f, [q, qd, p], to(b.w), allow_unused=True, materialize_grads=True)
        return f.detach(), gq, gqd, gp
    if call == "adamw":
        return _exact_adamw(case, seed, x, q, qd)
    if call == "tangent":
        return x.assemble(q, qd, DT, 1.0)
    f = x.force(q, qd)
    if call == "force":
        return f
    if call == "upper":
        return f, x.assemble(q, qd, 1.0, 0.0, upper=True)
    if call == "assemble":
        return f, x.assemble(q, qd, DT, 1.0)
    v_prev, f_ext = (to(a) for a in _loads(case, seed, q.numel()))
    H = x.assemble(q, qd, DT, 1.0, mass_over_h=1.0 / DT, upper=call == "newton_upper")
    return f, H, x.gradient(qd, v_prev, f, f_ext)


def _exact_adamw(case, seed, x, q_n, v0):
    v_n, f_ext = (torch.from_numpy(a).to(q_n.device) for a in _loads(case, seed, q_n.numel()))
    v, p = v0.clone(), ADAMW
    g, m, s = torch.zeros_like(v), torch.zeros_like(v), torch.zeros_like(v)
    for it in range(1, case["iters"] + 1):
        m = p["beta1"] * m + (1 - p["beta1"]) * g
        s = p["beta2"] * s + (1 - p["beta2"]) * g * g
        step = (m / (1 - p["beta1"] ** it)) / (torch.sqrt(s / (1 - p["beta2"] ** it)) + p["eps"])
        v = v - p["lr"] * (step + p["weight_decay"] * v)
        q = q_n + DT * v
        g = x.gradient(v, v_n, x.force(q, v), f_ext)
    return v, q, g, case["iters"]
