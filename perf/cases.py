"""Workloads by which the speed of the solver's public entry points is followed.

Each case is a dict of plain values: the operation ("op"), the lattice of the
mesh (a x b x c hexahedra of 6 quadratic tetrahedra), the number of load cases
and the type and options of the call.  ``prepare`` makes the mesh handle and
the inputs from a seed, ``run`` does one call, ``work`` says what the call
cannot do without, and ``exact`` gives the result in 64 bits from the
definition of the operators (quadrature of B^T D B), with torch alone.

The element topology of a lattice is made once and kept; the moduli and every
vector come from the seed, and each state has a mesh handle of its own.
"""
import functools
import math

import numpy as np
import torch

from paper_1710_08679_amd import ebe, meshgen

DTYPES = {"f64": torch.float64, "f32": torch.float32}
EDGES = ((0, 1), (1, 2), (0, 2), (0, 3), (1, 3), (2, 3))


def listed():
    return [
        # The smallest call: one product of the 4^3 cube (384 tetrahedra, bottom
        # fixed, one case) by a program that wrote its own CG: launches only.
        {"name": "product f64 n=1 cube 4", "op": "product", "mesh": "cube", "a": 4, "b": 4, "c": 4,
         "dtype": "f64", "n": 1, "bc": True, "tuned": False},
        # A ragged crust block with an odd number of cases, P K P, default form.
        {"name": "product f32 n=5 crust 29x23x17", "op": "product", "mesh": "crust", "a": 29, "b": 23, "c": 17,
         "dtype": "f32", "n": 5, "bc": True, "tuned": False},
        # One case on the 64^3 cube: an ordinary single right-hand side solve's product.
        {"name": "product f64 n=1 cube 64", "op": "product", "mesh": "layered", "a": 64, "b": 64, "c": 64,
         "dtype": "f64", "n": 1, "bc": False, "tuned": True},
        # The four load cases of the inverse analysis, in FP32.
        {"name": "product f32 n=4 box 64x64x32", "op": "product", "mesh": "layered", "a": 64, "b": 64, "c": 32,
         "dtype": "f32", "n": 4, "bc": False, "tuned": True},
        # Sixteen cases on the 64^3 cube: the FP32 product of the preconditioner ...
        {"name": "product f32 n=16 cube 64", "op": "product", "mesh": "layered", "a": 64, "b": 64, "c": 64,
         "dtype": "f32", "n": 16, "bc": False, "tuned": True},
        # ... and the FP64 product of the outer loop: the largest call.
        {"name": "product f64 n=16 cube 64", "op": "product", "mesh": "layered", "a": 64, "b": 64, "c": 64,
         "dtype": "f64", "n": 16, "bc": False, "tuned": True},
        # Curved (isoparametric) elements, sixteen cases.
        {"name": "curved product f32 n=16 cube 40", "op": "product", "mesh": "curved", "a": 40, "b": 40, "c": 40,
         "dtype": "f32", "n": 16, "bc": False, "tuned": True},
        # The coarse operator of the multigrid preconditioner.
        {"name": "linear product f32 n=16 crust 64x64x32", "op": "linear", "mesh": "crust", "a": 64, "b": 64, "c": 32,
         "dtype": "f32", "n": 16, "bc": True, "tuned": True},
        # Both grid transfers of a multigrid cycle.
        {"name": "transfers f32 n=16 crust 48x48x24", "op": "transfers", "mesh": "crust", "a": 48, "b": 48, "c": 24,
         "dtype": "f32", "n": 16, "bc": True, "tuned": False},
        # The backward pass of the inverse analysis: the element gradient, four cases.
        {"name": "adjoint f64 n=4 box 64x64x32", "op": "adjoint", "mesh": "layered", "a": 64, "b": 64, "c": 32,
         "dtype": "f64", "n": 4, "bc": False, "tuned": False},
        # Whole solves: the small cube by plain CG (launches and host checks) ...
        {"name": "solve pcge f64 n=1 cube 4", "op": "solve", "mesh": "cube", "a": 4, "b": 4, "c": 4,
         "dtype": "f64", "n": 1, "bc": True, "tuned": False, "precond": "pcge", "mode": "fp64", "tol": 1e-10},
        # ... and sixteen cases on a crust block by the mixed-precision three-level solver.
        {"name": "solve mg3 mixed n=16 crust 48x48x24", "op": "solve", "mesh": "crust", "a": 48, "b": 48, "c": 24,
         "dtype": "f64", "n": 16, "bc": True, "tuned": False, "precond": "mg3", "mode": "mixed", "tol": 1e-10},
    ]


def _axes(rng, hexes_lo, hexes_hi):
    """Three axis lengths whose product lies between the bounds, log-uniformly, in odd proportions."""
    h = math.exp(rng.uniform(math.log(hexes_lo), math.log(hexes_hi)))
    side = h ** (1.0 / 3.0)
    a = max(2, min(96, round(side * rng.uniform(0.8, 1.3))))
    b = max(2, min(96, round(side * rng.uniform(0.8, 1.3))))
    c = max(2, min(64, int(h / (a * b))))
    return a, b, c


def draw(rng):
    op = rng.choice(["product"] * 8 + ["linear", "linear", "transfers", "adjoint", "adjoint", "solve", "solve"])
    n = rng.choice([1, 2, 3, 4, 5, 6, 7, 8, 11, 12, 13, 16, 16, 16])
    case = {"op": op, "dtype": rng.choice(["f64", "f32"]), "n": n, "bc": False, "tuned": False}
    if op == "solve":
        a, b, c = _axes(rng, 4 * 4 * 4, 40 * 40 * 24)
        case.update(mesh="crust", dtype="f64", bc=True, precond=rng.choice(["mg3", "mg3", "mg2"]),
                    mode=rng.choice(["mixed", "mixed", "fp64"]), tol=1e-10)
    else:
        a, b, c = _axes(rng, 4 * 4 * 4, 60 * 60 * 60)
        kinds = {"product": ["layered", "crust", "crust", "curved"], "linear": ["crust"], "transfers": ["crust"],
                 "adjoint": ["layered"]}[op]
        case.update(mesh=rng.choice(kinds))
        case["bc"] = case["mesh"] == "crust"
        case["tuned"] = op in ("product", "linear") and rng.random() < 0.7
    case.update(a=a, b=b, c=c)
    return case


# ---- inputs ------------------------------------------------------------------
@functools.lru_cache(maxsize=3)
def _lattice(mesh, a, b, c):
    rng = meshgen.rng_for(2, 8000 + a * 97 + b * 31 + c)
    if mesh == "crust":
        return meshgen.crust_mesh(a, b, c)
    if mesh == "cube":
        m = meshgen.kuhn_mesh(a, b, c)
        meshgen.fix_faces(m, [(2, 0)])
        return m
    m = meshgen.kuhn_mesh(a, b, c, jitter=0.2, rng=rng)
    meshgen.set_layers_flat(m)
    return meshgen.quadratic_map(m, 0.25) if mesh == "curved" else m


def _host(case, seed):
    """The lattice, and its elements' moduli for this seed."""
    m = _lattice(case["mesh"], case["a"], case["b"], case["c"])
    young = m.young * np.random.default_rng(seed).uniform(0.8, 1.25, m.n_elem)
    return m, young


def _vectors(case, m, seed):
    """The call's input vectors: N(0, 1) values; for a solve, nodal loads on the top surface."""
    gen = torch.Generator(device="cuda").manual_seed(seed)

    def randn(rows):
        return torch.randn((rows, 3, case["n"]), generator=gen, dtype=torch.float64,
                           device="cuda").to(DTYPES[case["dtype"]])

    if case["op"] == "linear":
        return [randn(m.n_vertices)]
    if case["op"] == "transfers":
        return [randn(m.n_vertices), randn(m.n_nodes)]
    if case["op"] == "adjoint":
        return [randn(m.n_nodes), randn(m.n_nodes)]
    if case["op"] == "solve":
        f = randn(m.n_nodes)
        top = torch.from_numpy(m.xyz[:, 2] > m.xyz[:, 2].max() - 1e-9).cuda()
        return [torch.where(top[:, None, None], f, torch.zeros((), dtype=f.dtype, device="cuda"))]
    return [randn(m.n_nodes)]


def prepare(case, seed):
    m, young = _host(case, seed)
    fixed = m.fixed if m.fixed.any() else None
    mesh = ebe.Mesh(m.xyz, m.conn, m.n_vertices, young, m.poisson, fixed, curved=case["mesh"] == "curved")
    state = {"case": case, "mesh": mesh, "in": _vectors(case, m, seed)}
    dt = DTYPES[case["dtype"]]
    if case["tuned"]:
        mesh.autotune(1 if case["op"] == "linear" else 0, dt, case["n"])
    if case["op"] == "adjoint":
        state["out"] = [torch.empty((m.n_elem,), dtype=dt, device="cuda")]
    elif case["op"] == "transfers":
        state["out"] = [torch.empty_like(state["in"][1]), torch.empty_like(state["in"][0])]
    else:
        state["out"] = [torch.empty_like(state["in"][0])]
    if case["op"] == "solve":
        precond = {"pcge": ebe.PREC_PCGE, "mg2": ebe.PREC_MG2, "mg3": ebe.PREC_MG3}[case["precond"]]
        mode = {"fp64": ebe.MODE_FP64, "mixed": ebe.MODE_MIXED}[case["mode"]]
        state["opts"] = ebe.default_opts(precond=precond, mode=mode, tol=case["tol"])
    return state


def run(state):
    case, mesh, vin, out = state["case"], state["mesh"], state["in"], state["out"]
    op, bc = case["op"], case["bc"]
    if op == "product":
        return mesh.matvec(vin[0], apply_bc=bc, out=out[0])
    if op == "linear":
        return mesh.matvec_p1(vin[0], apply_bc=bc, out=out[0])
    if op == "transfers":
        return [mesh.prolong(vin[0], apply_bc=bc, out=out[0]), mesh.restrict(vin[1], apply_bc=bc, out=out[1])]
    if op == "adjoint":
        return mesh.adjoint_grad(vin[0], vin[1], out=out[0])
    return mesh.solve(vin[0], u=out[0], opts=state["opts"])[0]


# ---- what a call cannot do without ----------------------------------------------
def work(case):
    a, b, c, n = case["a"], case["b"], case["c"], case["n"]
    p = 8 if case["dtype"] == "f64" else 4
    elems = 6 * a * b * c
    corners = (a + 1) * (b + 1) * (c + 1)
    nodes = (2 * a + 1) * (2 * b + 1) * (2 * c + 1)
    # quadratic element: 440 flops for the operator and 30 additions per case, 80 for its geometry
    # (curved: 710, and 4 x 100); a linear one: 90 and 40
    per_case, per_elem = (710 + 30, 400) if case["mesh"] == "curved" else (440 + 30, 80)
    geometry = 40 * elems + 24 * (nodes if case["mesh"] == "curved" else corners) + 2 * p * elems
    if case["op"] == "linear":
        return {"bytes": 2 * 3 * corners * n * p + 16 * elems + 24 * corners + 2 * p * elems,
                "flops": elems * (90 * n + 40)}
    if case["op"] == "transfers":  # each vector once, and the two ends of every edge node for each direction
        return {"bytes": 2 * 3 * (corners + nodes) * n * p + 2 * 8 * (nodes - corners),
                "flops": 3 * n * 4 * (nodes - corners)}
    if case["op"] == "adjoint":
        return {"bytes": 2 * 3 * nodes * n * p + geometry + p * elems, "flops": elems * (500 * n + per_elem)}
    # a product; a solve cannot do without the loads, the solution and one product that shows the residual
    return {"bytes": 2 * 3 * nodes * n * p + geometry, "flops": elems * (per_case * n + per_elem)}


# ---- the same results in 64 bits, from the definitions --------------------------------
def _shape_gradients(L):
    """dN_a/dL_k (10, 4) of the quadratic shape functions at barycentric point L."""
    d = torch.zeros((10, 4), dtype=torch.float64)
    for k in range(4):
        d[k, k] = 4.0 * L[k] - 1.0
    for e, (i, j) in enumerate(EDGES):
        d[4 + e, i] = 4.0 * L[j]
        d[4 + e, j] = 4.0 * L[i]
    return d


def _element_matrices(x, young, poisson, linear):
    """K_e (E, 3 m, 3 m), m = 4 or 10 nodes (row 3 a + i), by quadrature of B^T D B."""
    if linear:
        points = [(torch.eye(4, dtype=torch.float64), 1.0 / 6.0)]
    else:
        qa, qb = (5.0 + 3.0 * math.sqrt(5.0)) / 20.0, (5.0 - math.sqrt(5.0)) / 20.0
        points = [(_shape_gradients([qa if k == q else qb for k in range(4)]), 1.0 / 24.0) for q in range(4)]
    lam = young * poisson / ((1 + poisson) * (1 - 2 * poisson))
    mu = young / (2 * (1 + poisson))
    m = x.shape[1]
    K = torch.zeros((x.shape[0], m, 3, m, 3), dtype=torch.float64, device=x.device)
    eye = torch.eye(3, dtype=torch.float64, device=x.device)
    for dL, w in points:
        dr = (dL[:, 1:] - dL[:, :1]).to(x.device)  # (m, 3): derivatives by L_1..L_3, L_0 = 1 - L_1 - L_2 - L_3
        J = torch.matmul(x.transpose(1, 2).contiguous(), dr)  # dx_i/dr_j
        g = torch.matmul(dr, torch.linalg.inv(J))  # (E, m, 3): grad N_a
        s = w * torch.linalg.det(J)
        gg = g[:, :, :, None, None] * g[:, None, None, :, :]  # (a, i, b, j): g_a,i g_b,j
        K += (lam * s)[:, None, None, None, None] * gg
        K += (mu * s)[:, None, None, None, None] * gg.permute(0, 1, 4, 3, 2)
        dot = torch.matmul(g, g.transpose(1, 2).contiguous())  # (a, b)
        K += (mu * s)[:, None, None, None, None] * dot[:, :, None, :, None] * eye[None, None, :, None, :]
    return K.reshape(x.shape[0], 3 * m, 3 * m)


class _Operator:
    """Element matrices and connectivity, in chunks (kept for a solve, else formed as they are used)."""

    def __init__(self, m, young, linear, keep):
        self.m, self.young, self.linear, self.keep = m, young, linear, {} if keep else None
        self.loc, self.chunk = (4 if linear else 10), 65536
        self.xyz = torch.from_numpy(m.xyz).cuda()

    def parts(self):
        for s in range(0, self.m.n_elem, self.chunk):
            if self.keep is not None and s in self.keep:
                yield (s,) + self.keep[s]
                continue
            conn = torch.from_numpy(self.m.conn[s:s + self.chunk, :self.loc].astype(np.int64)).cuda()
            young, poisson = (torch.from_numpy(v[s:s + self.chunk]).cuda() for v in (self.young, self.m.poisson))
            K = _element_matrices(self.xyz[conn], young, poisson, self.linear)
            if self.keep is not None:
                self.keep[s] = (conn, K)
            yield s, conn, K

    def product(self, x):
        y = torch.zeros_like(x)
        for _, conn, K in self.parts():
            ye = torch.matmul(K, x[conn].reshape(conn.shape[0], 3 * self.loc, -1))
            y.index_add_(0, conn.reshape(-1), ye.reshape(-1, 3, x.shape[2]))
        return y

    def diagonal(self, rows):
        d = torch.zeros((rows, 3, 3), dtype=torch.float64, device="cuda")
        for _, conn, K in self.parts():
            K5 = K.reshape(-1, self.loc, 3, self.loc, 3)
            for a in range(self.loc):
                d.index_add_(0, conn[:, a], K5[:, a, :, a, :].contiguous())
        return d


def _solve(op, f, free):
    """Block-Jacobi CG in FP64 on the free DOFs, to a residual far below any solve's tolerance."""
    eye = torch.eye(3, dtype=torch.float64, device="cuda")
    keep = free[:, :, None] * free[:, None, :]
    minv = torch.linalg.inv(op.diagonal(f.shape[0]) * keep + eye * (1 - free)[:, :, None])
    mask = free[:, :, None]
    u, r = torch.zeros_like(f), f * mask
    target = 1e-13 * r.square().sum((0, 1)).sqrt()
    z = torch.matmul(minv, r)
    p, rho = z.clone(), (r * z).sum((0, 1))
    for _ in range(4000):
        q = op.product(p) * mask
        alpha = rho / (p * q).sum((0, 1)).clamp_min(1e-300)
        u += alpha * p
        r -= alpha * q
        if bool((r.square().sum((0, 1)).sqrt() <= target).all()):
            break
        z = torch.matmul(minv, r)
        new = (r * z).sum((0, 1))
        p = z + (new / rho.clamp_min(1e-300)) * p
        rho = new
    return u


def exact(case, seed):
    m, young = _host(case, seed)
    vin = [v.double() for v in _vectors(case, m, seed)]
    free = torch.from_numpy(1.0 - m.fixed.astype(np.float64)).cuda()
    op = case["op"]
    if op == "transfers":
        ends = np.zeros((m.n_nodes - m.n_vertices, 2), dtype=np.int64)
        for e, (i, j) in enumerate(EDGES):
            ends[m.conn[:, 4 + e] - m.n_vertices, 0] = m.conn[:, i]
            ends[m.conn[:, 4 + e] - m.n_vertices, 1] = m.conn[:, j]
        ends = torch.from_numpy(ends).cuda()
        up = torch.cat([vin[0], 0.5 * (vin[0][ends[:, 0]] + vin[0][ends[:, 1]])])
        down = vin[1][:m.n_vertices].clone()
        half = 0.5 * vin[1][m.n_vertices:]
        down.index_add_(0, ends[:, 0], half)
        down.index_add_(0, ends[:, 1], half)
        if case["bc"]:
            up, down = up * free[:, :, None], down * free[:m.n_vertices, :, None]
        return [up, down]
    if op == "adjoint":
        A = _Operator(m, np.ones_like(young), False, False)
        g = torch.empty((m.n_elem,), dtype=torch.float64, device="cuda")
        for s, conn, K in A.parts():
            ue, le = (v[conn].reshape(conn.shape[0], 30, -1) for v in vin)
            g[s:s + conn.shape[0]] = -(le * torch.matmul(K, ue)).sum((1, 2))
        return g
    if op == "solve":
        return _solve(_Operator(m, young, False, True), vin[0], free)
    A = _Operator(m, young, op == "linear", False)
    x = vin[0]
    if not case["bc"]:
        return A.product(x)
    mask = free[:x.shape[0], :, None]
    return A.product(x * mask) * mask
