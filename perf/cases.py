"""The work a user of this library has it do, as measurable cases.

Every case is one pass through the public calls of `paper_2107_11541_amd` on a
jittered unit cube: assembling the operators (each element type, FP64 and
mixed), the explicit step's passes, the pressure solve, a whole time step, the
serving runtime, and the solver kernels on their own.  `prepare` builds what a
program holds before the call (the mesh uploaded, the fields in HBM); `run` is
the call.  Meshes are either ordered by the program itself along a Morton
curve and uploaded as they are (`shuffled` false: results come in the
program's own numbering), or arrive in random order and are renumbered by the
library (`shuffled` true).
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2107_11541_amd as fe

HEX, PRISM, PYRAMID, TET, HYBRID = "hex", "prism", "pyramid", "tet", "hybrid"
PER_CUBE = {HEX: 1, PRISM: 2, PYRAMID: 6, TET: 6, HYBRID: 3.8}       # elements per cube of the grid
PATTERN = {HEX: 27, PRISM: 21, PYRAMID: 26, TET: 15, HYBRID: 19.5}   # CSR entries per row, about
NEN = {HEX: 8, PRISM: 6, PYRAMID: 5, TET: 4, HYBRID: 5}
CODE = {HEX: fe.HEX08, PRISM: fe.PEN06, PYRAMID: fe.PYR05, TET: fe.TET04, HYBRID: fe.HYBRID}
OPERATOR = {"momentum": fe.MOMENTUM, "scalar": fe.SCALAR, "poisson": fe.POISSON}


def listed():
    return [
        # The smallest mesh of the tests and the smoke run: every launch and every wait counts.
        dict(name="step_hex_10", kind="step", mesh=HEX, n=10, shuffled=False, rtol=1e-10, iterations=1000),
        # The benchmark's time step: momentum and pressure operators, Dirichlet, exactly 200 CG iterations.
        dict(name="step_hex_128", kind="step", mesh=HEX, n=128, shuffled=True, rtol=0.0, iterations=200),
        # The implicit momentum operator on a tetrahedral flame mesh (547 k elements).
        dict(name="momentum_tet_45", kind="assemble", mesh=TET, n=45, shuffled=False, operator="momentum",
             scalars=0, mixed=False),
        # Five species equations in one call, with mixed-precision quadrature.
        dict(name="scalars_mixed_hex_72", kind="assemble", mesh=HEX, n=72, shuffled=False, operator="scalar",
             scalars=5, mixed=True),
        # The momentum operator on a mesh of prisms, hexahedra, pyramids and tetrahedra, as burner meshes are.
        dict(name="momentum_hybrid_64", kind="assemble", mesh=HYBRID, n=64, shuffled=True, operator="momentum",
             scalars=0, mixed=False),
        # The pressure Laplacian of a boundary-layer mesh of prisms.
        dict(name="poisson_prism_57", kind="assemble", mesh=PRISM, n=57, shuffled=False, operator="poisson",
             scalars=0, mixed=False),
        # The 3x3-block momentum operator with full stress and EMAC convection.
        dict(name="block_hex_40", kind="block", mesh=HEX, n=40, shuffled=False, form=3),
        # One Runge-Kutta stage's matrix-free residual.
        dict(name="residual_hex_101", kind="residual", mesh=HEX, n=101, shuffled=False, form=0),
        # A whole explicit step: three stages, divergence, pressure solve, correction.
        dict(name="fractional_hex_64", kind="fractional", mesh=HEX, n=64, shuffled=False, form=3, rtol=1e-8),
        # The pressure solve by single-precision CG inside double-precision refinement.
        dict(name="solve_mixed_hex_80", kind="solve", mesh=HEX, n=80, shuffled=False, mixed=True, rtol=1e-11),
        # A dozen independent requests through the serving runtime: host meshes in, host pressures out.
        dict(name="serve_12", kind="serve", mesh=HEX, requests=12, lo=8, hi=48, stream=3),
        # The solver's own kernels in a program that writes its own iteration.
        dict(name="kernels_pyramid_40", kind="kernels", mesh=PYRAMID, n=40, shuffled=False),
    ]


# kind -> (largest number of elements, meshes)
RANGE = {"step": (1_000_000, (HEX, TET, PRISM, PYRAMID, HYBRID)), "assemble": (2_000_000, (HEX, TET, PRISM, PYRAMID, HYBRID)),
         "block": (120_000, (HEX, TET, HYBRID)), "residual": (2_000_000, (HEX, TET, PRISM, PYRAMID, HYBRID)),
         "fractional": (400_000, (HEX, TET, HYBRID)), "solve": (1_000_000, (HEX, TET, HYBRID)),
         "kernels": (2_000_000, (HEX, TET, PRISM, PYRAMID, HYBRID))}


def draw(rng):
    kind = rng.choice(["step", "assemble", "assemble", "assemble", "block", "residual", "fractional", "solve", "solve",
                       "serve", "kernels"])
    if kind == "serve":
        return dict(kind=kind, mesh=HEX, requests=rng.randint(1, 12), lo=8, hi=rng.randint(12, 48),
                    stream=rng.randrange(1 << 30))
    most, meshes = RANGE[kind]
    mesh = rng.choice(meshes)
    elements = math.exp(rng.uniform(math.log(600), math.log(most)))
    n = max(5, int((elements / PER_CUBE[mesh]) ** (1 / 3)))
    case = dict(kind=kind, mesh=mesh, n=n, shuffled=mesh == HYBRID or rng.random() < 0.4)
    if kind == "step":
        # a fixed count stays below what converges to the last bit
        fixed = rng.random() < 0.5
        case.update(rtol=0.0 if fixed else 1e-10, iterations=rng.randint(n, 2 * n) if fixed else 2000)
    elif kind == "assemble":
        op = rng.choice(list(OPERATOR))
        case.update(operator=op, scalars=rng.randint(1, 5) if op == "scalar" else 0, mixed=rng.random() < 0.3)
    elif kind in ("block", "residual"):
        case.update(form=rng.randint(0, 3))
    elif kind == "fractional":
        case.update(form=rng.randint(0, 3), rtol=1e-8)
    elif kind == "solve":
        mixed = rng.random() < 0.4
        case.update(mixed=mixed, rtol=1e-11 if mixed else rng.choice([1e-8, 1e-10]))
    return case


# --- meshes -------------------------------------------------------------------------------------------------------
# The cube's corners 0:(-,-,-) 1:(+,-,-) 2:(+,+,-) 3:(-,+,-) and 4..7 above them; splits that conform.
KUHN = np.array([[0, 1, 2, 6], [0, 2, 3, 6], [0, 3, 7, 6], [0, 7, 4, 6], [0, 4, 5, 6], [0, 5, 1, 6]])
HALVES = np.array([[0, 1, 2, 4, 5, 6], [0, 2, 3, 4, 6, 7]])
FACES = np.array([[0, 1, 2, 3], [4, 7, 6, 5], [0, 4, 5, 1], [3, 2, 6, 7], [0, 3, 7, 4], [1, 5, 6, 2]])


def spread(v):
    """The bits of v (< 1024) three places apart."""
    v = v.astype(np.int64)
    v = (v | v << 16) & 0x030000FF
    v = (v | v << 8) & 0x0300F00F
    v = (v | v << 4) & 0x030C30C3
    return (v | v << 2) & 0x09249249


def build_mesh(mesh, n, rng, shuffled):
    """coords [N, 3], conn [E, nen] ([E, 8] padded with -1 for a hybrid), types (hybrid), boundary nodes."""
    h, m = 1.0 / n, n + 1
    i, j, k = (a.ravel() for a in np.meshgrid(*[np.arange(m)] * 3, indexing="ij"))
    at = np.stack([k, j, i], axis=1)                        # x fastest
    move = rng.uniform(-0.12 * h, 0.12 * h, at.shape)
    move[(at == 0) | (at == n)] = 0.0                       # boundary nodes stay on their faces
    coords = at * h + move
    boundary = ((at == 0) | (at == n)).any(axis=1)
    z, y, x = (a.ravel() for a in np.meshgrid(*[np.arange(n)] * 3, indexing="ij"))
    order = np.argsort(spread(x) | spread(y) << 1 | spread(z) << 2, kind="stable")
    x, y, z = x[order], y[order], z[order]
    base = x + m * (y + m * z)
    cubes = base[:, None] + np.array([0, 1, m + 1, m, m * m, m * m + 1, m * m + m + 1, m * m + m])
    types = None
    if mesh == HEX:
        conn = cubes
    elif mesh == TET:
        conn = cubes[:, KUHN].reshape(-1, 4)
    elif mesh == PRISM:
        conn = cubes[:, HALVES].reshape(-1, 6)
    elif mesh == PYRAMID:
        centre = len(coords) + np.arange(len(cubes))
        coords = np.concatenate([coords, coords[cubes].mean(axis=1)])
        apex = np.broadcast_to(centre[:, None, None], (len(cubes), 6, 1))
        conn = np.concatenate([cubes[:, FACES], apex], axis=2).reshape(-1, 5)
    else:
        # slabs along x: prisms, hexahedra, one slab of pyramids and tetrahedra around a centre node, tetrahedra
        turn = np.flatnonzero(x == n // 2)
        centre = len(coords) + np.arange(len(turn))
        coords = np.concatenate([coords, coords[cubes[turn]].mean(axis=1)])
        t, apex = cubes[turn], centre[:, None]
        parts = [(6, cubes[x < n // 4][:, HALVES].reshape(-1, 6)),
                 (8, cubes[(x >= n // 4) & (x < n // 2)]),
                 (5, np.concatenate([t[:, FACES[4]], apex], axis=1))]
        parts += [(4, np.concatenate([t[:, FACES[f][list(c)]], apex], axis=1))
                  for f in (0, 1, 2, 3, 5) for c in ((0, 1, 2), (0, 2, 3))]
        parts += [(4, cubes[x > n // 2][:, KUHN].reshape(-1, 4))]
        conn = np.concatenate([np.pad(c, ((0, 0), (0, 8 - w)), constant_values=-1) for w, c in parts])
        types = np.concatenate([np.full(len(c), w, np.uint8) for w, c in parts])
    boundary = np.concatenate([boundary, np.zeros(len(coords) - len(boundary), bool)])
    if shuffled:
        old = rng.permutation(len(coords))                  # new node -> old
        elems = rng.permutation(len(conn))
        conn, types = conn[elems], None if types is None else types[elems]
    else:                                                   # nodes in the order in which the elements meet them
        first = np.full(len(coords), conn.size)
        np.minimum.at(first, conn.ravel(), np.arange(conn.size))
        old = np.argsort(first, kind="stable")
    new = np.empty(len(old), np.int64)
    new[old] = np.arange(len(old))
    conn = np.where(conn >= 0, new[conn], -1).astype(np.int32)
    return coords[old], np.ascontiguousarray(conn), types, np.flatnonzero(boundary[old]).astype(np.int32)


def build_fields(coords, n, rng, scalars=0):
    """Taylor-Green velocity with noise, a hot kernel's density and viscosity, species."""
    x, y, z = (2 * math.pi * coords).T
    u = np.stack([np.sin(x) * np.cos(y) * np.cos(z), -np.cos(x) * np.sin(y) * np.cos(z), np.zeros_like(x)])
    u += rng.normal(0.0, 0.01, u.shape)
    hot = 0.5 * (1.0 - np.tanh((np.linalg.norm(coords - 0.5, axis=1) - 0.25) / 0.03))
    T = 300.0 + 1700.0 * hot
    rho = 101325.0 / (287.05 * T)
    mu = 1.716e-5 * (T / 273.15) ** 1.5 * (273.15 + 110.4) / (T + 110.4)
    Y = rng.uniform(0.0, 1.0, (scalars, len(coords)))
    D = 10.0 ** rng.uniform(-6.0, -4.0, scalars)
    return dict(u=u, rho=rho, mu=mu, Y=Y, D=D, dt=0.5 / n)


def sides(case):
    r = np.random.default_rng(case["stream"])
    return np.rint(np.exp(r.uniform(math.log(case["lo"]), math.log(case["hi"]), case["requests"]))).astype(int).tolist()


def inputs(case, seed):
    """The case's host inputs: one mesh and its fields, or one of each per request."""
    if case["kind"] == "serve":
        out = []
        for q, n in enumerate(sides(case)):
            r = np.random.default_rng([seed, q])
            m = build_mesh(HEX, n, r, False)
            out.append((m, build_fields(m[0], n, r)))
        return out
    r = np.random.default_rng(seed)
    m = build_mesh(case["mesh"], case["n"], r, case["shuffled"])
    return m, build_fields(m[0], case["n"], r, case.get("scalars", 0))


# --- the calls ----------------------------------------------------------------------------------------------------
def context(_kept=[]):
    """A program's one context."""
    if not _kept:
        _kept.append(fe.Context(0))
    return _kept[0]


def prepare(case, seed):
    kind, ctx = case["kind"], context()
    given = inputs(case, seed)
    if kind == "serve":
        return dict(kind=kind, given=given, server=fe.Server(ctx, hbm_budget=2 << 30, max_slots=16, host_threads=8))
    (coords, conn, types, boundary), f = given
    mesh = fe.Mesh(ctx, CODE[case["mesh"]], coords, conn, boundary, renumber=case["shuffled"], types=types)
    s = dict(kind=kind, mesh=mesh, dt=f["dt"], shuffled=case["shuffled"])
    for name in ("u", "rho", "mu", "Y"):
        a = torch.as_tensor(np.ascontiguousarray(f[name]), device="cuda")
        s[name] = mesh.to_mesh(a) if a.numel() else a
    new = lambda *shape: torch.empty(shape, dtype=torch.float64, device="cuda")  # noqa: E731
    N, nnz = mesh.n_nodes, mesh.nnz
    if kind == "step":
        s.update(V=new(1, nnz), B=new(3, N), L=new(1, nnz), f=new(1, N), rtol=case["rtol"], iterations=case["iterations"])
    elif kind == "assemble":
        k = max(1, case["scalars"])
        s.update(op=OPERATOR[case["operator"]], D=f["D"], precision=fe.MIXED if case["mixed"] else fe.FP64,
                 V=new(k, nnz), B=new(3 if case["operator"] == "momentum" else k, N))
    elif kind == "block":
        s.update(form=case["form"], V=new(nnz, 3, 3), B=new(3, N))
    elif kind == "residual":
        s.update(form=case["form"], out=new(4, N))
    elif kind in ("solve", "fractional"):
        L, b, _ = fe.assemble(mesh, fe.POISSON, s["dt"], s["u"], s["rho"])
        fe.apply_dirichlet(mesh, L, b)
        s.update(L=L[0], f=b[0], rtol=case["rtol"], form=case.get("form", 0))
        s["precision"] = fe.MIXED if case.get("mixed") else fe.FP64
        if kind == "fractional":
            s.update(u0=s["u"].clone(), p=new(N))
    elif kind == "kernels":
        r = np.random.default_rng([seed, 1])
        s["A"] = torch.as_tensor(r.standard_normal(nnz), device="cuda")
        s["x"] = torch.as_tensor(r.standard_normal(N), device="cuda")
        s["w"] = torch.as_tensor(r.standard_normal(N), device="cuda")
        s["y"], s["z"] = new(N), new(N)
    return s


def in_program_order(s, t):
    """A nodal result in the numbering the program gave its mesh in."""
    return s["mesh"].to_user(t) if s["shuffled"] else t


def run(s):
    kind = s["kind"]
    if kind == "serve":
        server = s["server"]
        tickets = [server.submit(fe.HEX08, m[0], m[1], m[3], f["dt"], f["u"], f["rho"], f["mu"], rtol=1e-8,
                                 want_mom_rhs=True) for m, f in s["given"]]
        done = [server.wait(t) for t in tickets]
        return [[d["x"], d["mom_rhs"]] for d in done]
    mesh = s["mesh"]
    if kind == "step":
        V, B, _ = fe.assemble(mesh, fe.MOMENTUM, s["dt"], s["u"], s["rho"], s["mu"], values=s["V"], rhs=s["B"])
        L, f, _ = fe.assemble(mesh, fe.POISSON, s["dt"], s["u"], s["rho"], values=s["L"], rhs=s["f"])
        fe.apply_dirichlet(mesh, L, f)
        x, _ = fe.cg_solve(mesh, L[0], f[0], rtol=s["rtol"], max_iter=s["iterations"])
        return dict(V=V, B=B, L=L, f=f, x=in_program_order(s, x))
    if kind == "assemble":
        mu = s["mu"] if s["op"] == fe.MOMENTUM else None
        Y, D = (s["Y"], s["D"]) if s["op"] == fe.SCALAR else (None, None)
        V, B, _ = fe.assemble(mesh, s["op"], s["dt"], s["u"], s["rho"], mu, Y, D, precision=s["precision"],
                              values=s["V"], rhs=s["B"])
        return dict(V=V, B=B)
    if kind == "block":
        V, B, _ = fe.assemble_block(mesh, s["form"], s["dt"], s["u"], s["rho"], s["mu"], values=s["V"], rhs=s["B"])
        return dict(V=V, B=B)
    if kind == "residual":
        return dict(r=in_program_order(s, fe.residual(mesh, s["u"], s["rho"], s["mu"], out=s["out"], form=s["form"])))
    if kind == "fractional":
        s["u"].copy_(s["u0"])
        s["p"].zero_()
        fe.fractional_step(mesh, s["dt"], s["rho"], s["mu"], s["L"], s["u"], s["p"], rtol=s["rtol"], form=s["form"])
        return dict(u=in_program_order(s, s["u"]), p=in_program_order(s, s["p"]))
    if kind == "solve":
        x, _ = fe.cg_solve(mesh, s["L"], s["f"], rtol=s["rtol"], precision=s["precision"])
        return dict(x=in_program_order(s, x))
    y = fe.spmv(mesh, s["A"], s["x"], s["y"])
    d = fe.dot(mesh.ctx, s["w"], y)
    s["z"].copy_(s["w"])
    fe.axpy(mesh.ctx, 0.25, y, s["z"])
    return dict(y=y, d=d, z=s["z"])


# --- what a pass cannot do without --------------------------------------------------------------------------------
def size(mesh, n):
    """(nodes, elements, CSR entries), near enough for counting bytes."""
    N = (n + 1) ** 3 + (n ** 3 if mesh == PYRAMID else n * n if mesh == HYBRID else 0)
    nnz = {HEX: (3 * n + 1) ** 3, TET: N + 6 * n * (n + 1) ** 2 + 6 * n * n * (n + 1) + 2 * n ** 3}.get(mesh, PATTERN[mesh] * N)
    return N, PER_CUBE[mesh] * n ** 3, nnz


def operator_work(mesh, n, nodal_in, rhs, mats=1, per_entry=1):
    N, E, nnz = size(mesh, n)
    a = NEN[mesh]
    points = 8 if a in (8, 5) else 6 if a == 6 else 4
    return dict(bytes=8 * N * (3 + nodal_in + rhs) + 4 * a * E + 8 * nnz * mats * per_entry,
                flops=E * points * (100 + mats * per_entry * 8 * a * a))


def cg_work(mesh, n, iterations):
    N, _, nnz = size(mesh, n)
    # the matrix and its column of indices once per iteration, x, r, p, q and the diagonal
    return dict(bytes=iterations * (12 * nnz + 20 * N + 64 * N), flops=iterations * (2 * nnz + 12 * N))


def iterations_of(n):
    """CG iterations to 1e-8 on these cubes, about (1.9 per cell along a side)."""
    return 10 + int(1.8 * n)


def add(*parts):
    return {k: sum(p[k] for p in parts) for k in ("bytes", "flops")}


def work(case):
    kind, mesh = case["kind"], case["mesh"]
    if kind == "serve":
        return add(*[add(operator_work(HEX, n, 5, 3), operator_work(HEX, n, 4, 1), cg_work(HEX, n, iterations_of(n)))
                     for n in sides(case)])
    n = case["n"]
    if kind == "step":
        its = case["iterations"] if case["rtol"] <= 0 else int(1.25 * iterations_of(n))
        return add(operator_work(mesh, n, 5, 3), operator_work(mesh, n, 4, 1), cg_work(mesh, n, its))
    if kind == "assemble":
        k = case["scalars"]
        if k:
            return operator_work(mesh, n, 4 + k, k, k)
        return operator_work(mesh, n, 5, 3) if case["operator"] == "momentum" else operator_work(mesh, n, 4, 1)
    if kind == "block":
        return operator_work(mesh, n, 5, 3, per_entry=9)
    if kind == "residual":
        return operator_work(mesh, n, 5, 4, mats=0)
    if kind == "fractional":
        passes = [operator_work(mesh, n, 5, 4, mats=0)] * 3 + [operator_work(mesh, n, 4, 1, mats=0)] * 2
        return add(*passes, cg_work(mesh, n, iterations_of(n)))
    if kind == "solve":
        w = cg_work(mesh, n, int(1.4 * iterations_of(n)))
        return dict(bytes=w["bytes"] * 0.6, flops=w["flops"]) if case["mixed"] else w
    N, _, nnz = size(mesh, n)
    return dict(bytes=12 * nnz + 20 * N + 16 * N + 24 * N, flops=2 * nnz + 4 * N)


# --- the same in plain torch, FP64 --------------------------------------------------------------------------------
def reference(a):
    """Shape functions [g][a], reference gradients [g][a][3] and weights [g] of an element with a nodes."""
    s = 1 / math.sqrt(3)
    N, dN, w = [], [], []
    if a == 8:
        sg = np.array([[-1, -1, -1], [1, -1, -1], [1, 1, -1], [-1, 1, -1], [-1, -1, 1], [1, -1, 1], [1, 1, 1], [-1, 1, 1]])
        for p in s * sg:
            f = 1 + sg * p
            N.append(f.prod(axis=1) / 8)
            dN.append(np.stack([sg[:, 0] * f[:, 1] * f[:, 2], sg[:, 1] * f[:, 0] * f[:, 2], sg[:, 2] * f[:, 0] * f[:, 1]], 1) / 8)
            w.append(1.0)
    elif a == 4:
        q = (5 - math.sqrt(5)) / 20
        for g in range(4):
            N.append(np.where(np.arange(4) == g, 1 - 3 * q, q))
            dN.append(np.array([[-1.0, -1, -1], [1, 0, 0], [0, 1, 0], [0, 0, 1]]))
            w.append(1 / 24)
    elif a == 6:
        for z in (-s, s):
            for px, py in ((1 / 6, 1 / 6), (2 / 3, 1 / 6), (1 / 6, 2 / 3)):
                L, dL = np.array([1 - px - py, px, py]), np.array([[-1.0, -1], [1, 0], [0, 1]])
                N.append(np.concatenate([L * (1 - z) / 2, L * (1 + z) / 2]))
                dN.append(np.concatenate([np.column_stack([dL * (1 - z) / 2, -L / 2]), np.column_stack([dL * (1 + z) / 2, L / 2])]))
                w.append(1 / 6)
    else:
        sx, sy = np.array([-1.0, 1, 1, -1]), np.array([-1.0, -1, 1, 1])
        r = math.sqrt(10)
        for z, wz in ((1 / 3 - r / 15, 1 / 6 + r / 48), (1 / 3 + r / 15, 1 / 6 - r / 48)):
            m = 1 - z
            for ex in (-s, s):
                for ey in (-s, s):
                    p, q = m + sx * ex * m, m + sy * ey * m
                    N.append(np.append(p * q / (4 * m), z))
                    d = np.column_stack([sx * q, sy * p, (sx * sy * ex * ey * m * m - m * m) / m]) / (4 * m)
                    dN.append(np.concatenate([d, [[0, 0, 1.0]]]))
                    w.append(wz)
    return np.array(N), np.array(dN), np.array(w)


class Exact:
    """The operators on one host mesh, element by element in torch's FP64, in the mesh's own numbering."""

    def __init__(self, m, f):
        t = lambda a: torch.as_tensor(np.ascontiguousarray(a), device=self.dev)  # noqa: E731
        self.dev = "cuda" if torch.cuda.is_available() else "cpu"
        coords, conn, types, boundary = m
        self.N, self.x, self.dt, self.D = len(coords), t(coords), f["dt"], f["D"]
        self.u, self.rho, self.mu, self.Y = t(f["u"]), t(f["rho"]), t(f["mu"]), t(f["Y"])
        types = np.full(len(conn), conn.shape[1]) if types is None else types
        self.parts = [(a, t(conn[types == a][:, :a].astype(np.int64))) for a in (4, 5, 6, 8) if (types == a).any()]
        self.free = torch.ones(self.N, dtype=torch.bool, device=self.dev)
        self.free[t(boundary.astype(np.int64))] = False

    def points(self, a, c):
        """Per Gauss point: N [a], grad N [e][a][3], dV [e]."""
        N, dN, w = reference(a)
        for g in range(len(w)):
            d = torch.as_tensor(dN[g], device=self.dev)
            J = torch.einsum("eai,aj->eij", self.x[c], d)
            yield torch.as_tensor(N[g], device=self.dev), torch.einsum("aj,eji->eai", d, torch.linalg.inv(J)), w[g] * torch.linalg.det(J)

    def chunks(self, most=200_000):
        for a, c in self.parts:
            for q in range(0, len(c), most):
                yield a, c[q:q + most]

    def pattern(self):
        """CSR of the node pairs that share an element, columns ascending."""
        if not hasattr(self, "keys"):
            self.keys = torch.unique(torch.cat([torch.unique((c[:, :, None] * self.N + c[:, None, :]).reshape(-1))
                                                for _, c in self.chunks(1_000_000)]))
            rows = torch.div(self.keys, self.N, rounding_mode="floor")
            self.rowptr = torch.cat([rows.new_zeros(1), torch.bincount(rows, minlength=self.N).cumsum(0)])
            self.rows, self.cols = rows, self.keys - rows * self.N
        return self.keys

    def assemble(self, matrix, vector, shape=(), comps=1):
        """values [nnz, *shape] and rhs [comps, N] from matrix(...) -> [e][a][b][*shape] and vector(...) -> [comps][e][a] a point."""
        V = None if matrix is None else torch.zeros((len(self.pattern()),) + shape, dtype=torch.float64, device=self.dev)
        B = torch.zeros((comps, self.N), dtype=torch.float64, device=self.dev)
        for a, c in self.chunks(100_000):
            A = b = 0
            for N, g, dV in self.points(a, c):
                if matrix is not None:
                    A = A + matrix(c, N, g, dV)
                b = b + vector(c, N, g, dV)
            if matrix is not None:
                at = torch.searchsorted(self.keys, (c[:, :, None] * self.N + c[:, None, :]).reshape(-1))
                V.index_add_(0, at, A.reshape((-1,) + shape))
            B.index_add_(1, c.reshape(-1), b.reshape(comps, -1))
        return V, B

    def transport(self, diffusivity, source):
        """M/dt + C + K and M source / dt; diffusivity(c, N) at the points."""
        def matrix(c, N, g, dV):
            r, adv = self.rho[c] @ N, (g * (self.u[:, c] @ N).T[:, None, :]).sum(2)
            s = (dV * r)[:, None] * (N / self.dt + adv)
            return N[:, None] * s[:, None, :] + (dV * diffusivity(c, N))[:, None, None] * (g @ g.transpose(1, 2).contiguous())

        def vector(c, N, g, dV):
            return (dV * (self.rho[c] @ N) / self.dt * (source[:, c] @ N))[:, :, None] * N
        return self.assemble(matrix, vector, comps=len(source))

    def momentum(self):
        return self.transport(lambda c, N: self.mu[c] @ N, self.u)

    def scalars(self):
        got = [self.transport(lambda c, N, k=k: float(self.D[k]) * (self.rho[c] @ N), self.Y[k:k + 1]) for k in range(len(self.D))]
        return torch.stack([v for v, _ in got]), torch.cat([b for _, b in got])

    def flux(self, c, N, g, dV):
        ru = ((self.rho[c] @ N) * (self.u[:, c] @ N)).T
        return (dV / self.dt)[None, :, None] * (g * ru[:, None, :]).sum(2)[None]

    def poisson(self, fixed=False):
        V, B = self.assemble(lambda c, N, g, dV: dV[:, None, None] * (g @ g.transpose(1, 2).contiguous()), self.flux)
        if fixed:
            V = V * ((self.free[self.rows] & self.free[self.cols]) | (self.rows == self.cols))
            B = B * self.free
        return V, B

    def block(self, form):
        def matrix(c, N, g, dV):
            r, uq = self.rho[c] @ N, (self.u[:, c] @ N).T
            s = (dV * r)[:, None] * (N / self.dt + (g * uq[:, None, :]).sum(2))
            wm = dV * (self.mu[c] @ N)
            S = N[:, None] * s[:, None, :] + wm[:, None, None] * (g @ g.transpose(1, 2).contiguous())
            if form & 2:
                div = (g * self.u[:, c].permute(1, 2, 0)).sum((1, 2))
                S = S + (dV * r * div)[:, None, None] * torch.outer(N, N)
            A = S[..., None, None] * torch.eye(3, dtype=torch.float64, device=self.dev)
            if form & 1:
                A = A + wm[:, None, None, None, None] * g[:, None, :, :, None] * g[:, :, None, None, :]
            return A

        def vector(c, N, g, dV):
            return (dV * (self.rho[c] @ N) / self.dt * (self.u[:, c] @ N))[:, :, None] * N
        return self.assemble(matrix, vector, (3, 3), 3)

    def residual(self, form):
        def vector(c, N, g, dV):
            uc = self.u[:, c]
            uq, du = uc @ N, torch.einsum("iea,eaj->ije", uc, g)
            adv = (uq[None] * du).sum(1)
            sym = du + (du.transpose(0, 1) if form & 1 else 0)
            if form & 2:
                adv = adv + (du[0, 0] + du[1, 1] + du[2, 2]) * uq
            wr, wm = dV * (self.rho[c] @ N), dV * (self.mu[c] @ N)
            r = -(wr * adv)[:, :, None] * N - torch.einsum("eaj,ije->iea", g, wm * sym)
            return torch.cat([r, (wr[:, None] * N)[None]])
        return self.assemble(None, vector, comps=4)[1]

    def multiply(self, V):
        A = torch.sparse_csr_tensor(self.rowptr, self.cols, V, (self.N, self.N))
        return lambda x: A @ x

    def solve(self, V, b, iterations=None):
        """Jacobi-CG from zero: that many iterations, or as far as FP64 goes."""
        A, d = self.multiply(V), V[self.rows == self.cols]
        x, r = torch.zeros_like(b), b.clone()
        z = r / d
        p, rz = z.clone(), torch.dot(r, z)
        for _ in range(iterations or 20 * int(round(self.N ** (1 / 3))) + 200):
            if iterations is None and float(r.norm()) <= 1e-14 * float(b.norm()):
                break
            q = A(p)
            alpha = rz / torch.dot(p, q)
            x += alpha * p
            r -= alpha * q
            z = r / d
            rz, old = torch.dot(r, z), rz
            p = z + (rz / old) * p
        return x

    def step(self, form):
        """One explicit step from u and p = 0."""
        V, _ = self.poisson(fixed=True)
        u0 = self.u
        for a, b in ((0.0, 1.0), (0.75, 0.25), (1 / 3, 2 / 3)):
            r = self.residual(form)
            self.u = torch.where(self.free, a * u0 + b * (self.u + self.dt * r[:3] / r[3]), u0)
        p = self.solve(V, self.assemble(None, self.flux)[1][0] * self.free)
        grad = self.assemble(None, lambda c, N, g, dV: (dV * torch.einsum("eaj,ea->je", g, p[c]))[:, :, None] * N, comps=3)[1]
        return torch.where(self.free, self.u - self.dt * grad / r[3], self.u), p


def exact(case, seed):
    kind = case["kind"]
    if kind == "serve":
        out = []
        for m, f in inputs(case, seed):
            e = Exact(m, f)
            V, b = e.poisson(fixed=True)
            out.append([e.solve(V, b[0]).cpu().numpy(), e.momentum()[1].cpu().numpy()])
        return out
    e = Exact(*inputs(case, seed))
    # the library numbers a shuffled mesh itself: only what comes back in the program's numbering can be told
    own = lambda v: None if case["shuffled"] else v  # noqa: E731
    if kind == "step":
        L, f = e.poisson(fixed=True)
        x = e.solve(L, f[0], case["iterations"] if case["rtol"] <= 0 else None)
        V, B = (None, None) if case["shuffled"] else e.momentum()
        return dict(V=own(V), B=own(B), L=own(L), f=own(f), x=x)
    if kind == "assemble":
        if case["shuffled"]:
            return None
        V, B = {"momentum": e.momentum, "scalar": e.scalars, "poisson": e.poisson}[case["operator"]]()
        return dict(V=V.reshape(-1, V.shape[-1]), B=B)
    if kind == "block":
        if case["shuffled"]:
            return None
        V, B = e.block(case["form"])
        return dict(V=V, B=B)
    if kind == "residual":
        return dict(r=e.residual(case["form"]))
    if kind == "fractional":
        u, p = e.step(case["form"])
        return dict(u=u, p=p)
    if kind == "solve":
        V, b = e.poisson(fixed=True)
        return dict(x=e.solve(V, b[0]))
    if case["shuffled"]:
        return None
    r = np.random.default_rng([seed, 1])
    A, x, w = (torch.as_tensor(r.standard_normal(k), device=e.dev) for k in (len(e.pattern()), e.N, e.N))
    y = e.multiply(A)(x)
    return dict(y=y, d=float(torch.dot(w, y)), z=w + 0.25 * y)
