"""The work that a user of the library has it do, as cases that can be timed and checked.

listed() names the fixed cases, draw() gives more of the same ranges, prepare() makes what a
program holds before the call, run() is one pass through the public entry points, work() what a
pass cannot do without, exact() what it should return, from plain torch in 64 bits.

Meshes are unit-cube (unit-square) lattices with 5 % jitter of the interior vertices, as in the
benchmark, or its lattice with quadratic geometry; coefficients are lognormal (sigma 1) per
quadrature point.  All vectors are standard normal.
"""
import math

import numpy as np
import torch

from paper_1911_09220_amd import pafem as P

# scalars of input and output per dof, stored values per quadrature point, space family
KINDS = {
    "mass": (P.MASS, 1, 1, 1, "h1"),
    "diffusion": (P.DIFFUSION, 1, 1, 6, "h1"),
    "diffusion_geom": (P.DIFFUSION_GEOM, 1, 1, 1, "h1"),
    "convection": (P.CONVECTION, 1, 1, 3, "h1"),
    "gradient": (P.GRADIENT, 1, 3, 9, "h1"),
    "divergence": (P.DIVERGENCE, 3, 1, 9, "h1"),
    "elasticity": (P.ELASTICITY, 3, 3, 11, "h1"),
    "maxwell": (P.HCURL_MAXWELL, 1, 1, 12, "nd"),
    "dg": (P.DG_CONVECTION, 1, 1, 3, "l2"),
}
UNCONSTRAINED = ("mass", "convection", "gradient", "divergence", "dg")  # the others eliminate the boundary
BETA = (1.0, 0.5, 0.25)  # transport velocity


def listed():
    return [
        # one operator action on the small Poisson mesh: a call's latency and launches
        {"name": "diffusion-p2-small", "path": "apply", "kind": "diffusion", "p": 2, "nx": 8, "ny": 8, "nz": 8},
        # the headline action, on a mesh well past every cache
        {"name": "diffusion-p3-large", "path": "apply", "kind": "diffusion", "p": 3, "nx": 52, "ny": 52, "nz": 52},
        # mass action (time stepping, projections) on a box with odd sides
        {"name": "mass-p4-ragged", "path": "apply", "kind": "mass", "p": 4, "nx": 23, "ny": 31, "nz": 37},
        # the vector-valued operator of solid mechanics, at the order it is mostly used at
        {"name": "elasticity-p2", "path": "apply", "kind": "elasticity", "p": 2, "nx": 40, "ny": 40, "nz": 40},
        # definite Maxwell on edge elements
        {"name": "maxwell-p3", "path": "apply", "kind": "maxwell", "p": 3, "nx": 32, "ny": 33, "nz": 31},
        # upwind transport on a discontinuous space: one stage of an explicit time step
        {"name": "dg-p4", "path": "apply", "kind": "dg", "p": 4, "nx": 40, "ny": 40, "nz": 40},
        # 16 right-hand sides on independent meshes of uneven size and order
        {"name": "batch-uneven", "path": "batch", "meshes": 8, "dofs_min": 10000, "dofs_max": 300000,
         "pmin": 2, "pmax": 6, "nrhs": 16, "mesh_seed": 4, "f32": False},
        # a whole small solve: latency of an iteration
        {"name": "pcg-p2-small", "path": "pcg", "p": 2, "n": 8, "rel_tol": 1e-10, "its": 72},
        # the paper's experiment: 2D Poisson, 1.3M dofs, 200 unpreconditioned CG iterations
        {"name": "cg200-2d-p4", "path": "cg2d", "p": 4, "n": 285, "its": 200},
        # FP32 operator inside FP64 refinement, on quadratic geometry
        {"name": "refine-p6-q2", "path": "ir", "p": 6, "n": 12, "rel_tol": 1e-10, "its": 1050},
        # multigrid in the order: flexible CG around V-cycles
        {"name": "multigrid-p3", "path": "pmg", "p": 3, "n": 28, "rel_tol": 1e-10, "its": 33},
        # a new coefficient on a kept space: quadrature data, diagonal and load vector
        {"name": "assemble-p3", "path": "assemble", "p": 3, "nx": 40, "ny": 40, "nz": 40},
    ]


def _box(rng, p, dofs, per_elem):
    """Sides of a box, odd ones among them, of about dofs dofs at per_elem of them an element."""
    e = max(8.0, dofs / per_elem)
    side = e ** (1.0 / 3.0)
    nx = max(2, round(side * rng.uniform(0.7, 1.4)))
    ny = max(2, round(side * rng.uniform(0.7, 1.4)))
    return {"nx": nx, "ny": ny, "nz": max(2, round(e / (nx * ny)))}


def draw(rng):
    def logu(a, b):
        return math.exp(rng.uniform(math.log(a), math.log(b)))

    path = rng.choice(["apply"] * 8 + ["batch", "pcg", "cg2d", "assemble"])
    if path == "apply":
        kind = rng.choice(["diffusion", "diffusion", "mass", "mass", "elasticity", "maxwell", "dg",
                           "convection", "gradient", "divergence", "diffusion_geom"])
        p = rng.randint(1, 8)
        top = min(2e6, 6e4 * p ** 3 / (3 if kind in ("elasticity", "maxwell", "gradient", "divergence") else 1))
        per = (p + 1) ** 3 if kind == "dg" else 3 * p ** 3 if kind == "maxwell" else p ** 3
        return {"path": path, "kind": kind, "p": p, **_box(rng, p, logu(4e3, top * per / p ** 3), per)}
    if path == "batch":
        return {"path": path, "meshes": rng.randint(2, 6), "dofs_min": 10000,
                "dofs_max": round(logu(3e4, 2e5)), "pmin": rng.randint(1, 4), "pmax": rng.randint(4, 6),
                "nrhs": rng.choice([2, 8, 16, 16]), "mesh_seed": rng.randint(0, 9999), "f32": rng.random() < 0.3}
    if path == "pcg":
        p = rng.randint(1, 5)
        n = max(2, round(logu(6, 24) / p))
        return {"path": path, "p": p, "n": n, "rel_tol": 1e-10, "its": 5 * p * n}
    if path == "cg2d":
        p = rng.randint(1, 8)
        return {"path": path, "p": p, "n": max(4, round(logu(60, 1000) / p)), "its": rng.choice([50, 100, 200])}
    p = rng.randint(1, 6)
    return {"path": path, "p": p, **_box(rng, p, logu(5e3, min(1e6, 6e4 * p ** 3)), p ** 3)}


# ---- meshes and inputs ----------------------------------------------------------------------

def _lattice(n, seed, jitter=0.05):
    """Vertices, lexicographic elements: of the box n = (nx, ny[, nz]) as in the unit cube."""
    dim, h = len(n), 1.0 / max(n)
    axes = [np.arange(k + 1) / k for k in n]
    verts = np.stack([g.ravel() for g in np.meshgrid(*axes[::-1], indexing="ij")[::-1]], axis=1)
    rng = np.random.default_rng(seed)
    disp = rng.uniform(-jitter * h / math.sqrt(dim), jitter * h / math.sqrt(dim), size=verts.shape)
    inner = np.all((verts > 0.0) & (verts < 1.0), axis=1)
    verts[inner] += disp[inner]
    low = _low_vertices(n)
    st = np.cumprod([1] + [k + 1 for k in n[:-1]])
    order = [0, 1, 3, 2] if dim == 2 else [0, 1, 3, 2, 4, 5, 7, 6]  # corner bits of each slot
    conn = np.stack([low + sum(((c >> a) & 1) * st[a] for a in range(dim)) for c in order], axis=1)
    return verts, conn


def _low_vertices(n):
    """First vertex of every element, elements x fastest."""
    st = np.cumprod([1] + [k + 1 for k in n[:-1]])
    idx = np.meshgrid(*[np.arange(k) for k in n][::-1], indexing="ij")[::-1]
    return sum(i.ravel() * s for i, s in zip(idx, st))


def _warped(n, amp=0.05):
    """Quadratic-geometry lattice: 27 nodes an element, x + amp sin sin sin (1, 1, 1)."""
    def warp(x):
        return x + amp * np.prod(np.sin(2.0 * np.pi * x), axis=-1, keepdims=True)

    verts, conn = _lattice((n, n, n), 0, 0.0)
    t = np.array([0.0, 0.5, 1.0]) / n
    off = np.stack([g.ravel() for g in np.meshgrid(t, t, t, indexing="ij")[::-1]], axis=1)
    nodes = warp(verts[conn[:, 0]][:, None, :] + off[None])
    return warp(verts), conn, nodes


def _normal(seed, k, shape, device):
    g = torch.Generator(device=device)
    g.manual_seed(int(seed) * 64 + k)
    return torch.randn(shape, dtype=torch.float64, device=device, generator=g)


def _device():
    return "cuda" if torch.cuda.is_available() else "cpu"


def _sides(case):
    return (case["nx"], case["ny"], case["nz"])


def _coeff(kind, seed, ne, q3, device):
    """Coefficient of an operator kind per element (lexicographic) and point."""
    if kind == "dg":
        return torch.tensor(BETA, dtype=torch.float64, device=device)
    if kind == "convection":
        return torch.tensor(BETA, dtype=torch.float64, device=device).expand(ne, q3, 3).contiguous()
    if kind in ("elasticity", "maxwell"):
        return _normal(seed, 1, (ne, q3, 2), device).exp_()
    return _normal(seed, 1, (ne, q3), device).exp_()


def _batch_sizes(case):
    rng = np.random.default_rng(case["mesh_seed"])
    out = []
    for _ in range(case["meshes"]):
        dofs = math.exp(rng.uniform(math.log(case["dofs_min"]), math.log(case["dofs_max"])))
        p = int(rng.integers(case["pmin"], case["pmax"] + 1))
        out.append((p, max(1, round((dofs ** (1.0 / 3.0) - 1.0) / p))))
    return out


def prepare(case, seed):
    dev, path = "cuda", case["path"]
    if path in ("apply", "assemble"):
        verts, conn = _lattice(_sides(case), seed)
        kind = case.get("kind", "diffusion")
        code, nin, nout, _, family = KINDS[kind]
        S = P.Space(P.Mesh(verts, conn), case["p"], family=family)
        q3 = (case["p"] + 2) ** 3
        coeff = _coeff(kind, seed, S.nelem, q3, dev)
        if path == "assemble":
            return {"path": path, "space": S, "coeff": coeff, "f": _normal(seed, 2, (S.nelem * q3,), dev)}
        A = P.Operator(S, code, S.qdata(code, coeff=coeff), constrained=kind not in UNCONSTRAINED)
        return {"path": path, "op": A, "x": _normal(seed, 0, (nin * S.ndofs,), dev),
                "y": torch.empty(nout * S.ndofs, dtype=torch.float64, device=dev)}
    if path == "batch":
        ops, xs, ys = [], [], []
        for k, (p, n) in enumerate(_batch_sizes(case)):
            verts, conn = _lattice((n, n, n), seed + k)
            S = P.Space(P.Mesh(verts, conn), p)
            qd = S.qdata(P.DIFFUSION, coeff=_coeff("diffusion", seed + 1000 * k, S.nelem, (p + 2) ** 3, dev))
            if case["f32"]:
                qd = P.lowered_qdata(qd, P.F32)
            ops.append(P.Operator(S, P.DIFFUSION, qd, qdata_dtype=P.F32 if case["f32"] else P.F64))
            x = _normal(seed + 1000 * k, 0, (S.ndofs, case["nrhs"]), dev)
            xs.append(x.float() if case["f32"] else x)
            ys.append(torch.empty_like(xs[-1]))
        B = P.Batch(ops, nrhs=case["nrhs"])
        B.autotune(xs, ys, reps=3)
        return {"path": path, "batch": B, "xs": xs, "ys": ys}
    if path == "cg2d":
        verts, conn = _lattice((case["n"], case["n"]), seed)
        S = P.Space(P.Mesh(verts, quads=conn), case["p"])
        A = P.Operator(S, P.DIFFUSION, S.qdata(P.DIFFUSION))
        return {"path": path, "op": A, "b": S.linear_form(P.SOURCE_SINE), "its": case["its"]}
    n, p = case["n"], case["p"]
    if path == "ir":
        verts, conn, nodes = _warped(n)
        S = P.Space(P.Mesh(verts, conn, 2, nodes), p)
    else:
        verts, conn = _lattice((n, n, n), seed)
        S = P.Space(P.Mesh(verts, conn), p)
    coeff = _coeff("diffusion", seed, S.nelem, (p + 2) ** 3, dev)
    qd = S.qdata(P.DIFFUSION, coeff=coeff)
    A = P.Operator(S, P.DIFFUSION, qd)
    diag, b = A.diagonal(), S.linear_form(P.SOURCE_SINE)
    state = {"path": path, "op": A, "diag": diag, "b": b, "rel_tol": case["rel_tol"]}
    if path == "ir":
        state["lo"] = P.Operator(S, P.DIFFUSION, P.lowered_qdata(qd, P.F32), qdata_dtype=P.F32)
    if path == "pmg":
        Sc = P.Space(S.mesh, 1)
        Ac = P.Operator(Sc, P.DIFFUSION, Sc.qdata(P.DIFFUSION, coeff=S.coeff_mean(coeff.reshape(-1), q1d_out=3)))
        ops, diags = [A, Ac], [diag, Ac.diagonal()]
        lmax = [o.lambda_max(d, _normal(seed, 3 + k, (o.space.ndofs,), dev), 20)
                for k, (o, d) in enumerate(zip(ops, diags))]
        state["pmg"] = P.PMG(ops, diags, lmax, degree=2, coarse_iters=10)
    return state


def run(state):
    path = state["path"]
    if path == "apply":
        return state["op"].apply(state["x"], state["y"])
    if path == "batch":
        return state["batch"].apply(state["xs"], state["ys"])
    if path == "assemble":
        S = state["space"]
        A = P.Operator(S, P.DIFFUSION, S.qdata(P.DIFFUSION, coeff=state["coeff"]))
        return {"diagonal": A.diagonal(), "load": S.linear_form(P.SOURCE_ARRAY, f_qp=state["f"])}
    if path == "cg2d":
        return state["op"].pcg(state["b"], rel_tol=0.0, max_iter=state["its"], precond=P.PRECOND_NONE,
                               check_every=state["its"], history=False)[0]
    if path == "pcg":
        return state["op"].pcg(state["b"], diag=state["diag"], rel_tol=state["rel_tol"])[0]
    if path == "ir":
        return state["op"].ir_solve(state["lo"], state["b"], diag=state["diag"], rel_tol=state["rel_tol"])[0]
    return state["pmg"].fcg(state["b"], rel_tol=state["rel_tol"])[0]


# ---- what a pass cannot do without ------------------------------------------------------------

def _ndofs(n, p, family="h1"):
    if family == "l2":
        return math.prod(n) * (p + 1) ** len(n)
    if family == "nd":
        return sum(math.prod(n[b] * p + (b != a) for b in range(3)) for a in range(3))
    return math.prod(k * p + 1 for k in n)


def _action(n, p, kind, nrhs=1, size=8):
    """Bytes and flops of one action: vectors, stored values and the element-to-dof map once."""
    _, nin, nout, nc, family = KINDS[kind]
    dim = len(n)
    nc = 3 if dim == 2 else nc
    ne, D, Q = math.prod(n), p + 1, p + 2
    dofs = _ndofs(n, p, family)
    per = D ** dim if family != "nd" else 3 * p * D * D
    nbytes = size * ((nin + nout) * nrhs * dofs + nc * ne * Q ** dim)
    nbytes += 0 if family == "l2" else 4 * ne * per
    lines = 2 * D ** 3 * Q + 3 * D * D * Q * Q + 3 * D * Q ** 3 if dim == 3 else 2 * D * D * Q + 2 * D * Q * Q
    both = {"mass": 2 * (D ** 3 * Q + D * D * Q * Q + D * Q ** 3), "maxwell": 3 * 2 * lines, "elasticity": 3 * 2 * lines,
            "gradient": 2 * lines, "divergence": 2 * lines}.get(kind, 2 * lines)
    return {"bytes": float(nbytes), "flops": float(nrhs * ne * (2 * both + 2 * nc * Q ** dim))}


def work(case):
    path, p = case["path"], case["p"] if "p" in case else 0
    if path == "apply":
        return _action(_sides(case), p, case["kind"])
    if path == "batch":
        parts = [_action((n, n, n), pp, "diffusion", case["nrhs"], 4 if case["f32"] else 8)
                 for pp, n in _batch_sizes(case)]
        return {k: sum(w[k] for w in parts) for k in ("bytes", "flops")}
    if path == "assemble":
        n = _sides(case)
        ne, q3 = math.prod(n), (p + 2) ** 3
        one = _action(n, p, "diffusion")
        return {"bytes": 8.0 * (2 * ne * q3 + 2 * 6 * ne * q3 + 2 * _ndofs(n, p)) + 4.0 * ne * (p + 1) ** 3,
                "flops": 2.0 * one["flops"]}
    n = (case["n"],) * (2 if path == "cg2d" else 3)
    one = _action(n, p, "diffusion", size=4 if path == "ir" else 8)
    # an iteration: one action, and x, r, d read and written, the diagonal read
    vec = 8.0 * _ndofs(n, p) * (6 + (path != "cg2d"))
    applies = case["its"] * (5 if path == "pmg" else 1)
    return {"bytes": applies * one["bytes"] + case["its"] * vec, "flops": applies * one["flops"]}


# ---- the same from plain torch in 64 bits -------------------------------------------------------

def _rule(q):
    x, w = np.polynomial.legendre.leggauss(q)
    return 0.5 * (x + 1.0), 0.5 * w


def _lobatto(n):
    inner = np.polynomial.legendre.Legendre.basis(n - 1).deriv().roots() if n > 2 else np.empty(0)
    return 0.5 * (np.concatenate([[-1.0], np.sort(inner.real), [1.0]]) + 1.0)


def _basis(nodes, pts):
    """Lagrange values and derivatives [points, nodes]."""
    n = len(nodes)
    val, der = np.ones((len(pts), n)), np.zeros((len(pts), n))
    for j in range(n):
        for m in range(n):
            if m != j:
                val[:, j] *= (pts - nodes[m]) / (nodes[j] - nodes[m])
                rest = np.ones(len(pts))
                for k in range(n):
                    if k not in (j, m):
                        rest *= (pts - nodes[k]) / (nodes[j] - nodes[k])
                der[:, j] += rest / (nodes[j] - nodes[m])
    return val, der


def _first_seen(codes):
    """Numbers 0.. of the distinct codes in the order of their first appearance."""
    _, first, inv = np.unique(codes.ravel(), return_index=True, return_inverse=True)
    rank = np.empty(len(first), dtype=np.int64)
    rank[np.argsort(first)] = np.arange(len(first))
    return rank[inv].reshape(codes.shape), len(first)


def _entities(n):
    """Edge numbers by (axis, low corner bits) and face numbers by (axis, side), per element."""
    st = np.cumprod([1] + [k + 1 for k in n[:-1]])
    dim, nv, low = len(n), math.prod(k + 1 for k in n), _low_vertices(n)
    slots = [(a, c) for a in range(dim) for c in range(1 << dim) if not (c >> a) & 1]
    codes = [a * nv + low + sum(((c >> b) & 1) * st[b] for b in range(dim)) for a, c in slots]
    eid, n_edges = _first_seen(np.stack(codes, axis=1))
    edges = {s: eid[:, k] for k, s in enumerate(slots)}
    if dim == 2:
        return edges, n_edges, {}, 0
    codes = [a * nv + low + s * st[a] for a in range(3) for s in (0, 1)]
    fid, n_faces = _first_seen(np.stack(codes, axis=1))
    return edges, n_edges, {(k // 2, k % 2): fid[:, k] for k in range(6)}, n_faces


def _h1_map(n, p):
    """Element-to-dof map [E, i3, i2, i1] (2D: [E, i2, i1]), numbered vertices, edges, faces, interiors."""
    dim, ne, m = len(n), math.prod(n), p - 1
    st = np.cumprod([1] + [k + 1 for k in n[:-1]])
    low = _low_vertices(n)
    edges, n_edges, faces, n_faces = _entities(n)
    ebase = math.prod(k + 1 for k in n)
    fbase = ebase + n_edges * m
    ibase = fbase + n_faces * m * m
    g = np.empty((ne,) + (p + 1,) * dim, dtype=np.int64)
    for idx in np.ndindex(*(p + 1,) * dim):
        i = idx[::-1]
        inner = [a for a in range(dim) if 0 < i[a] < p]
        bits = sum((i[a] == p) << a for a in range(dim))
        if not inner:
            d = low + sum(((bits >> a) & 1) * st[a] for a in range(dim))
        elif len(inner) == 1:
            d = ebase + edges[(inner[0], bits)] * m + i[inner[0]] - 1
        elif len(inner) == 2 and dim == 3:
            (a,) = [a for a in range(3) if a not in inner]
            d = fbase + faces[(a, int(i[a] == p))] * m * m + (i[inner[0]] - 1) + m * (i[inner[1]] - 1)
        else:
            d = ibase + np.arange(ne) * m ** dim + sum((i[a] - 1) * m ** a for a in range(dim))
        g[(slice(None),) + idx] = d
    return g


def _boundary(n, g):
    """Marks the dofs of map g on the boundary (axes of g after the first: last axis is x)."""
    dim = len(n)
    ends = np.zeros(int(g.max()) + 1, dtype=bool)
    pos = np.unravel_index(np.arange(math.prod(n)), n[::-1])[::-1]
    for a in range(dim):
        for side, at in ((0, 0), (-1, n[a] - 1)):
            ends[np.take(g[pos[a] == at], side, axis=dim - a)] = True
    return ends


def _nd_maps(n, p):
    """The three components' maps [E, i2, i1, i0] of the edge-element space (open index along a)."""
    ne, m = math.prod(n), p - 1
    edges, n_edges, faces, n_faces = _entities(n)
    fbase = n_edges * p
    ibase = fbase + n_faces * 2 * p * m
    out = []
    for a in range(3):
        size = [p if b == a else p + 1 for b in range(3)]
        g = np.empty((ne, size[2], size[1], size[0]), dtype=np.int64)
        for idx in np.ndindex(*size[::-1]):
            i = idx[::-1]
            ends = [b for b in range(3) if b != a and i[b] in (0, p)]
            if len(ends) == 2:
                d = edges[(a, sum((i[b] == p) << b for b in ends))] * p + i[a]
            elif len(ends) == 1:
                u, v = [b for b in range(3) if b != ends[0]]
                loc = (i[v] - 1) * p + i[u] if a == u else p * m + i[v] * m + i[u] - 1
                d = fbase + faces[(ends[0], int(i[ends[0]] == p))] * 2 * p * m + loc
            else:
                j = [i[b] - (b != a) for b in range(3)]
                w = [p if b == a else m for b in range(3)]
                d = ibase + np.arange(ne) * 3 * p * m * m + a * p * m * m + j[0] + w[0] * (j[1] + w[1] * j[2])
            g[(slice(None),) + idx] = d
        out.append(g)
    return out


def _along(T, u, axis):
    return torch.movedim(torch.movedim(u, axis, -1) @ T.T, -1, axis)


def _tensor(mats, u):
    """mats[0] along the last axis (x), mats[1] along the one before, ..."""
    for a, T in enumerate(mats):
        u = _along(T, u, u.dim() - 1 - a)
    return u


class _Problem:
    """Action of one operator kind on one mesh, element by element in torch."""

    def __init__(self, n, p, kind, coeff, verts=None, conn=None, nodes=None):
        self.n, self.p, self.kind, self.dim = n, p, kind, len(n)
        dev = self.dev = coeff.device if coeff is not None else torch.device(_device())
        Q, dim, ne = p + 2, len(n), math.prod(n)
        x, w = _rule(Q)
        t = lambda v: torch.as_tensor(v, device=dev)  # noqa: E731
        B, G = _basis(_lobatto(p + 1), x)
        self.B, self.G, self.Bo = t(B), t(G), None
        family = KINDS[kind][4]
        lex = [0, 1, 3, 2] if dim == 2 else [0, 1, 3, 2, 4, 5, 7, 6]
        if nodes is None:
            gn, X = np.array([0.0, 1.0]), t(verts)[t(conn[:, lex])].reshape((ne,) + (2,) * dim + (dim,))
        else:
            gn, X = np.array([0.0, 0.5, 1.0]), t(nodes).reshape(ne, 3, 3, 3, 3)
        gB, gG = (t(v) for v in _basis(gn, x))
        self.gn, self.X, self.x1, self.w1 = gn, X, x, t(w)
        cols = []
        for b in range(dim):
            mats = [gG if a == b else gB for a in range(dim)]
            cols.append(torch.stack([_tensor(mats, X[..., c]) for c in range(dim)], dim=-1))
        J = torch.stack(cols, dim=-1)  # [E, q.., a, b] = dx_a / dxi_b
        W = t(w)
        for _ in range(dim - 1):
            W = W[..., None] * t(w)
        self.det = torch.linalg.det(J)
        self.J, self.Ji, self.W = J, torch.linalg.inv(J), W
        shape = (ne,) + (Q,) * dim
        self.c = None if coeff is None else coeff if kind == "dg" else coeff.reshape(shape + tuple(coeff.shape[2:]))
        if family == "h1":
            g = _h1_map(n, p)
            self.maps, self.ndofs = [t(g)], int(g.max()) + 1
            self.ess = t(_boundary(n, g))
        elif family == "nd":
            gs = _nd_maps(n, p)
            self.ndofs = max(int(g.max()) for g in gs) + 1
            self.Bo = t(_basis(_rule(p)[0], x)[0])
            ess = np.zeros(self.ndofs, dtype=bool)
            pos = np.unravel_index(np.arange(ne), n[::-1])[::-1]
            for a, g in enumerate(gs):
                for b in range(3):
                    for side, at in ((0, 0), (-1, n[b] - 1)):
                        if b != a:
                            ess[np.take(g[pos[b] == at], side, axis=3 - b)] = True
            self.maps, self.ess = [t(g) for g in gs], t(ess)
        else:
            self.ndofs = ne * (p + 1) ** 3
            self.maps, self.ess = [torch.arange(self.ndofs, device=dev).reshape(ne, p + 1, p + 1, p + 1)], None
        self.constrained = kind not in UNCONSTRAINED

    def grad(self, u):
        """Reference gradient at the points, [E, q.., b]."""
        return torch.stack([_tensor([self.G if a == b else self.B for a in range(self.dim)], u)
                            for b in range(self.dim)], dim=-1)

    def grad_t(self, v):
        return sum(_tensor([(self.G if a == b else self.B).T for a in range(self.dim)], v[..., b])
                   for b in range(self.dim))

    def val(self, u):
        return _tensor([self.B] * self.dim, u)

    def val_t(self, v):
        return _tensor([self.B.T] * self.dim, v)

    def add(self, ye, k=0):
        y = torch.zeros(self.ndofs, dtype=torch.float64, device=self.dev)
        return y.index_add_(0, self.maps[k].reshape(-1), ye.reshape(-1))

    def apply(self, x):
        N, kind = self.ndofs, self.kind
        xs = x.reshape(-1, N)
        if self.constrained:
            xs = torch.where(self.ess, torch.zeros_like(xs), xs)
        g, Ji, wd = self.maps[0], self.Ji, self.W * self.det
        mv = lambda M, v: (M @ v[..., None])[..., 0]  # noqa: E731
        tr = lambda M: M.transpose(-1, -2)  # noqa: E731
        if kind == "mass":
            y = [self.add(self.val_t(self.c * wd * self.val(xs[0][g])))]
        elif kind in ("diffusion", "diffusion_geom"):
            k = wd if self.c is None else self.c * wd
            y = [self.add(self.grad_t(k[..., None] * mv(Ji, mv(tr(Ji), self.grad(xs[0][g])))))]
        elif kind == "convection":
            y = [self.add(self.val_t(wd * (mv(Ji, self.c) * self.grad(xs[0][g])).sum(-1)))]
        elif kind == "gradient":
            v = (self.c * wd)[..., None] * mv(tr(Ji), self.grad(xs[0][g]))
            y = [self.add(self.val_t(v[..., c])) for c in range(3)]
        elif kind == "divergence":
            d = sum(mv(tr(Ji), self.grad(xs[c][g]))[..., c] for c in range(3))
            y = [self.add(self.val_t(self.c * wd * d))]
        elif kind == "elasticity":
            F = torch.stack([mv(tr(Ji), self.grad(xs[c][g])) for c in range(3)], dim=-2)
            lam, mu = self.c[..., 0] * wd, self.c[..., 1] * wd
            sig = mu[..., None, None] * (F + tr(F))
            div = lam * torch.diagonal(F, dim1=-2, dim2=-1).sum(-1)
            for c in range(3):
                sig[..., c, c] += div
            y = [self.add(self.grad_t(mv(Ji, sig[..., c, :]))) for c in range(3)]
        elif kind == "maxwell":
            y = [self._maxwell(xs[0])]
        else:
            y = [self._dg(xs[0])]
        y = torch.cat(y)
        if self.constrained:
            y = torch.where(self.ess.repeat(len(y) // N), x, y)
        return y

    def _nd_tab(self, a, d=None):
        return [self.Bo if b == a else self.G if b == d else self.B for b in range(3)]

    def _maxwell(self, x):
        u, curl = [None] * 3, [0.0] * 3
        for a in range(3):
            xe = x[self.maps[a]]
            u[a] = _tensor(self._nd_tab(a), xe)
            b, c = (a + 1) % 3, (a + 2) % 3  # curl of f e_a: df/dx_c along b, -df/dx_b along c
            curl[b] = curl[b] + _tensor(self._nd_tab(a, c), xe)
            curl[c] = curl[c] - _tensor(self._nd_tab(a, b), xe)
        mv = lambda M, v: (M @ v[..., None])[..., 0]  # noqa: E731
        u, curl = torch.stack(u, dim=-1), torch.stack(curl, dim=-1)
        alpha, beta = self.c[..., 0], self.c[..., 1]
        m = (self.W * self.det * beta)[..., None] * mv(self.Ji, mv(self.Ji.transpose(-1, -2), u))
        k = (self.W * alpha / self.det)[..., None] * mv(self.J.transpose(-1, -2), mv(self.J, curl))
        y = 0.0
        tt = lambda tab: [T.T for T in tab]  # noqa: E731
        for a in range(3):
            b, c = (a + 1) % 3, (a + 2) % 3
            ye = _tensor(tt(self._nd_tab(a)), m[..., a])
            ye = ye + _tensor(tt(self._nd_tab(a, c)), k[..., b]) - _tensor(tt(self._nd_tab(a, b)), k[..., c])
            y = y + self.add(ye, a)
        return y

    def _dg(self, x):
        n, D, Q = self.n, self.p + 1, self.p + 2
        beta = self.c
        u = x[self.maps[0]]
        vel = (self.W * self.det)[..., None] * (self.Ji @ beta)
        y = self.grad_t(-self.val(u)[..., None] * vel).reshape(n[::-1] + (D,) * 3)
        u = u.reshape(n[::-1] + (D,) * 3)
        X = self.X.reshape(n[::-1] + tuple(self.X.shape[1:]))
        gB, gG = (torch.as_tensor(v, device=self.dev) for v in _basis(self.gn, self.x1))
        ww = self.w1[:, None] * self.w1
        for a in range(3):
            b, c = [d for d in range(3) if d != a]
            el, nd = 2 - a, 5 - a  # axes of the elements and of the nodes along a

            def flow(Xs, end):
                """w beta . N of the faces at the end of axis a, N along +a."""
                Xf = torch.select(Xs, nd, end)
                Tb = torch.stack([_tensor([gG, gB], Xf[..., k]) for k in range(3)], dim=-1)
                Tc = torch.stack([_tensor([gB, gG], Xf[..., k]) for k in range(3)], dim=-1)
                N = torch.cross(Tb, Tc, dim=-1) * (-1.0 if a == 1 else 1.0)
                return ww * (N @ beta)

            trace = lambda v, end: _tensor([self.B, self.B], torch.select(v, nd, end))  # noqa: E731
            back = lambda f: _tensor([self.B.T, self.B.T], f)  # noqa: E731
            k = n[a]
            lo, hi = u.narrow(el, 0, k - 1), u.narrow(el, 1, k - 1)
            w = flow(X.narrow(el, 0, k - 1), -1)
            f = back(torch.where(w > 0, w * trace(lo, -1), w * trace(hi, 0)))
            torch.select(y.narrow(el, 0, k - 1), nd, -1).add_(f)
            torch.select(y.narrow(el, 1, k - 1), nd, 0).sub_(f)
            for at, end, sign in ((0, 0, -1.0), (k - 1, -1, 1.0)):
                w = sign * flow(X.narrow(el, at, 1), end)
                f = back(torch.clamp(w, min=0.0) * trace(u.narrow(el, at, 1), end))
                torch.select(y.narrow(el, at, 1), nd, end).add_(f)
        return y.reshape(-1)

    def diagonal(self):
        """Diagonal of the constrained diffusion operator."""
        D = (self.c * self.W * self.det)[..., None, None] * (self.Ji @ self.Ji.transpose(-1, -2))
        ye = 0.0
        for a in range(3):
            for b in range(3):
                mats = [((self.G if d == a else self.B) * (self.G if d == b else self.B)).T for d in range(3)]
                ye = ye + _tensor(mats, D[..., a, b])
        return torch.where(self.ess, 1.0, self.add(ye))

    def load(self, f):
        """(f, v), 0 on the boundary, f [E, points]."""
        b = self.add(self.val_t(self.W * self.det * f.reshape(self.det.shape)))
        return torch.where(self.ess, 0.0, b)

    def sine(self):
        B = torch.as_tensor(_basis(self.gn, self.x1)[0], device=self.dev)
        x = torch.stack([_tensor([B] * self.dim, self.X[..., a]) for a in range(self.dim)], dim=-1)
        return self.dim * math.pi ** 2 * torch.sin(math.pi * x).prod(-1)

    def solve(self, b, its=None):
        """Jacobi-preconditioned CG to 1e-13, or its iterations without a preconditioner."""
        d = self.diagonal() if its is None else 1.0
        x = torch.zeros_like(b)
        r = b.clone()
        z = r / d
        s, rz, stop = z.clone(), float(r @ z), 1e-26 * float(b @ b)
        for k in range(6000 if its is None else its):
            q = self.apply(s)
            alpha = rz / float(s @ q)
            x += alpha * s
            r -= alpha * q
            if its is None and k % 10 == 0 and float(r @ r) <= stop:
                break
            z = r / d
            rz, old = float(r @ z), rz
            s = z + (rz / old) * s
        return x


def exact(case, seed):
    path, dev = case["path"], _device()
    p = case.get("p", 0)
    if path in ("apply", "assemble"):
        n, kind = _sides(case), case.get("kind", "diffusion")
        verts, conn = _lattice(n, seed)
        A = _Problem(n, p, kind, _coeff(kind, seed, math.prod(n), (p + 2) ** 3, dev), verts, conn)
        if path == "assemble":
            f = _normal(seed, 2, (math.prod(n) * (p + 2) ** 3,), dev)
            return {"diagonal": A.diagonal(), "load": A.load(f)}
        return A.apply(_normal(seed, 0, (KINDS[kind][1] * A.ndofs,), dev))
    if path == "batch":
        out = []
        for k, (pp, m) in enumerate(_batch_sizes(case)):
            verts, conn = _lattice((m, m, m), seed + k)
            c = _coeff("diffusion", seed + 1000 * k, m ** 3, (pp + 2) ** 3, dev)
            A = _Problem((m, m, m), pp, "diffusion", c, verts, conn)
            x = _normal(seed + 1000 * k, 0, (A.ndofs, case["nrhs"]), dev)
            x = x.float().double() if case["f32"] else x
            out.append(torch.stack([A.apply(v.contiguous()) for v in x.T], dim=1))
        return out
    n = case["n"]
    if path == "cg2d":
        verts, conn = _lattice((n, n), seed)
        A = _Problem((n, n), p, "diffusion", None, verts, conn)
        return A.solve(A.load(A.sine()), case["its"])
    c = _coeff("diffusion", seed, n ** 3, (p + 2) ** 3, dev)
    if path == "ir":
        verts, conn, nodes = _warped(n)
        A = _Problem((n, n, n), p, "diffusion", c, verts, conn, nodes)
    else:
        verts, conn = _lattice((n, n, n), seed)
        A = _Problem((n, n, n), p, "diffusion", c, verts, conn)
    return A.solve(A.load(A.sine()))
