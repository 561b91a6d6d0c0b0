"""Measured workloads of the library: what a program that uses it runs.

A case is a dict of plain values.  Kinds:

* ``solve``: one right-hand side against a kept hierarchy, ``Solver.solve`` to
  a relative residual of 1e-10 from a zero guess (FP64 PCG, or the FP32 V-cycle
  inside FP64 flexible CG);
* ``batch``: k right-hand sides against a kept hierarchy, ``Solver.solve_batch``;
* ``setup``: a mesh seen for the first time: ``Solver(...)``, one solve, close;
* ``serve``: requests for several resident hierarchies submitted to a
  ``Server`` together, then waited for.

The problem is always -lap u + lambda u = f on n^3 hexahedra of order p in the
unit cube, interior vertices moved by up to a tenth of the spacing, i.i.d.
N(0, 1) right-hand sides, and the output is the solution.
"""
import math

import numpy as np
import torch

import synth
from paper_2512_15121_amd import Options, Server, Solver

DEV = "cuda:0"
TOL = 1e-10


def _solve(name, n, p, lam, **kw):
    return {"name": name, "kind": "solve", "n": n, "p": p, "lam": lam, **kw}


def listed():
    return [
        # the smallest call: 729 dofs, weighted-Jacobi smoothing; launches and
        # synchronisations only
        _solve("solve_4_p2_jacobi", 4, 2, 1.0, smoother="jacobi"),
        # an ordinary small problem, as in the small serving trace
        _solve("solve_8_p4", 8, 4, 10.0),
        # an odd size of higher order (6 -> 3 -> 1), FP32 V-cycle, three smoothing steps
        _solve("solve_9_p6_mixed_deg3", 9, 6, 0.5, precision="mixed", degree=3),
        # the benchmark's 16^3 workload, FP64
        _solve("solve_16_p4", 16, 4, 10.0),
        # the headline workload (2.1 M dofs, 424 M nonzeros), both precisions
        _solve("solve_32_p4", 32, 4, 39.3),
        _solve("solve_32_p4_mixed", 32, 4, 39.3, precision="mixed"),
        # the parameter study's fastest setting at p = 5: explicit schedule 5 -> 3 -> 1
        _solve("solve_13_p5_s31", 13, 5, 10.0, schedule="3,1"),
        # the paper's hierarchical modal basis: injection transfers, many iterations
        _solve("solve_9_p4_modal", 9, 4, 10.0, basis="modal"),
        # the pressure-Poisson batch: pure Neumann, one pinned node, 64 right-hand sides
        {"name": "batch_20_p3_k64_mixed", "kind": "batch", "n": 20, "p": 3, "lam": 0.0, "k": 64,
         "bc": "pin", "precision": "mixed"},
        # a batch as wide as the server's slots, odd mesh, FP64
        {"name": "batch_11_p4_k8", "kind": "batch", "n": 11, "p": 4, "lam": 10.0, "k": 8},
        # a mesh seen for the first time (a cache miss of the server, a new lambda)
        {"name": "setup_12_p4", "kind": "setup", "n": 12, "p": 4, "lam": 10.0},
        # three resident hierarchies, eight requests each, arriving together
        {"name": "serve_4_6_8_mixed", "kind": "serve", "n": 4, "p": 4, "lam": 3.0, "requests": 8,
         "precision": "mixed"},
    ]


def draw(rng):
    """One more case: any kind, order 2 to 6, sizes spread over the logarithm
    of the node count between 729 and the headline's 2.1 M (fewer where the
    call holds several columns or builds the hierarchy)."""
    kind = rng.choices(["solve", "batch", "setup", "serve"], [8, 3, 1, 1])[0]
    p = rng.randint(2, 6)
    lam = round(math.exp(rng.uniform(math.log(0.1), math.log(100.0))), 3)
    most = {"solve": 2.1e6, "batch": 2.2e5, "setup": 1.2e5, "serve": 2e4}[kind]
    nodes = math.exp(rng.uniform(math.log(729.0), math.log(most)))
    # no more nonzeros than the headline's: (p + 2)^3 per row
    n = max(2, min(int(round((nodes ** (1 / 3) - 1) / p)), int((4.2e8 / (p * (p + 2)) ** 3) ** (1 / 3))))
    case = {"kind": kind, "n": n, "p": p, "lam": lam,
            "precision": rng.choice(["fp64", "mixed"])}
    if kind == "serve":
        case["n"] = min(n, 8)
        case["p"] = min(p, 4)
        case["requests"] = rng.randint(2, 9)
        return case
    if kind == "batch":
        case["k"] = rng.choice([2, 3, 5, 8, 16, 27, 48, 64])
    if rng.random() < 0.2:
        case["bc"], case["lam"] = "pin", 0.0
    if kind != "setup" and rng.random() < 0.3:
        case["degree"] = rng.randint(1, 4)
    if rng.random() < 0.15:
        case["smoother"] = "jacobi"
    elif p == 5 and rng.random() < 0.5:
        case["schedule"] = rng.choice(["3,1", "4,3,2,1"])
    return case


def _options(case):
    sched = tuple(int(q) for q in case["schedule"].split(",")) if case.get("schedule") else ()
    return Options(smoother=case.get("smoother", "chebyshev"), degree=case.get("degree", 2),
                   precision=case.get("precision", "fp64"), bc=case.get("bc", "dirichlet"),
                   basis=case.get("basis", "nodal"), schedule=sched, maxit=2000)


def _mesh(case, seed, n=None):
    return synth.hex_mesh(n or case["n"], case["p"], perturb=0.1, seed=seed,
                          basis=case.get("basis", "nodal"))


def _rhs(case, mesh, seed, k=1):
    """float64 [n_nodes, k]"""
    if case.get("bc") == "pin":
        return synth.pinned_normal_batch(mesh.n_nodes, k, seed)
    return synth.normal_rhs(mesh.n_nodes * k, seed).reshape(mesh.n_nodes, k)


def _serve_sizes(case):
    return [case["n"], case["n"] + 2, case["n"] + 4]


def prepare(case, seed):
    if case["kind"] == "serve":
        srv = Server(hbm_budget=20_000_000_000, slots=8, chunk=2, tol=TOL)
        requests = []
        for i, n in enumerate(_serve_sizes(case)):
            mesh = _mesh(case, seed + i, n)
            pid = srv.add_problem(mesh.coords, mesh.l2g, case["p"], case["lam"], _options(case))
            B = _rhs(case, mesh, seed + 100 + i, case["requests"])
            requests += [(pid, np.ascontiguousarray(B[:, j])) for j in range(case["requests"])]
            srv.wait(srv.submit(pid, requests[-1][1]))   # the hierarchy is resident from here on
        return {"kind": "serve", "server": srv, "requests": requests}
    mesh = _mesh(case, seed)
    b = torch.from_numpy(np.ascontiguousarray(_rhs(case, mesh, seed + 100, case.get("k", 1)))).to(DEV)
    state = {"kind": case["kind"], "b": b if case["kind"] == "batch" else b[:, 0].contiguous()}
    if case["kind"] == "setup":
        return {**state, "args": (mesh.coords, mesh.l2g, case["p"], case["lam"], _options(case))}
    state["solver"] = Solver(mesh.coords, mesh.l2g, case["p"], case["lam"], _options(case))
    return state


def run(state):
    kind = state["kind"]
    if kind == "solve":
        return state["solver"].solve(state["b"], tol=TOL)[0]
    if kind == "batch":
        return state["solver"].solve_batch(state["b"], tol=TOL)[0]
    if kind == "setup":
        solver = Solver(*state["args"])
        x = solver.solve(state["b"], tol=TOL)[0]
        solver.close()
        return x
    srv = state["server"]
    ids = [srv.submit(pid, b) for pid, b in state["requests"]]
    return [srv.wait(i)[0] for i in ids]


def work(case):
    """Bytes: the mesh (element corners and element map), the right-hand sides
    and the solutions once.  Flops: ten iterations of five applications of the
    fine operator per column, each by contractions of one direction at a time
    (values and gradient to the (p + 2)^3 quadrature points and back)."""
    def one(n, cols):
        p = case["p"]
        n1, q, ne, nodes = p + 1, p + 2, n ** 3, (n * p + 1) ** 3
        mac = 2 * q * n1 ** 3 + 3 * q * q * n1 * n1 + 4 * q ** 3 * n1
        return (ne * (24 * 8 + 4 * n1 ** 3) + 16 * nodes * cols, 50.0 * cols * ne * (4 * mac + 14 * q ** 3))

    if case["kind"] == "serve":
        parts = [one(n, case["requests"]) for n in _serve_sizes(case)]
    else:
        parts = [one(case["n"], case.get("k", 1))]
    return {"bytes": sum(b for b, _ in parts), "flops": sum(f for _, f in parts)}


# ---- the same systems in plain 64-bit torch ---------------------------------
def _basis(p, basis):
    """Values and derivatives [p + 1, p + 2] of the 1-D basis at the Gauss
    points, and the Gauss points and weights."""
    leg = np.polynomial.legendre
    g, w = leg.leggauss(p + 2)
    if basis == "modal":   # (1 - a)/2, (1 + a)/2, then (1 - a)/2 (1 + a)/2 P_m^{1,1}
        V, D = [(1 - g) / 2, (1 + g) / 2], [np.full(p + 2, -0.5), np.full(p + 2, 0.5)]
        for m in range(p - 1):
            # P_m^{1,1} = 2/(m + 2) P'_{m + 1}, and (1 - a^2) P' has the derivative -l(l + 1) P_l
            c = np.zeros(m + 2)
            c[-1] = 1.0
            V.append((1 - g * g) / 4 * (2 / (m + 2)) * leg.legval(g, leg.legder(c)))
            D.append(-(m + 1) * (m + 2) / 4 * (2 / (m + 2)) * leg.legval(g, c))
        return np.array(V), np.array(D), g, w
    c = np.zeros(p + 1)
    c[-1] = 1.0
    x = np.concatenate([[-1.0], np.sort(leg.legroots(leg.legder(c)).real) if p > 1 else [], [1.0]])
    V, D = np.ones((p + 1, p + 2)), np.zeros((p + 1, p + 2))
    for i in range(p + 1):
        for j in range(p + 1):
            if j != i:
                V[i] *= (g - x[j]) / (x[i] - x[j])
        for m in range(p + 1):
            if m != i:
                t = np.full(p + 2, 1.0 / (x[i] - x[m]))
                for j in range(p + 1):
                    if j not in (i, m):
                        t *= (g - x[j]) / (x[i] - x[j])
                D[i] += t
    return V, D, g, w


def _element_matrices(mesh, p, lam, basis):
    """Stiffness plus lam mass, float64 [elements, (p + 1)^3, (p + 1)^3]."""
    V, D, g, w = _basis(p, basis)
    q = p + 2
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)  # noqa: E731
    kron = lambda a, b, c: np.einsum("iq,jr,ks->ijkqrs", a, b, c).reshape((p + 1) ** 3, q ** 3)  # noqa: E731
    G = [t(kron(D, V, V)), t(kron(V, D, V)), t(kron(V, V, D))]
    M = t(kron(V, V, V))
    H, dH = np.array([(1 - g) / 2, (1 + g) / 2]), np.array([np.full(q, -0.5), np.full(q, 0.5)])
    corner = lambda a, b, c: t(np.einsum("iq,jr,ks->ijkqrs", a, b, c).reshape(8, q ** 3))  # noqa: E731
    dN = torch.stack([corner(dH, H, H), corner(H, dH, H), corner(H, H, dH)])
    wq = t(np.einsum("q,r,s->qrs", w, w, w).reshape(-1))
    ends = [0, 1] if basis == "modal" else [0, p]
    loc = [((p + 1) * i + j) * (p + 1) + k for i in ends for j in ends for k in ends]
    X = t(mesh.coords[mesh.l2g[:, loc]])                          # [ne, 8, 3]
    out = []
    for Xc in X.split(512):
        # J[e, q, a, d] = d x_a / d xi_d, one product per (a, d)
        J = torch.stack([torch.stack([Xc[:, :, a] @ dN[d] for d in range(3)], -1) for a in range(3)], -2)
        Ji = torch.linalg.inv(J)
        wd = wq * torch.linalg.det(J)
        # K = sum_de G_d diag(wd Ji_d . Ji_e) G_e^T, column factors summed first
        K = torch.zeros(Xc.shape[0], (p + 1) ** 3, (p + 1) ** 3, dtype=torch.float64, device=DEV)
        for d in range(3):
            F = sum(((Ji[:, :, d, :] * Ji[:, :, e, :]).sum(-1) * wd)[:, None, :] * G[e][None] for e in range(3))
            K += (F.reshape(-1, q ** 3) @ G[d].T).reshape(K.shape).transpose(1, 2)
        F = (lam * wd)[:, None, :] * M[None]
        K += (F.reshape(-1, q ** 3) @ M.T).reshape(K.shape)
        out.append(K)
    return torch.cat(out)


def _constrained(case, mesh):
    L = mesh.n * mesh.p + 1
    mask = np.zeros((L, L, L), dtype=bool)
    if case.get("bc") == "pin":
        mask.reshape(-1)[0] = True
    else:
        for axis in range(3):
            side = np.moveaxis(mask, axis, 0)
            side[0] = side[-1] = True
    return torch.from_numpy(mask.reshape(-1)).to(DEV)


def _cg(case, mesh, B):
    """A X = B by diagonally preconditioned CG on every column, until the
    residual stops falling."""
    K = _element_matrices(mesh, mesh.p, case["lam"], case.get("basis", "nodal"))
    ids = torch.from_numpy(mesh.l2g.astype(np.int64)).to(DEV)
    cons = _constrained(case, mesh)[:, None]
    n, k = B.shape

    def apply(v):
        y = (K @ torch.where(cons, 0.0, v)[ids]).reshape(-1, k)
        return torch.where(cons, v, torch.zeros(n, k, dtype=v.dtype, device=DEV).index_add_(0, ids.reshape(-1), y))

    diag = torch.zeros(n, dtype=torch.float64, device=DEV)
    diag.index_add_(0, ids.reshape(-1), torch.diagonal(K, dim1=1, dim2=2).reshape(-1))
    diag = torch.where(cons, 1.0, diag[:, None])
    X, R = torch.zeros_like(B), B.clone()
    P = Z = R / diag
    rz = (R * Z).sum(0)
    bb = B.norm(dim=0)
    for it in range(20000):
        Q = apply(P)
        alpha = rz / (P * Q).sum(0)
        X += alpha * P
        R -= alpha * Q
        if it % 20 == 0 and bool((R.norm(dim=0) < 1e-15 * bb).all()):
            break
        Z = R / diag
        new = (R * Z).sum(0)
        P = Z + (new / rz) * P
        rz = new
    return X


def exact(case, seed):
    if case["kind"] == "serve":
        out = []
        for i, n in enumerate(_serve_sizes(case)):
            mesh = _mesh(case, seed + i, n)
            B = torch.from_numpy(_rhs(case, mesh, seed + 100 + i, case["requests"])).to(DEV)
            X = _cg(case, mesh, B).cpu().numpy()
            out += [np.ascontiguousarray(X[:, j]) for j in range(case["requests"])]
        return out
    mesh = _mesh(case, seed)
    k = case.get("k", 1)
    # the batched product needs the element blocks of every column: a few at a time
    B = torch.from_numpy(np.ascontiguousarray(_rhs(case, mesh, seed + 100, k))).to(DEV)
    X = torch.cat([_cg(case, mesh, b.contiguous()) for b in B.split(16, dim=1)], 1)
    return X if case["kind"] == "batch" else X[:, 0].contiguous()
