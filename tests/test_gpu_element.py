"""The element form of the fine operator (sum factorisation over the elements)
against the assembled rows of the same handle, at every order it serves.

Bounds.  A product by sum factorisation rounds about 2 (3 (p + 2)) multiply-adds
per value along its six contractions and 40 more at a quadrature point, on
quantities up to the size of |B|^T |D| |B| |x|, which exceeds |A| |x| by the
interpolation's Lebesgue constants (below 2 per direction and pass, 2^6
together): max |y - A x| <= (6 (p + 2) + 40) 64 eps max(|A| |x|), eps the unit
roundoff of the precision.
"""
import numpy as np
import pytest
import scipy.sparse as sp

import synth

pytestmark = pytest.mark.gpu

# (n, p, basis, bc): one per order, above the size from which the form is used
# (0.15 M p^2 and 4 M nonzeros); element counts that leave the last block of
# several elements ragged, few and many elements per order, both block shapes
CASES = [(21, 2, "nodal", "dirichlet"), (13, 3, "nodal", "pin"), (17, 3, "modal", "dirichlet"),
         (9, 4, "nodal", "dirichlet"), (9, 4, "modal", "pin"), (13, 4, "nodal", "dirichlet"),
         (7, 5, "nodal", "dirichlet"), (12, 5, "nodal", "dirichlet"), (6, 6, "modal", "dirichlet"),
         (5, 7, "nodal", "pin"), (10, 7, "nodal", "dirichlet"), (4, 8, "nodal", "dirichlet"),
         (9, 8, "nodal", "dirichlet"), (4, 9, "nodal", "dirichlet"), (3, 10, "nodal", "pin")]


@pytest.mark.parametrize("n,p,basis,bc", CASES)
def test_element_products_match_assembled_rows(n, p, basis, bc):
    import torch
    from paper_2512_15121_amd import Options, Solver
    m = synth.hex_mesh(n, p, perturb=0.1, seed=5, basis=basis)
    # mixed handles with a pinned node keep the assembled rows (the constant's mode)
    precision = "fp64" if bc == "pin" else "mixed"
    s = Solver(m.coords, m.l2g, p, 2.0, Options(precision=precision, basis=basis, bc=bc))
    _, by = s.time_kernel("spmv", 0, 1)
    d = s.level(0)
    assert by < 8 * d["nnz_A"], "the product reads the assembled values"
    rp, ci, val = s.level_csr(0)
    A = sp.csr_matrix((val, ci, rp), shape=(d["rows"],) * 2)
    rng = np.random.default_rng(7)
    x, f = rng.standard_normal(d["rows"]), rng.standard_normal(d["rows"])
    for dt, eps, fp32 in ((torch.float64, 2.0 ** -53, False), (torch.float32, 2.0 ** -24, True)):
        if fp32 and precision != "mixed":
            continue
        xt, ft = (torch.from_numpy(v).to(dt).to("cuda:0") for v in (x, f))
        xh, fh = xt.double().cpu().numpy(), ft.double().cpu().numpy()
        bound = (6 * (p + 2) + 40) * 64 * eps * np.max(abs(A) @ np.abs(xh))
        y = torch.zeros_like(xt)
        s.apply("spmv", 0, xt, out=y, fp32=fp32)
        got = y.double().cpu().numpy()
        assert np.max(np.abs(got - A @ xh)) <= bound
        cons = s.constrained()
        assert np.array_equal(got[cons], xh[cons])          # identity rows
        s.apply("residual", 0, ft, xt, out=y, fp32=fp32)
        assert np.max(np.abs(y.double().cpu().numpy() - (fh - A @ xh))) <= bound + 4 * eps * np.max(np.abs(fh))
        z = torch.zeros_like(xt)
        s.apply("residual", 0, ft, xt, out=z, fp32=fp32)
        assert torch.equal(y, z)                             # the same bits every time
    s.close()


# (n, p, basis, precision): every order of the block products' element form (matrix
# instructions up to p = 4, sum factorisation above)
BATCHES = [(5, 2, "nodal", "mixed"), (4, 2, "modal", "fp64"), (3, 3, "nodal", "mixed"), (4, 3, "nodal", "fp64"),
           (4, 4, "nodal", "mixed"), (3, 4, "modal", "fp64"), (4, 5, "nodal", "mixed"), (3, 6, "modal", "fp64"), (3, 7, "nodal", "mixed"), (2, 8, "nodal", "fp64"),
           (2, 9, "nodal", "mixed"), (2, 10, "nodal", "fp64")]


@pytest.mark.parametrize("n,p,basis,precision", BATCHES)
def test_element_block_columns_alone_and_together(n, p, basis, precision):
    """A column gives the same bits alone, among 2, 20 and 70 (each split of rows
    and columns over waves, tiles of 16 and 64 columns that end ragged, blocks
    of (element, column) pairs that cross elements; vectors of one and of four
    columns in the node step), and agrees with the single solve of the same system: both
    stop at a relative residual of 1e-10 of the same operator, 1e-8 apart at
    most."""
    import torch
    from paper_2512_15121_amd import Options, Solver
    m = synth.hex_mesh(n, p, perturb=0.1, seed=6, basis=basis)
    s = Solver(m.coords, m.l2g, p, 2.0, Options(precision=precision, basis=basis))
    B = torch.from_numpy(synth.normal_rhs(m.n_nodes * 70, 8).reshape(m.n_nodes, 70)).to("cuda:0")
    X, infos = s.solve_batch(B)
    assert all(i.status == 0 and i.true_relres < 1e-9 for i in infos)
    for cols in ((0,), (41,), (69, 3), tuple(range(45, 65))):
        Xc, ic = s.solve_batch(B[:, list(cols)].contiguous())
        for j, c in enumerate(cols):
            assert ic[j].iters == infos[c].iters and torch.equal(Xc[:, j], X[:, c]), (cols, c)
    x, _ = s.solve(B[:, 41].contiguous())
    assert torch.linalg.norm(x - X[:, 41]) <= 1e-8 * torch.linalg.norm(x)
    s.close()


def test_pinned_mixed_handles_keep_the_assembled_rows():
    """One pinned node holds the constant of a pure Neumann problem: in mixed
    precision the FP32 cycle's rounding decides the solution's shift, so single
    and batched products of such handles stay with the assembled rows, whose
    bits direct_gathers = 1 and the forced block shapes share."""
    import torch
    from paper_2512_15121_amd import Options, Solver
    m = synth.hex_mesh(8, 5, perturb=0.1, seed=5)
    B = torch.from_numpy(synth.pinned_normal_batch(m.n_nodes, 3, 9)).to("cuda:0")
    x, X = [], []
    for kw in ({}, {"direct_gathers": True, "batch_kernel": "lanes"}):
        s = Solver(m.coords, m.l2g, 5, 0.0, Options(precision="mixed", bc="pin", **kw))
        assert s.time_kernel("spmv", 0, 1)[1] >= 8 * s.level(0)["nnz_A"]
        x.append(s.solve(B[:, 1].contiguous())[0])
        X.append(s.solve_batch(B)[0])
        s.close()
    assert torch.equal(x[0], x[1]) and torch.equal(X[0], X[1])


# (n, p, schedule): every order the transfers' element form takes (a million entries of P), with
# divisor and other coarse orders, meshes whose last block of elements is partly filled
TRANSFERS = [(35, 2, ()), (22, 3, ()), (14, 4, ()), (9, 4, (3, 1)), (7, 5, (3, 1)), (7, 5, (4, 2, 1)), (6, 6, ()),
             (9, 7, ()), (4, 8, ()), (4, 9, ()), (3, 10, ())]


@pytest.mark.parametrize("n,p,schedule", TRANSFERS)
def test_element_transfers_match_the_assembled_ones(n, p, schedule):
    """x + P e and R t against the stored P and R = P^T.  An entry sums along
    three axes of at most 11 terms and over 8 elements, and the 1-D factors' moduli
    multiply to |P|: 64 roundings of |P| |e| and |R| |t| bound the difference."""
    import torch
    from paper_2512_15121_amd import Options, Solver
    m = synth.hex_mesh(n, p, perturb=0.1, seed=7)
    for precision in ("fp64", "mixed"):
        s = Solver(m.coords, m.l2g, p, 2.0, Options(precision=precision, schedule=schedule))
        d, c = s.level(0), s.level(1)
        assert s.time_kernel("prolong", 0, 1)[1] < 8 * d["nnz_P"] + 24 * d["rows"]   # not the stored values
        rp, ci, val = s.level_csr(0, "P")
        P = sp.csr_matrix((val, ci, rp), shape=(d["rows"], c["rows"]))
        rng = np.random.default_rng(p)
        e, t = rng.standard_normal(c["rows"]), rng.standard_normal(d["rows"])
        fp32 = precision == "mixed"
        dt = torch.float32 if fp32 else torch.float64
        eps = 2.0 ** -23 if fp32 else 2.0 ** -52
        et, tt = torch.from_numpy(e).to("cuda:0", dt), torch.from_numpy(t).to("cuda:0", dt)
        e, t = et.double().cpu().numpy(), tt.double().cpu().numpy()
        x = tt.clone()
        s.apply("prolong_add", 0, et, out=x, fp32=fp32)
        got = x.double().cpu().numpy()
        assert np.all(np.abs(got - (t + P @ e)) <= 64 * eps * (np.abs(t) + abs(P) @ np.abs(e)))
        f = torch.zeros(c["rows"], dtype=dt, device="cuda:0")
        s.apply("restrict", 0, tt, out=f, fp32=fp32)
        assert np.all(np.abs(f.double().cpu().numpy() - P.T @ t) <= 64 * eps * (abs(P).T @ np.abs(t)))
        s.close()


def _turned(n, p):
    """Every third element turned by half a turn about its third axis."""
    m = synth.hex_mesh(n, p, perturb=0.1, seed=7)
    l2g = m.l2g.reshape(-1, p + 1, p + 1, p + 1).copy()
    l2g[::3] = l2g[::3, ::-1, ::-1, :]
    return m.coords, np.ascontiguousarray(l2g.reshape(m.l2g.shape))


def _sector(n, p):
    """A quarter of a cylinder: the elements at its axis list each node there p + 1 times."""
    m = synth.hex_mesh(n, p)
    r, t = m.coords[:, 0], m.coords[:, 1] * np.pi / 2
    coords = np.stack([r * np.cos(t), r * np.sin(t), m.coords[:, 2]], 1)
    L = n * p + 1
    ids = np.arange(L ** 3).reshape(L, L, L)
    ids[0] = ids[0, :1]
    used, l2g = np.unique(ids.reshape(-1)[m.l2g], return_inverse=True)
    return np.ascontiguousarray(coords[used]), l2g.reshape(m.l2g.shape).astype(np.int32)


# order 2 keeps an order-5 element's nodes unevenly, order 3 evenly
@pytest.mark.parametrize("mesh,n,p,schedule,form", [(_turned, 9, 5, (2, 1), False), (_turned, 7, 5, (3, 1), True),
                                                    (_sector, 14, 4, (), False)])
def test_transfers_on_turned_and_collapsed_elements(mesh, n, p, schedule, form):
    """P's rows are unions over a node's elements with the first weight of a coarse
    node kept: where an element alone does not give them, the transfers keep the
    stored rows (bound as above).  Products run over the elements on these meshes
    too, against the assembled rows to the bound of the module."""
    import torch
    from paper_2512_15121_amd import Options, Solver
    coords, l2g = mesh(n, p)
    s = Solver(coords, l2g, p, 2.0, Options(schedule=schedule, bc="pin"))
    d, c = s.level(0), s.level(1)

    def rows(which, cols):
        rp, ci, val = s.level_csr(0, which)
        return sp.csr_matrix((val, ci, rp), shape=(d["rows"], cols))
    P, A = rows("P", c["rows"]), rows("A", d["rows"])
    assert P.nnz > 1000000 and s.time_kernel("spmv", 0, 1)[1] < 8 * A.nnz
    assert (s.time_kernel("prolong", 0, 1)[1] < 8 * P.nnz + 24 * d["rows"]) == form
    rng = np.random.default_rng(p)
    e, t = rng.standard_normal(c["rows"]), rng.standard_normal(d["rows"])
    dev = lambda v: torch.from_numpy(v).to("cuda:0")  # noqa: E731
    eps = 2.0 ** -52
    x = dev(t).clone()
    s.apply("prolong_add", 0, dev(e), out=x)
    assert np.all(np.abs(x.cpu().numpy() - (t + P @ e)) <= 64 * eps * (np.abs(t) + abs(P) @ np.abs(e)))
    f = torch.zeros(c["rows"], dtype=torch.float64, device="cuda:0")
    s.apply("restrict", 0, dev(t), out=f)
    assert np.all(np.abs(f.cpu().numpy() - P.T @ t) <= 64 * eps * (abs(P).T @ np.abs(t)))
    y = torch.zeros_like(x)
    s.apply("spmv", 0, dev(t), out=y)
    assert np.max(np.abs(y.cpu().numpy() - A @ t)) <= (6 * (p + 2) + 40) * 32 * eps * np.max(abs(A) @ np.abs(t))
    s.close()


# single products over the elements (p = 4, 2), and block products of order 5
@pytest.mark.parametrize("n,p,batch", [(9, 4, False), (21, 2, False), (4, 5, True)])
def test_fp32_cycle_in_any_unit_of_length(n, p, batch):
    """The entries go as the element size h (lambda h^2 kept): with h scaled by a power
    of two every number of a mixed solve is scaled by one too (identity rows apart,
    whose right-hand sides are zero here), so the solution times it is the same to the
    last bit.  2^-47 and 2^47 take (h / 2)^3 out of FP32's range, the entries not."""
    import torch
    from paper_2512_15121_amd import Options, Solver
    m = synth.hex_mesh(n, p, perturb=0.1, seed=3)
    x = {}
    for e in (0, -47, 47):
        h = 2.0 ** e
        s = Solver(m.coords * h, m.l2g, p, 3.0 / (h * h), Options(precision="mixed"))
        if not batch:
            assert s.time_kernel("spmv", 0, 1)[1] < 8 * s.level(0)["nnz_A"]
        b = synth.normal_rhs(m.n_nodes, 5) * ~s.constrained()
        bt = torch.from_numpy(b).to("cuda:0")
        if batch:
            X, (info,) = s.solve_batch(bt.reshape(-1, 1).contiguous())
            x[e] = X[:, 0] * h
        else:
            xs, info = s.solve(bt)
            x[e] = xs * h
        assert info.status == 0 and info.true_relres < 1e-9, e
        s.close()
    assert torch.equal(x[0], x[-47]) and torch.equal(x[0], x[47])


@pytest.mark.parametrize("shear,form", [(100.0, True), (1e4, False)])
def test_sheared_elements_keep_the_precision_of_the_fp32_products(shear, form):
    """Elements sheared so far that FP32 loses their determinant keep the assembled
    rows in mixed precision (their FP32 products round (p + 2)^3 multiply-adds at
    most); the form serves those it is good for, to the bound of the module times the
    growth of a determinant's rounding, the shear."""
    import torch
    from paper_2512_15121_amd import Options, Solver
    n, p = 9, 4
    m = synth.hex_mesh(n, p)
    rng = np.random.default_rng(2)
    turn, _ = np.linalg.qr(rng.standard_normal((3, 3)))
    turn *= np.linalg.det(turn)
    S = np.eye(3)
    S[0, 1] = shear
    s = Solver(m.coords @ (turn @ S).T, m.l2g, p, 2.0, Options(precision="mixed"))
    d = s.level(0)
    rp, ci, val = s.level_csr(0)
    A = sp.csr_matrix((val, ci, rp), shape=(d["rows"],) * 2)
    assert (s.time_kernel("spmv", 0, 1)[1] < 8 * A.nnz) == form
    x = torch.from_numpy(rng.standard_normal(d["rows"])).to("cuda:0", torch.float32)
    y = torch.zeros_like(x)
    s.apply("spmv", 0, x, out=y, fp32=True)
    s.close()
    xh = x.double().cpu().numpy()
    bound = ((6 * (p + 2) + 40) * 64 * shear if form else 2 * (p + 2) ** 3) * 2.0 ** -24 * np.max(abs(A) @ np.abs(xh))
    assert np.max(np.abs(y.double().cpu().numpy() - A @ xh)) <= bound


@pytest.mark.parametrize("n,p", [(16, 4), (41, 2)])
def test_element_matrices_of_several_launches(n, p):
    """73 k and 116 k blocks form the matrices, two launches of at most 65536.  Batched
    against the single solve, which has no matrices: both stop at a relative residual
    of 1e-10 of the same operator, 1e-8 apart at most, for every column."""
    import torch
    from paper_2512_15121_amd import Options, Solver
    m = synth.hex_mesh(n, p, perturb=0.1, seed=6)
    s = Solver(m.coords, m.l2g, p, 2.0, Options())
    B = torch.from_numpy(synth.normal_rhs(m.n_nodes * 3, 8).reshape(m.n_nodes, 3)).to("cuda:0")
    X, infos = s.solve_batch(B)
    for j in range(3):
        x, info = s.solve(B[:, j].contiguous())
        assert infos[j].status == 0 and infos[j].true_relres < 1e-9 and abs(infos[j].iters - info.iters) <= 1
        assert torch.linalg.norm(x - X[:, j]) <= 1e-8 * torch.linalg.norm(x)
    s.close()


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("n,p", [(14, 4), (22, 3), (7, 5)])
def test_handles_keep_nothing_that_their_products_do_not_read(n, p, precision):
    """With the products over the elements a handle's memory is bounded by the FP64
    rows of A (level_csr), P and R and their FP32 copies, the coarse levels with A P
    and tables (2 bytes per entry and precision), the element and transfer forms, and
    vectors: no FP32 copy of A, no A P, no tables of either.  level_csr still gives
    A P, and a level's description the tables' counts."""
    import torch
    from paper_2512_15121_amd import Options, Solver, giamg
    m = synth.hex_mesh(n, p, perturb=0.1, seed=5)
    live = {}

    def alloc(nbytes, stream):
        q = torch.cuda.caching_allocator_alloc(nbytes, 0, stream)
        live[q] = nbytes
        return q

    def release(q):
        live.pop(q)
        torch.cuda.caching_allocator_delete(q)

    giamg.set_allocator(alloc, release)
    try:
        s = Solver(m.coords, m.l2g, p, 2.0, Options(precision=precision, coarse_max=300))
        held = sum(live.values())
        d = [s.level(l) for l in range(s.num_levels())]
        assert s.time_kernel("spmv", 0, 1)[1] < 8 * d[0]["nnz_A"]
        f32 = 4 if precision == "mixed" else 0
        nl, nodes = (p + 1) ** 3, sum(lv["rows"] for lv in d)
        bound = 12 * d[0]["nnz_A"] + (12 + f32) * (d[0]["nnz_P"] + d[0]["nnz_R"])
        bound += sum((12 + f32 + 2 + f32 // 2) * lv["nnz_" + q] for lv in d[1:] for q in ("A", "P", "R", "AP"))
        bound += m.n_elem * (4 * nl + 8 * nl + 4 * nl + 21 * 8 + 23 * f32)      # map, results, entries, geometry
        bound += m.n_elem * (4 * nl + 2 * 4 * (nl // 2))                        # transfers' maps and entries
        bound += nodes * (4 * 8 + 4 * 4 + 7 * (8 + f32)) + 7 * 8 * m.n_nodes    # row pointers, lists, vectors
        bound += 8 * d[-1]["rows"] ** 2 + nodes * 8                             # coarse inverse, row blocks, partials
        print(f"n = {n}, p = {p}, {precision}: {held} bytes, bound {bound}")
        assert held <= bound
        if d[0]["nnz_A"] > 2000000:
            assert d[0]["staged_nnz_A"] == d[0]["nnz_A"]
        mats = []
        for which, cols in (("A", d[0]["rows"]), ("P", d[1]["rows"]), ("AP", d[1]["rows"])):
            rp, ci, val = s.level_csr(0, which)
            mats.append(sp.csr_matrix((val, ci, rp), shape=(d[0]["rows"], cols)))
        A, P, AP = mats
        assert d[0]["nnz_AP"] == AP.nnz
        assert abs(AP - A @ P).max() <= 1e-12 * (abs(A) @ abs(P)).max()
        s.close()
        assert live == {}
    finally:
        giamg.set_allocator()
