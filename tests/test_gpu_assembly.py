"""Fine-level assembly on the device against the host assembly and the
oracle: the same CSR pattern bit for bit, values to rounding (the element
integrals are contracted in another order), for nodal and modal bases,
Dirichlet and pinned constraints, several orders; and the AUTO / DEVICE /
HOST choice of where the operator is built."""
import numpy as np
import pytest

import synth
from oracle import assembly as oasm

pytestmark = pytest.mark.gpu

CASES = {
    # name: (n, p, lambda, bc, perturb, basis)
    "p1_5cube": (5, 1, 2.0, "dirichlet", 0.2, "nodal"),
    "p2_4cube": (4, 2, 0.5, "dirichlet", 0.15, "nodal"),
    "p3_3cube_pin": (3, 3, 0.0, "pin", 0.1, "nodal"),
    "p4_3cube": (3, 4, 10.0, "dirichlet", 0.1, "nodal"),
    "p5_2cube": (2, 5, 1.0, "dirichlet", 0.1, "nodal"),
    "p6_2cube_pin": (2, 6, 3.0, "pin", 0.1, "nodal"),
    "p4_3cube_modal": (3, 4, 1.0, "dirichlet", 0.1, "modal"),
    "p8_2cube": (2, 8, 1.0, "dirichlet", 0.0, "nodal"),
}


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2512_15121_amd import giamg
    giamg.library()
    return torch


def _solver(m, p, lam, bc, basis, assembly):
    from paper_2512_15121_amd import Solver, Options
    return Solver(m.coords, m.l2g, p, lam,
                  Options(bc=bc, basis=basis, assembly=assembly, preconditioner="jacobi"))


@pytest.mark.parametrize("name", list(CASES))
def test_device_assembly_matches_host_and_oracle(torch_dev, name):
    n, p, lam, bc, pert, basis = CASES[name]
    print(f"case {name}", flush=True)
    m = synth.hex_mesh(n, p, perturb=pert, seed=5, basis=basis)
    sd = _solver(m, p, lam, bc, basis, "device")
    sh = _solver(m, p, lam, bc, basis, "host")
    assert sd.level(0)["device_assembly"] and not sh.level(0)["device_assembly"]
    rp_d, ci_d, v_d = sd.level_csr(0, "A")
    rp_h, ci_h, v_h = sh.level_csr(0, "A")
    assert np.array_equal(rp_d, rp_h) and np.array_equal(ci_d, ci_h)
    scale = np.max(np.abs(v_h))
    assert np.max(np.abs(v_d - v_h)) <= 1e-13 * scale
    # against the oracle's assembly of the same operator
    A, _ = oasm.assemble(m.coords, m.l2g, p, lam, bc=bc, basis=basis)
    assert np.array_equal(rp_d, A.indptr) and np.array_equal(ci_d, A.indices)
    assert np.max(np.abs(v_d - A.data)) <= 1e-12 * np.max(np.abs(A.data))
    sd.close()
    sh.close()


def test_auto_assembly_is_on_the_device_and_solves_match(torch_dev):
    torch = torch_dev
    from paper_2512_15121_amd import Solver, Options
    m = synth.hex_mesh(4, 3, perturb=0.1, seed=9)
    b = torch.from_numpy(synth.normal_rhs(m.n_nodes, 3)).to("cuda:0")
    out = {}
    for where in ("auto", "host"):
        s = Solver(m.coords, m.l2g, 3, 1.0, Options(assembly=where))
        assert s.level(0)["device_assembly"] == (where == "auto")
        x, info = s.solve(b, tol=1e-10)
        assert info.status == 0
        out[where] = (x, info.iters)
        s.close()
    (xa, ia), (xh, ih) = out["auto"], out["host"]
    assert abs(ia - ih) <= 1
    assert (torch.linalg.norm(xa - xh) / torch.linalg.norm(xh)).item() <= 1e-9


def test_device_assembly_beyond_its_lds_lists(torch_dev):
    """p = 10 on 2^3 elements: the centre row has 21^3 columns, more than the
    fill kernel's LDS lists hold with the order-10 element-row work: DEVICE
    reports GIAMG_ENOTSUP, AUTO builds the operator on the host."""
    from paper_2512_15121_amd import Solver, Options, giamg
    m = synth.hex_mesh(2, 10, perturb=0.0, seed=1)
    with pytest.raises(giamg.GiamgError) as e:
        Solver(m.coords, m.l2g, 10, 1.0, Options(assembly="device", preconditioner="jacobi"))
    assert e.value.code == giamg.ENOTSUP
    s = Solver(m.coords, m.l2g, 10, 1.0, Options(assembly="auto", preconditioner="jacobi"))
    assert not s.level(0)["device_assembly"]
    s.close()


def test_device_assembly_full_size_16cube_p4(torch_dev):
    """The benchmark's 16^3, p = 4 operator (274,625 rows, 49.5 M nonzeros):
    device and host assembly give the same pattern bit for bit and values to
    1e-13 of the largest entry, and the device operator is symmetric to the
    same bar (each entry and its mirror are separate element-row sums)."""
    import scipy.sparse as sp
    m = synth.hex_mesh(16, 4, perturb=0.1, seed=2)
    sd = _solver(m, 4, 10.0, "dirichlet", "nodal", "device")
    sh = _solver(m, 4, 10.0, "dirichlet", "nodal", "host")
    rp_d, ci_d, v_d = sd.level_csr(0, "A")
    rp_h, ci_h, v_h = sh.level_csr(0, "A")
    sd.close()
    sh.close()
    assert rp_d[-1] == 49455441
    assert np.array_equal(rp_d, rp_h) and np.array_equal(ci_d, ci_h)
    scale = np.max(np.abs(v_h))
    assert np.max(np.abs(v_d - v_h)) <= 1e-13 * scale
    A = sp.csr_matrix((v_d, ci_d, rp_d), shape=(m.n_nodes, m.n_nodes))
    assert abs(A - A.T).max() <= 1e-13 * scale


TRANSFER_CASES = {
    # name: (n, p, bc, basis, schedule, keep_boundary)
    "p4_dirichlet": (4, 4, "dirichlet", "nodal", (), False),
    "p6_pin": (3, 6, "pin", "nodal", (), False),
    "p5_by_one": (3, 5, "dirichlet", "nodal", (4, 3, 2, 1), False),
    "p5_non_divisor": (3, 5, "dirichlet", "nodal", (4, 2, 1), False),
    "p4_modal": (3, 4, "dirichlet", "modal", (), False),
    "p8_keep_boundary": (2, 8, "dirichlet", "nodal", (), True),
}


@pytest.mark.parametrize("name", list(TRANSFER_CASES))
def test_device_p_transfer_matches_host_bitwise(torch_dev, name):
    """P and R = P^T of every p-level built on the device equal the host
    build bit for bit (rows, columns, values), and so do the coarse element
    maps."""
    from paper_2512_15121_amd import Solver, Options
    n, p, bc, basis, sched, keep = TRANSFER_CASES[name]
    print(f"case {name}", flush=True)
    m = synth.hex_mesh(n, p, perturb=0.1, seed=3, basis=basis)
    out = {}
    for where in ("device", "host"):
        s = Solver(m.coords, m.l2g, p, 1.0, Options(bc=bc, basis=basis, schedule=sched, keep_boundary=keep,
                                                     assembly=where, coarse_max=50))
        levels = []
        for l in range(s.num_levels() - 1):
            d = s.level(l)
            if d["kind"] != "p" or s.level(l + 1)["kind"] != "p":
                break
            levels.append((s.level_csr(l, "P"), s.level_csr(l, "R"), s.level_l2g(l + 1)))
        out[where] = levels
        s.close()
    assert len(out["device"]) == len(out["host"]) > 0
    for (pd, rd, gd), (ph, rh, gh) in zip(out["device"], out["host"]):
        for a, b in ((pd, ph), (rd, rh)):
            assert all(np.array_equal(x, y) for x, y in zip(a, b))
        assert np.array_equal(gd, gh)


# (mesh size, boundary condition) of an order-1 operator that is its own coarsest
# level, (n + 1)^3 rows: 2 tiles of 64 rows with 61 in the last, 6 with 23, 8 full
# ones, 12 with 25
@pytest.mark.parametrize("n,bc", [(4, "dirichlet"), (6, "dirichlet"), (6, "pin"), (7, "dirichlet"), (8, "dirichlet")])
def test_coarsest_inverse_on_the_device(n, bc):
    """Against LAPACK's inverse, to the bound of the host's inverse (n eps cond,
    with cond below 1e3: 1e-11), and exactly symmetric."""
    import scipy.sparse as sp
    import torch
    from paper_2512_15121_amd import Options, Solver
    m = synth.hex_mesh(n, 1, perturb=0.1, seed=3)
    s = Solver(m.coords, m.l2g, 1, 2.0, Options(bc=bc, coarse_max=2000))
    l = s.num_levels() - 1
    rp, ci, val = s.level_csr(l)
    A = sp.csr_matrix((val, ci, rp)).toarray()
    nc = A.shape[0]
    f = torch.zeros(nc, dtype=torch.float64, device="cuda:0")
    out = torch.zeros_like(f)
    X = np.empty((nc, nc))
    for c in range(nc):
        f[c] = 1.0
        s.apply("coarse", l, f, out=out)
        X[:, c] = out.cpu().numpy()
        f[c] = 0.0
    s.close()
    ref = np.linalg.inv(A)
    assert np.array_equal(X, X.T)
    assert np.max(np.abs(X - ref)) <= 1e-11 * np.max(np.abs(ref))
