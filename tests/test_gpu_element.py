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
    s = Solver(m.coords, m.l2g, p, 2.0, Options(precision="mixed", basis=basis, bc=bc))
    _, by = s.time_kernel("spmv", 0, 1)
    d = s.level(0)
    assert by < 8 * d["nnz_A"], "the product reads the assembled values"
    rp, ci, val = s.level_csr(0)
    A = sp.csr_matrix((val, ci, rp), shape=(d["rows"],) * 2)
    rng = np.random.default_rng(7)
    x, f = rng.standard_normal(d["rows"]), rng.standard_normal(d["rows"])
    for dt, eps, fp32 in ((torch.float64, 2.0 ** -53, False), (torch.float32, 2.0 ** -24, True)):
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
