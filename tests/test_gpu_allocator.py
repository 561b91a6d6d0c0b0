"""Device memory through a caller's allocator (giamg_set_allocator): every
block the library takes comes from the registered allocator and goes back
to it, and results do not depend on where the memory came from."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def test_torch_allocator_routes_all_device_memory():
    import torch
    from paper_2512_15121_amd import Solver, Options, giamg
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    m = synth.hex_mesh(5, 3, perturb=0.1, seed=4)
    b = torch.from_numpy(synth.normal_rhs(m.n_nodes, 3)).to("cuda:0")
    B = torch.from_numpy(synth.normal_rhs(m.n_nodes * 4, 5).reshape(m.n_nodes, 4)).to("cuda:0")
    live, total = {}, [0, 0]

    def alloc(n, stream):
        p = torch.cuda.caching_allocator_alloc(n, 0, stream)
        live[p] = n
        total[0] += 1
        total[1] += n
        return p

    def release(p):
        live.pop(p)
        torch.cuda.caching_allocator_delete(p)

    giamg.set_allocator(alloc, release)
    try:
        s = Solver(m.coords, m.l2g, 3, 2.0, Options(precision="mixed"))
        after_setup = total[0]
        x1, i1 = s.solve(b, tol=1e-10)
        X1, _ = s.solve_batch(B, tol=1e-10)
        torch.cuda.synchronize()
        assert after_setup > 10 and total[0] >= after_setup and live
        assert all(p % 256 == 0 for p in live)
        s.close()
        assert live == {}, f"{len(live)} blocks not returned"
    finally:
        giamg.set_allocator()
    s2 = Solver(m.coords, m.l2g, 3, 2.0, Options(precision="mixed"))
    x2, i2 = s2.solve(b, tol=1e-10)
    X2, _ = s2.solve_batch(B, tol=1e-10)
    assert i1.iters == i2.iters and torch.equal(x1, x2) and torch.equal(X1, X2)
    s2.close()
    n_before = total[0]
    s3 = Solver(m.coords, m.l2g, 3, 2.0, Options())   # hipMalloc again
    s3.close()
    assert total[0] == n_before


def test_failing_allocator_is_an_allocation_error():
    import torch
    from paper_2512_15121_amd import Solver, Options, giamg
    m = synth.hex_mesh(3, 2, seed=1)
    giamg.set_allocator(lambda n, s: 0, lambda p: None)
    try:
        with pytest.raises(giamg.GiamgError) as e:
            Solver(m.coords, m.l2g, 2, 1.0, Options())
        assert e.value.code == giamg.ENOMEM
    finally:
        giamg.set_allocator()
    s = Solver(m.coords, m.l2g, 2, 1.0, Options())
    s.close()


# (in mixed precision the tuning of the rows' products at p = 5 needs more than the element form)
@pytest.mark.parametrize("n,p,k,session,precision", [(6, 4, 8, False, "fp64"), (6, 4, 8, False, "mixed"),
                                                     (9, 4, 4, False, "fp64"), (9, 4, 4, False, "mixed"),
                                                     (5, 3, 64, True, "fp64"), (5, 3, 64, True, "mixed"),
                                                     (4, 5, 64, False, "fp64")])
def test_batches_without_memory_for_the_element_form(n, p, k, session, precision):
    """With one byte less than the block products' element form needs at its peak, a
    batch takes the rows' products instead: the same solutions to the tolerance (both
    stop at a relative residual of 1e-10 of the same operator, 1e-8 apart at most),
    and a column's bits alone are those in the batch, then too."""
    import torch
    from paper_2512_15121_amd import Options, Session, Solver, giamg
    m = synth.hex_mesh(n, p, perturb=0.1, seed=6)
    B = torch.from_numpy(synth.normal_rhs(m.n_nodes * k, 8).reshape(m.n_nodes, k)).to("cuda:0")
    live, state = {}, {"sum": 0, "peak": 0, "cap": None}

    def alloc(nbytes, stream):
        if state["cap"] is not None and state["sum"] + nbytes > state["cap"]:
            return 0
        p_ = torch.cuda.caching_allocator_alloc(nbytes, 0, stream)
        live[p_] = nbytes
        state["sum"] += nbytes
        state["peak"] = max(state["peak"], state["sum"])
        return p_

    def release(p_):
        state["sum"] -= live.pop(p_)
        torch.cuda.caching_allocator_delete(p_)

    def solutions(s):
        if not session:
            return s.solve_batch(B)[0]
        ses = Session(s, k)
        ses.admit(list(range(k)), [B[:, j].contiguous() for j in range(k)])
        running = [1]
        while any(running):
            ses.step(2)
            running, infos = ses.poll()
        X = torch.empty_like(B)
        for j in range(k):
            x = torch.zeros(m.n_nodes, dtype=torch.float64, device="cuda:0")
            X[:, j] = ses.retire(j, x)
        ses.close()
        return X

    giamg.set_allocator(alloc, release)
    try:
        X = []
        for capped in (False, True):
            s = Solver(m.coords, m.l2g, p, 2.0, Options(precision=precision))
            after_setup, state["peak"] = state["sum"], 0
            if capped:
                state["cap"] = peak - 1
            X.append(solutions(s))
            peak = state["peak"]
            assert peak > after_setup
            if capped:
                alone, _ = s.solve_batch(B[:, 3:4].contiguous())
                assert torch.equal(alone[:, 0], X[1][:, 3])
            state["cap"] = None
            s.close()
        assert live == {}
    finally:
        giamg.set_allocator()
    assert not torch.equal(X[0], X[1])          # another form ran
    assert torch.all(torch.linalg.norm(X[0] - X[1], dim=0) <= 1e-8 * torch.linalg.norm(X[0], dim=0))
