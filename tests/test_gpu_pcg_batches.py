"""Jacobi-PCG batches of iterations: what the host does between them must not
show in the result."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from paper_2104_05829_amd import Sem, inputs  # noqa: E402

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


def _dev(a):
    return torch.tensor(a, dtype=torch.float64, device="cuda")


# every number of lanes that sums the records, the forms on both sides of 2^18 points
@pytest.mark.parametrize("N,shape", [(2, (7, 6, 5)), (3, (9, 9, 9)), (3, (16, 17, 16)), (4, (9, 11, 11)), (4, (13, 13, 14)),
                                     (5, (6, 6, 6)), (5, (10, 11, 12)), (6, (7, 7, 6)), (6, (9, 9, 10)),
                                     (7, (5, 5, 5)), (7, (9, 8, 9)), (9, (5, 5, 5))])
def test_result_does_not_depend_on_check_every(N, shape):
    """Where a batch of iterations ends must not show: the same solution,
    count and residual to the last bit, however often the host looks."""
    print(f"[gpu] pcg check_every N={N} {shape}", flush=True)
    xi, _ = oracle.gll(N)
    m = inputs.box_mesh(*shape, xi, deform="cyclic", amp=0.05)
    s = Sem(m)
    b = s.rhs(_dev(inputs.gaussian_per_node(m.gid, 31)))
    # a residual to compare at many different iterations: ends at a batch's end
    # (1), inside a batch
    for tol in np.geomspace(0.3, 1e-8, 40):
        ref = None
        for every in (1, 7, 64):
            x, st, rc = s.solve(b, tol=float(tol), h2=10.0, check_every=every, maxit=2000)
            got = (st["iters"], st["rel_res"], st["true_rel_res"])
            if ref is None:
                ref = (got, x)
            assert rc == 0 and got == ref[0] and torch.equal(x, ref[1]), (tol, every, got, ref[0])
    s.free()


@pytest.mark.parametrize("case", ["zero", "converged", "maxit"])
def test_no_iterations_past_the_need(case):
    """A right-hand side of zero, a start that has converged and a small maxit
    take no batch of check_every: 20000 iterations of two launches or more
    cannot be enqueued in 20 ms, so 10 ms tell them from the few that are due."""
    print(f"[gpu] pcg no iterations past the need, {case}", flush=True)
    xi, _ = oracle.gll(7)
    m = inputs.box_mesh(4, 4, 4, xi)
    s = Sem(m)
    b = s.rhs(_dev(inputs.gaussian_per_node(m.gid, 4)))
    kw = dict(h2=10.0, check_every=20000, maxit=20000, tol=1e-8, raise_on_error=False)
    x, st, rc = s.solve(b, **dict(kw, check_every=8))
    its = st["iters"]
    assert rc == 0 and its > 20
    for _ in range(3):  # the first call may build what later ones keep
        if case == "zero":
            y, st, rc = s.solve(torch.zeros_like(b), **kw)
            assert rc == 0 and st["iters"] == 0 and not y.any()
        elif case == "converged":
            y, st, rc = s.solve(b, x.clone(), **dict(kw, zero_guess=0, tol=1e-6))
            assert rc == 0 and st["iters"] == 0
        else:
            y, st, rc = s.solve(b, **dict(kw, maxit=3))
            assert rc == -4 and st["iters"] == 3
    assert st["ms_solve"] < 10.0, st
    s.free()


@pytest.mark.parametrize("nf", [1, 3])
def test_batch_lengths_and_limits(nf):
    """maxit before, at and after the ends of batches and of the iterations
    enqueued ahead of the host, rows that end at different iterations: the
    same iterates for every check_every."""
    print(f"[gpu] pcg batch lengths nf={nf}", flush=True)
    xi, _ = oracle.gll(5)
    m = inputs.box_mesh(4, 3, 5, xi, deform="cyclic", amp=0.05)
    s = Sem(m)
    B = torch.stack([s.rhs(_dev(inputs.gaussian_per_node(m.gid, 50 + q))) for q in range(nf)])
    X0 = torch.zeros_like(B)
    if nf > 1:  # a row that has converged, and one that is nearly there
        X0[1], _, _ = s.solve(B[1].contiguous(), h2=10.0, tol=1e-12)
        X0[2], _, _ = s.solve(B[2].contiguous(), h2=10.0, tol=1e-7)
    for maxit in (1, 2, 3, 4, 5, 8, 9, 10, 11, 17, 500):
        ref = None
        for every in (1, 2, 3, 8, 9, 500):
            X, sts, rc = s.solve_multi(B, X0.clone(), h2=10.0, zero_guess=0, tol=1e-9, maxit=maxit,
                                       check_every=every, raise_on_error=False)
            got = [(st["iters"], st["rel_res"], st["converged"]) for st in sts]
            assert all(st["iters"] <= maxit for st in sts) and rc in (0, -4)
            if nf > 1:
                assert sts[1]["iters"] == 0 and (rc == 0) == (maxit == 500)
            if ref is None:
                ref = (got, X)
            assert got == ref[0] and torch.equal(X, ref[1]), (maxit, every, got, ref[0])
    s.free()


@pytest.mark.parametrize("shape,every", [((4, 4, 4), 2), ((4, 4, 4), 8), ((9, 9, 9), 2), ((4, 4, 4), 400)])
def test_timers_leave_the_launch_sequence_alone(shape, every):
    """With timers the host still works ahead of the stream: apart from its look
    at the start (some 20 us) the phases follow each other without a gap, so
    they add up to all but a few percent of a solve of milliseconds.  400: more
    phase boundaries between two looks than the event pool starts with."""
    print(f"[gpu] pcg timers {shape} every={every}", flush=True)
    xi, _ = oracle.gll(7)
    m = inputs.box_mesh(*shape, xi, deform="cyclic", amp=0.05)
    s = Sem(m)
    b = s.rhs(_dev(inputs.gaussian_per_node(m.gid, 8)))
    kw = dict(h2=10.0, tol=1e-9, check_every=every, maxit=2000)
    x0, st0, _ = s.solve(b, **kw)
    part = 0.0
    for _ in range(3):
        x1, st1, _ = s.solve(b, timers=1, **kw)
        assert torch.equal(x0, x1) and st0["iters"] == st1["iters"] and st0["rel_res"] == st1["rel_res"]
        total = st1["ms_ax"] + st1["ms_gs"] + st1["ms_vec"]
        assert min(st1["ms_ax"], st1["ms_gs"], st1["ms_vec"]) > 0.0 and total <= st1["ms_solve"] * 1.05 + 0.05
        part = max(part, total / st1["ms_solve"])
    print(f"  phases {part:.3f} of the solve", flush=True)
    assert part >= 0.85
    s.free()
