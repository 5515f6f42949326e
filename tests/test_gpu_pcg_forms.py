"""Jacobi-PCG on both sides of the lines between its forms (the update that
sums the copies of a node itself, one or two copies a thread; the direction
update inside the spread and the column operator), with ragged last blocks,
against the oracle's PCG: iterations within 2, solution within 1e-9 of its
largest value at a residual of 1e-12 (the bounds of the solver's tests)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from oracle import solvers  # noqa: E402
from paper_2104_05829_amd import Sem, inputs  # noqa: E402

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


def _dev(a):
    return torch.tensor(a, dtype=torch.float64, device="cuda")


# up to and above 2^16 (copies per thread), 2^17 (spread operator) and 2^18
# points (own sums), orders wider than a wavefront, several planes a thread
CASES = [(7, (5, 5, 5)), (7, (6, 5, 5)), (7, (6, 6, 8)), (7, (8, 8, 8)), (7, (9, 8, 8)), (3, (9, 9, 9)),
         (2, (7, 6, 5)), (4, (9, 11, 11)), (9, (3, 3, 3)), (11, (4, 4, 3)), (12, (3, 2, 2)), (6, (7, 7, 6))]


@pytest.mark.parametrize("N,shape", CASES)
@pytest.mark.parametrize("check_every", [1, 8])
def test_pcg_matches_oracle(N, shape, check_every):
    print(f"[gpu] pcg forms N={N} {shape} every={check_every}", flush=True)
    xi, _ = oracle.gll(N)
    m = inputs.box_mesh(*shape, xi, deform="cyclic", amp=0.05)
    lv = solvers.Level(N, m.x, m.y, m.z, m.gid, m.dirichlet, 1.0, 10.0)
    b = lv.rhs(inputs.gaussian_per_node(m.gid, 30))
    xo, ito, _ = solvers.pcg_jacobi(lv, b, tol=1e-12)
    s = Sem(m)
    x, st, rc = s.solve(_dev(b), tol=1e-12, h2=10.0, check_every=check_every, maxit=5000)
    assert rc == 0 and st["converged"] and abs(st["iters"] - ito) <= 2, (st, ito)
    assert np.max(np.abs(x.cpu().numpy() - xo)) <= 1e-9 * np.max(np.abs(xo))
    # the allocation-free form takes the same kernels, lockstep rows the same records
    xn, stn, _ = s.solve_noalloc(_dev(b), torch.zeros_like(x), tol=1e-12, h2=10.0, maxit=5000,
                                 check_every=check_every)
    assert torch.equal(x, xn) and st["iters"] == stn["iters"]
    X, sts, _ = s.solve_multi(torch.stack([_dev(b), _dev(-b)]), tol=1e-12, h2=10.0, maxit=5000,
                              check_every=check_every)
    assert torch.equal(X[0], x) and torch.equal(X[1], -x) and sts[0]["iters"] == st["iters"]
    s.free()


def test_maxit_and_small_steps():
    """The limit falls inside a batch, at its end and after it."""
    print("[gpu] pcg maxit", flush=True)
    xi, _ = oracle.gll(7)
    m = inputs.box_mesh(3, 3, 3, xi)
    lv = solvers.Level(7, m.x, m.y, m.z, m.gid, m.dirichlet, 1.0, 0.0)
    b = lv.rhs(inputs.gaussian_per_node(m.gid, 3))
    s = Sem(m)
    ref = {}
    for maxit in (1, 2, 7, 8, 9, 16, 17):
        for every in (1, 3, 8):
            x, st, rc = s.solve(_dev(b), tol=1e-14, maxit=maxit, check_every=every)
            assert rc == -4 and st["iters"] == maxit, (maxit, every, st)
            assert torch.equal(x, ref.setdefault(maxit, x)), (maxit, every)
        xo, ito, _ = solvers.pcg_jacobi(lv, b, tol=1e-14, maxit=maxit)
        assert np.max(np.abs(ref[maxit].cpu().numpy() - xo)) <= 1e-10 * np.max(np.abs(xo))
    s.free()


@pytest.mark.parametrize("precond", ["jacobi", "pmg"])
def test_multiplicity_beyond_a_byte(precond):
    """300 coincident elements: the counting weight no longer fits a byte and
    is read in full (8 of its copies beyond 255 would lose 15% of each sum)."""
    print(f"[gpu] pcg 300 copies {precond}", flush=True)
    xi, _ = oracle.gll(3)
    one = inputs.box_mesh(1, 1, 1, xi)
    rep = lambda a: np.repeat(a, 300, axis=0)  # noqa: E731
    m = inputs.BoxMesh(N=3, shape=(300, 1, 1), x=rep(one.x), y=rep(one.y), z=rep(one.z), gid=rep(one.gid),
                       dirichlet=rep(one.dirichlet))
    lv = solvers.Level(3, m.x, m.y, m.z, m.gid, m.dirichlet, 1.0, 10.0)
    b = lv.rhs(inputs.gaussian_per_node(m.gid, 5))
    xo, _, _ = solvers.pcg_jacobi(lv, b, tol=1e-13)
    s = Sem(m, levels=(3, 1))
    x, st, rc = s.solve(_dev(b), tol=1e-12, h2=10.0, precond=precond)
    assert rc == 0 and np.max(np.abs(x.cpu().numpy() - xo)) <= 1e-9 * np.max(np.abs(xo)), st
    s.free()
