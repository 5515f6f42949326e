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
