"""Jacobi-PCG of several right-hand sides on meshes on which the operator with the
direction update takes the forms of many elements: a wavefront a field, several
fields a wavefront, workgroups that write several records of partial sums.  Each
row performs the arithmetic of a solve alone, so every iterate is the same to the
last bit, also beside a row that stops early."""
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from paper_2104_05829_amd import Sem, inputs  # noqa: E402

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


# just past 2^17 points (spread form or not), 2^18 (QQ^T inside the update or not) and 2.5 M
@pytest.mark.parametrize("N,shape,fields", [(7, (7, 7, 6), (2, 3, 4)), (7, (9, 8, 8), (2, 3, 4)),
                                            (7, (17, 17, 17), (2, 3, 4)), (6, (20, 19, 20), (2, 3)),
                                            (5, (9, 9, 8), (2, 3, 4)), (5, (23, 23, 22), (2, 3, 4)),
                                            (4, (11, 10, 10), (2, 3)), (4, (28, 27, 27), (2, 3, 4)),
                                            (3, (16, 17, 16), (2, 3)), (3, (34, 34, 34), (2, 3, 4)),
                                            (2, (17, 18, 17), (2, 4)), (2, (46, 45, 45), (2, 3, 4))])
def test_rows_match_single_solves(N, shape, fields):
    print(f"[gpu] pcg fields N={N} {shape}", flush=True)
    xi, _ = oracle.gll(N)
    m = inputs.box_mesh(*shape, xi, deform="cyclic", amp=0.05)
    s = Sem(m)
    B = torch.stack([s.rhs(torch.tensor(inputs.gaussian_per_node(m.gid, 70 + r), device="cuda"))
                     for r in range(max(fields))])
    for h2 in (10.0, 0.0):
        opts = dict(h2=h2, tol=1e-8, maxit=9, check_every=4, raise_on_error=False, zero_guess=0)
        X0 = torch.zeros_like(B)
        # a row that is nearly there and stops before the others do
        X0[1] = s.solve(B[1].contiguous(), h2=h2, tol=1.02e-8, maxit=4000)[0]
        alone = [s.solve(B[r].contiguous(), X0[r].clone(), **opts)[:2] for r in range(max(fields))]
        assert alone[1][1]["iters"] < 9 and alone[0][1]["iters"] == 9
        for nf in fields:
            X, sts, _ = s.solve_multi(B[:nf].contiguous(), X0[:nf].clone(), **opts)
            for r in range(nf):
                assert sts[r]["iters"] == alone[r][1]["iters"] and sts[r]["rel_res"] == alone[r][1]["rel_res"]
                assert torch.equal(X[r], alone[r][0]), (h2, nf, r)
    s.free()
