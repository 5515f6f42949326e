"""Both forms of the Schwarz smoother's element kernel at N = 2 and 3 (matrix
instructions below a number of elements, the vector unit from it on), at counts
of elements that no workgroup's divides: sampled elements (corner, edge, face,
interior) against the oracle's operator on the block of the mesh around each, on
which an element's output depends alone, within the 2e-5 of the largest value that
holds for the smoother elsewhere; and the rows of lockstep solves against the
solves alone, iterations within 1 and solutions within 1e-7 of the largest value
at a residual of 1e-9."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from oracle import asm, solvers  # noqa: E402
from paper_2104_05829_amd import Sem, inputs  # noqa: E402

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


def _mesh(shape, N):
    xi, _ = oracle.gll(N)
    return inputs.box_mesh(*shape, xi, deform="cyclic", amp=0.05)


@pytest.mark.parametrize("variant", ["asm", "ras"])
# 5832, 6137 and 13248 elements
@pytest.mark.parametrize("N,shape", [(2, (17, 19, 19)), (2, (23, 24, 24)), (3, (18, 18, 18)), (3, (17, 19, 19))])
def test_sampled_elements_match_oracle(N, shape, variant):
    print(f"[gpu] schwarz forms N={N} {shape} {variant}", flush=True)
    m = _mesh(shape, N)
    s = Sem(m, levels=(N, 1))
    r32 = (inputs.gaussian_per_node(m.gid, 21) * (1.0 - m.dirichlet.reshape(-1))).astype(np.float32)
    z = s.smoother_apply(0, torch.tensor(r32, device="cuda"), smoother=variant, h1=1.0, h2=10.0).cpu().numpy()
    s.free()
    pts = (N + 1) ** 3
    z, r32 = z.reshape(m.E, pts), r32.reshape(m.E, pts)
    top = [n - 1 for n in shape]
    for c in ((0, 0, 0), (top[0], 0, 5), (7, top[1], 13), (9, 4, 6), tuple(top)):
        box = [range(max(0, i - 2), min(n, i + 3)) for i, n in zip(c, shape)]
        idx = np.array([x + shape[0] * (y + shape[1] * k) for k in box[2] for y in box[1] for x in box[0]])
        x, y, zc, gid, dirichlet = (np.asarray(f)[idx] for f in (m.x, m.y, m.z, m.gid, m.dirichlet))
        lv = solvers.Level(N, x, y, zc, gid, dirichlet, 1.0, 10.0)
        op = asm.Schwarz(lv, tuple(len(b) for b in box), x, y, zc, dirichlet, variant)
        ref = op.apply(r32[idx].reshape(-1).astype(np.float64)).reshape(len(idx), pts)
        e = c[0] + shape[0] * (c[1] + shape[1] * c[2])
        err = np.max(np.abs(z[e] - ref[int(np.nonzero(idx == e)[0][0])])) / np.max(np.abs(ref))
        assert err <= 2e-5, (c, err)


# one vector and three on either side of the line, and both past it
@pytest.mark.parametrize("smoother", ["asm", "ras"])
@pytest.mark.parametrize("N,shape", [(2, (17, 19, 19)), (3, (17, 19, 19)), (2, (25, 25, 27)), (3, (29, 28, 28))])
def test_lockstep_rows_match_single_solves(N, shape, smoother):
    print(f"[gpu] schwarz forms lockstep N={N} {shape} {smoother}", flush=True)
    m = _mesh(shape, N)
    s = Sem(m, levels=(N, 1))
    B = torch.stack([s.rhs(torch.tensor(inputs.gaussian_per_node(m.gid, 90 + r), device="cuda")) for r in range(3)])
    opts = dict(h2=5.0, tol=1e-9, maxit=200, precond="pmg", smoother=smoother, cheb_lo=0.25)
    alone = [s.solve(B[r], **opts) for r in range(3)]
    for nf in (2, 3):
        X, sts, rc = s.solve_multi(B[:nf].contiguous(), **opts)
        assert rc == 0
        for r in range(nf):
            x, st, rc1 = alone[r]
            assert rc1 == 0 and abs(sts[r]["iters"] - st["iters"]) <= 1
            assert (X[r] - x).abs().max() <= 1e-7 * x.abs().max()
    s.free()
