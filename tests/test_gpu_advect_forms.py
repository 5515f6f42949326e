"""The velocity transform on both sides of the line between its forms (few
elements: three lane groups of an element share the fields and the points; many:
one field after the other), at every order and Gauss rule, on 16 elements spread
over the mesh against the oracle, within 1e-12 of the largest value (the bound of
the transform's other tests)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import advect as adv  # noqa: E402
import oracle  # noqa: E402
from paper_2104_05829_amd import Sem, inputs  # noqa: E402

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

TOL = 1e-12


@pytest.mark.parametrize("shape", [(1, 1, 1), (8, 8, 8), (9, 19, 3)])
@pytest.mark.parametrize("N,more", [(1, 0), (1, 1), (2, 0), (3, 1), (4, 0), (5, 0), (5, 1), (6, 0), (6, 1),
                                    (7, 0), (7, 1)])
def test_velocity_forms_match_oracle(shape, N, more):
    M = (3 * N + 2) // 2 + more
    print(f"[gpu] velocity forms {shape} N={N} M={M}", flush=True)
    xi, _ = oracle.gll(N)
    m = inputs.box_mesh(*shape, xi, deform="cyclic", amp=0.03, bc="neumann")
    rng = np.random.default_rng(17)
    c = rng.standard_normal((3, m.n_local))
    s = Sem(m)
    assert s.advect_setup(M) == M
    ct = s.advect_velocity(torch.tensor(c, device="cuda")).cpu().numpy()
    els = np.unique(np.linspace(0, m.E - 1, 16).astype(int))
    idx = (els[:, None] * (N + 1) ** 3 + np.arange((N + 1) ** 3)[None, :]).reshape(-1)
    ref = adv.conv_velocity(N, M, *[a.reshape(-1)[idx] for a in (m.x, m.y, m.z)],
                            [cd[idx] for cd in c]).reshape(len(els), 3, -1)
    assert np.max(np.abs(ct[els] - ref)) <= TOL * np.max(np.abs(ref))
    s.free()
