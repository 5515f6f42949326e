"""The velocity transform where a workgroup takes several elements (up to M = 5 by
their columns in one wavefront, from M = 9 on two side by side): element counts
around the multiples of its 8-apart groups, and grids that loop, against the
oracle, within 1e-12 of the largest value (the bound of the transform's tests)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import advect as adv  # noqa: E402
import oracle  # noqa: E402
from paper_2104_05829_amd import Sem, inputs  # noqa: E402

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

TOL = 1e-12
SMALL = [(769, 1, 1), (13, 10, 6), (7, 37, 3), (8, 16, 7), (32, 32, 1), (1031, 1, 1)]  # 769 .. 1031
PAIRS = [(257, 1, 1), (8, 11, 3), (5, 53, 1), (7, 73, 1), (8, 8, 8), (7, 183, 1), (1289, 1, 1), (12, 16, 8)]
LOOPS = [(1, (50, 41, 67)), (2, (33, 32, 32)), (3, (41, 40, 11)), (6, (13, 12, 11)), (7, (12, 11, 10))]


@pytest.mark.parametrize("N,shape", [(N, s) for N in (1, 2, 3) for s in SMALL]
                         + [(N, s) for N in (6, 7) for s in PAIRS] + [(5, (7, 61, 1)), (5, (8, 8, 8))] + LOOPS)
@pytest.mark.parametrize("more", [0, 1])
def test_velocity_groups_match_oracle(N, shape, more):
    M = (3 * N + 2) // 2 + more
    print(f"[gpu] velocity groups {shape} N={N} M={M}", flush=True)
    xi, _ = oracle.gll(N)
    m = inputs.box_mesh(*shape, xi, deform="cyclic", amp=0.03 / max(shape), bc="neumann")
    rng = np.random.default_rng(19)
    c = rng.standard_normal((3, m.n_local))
    s = Sem(m)
    assert s.advect_setup(M) == M
    ct = torch.full((m.E, 3, M ** 3), float("nan"), dtype=torch.float64, device="cuda")
    s.advect_velocity(torch.tensor(c, device="cuda"), ct)
    s.free()
    assert not bool(torch.isnan(ct).any())  # every element is written
    els = np.unique(np.r_[np.arange(min(m.E, 24)), np.linspace(0, m.E - 1, 24).astype(int), m.E - 1 - np.arange(24)])
    idx = (els[:, None] * (N + 1) ** 3 + np.arange((N + 1) ** 3)[None, :]).reshape(-1)
    ref = adv.conv_velocity(N, M, *[a.reshape(-1)[idx] for a in (m.x, m.y, m.z)],
                            [cd[idx] for cd in c]).reshape(len(els), 3, -1)
    got = ct[torch.tensor(els, device="cuda")].cpu().numpy()
    assert np.max(np.abs(got - ref)) <= TOL * np.max(np.abs(ref))
