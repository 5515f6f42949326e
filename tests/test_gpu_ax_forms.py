"""The element operator's forms on both sides of the lines between them: the
spread form (few points) against the column form, and a batch of fields
computed inside one wavefront, or by a wavefront each, against single calls.
Tolerance against the oracle: 1e-12 (2-norm, and largest value), the FP64
bound of the operator's parity tests; between forms: equal bits."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from paper_2104_05829_amd import Sem, inputs  # noqa: E402

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

TOL = 1e-12


def _mesh(shape, N):
    xi, _ = oracle.gll(N)
    return inputs.box_mesh(*shape, xi, deform="cyclic", amp=0.05)


# (N, shape): the largest box up to 2^18 points and the next one above, ragged
# last workgroups of the small orders, and orders with several planes a thread
SIDES = [(1, (31, 32, 33)), (1, (33, 32, 32)), (2, (21, 21, 22)), (2, (22, 21, 22)), (3, (16, 16, 16)),
         (3, (16, 16, 17)), (4, (13, 12, 13)), (5, (10, 11, 11)), (5, (11, 10, 12)), (6, (9, 9, 9)),
         (6, (9, 9, 10)), (7, (8, 8, 8)), (7, (8, 8, 9)), (8, (7, 7, 7)), (8, (7, 7, 8)), (9, (1, 1, 1)),
         (9, (6, 6, 8)), (10, (3, 2, 2)), (10, (6, 6, 5)), (10, (6, 6, 6)), (11, (5, 5, 6)), (11, (6, 5, 6)),
         (12, (3, 2, 2)), (13, (2, 2, 2)), (14, (2, 1, 2)), (15, (2, 2, 1))]


@pytest.mark.parametrize("N,shape", SIDES)
@pytest.mark.parametrize("h2,vark", [(0.0, False), (10.0, True)])
def test_forms_match_oracle(N, shape, h2, vark):
    print(f"[gpu] ax forms N={N} {shape} h2={h2} k={vark}", flush=True)
    m = _mesh(shape, N)
    u = inputs.uniform_lvector(m.n_local, 3)
    k = inputs.uniform_lvector(m.n_local, 4, 0.5, 2.0) if vark else None
    G, B, _ = oracle.geometry(N, m.x, m.y, m.z)
    xi, _ = oracle.gll(N)
    ref = oracle.ax(N, oracle.dhat(N, xi), G, u, h1=1.5, h2=h2, B=B, k=k)
    s = Sem(m)
    dev = lambda a: None if a is None else torch.tensor(a, device="cuda")  # noqa: E731
    w = s.ax(dev(u), h1=1.5, h2=h2, k=dev(k)).cpu().numpy()
    s.free()
    assert np.linalg.norm(w - ref) <= TOL * np.linalg.norm(ref)
    assert np.max(np.abs(w - ref)) <= TOL * np.max(np.abs(ref))


@pytest.mark.parametrize("N,shape", [(7, (6, 6, 5)), (7, (8, 8, 8)), (7, (17, 17, 17)), (4, (29, 27, 26)),
                                     (5, (22, 23, 23)), (9, (6, 6, 6))])
@pytest.mark.parametrize("nf", [2, 3, 4])
@pytest.mark.parametrize("f32", [False, True])
def test_batch_equals_single_fields(N, shape, nf, f32):
    """Around 2^18 points over all fields, and around the 2.5 M points from
    which the fields go inside one wavefront."""
    print(f"[gpu] ax batch N={N} {shape} nf={nf} f32={f32}", flush=True)
    s = Sem(_mesh(shape, N), levels=(N, 1))
    g = torch.Generator(device="cuda").manual_seed(5)
    U = torch.rand(nf, s.n_local, generator=g, device="cuda", dtype=torch.float64) * 2 - 1
    if f32:
        U = U.float()
        W = s.ax_level_multi(0, U, h1=1.0, h2=10.0)
        one = [s.ax_level(0, U[q].contiguous(), h1=1.0, h2=10.0) for q in range(nf)]
    else:
        W = s.ax_multi(U, h1=1.0, h2=10.0)
        one = [s.ax(U[q].contiguous(), h1=1.0, h2=10.0) for q in range(nf)]
    for q in range(nf):
        assert torch.equal(W[q], one[q]), q
    s.free()
