"""Error of the FP32 level operator against FP64, set against FP32 arithmetic in
the definition's order: each derivative a chain of fused multiply-adds, and D^T
of the three fluxes one chain of 3 (N + 1) of them (emulated here, every step
rounded to FP32).  Summing each direction by itself leaves the sum of the
partial results' roundings a third as large (chains a third as long, over a
third of the terms each), the rest of the roundings alike: the library has to
stay below the chain, by 5% (the rms over 10^4 points or more is known to 1%)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from paper_2104_05829_amd import Sem, inputs  # noqa: E402

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


def _fma(a, b, c):
    """round(a b + c) to FP32: the product is exact in FP64, and the double
    rounding of the sum is off by at most a part in 2^29."""
    return (a.astype(np.float64) * b + c).astype(np.float32)


def _ax_chain(N, D, G, B, u, h2):
    q = N + 1
    D, G, B = D.astype(np.float32), G.astype(np.float32), B.astype(np.float32)
    u = u.reshape(-1, q, q, q)  # [e][k][j][i]
    z = np.zeros_like(u)
    ur, us, ut = z, z, z
    for l in range(q):
        ur = _fma(D[:, l][None, None, None, :], u[..., l:l + 1], ur)
        us = _fma(D[:, l][None, None, :, None], u[:, :, l:l + 1, :], us)
        ut = _fma(D[:, l][None, :, None, None], u[:, l:l + 1], ut)
    g = [c.reshape(u.shape) for c in G]

    def flux(a, b, c):
        return _fma(c, ut, _fma(b, us, (a * ur).astype(np.float32)))

    wr, ws, wt = flux(g[0], g[1], g[2]), flux(g[1], g[3], g[4]), flux(g[2], g[4], g[5])
    acc = z
    for l in range(q):
        acc = _fma(D[l][None, :, None, None], wt[:, l:l + 1], acc)
    for l in range(q):
        acc = _fma(D[l][None, None, None, :], wr[..., l:l + 1], acc)
        acc = _fma(D[l][None, None, :, None], ws[:, :, l:l + 1, :], acc)
    if h2:
        acc = _fma((np.float32(h2) * B).astype(np.float32).reshape(u.shape), u, acc)
    return acc.reshape(-1)


# one element a workgroup and several, the column form by planes and in two
# phases, the spread form
@pytest.mark.parametrize("N,shape", [(2, (22, 21, 23)), (3, (9, 10, 8)), (3, (27, 26, 27)), (4, (8, 9, 8)),
                                     (4, (14, 14, 13)), (5, (6, 7, 6)), (5, (12, 11, 13)), (5, (20, 18, 17)),
                                     (6, (6, 7, 6)), (6, (10, 10, 11)), (7, (5, 6, 5)), (7, (9, 9, 9)),
                                     (8, (5, 5, 4)), (8, (9, 8, 9)), (9, (6, 7, 7)), (11, (4, 4, 4)),
                                     (11, (7, 7, 6)), (15, (3, 3, 4))])
@pytest.mark.parametrize("h2", [0.0, 10.0])
def test_fp32_error_below_the_plain_chain(N, shape, h2):
    print(f"[gpu] ax f32 N={N} {shape} h2={h2}", flush=True)
    xi, _ = oracle.gll(N)
    m = inputs.box_mesh(*shape, xi, deform="cyclic", amp=0.05)
    u = inputs.uniform_lvector(m.n_local, 7).astype(np.float32)
    G, B, _ = oracle.geometry(N, m.x, m.y, m.z)
    D = oracle.dhat(N, xi)
    exact = oracle.ax(N, D, G, u.astype(np.float64), h1=1.0, h2=h2, B=B)
    chain = _ax_chain(N, D, G, B, u, h2)
    s = Sem(m, levels=(N, 1))
    w = s.ax_level(0, torch.tensor(u, device="cuda"), h1=1.0, h2=h2).cpu().numpy()
    s.free()
    got = np.linalg.norm(w - exact)
    ref = np.linalg.norm(chain - exact)
    print(f"  error / chain {got / ref:.3f} ({got / np.linalg.norm(exact):.2e})", flush=True)
    assert got <= 0.95 * ref
