"""GPU: slices whose rows are far longer than everything else's, while the other wavefronts
wait.  64 hubs that each border every one of L leaves: level 0 is the leaves, level 1 one
slice of 64 rows of L entries.  The leaves' phi is S / (A + kappa V), a hub's
(sum of w phi + S) / (kappa V) (nothing leaves it along the direction), in FP64; summation in
FP32 over L terms allows L 2^-24 relative, and no wait may give up."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def _hubs(H, L, rng):
    a = np.arange(L * H)
    area = rng.random(L * H) + 0.5
    hub_twin = (a % L) * H + a // L
    nrm = np.zeros((2 * L * H, 3))
    nrm[:L * H, 0], nrm[L * H:, 0] = 1.0, -1.0
    return dict(face_ptr=np.concatenate([np.arange(L + 1) * H, L * H + np.arange(1, H + 1) * L]),
                face_nbr=np.concatenate([a % H + L, a % L]).astype(np.int32),
                face_twin=np.concatenate([L * H + (a % H) * L + a // H, hub_twin]).astype(np.int32),
                face_area=np.concatenate([area, area[hub_twin]]), face_normal=nrm,
                cell_volume=rng.random(H + L) + 0.5), area.reshape(L, H)


@pytest.mark.parametrize("L,G", [(3000, 1), (3001, 3), (20000, 1), (20000, 4)])
def test_hubs(L, G):
    import paper_2207_12848_amd as sw
    H = 64
    rng = np.random.default_rng(L)
    mesh, area = _hubs(H, L, rng)
    k, e = (rng.random((H + L, G)).astype(np.float32) + np.float32(0.1) for _ in range(2))
    dag = sw.build_dag([mesh], np.array([[1.0, 0.0, 0.0]]))
    J = sw.forward(dag, torch.tensor(k, device="cuda"), torch.tensor(e, device="cuda"), check=True, pack=G)[0]
    kV = k.astype(np.float64) * mesh["cell_volume"][:, None]
    phi = e[:L] / (area.sum(1)[:, None] + kV[:L])
    phi = np.concatenate([phi, (area.T @ phi + e[L:]) / kV[L:]]) / (4 * np.pi)
    assert np.allclose(J.cpu().numpy(), phi, rtol=L * 2.0 ** -24 + 1e-6, atol=0.0)
    dag.close()
