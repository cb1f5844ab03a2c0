"""GPU: the totals of the counts (row entries of either walk) over one and many tiles of 32
cells, for both transport schemes: every upwind dependency is an entry of either list, and
the in-degrees are the oracle's."""
import numpy as np
import pytest

pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

import oracle  # noqa: E402
from synth import workloads as W  # noqa: E402
from synth.directions import direction_set  # noqa: E402


@pytest.mark.parametrize("scheme", ["area", "aligned"])
@pytest.mark.parametrize("sizes", [(8,), (32,), (33,), (700, 40, 1500)])
def test_entries_are_counted(scheme, sizes):
    import paper_2207_12848_amd as sw
    rng = np.random.default_rng(len(sizes))
    meshes = [W.uniform_mesh(n, rng) for n in sizes]
    dirs = direction_set(24)[:9]
    dag = sw.build_dag(meshes, dirs, scheme=scheme)
    indeg = dag.export()[2]
    info = dag.info()
    assert info["n_up_entries"] == info["n_down_entries"] == int(indeg.sum(dtype=np.int64))
    if scheme == "area":
        for m, got in zip(meshes, dag.split(indeg)):
            assert np.array_equal(got, oracle.build_dag(m, dirs)[2])
    dag.close()


def test_tiles_of_cells_without_faces():
    """Cells without faces, enough of them for whole tiles: a cell's phi is its source over
    kappa V; the others' results are theirs alone, bit for bit."""
    import torch

    import paper_2207_12848_amd as sw
    w = W.small_random(200, 9, seed=12)
    m = w["meshes"][0]
    n = 100
    more = dict(m, face_ptr=np.concatenate([m["face_ptr"], np.full(n, m["face_ptr"][-1])]),
                cell_volume=np.concatenate([m["cell_volume"], np.full(n, 0.5)]))
    k, e = (np.concatenate([w[x], np.full((n, 1), 0.25, np.float32)]) for x in ("kappa", "emission"))
    out = []
    for mesh, kk, ee in ((m, w["kappa"], w["emission"]), (more, k, e)):
        dag = sw.build_dag([mesh], w["dirs"])
        out.append(sw.forward(dag, *(torch.tensor(x, device="cuda") for x in (kk, ee)), check=True)[0].cpu().numpy())
        dag.close()
    C = len(m["cell_volume"])
    assert np.array_equal(out[1][:C], out[0])
    assert np.allclose(out[1][C:], 0.25 / (0.25 * 0.5) / (4 * np.pi), rtol=1e-6, atol=0.0)
