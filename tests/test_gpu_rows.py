"""GPU parity of rows of very different lengths in one mesh, against the FP64 oracle.

The rows of a slice are assembled in LDS, 32 tasks at a time, with room for about twice
the mesh's mean number of faces per cell; a slice with a wider cell takes 16 tasks at a
time, one that does not fit that way either is written by a lane per row.  A random mesh
of 14.4 faces per cell is joined with cells that all border each other, of `wide` faces on
either side of those lines (28 to 29 and 54 to 56 faces, with the mean); in the last mesh all cells are such.

Tolerances as in test_gpu_parity: J and absorbed within 1e-5 relative per element and in
L1, gradients within 1e-5 in relative L2."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

import oracle  # noqa: E402
from synth import workloads as W  # noqa: E402


def _join(a, b):
    """One mesh of two unconnected ones."""
    n, f = len(a["cell_volume"]), len(a["face_nbr"])
    out = {}
    for k in a:
        x, y = a[k], b.get(k)
        if not isinstance(x, np.ndarray) or y is None:
            continue
        if k == "face_ptr":
            out[k] = np.concatenate([x, y[1:] + f])
        elif k == "face_nbr":
            out[k] = np.concatenate([x, np.where(y >= 0, y + n, y)]).astype(x.dtype)
        elif k == "face_twin":
            out[k] = np.concatenate([x, np.where(y >= 0, y + f, y)]).astype(x.dtype)
        else:
            out[k] = np.concatenate([x, y])
    return out


@pytest.mark.parametrize("cells,wide", [(2000, 28), (2000, 29), (2000, 30), (2000, 56), (2000, 57), (700, 120), (0, 260)])
def test_rows_of_mixed_lengths(cells, wide):
    import paper_2207_12848_amd as sw
    w = W.many_faces(wide - 5, 6, G=1, seed=wide)  # (five of a cell's faces are walls)
    if cells > 0:
        r = W.small_random(cells, 6, G=1, seed=cells)
        w = dict(r, meshes=[_join(r["meshes"][0], w["meshes"][0])],
                 **{k: np.concatenate([r[k], w[k]]) for k in ("kappa", "emission")})
    dag = sw.build_dag(w["meshes"], w["dirs"])
    k, e = (torch.tensor(np.asarray(w[x], np.float32), device="cuda") for x in ("kappa", "emission"))
    gJ = torch.rand(k.shape, generator=torch.Generator().manual_seed(3)).cuda()
    J, A, _, saved = sw.forward(dag, k, e, save_for_adjoint=True, check=True)
    dk, de = sw.adjoint(dag, k, e, saved, gJ, gJ, check=True)
    ref = oracle.forward(w)
    for x, r in ((J, ref["J"]), (A, ref["absorbed"])):
        x = x.cpu().numpy()
        big = np.abs(r) >= 1e-20 * np.abs(r).max()
        assert (np.abs(x - r)[big] / np.abs(r[big])).max() <= 1e-5
        assert np.abs(x - r).sum() <= 1e-5 * np.abs(r).sum()
    g = gJ.cpu().numpy()
    for x, r in zip((dk, de), oracle.adjoint(w, g, g)):
        assert np.linalg.norm(x.cpu().numpy() - r) <= 1e-5 * np.linalg.norm(r)
    dag.close()


@pytest.mark.parametrize("G", [1, 2, 3])
@pytest.mark.parametrize("n", [3, 5, 6, 8, 9, 10, 12, 13, 14, 16, 17])
def test_row_lengths_of_the_sweep_kernels(n, G):
    """Rows of up to n - 1 entries: the sweep holds two or eight pairs of entries per row in
    registers and sums the first four, six or eight."""
    import paper_2207_12848_amd as sw
    w = W.many_faces(n, 5, G=G, seed=200 + n)
    dag = sw.build_dag(w["meshes"], w["dirs"])
    k, e = (torch.tensor(np.asarray(w[x], np.float32), device="cuda") for x in ("kappa", "emission"))
    g = torch.ones_like(k)
    J, _, _, saved = sw.forward(dag, k, e, save_for_adjoint=True, check=True)
    dk, de = sw.adjoint(dag, k, e, saved, g, g, check=True)
    ref = oracle.forward(w)["J"]
    assert np.abs(J.cpu().numpy() - ref).sum() <= 1e-5 * np.abs(ref).sum()
    for x, r in zip((dk, de), oracle.adjoint(w, g.cpu().numpy(), g.cpu().numpy())):
        assert np.linalg.norm(x.cpu().numpy() - r) <= 1e-5 * np.linalg.norm(r)
    dag.close()
