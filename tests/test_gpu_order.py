"""GPU: the order within levels, as the device made it, at the widths where the way of sorting
changes: one, two and four cells per lane of a wavefront (up to 64, 128 and 256 cells), the
workgroup (up to 4,096) and wider levels, which are left as they are and sorted for the
export.  Lattices swept along an axis (n levels of n^2 cells) and their diagonals, several
graphs at once; levels and order bit for bit as the oracle's, J within 1e-5 of it."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

import oracle  # noqa: E402
from synth import workloads as W  # noqa: E402
from synth.directions import direction_set  # noqa: E402


@pytest.mark.parametrize("n", [1, 2, 7, 8, 9, 11, 12, 16, 17, 33, 63, 64, 65])
def test_order_within_levels(n):
    import paper_2207_12848_amd as sw
    dirs = np.concatenate([np.eye(3), -np.eye(3), direction_set(8)[:1]])[:2 if n > 40 else None]
    w = W.lattice_workload(n, dirs, 1.5, [n // 2 + n * (n // 2 + n * (n // 2)), 0], [1.0, 0.5], G=1)
    dag = sw.build_dag(w["meshes"], w["dirs"])
    level, order, indeg = (dag.split(x)[0] for x in dag.export())
    rl, ro, ri, rd = oracle.build_dag(w["meshes"][0], w["dirs"])
    assert np.array_equal(order, ro)
    assert np.array_equal(level, rl) and np.array_equal(indeg, ri) and np.array_equal(dag.depths()[0], rd)
    k, e = (torch.tensor(np.asarray(w[x], np.float32), device="cuda") for x in ("kappa", "emission"))
    J = sw.forward(dag, k, e, check=True)[0].cpu().numpy()
    ref = oracle.forward(w)["J"]
    assert np.abs(J - ref).sum() <= 1e-5 * np.abs(ref).sum()
    assert (np.abs(J - ref) <= 1e-5 * np.abs(ref) + 1e-25 * ref.max()).all()
    dag.close()
