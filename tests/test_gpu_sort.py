"""GPU: the levels' order at the widths where the way of sorting changes.

A lattice of n^3 cells swept along an axis has n levels of n^2 cells: one, two and four
cells per lane of a wavefront (up to 64, 128 and 256 cells), and by the workgroup above.
The depths are the lattice's planes and J agrees with the FP64 oracle within 1e-5 per
cell and in L1, as in test_gpu_parity."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

import oracle  # noqa: E402
from synth import workloads as W  # noqa: E402


@pytest.mark.parametrize("n", [7, 8, 9, 11, 12, 16, 17])
def test_levels_along_an_axis(n):
    import paper_2207_12848_amd as sw
    dirs = np.concatenate([np.eye(3), -np.eye(3)])
    w = W.lattice_workload(n, dirs, 1.5, [n // 2 + n * (n // 2 + n * (n // 2)), 0], [1.0, 0.5], G=1)
    dag = sw.build_dag(w["meshes"], w["dirs"])
    assert set(np.asarray(dag.depths()).ravel().tolist()) == {n}
    k, e = (torch.tensor(np.asarray(w[x], np.float32), device="cuda") for x in ("kappa", "emission"))
    J = sw.forward(dag, k, e, check=True)[0].cpu().numpy()
    ref = oracle.forward(w)["J"]
    assert np.abs(J - ref).sum() <= 1e-5 * np.abs(ref).sum()
    assert (np.abs(J - ref) <= 1e-5 * np.abs(ref) + 1e-25 * ref.max()).all()
    dag.close()
