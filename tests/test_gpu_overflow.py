"""GPU: sources whose intensities overflow FP32 give infinities downstream, and no NaN: no term
of a task's sum that the graph does not have takes part in it.  Rows of all lengths (odd ones
are padded), every kernel that holds them, small rings and packed groups.  Where J is finite
it agrees with the FP64 oracle within 1e-5."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

import oracle  # noqa: E402
from synth import workloads as W  # noqa: E402
from synth.directions import direction_set  # noqa: E402


@pytest.mark.parametrize("case,G", [("voronoi", 1), ("voronoi", 3), ("lattice", 1), ("lattice", 2), ("faces", 1), ("wide", 4)])
def test_infinities_stay_infinities(case, G):
    import paper_2207_12848_amd as sw
    if case == "voronoi":
        w = W.small_random(3000, 11, G=G, seed=31)
    elif case == "lattice":
        w = W.lattice_workload(14, direction_set(24)[:5], 1.5, [7, 900], [1.0, 0.5], G=G)
    else:
        w = W.many_faces(33 if case == "faces" else 180, 5, G=G, seed=32)
    C = len(w["kappa"])
    e = np.array(w["emission"], np.float32)
    e[C // 2] = 3e38
    m = w["meshes"][0]  # (a hundredth of its size: intensities ten thousand times as high)
    w = dict(w, emission=e, meshes=[dict(m, face_area=m["face_area"] * 1e-4, cell_volume=m["cell_volume"] * 1e-6)])
    ref = oracle.forward(w)["J"]
    dag = sw.build_dag(w["meshes"], w["dirs"])
    k, e = (torch.tensor(np.asarray(w[x], np.float32), device="cuda") for x in ("kappa", "emission"))
    for kw in (dict(), dict(ring=64, block=256), dict(pack=1)):
        J = sw.forward(dag, k, e, **kw)[0].cpu().numpy()
        assert not np.isnan(J).any() and np.isinf(J).any()
        fin = np.isfinite(J) & (ref > 1e-20)
        assert (np.abs(J - ref)[fin] <= 1e-5 * ref[fin]).all()
    dag.close()
