"""GPU levels, order and in-degrees against the oracle where the counters of large meshes lie:
in global memory with few graphs in flight, in the hash table from about 150 row entries of
all graphs per cell of the largest mesh on (directions x the mean row, for one mesh).  Small meshes with the counters
kept out of LDS by the option, on either side of that line: tables whose buckets overflow,
levels wider than the frontier's and the table's lists, cells of more dependencies than the
table counts.  Bit-exact."""
import numpy as np
import pytest

pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

import oracle  # noqa: E402
from synth import mesh as M  # noqa: E402
from synth import workloads as W  # noqa: E402
from synth.directions import direction_set  # noqa: E402
from tests.test_gpu_rows import _join  # noqa: E402


@pytest.mark.parametrize("case,copies,D", [("uniform", 1, 1), ("uniform", 1, 19), ("uniform", 1, 20), ("uniform", 1, 24),
                                           ("uniform", 6, 7), ("wide", 1, 3), ("wide", 14, 4), ("lattice", 1, 48),
                                           ("lattice", 1, 60), ("big 124", 1, 24), ("big 255", 1, 24), ("big 255", 3, 8)])
def test_levels_on_either_side(case, copies, D):
    import paper_2207_12848_amd as sw
    rng = np.random.default_rng(9)
    if case == "uniform":
        mesh = W.uniform_mesh(3001, rng)
    elif case == "lattice":
        mesh = M.lattice_mesh(12)
    elif case == "wide":  # up to 2,352 tasks per level
        mesh = M.lattice_mesh(56)
    else:
        mesh = _join(W.uniform_mesh(2500, rng), M.complete_graph_mesh(int(case.split()[1]), 5))
    dirs = direction_set(84)[:D] if D > 8 else direction_set(8)[:D]
    dag = sw.build_dag([mesh] * copies, dirs, kahn_counters="global")
    rl, ro, ri, rd = oracle.build_dag(mesh, dirs)
    for level, order, indeg, depth in zip(*(dag.split(x) for x in dag.export()), dag.depths()):
        assert np.array_equal(level, rl) and np.array_equal(order, ro) and np.array_equal(indeg, ri)
        assert np.array_equal(depth, rd)
    dag.close()
