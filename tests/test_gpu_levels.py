"""The level computation against the FP64 oracle, bit for bit, in every place its counters
may live: bytes in LDS, 4-bit fields in LDS (meshes whose bytes do not fit; tasks with 15
or more dependencies counted in global memory), the hash table of the cells being
counted (small meshes get small tables, whose buckets overflow into global memory), and
bytes in global memory (more dependencies than the table counts); with levels wider than
the frontier's and the table's lists in LDS."""
import numpy as np
import pytest

pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

import oracle  # noqa: E402
from synth import mesh as M  # noqa: E402
from synth import workloads as W  # noqa: E402
from synth.directions import direction_set  # noqa: E402

AXIS = np.array([[1.0, 0.0, 0.0], [0.0, 0.0, -1.0]])


@pytest.mark.parametrize("case,where,lds", [
    ("uniform", "lds", 1), ("uniform", "global", 0), ("one cell", "global", 0), ("one cell", "auto", 1),
    ("145k", "auto", 1), ("wide", "auto", 1), ("wide", "global", 0), ("many faces", "auto", 1),
    ("many faces", "global", 0)])
def test_levels_match_oracle(case, where, lds):
    import paper_2207_12848_amd as sw
    rng = np.random.default_rng(8)
    if case == "uniform":
        mesh, dirs = W.uniform_mesh(3001, rng), direction_set(24)[:7]
    elif case == "one cell":
        mesh, dirs = M.lattice_mesh(1), AXIS
    elif case == "145k":
        mesh, dirs = W.uniform_mesh(150_000, rng), direction_set(24)[:2]
    elif case == "wide":  # 3,136 tasks per level along the axes, up to 2,352 along the diagonals
        mesh, dirs = M.lattice_mesh(56), np.concatenate([AXIS, direction_set(8)[:2]])
    else:
        mesh, dirs = M.complete_graph_mesh(150, 5), direction_set(24)[:3]
    dag = sw.build_dag([mesh], dirs, kahn_counters=where)
    assert dag.info()["kahn_lds_counters"] == lds
    level, order, indeg = (dag.split(x)[0] for x in dag.export())
    rl, ro, ri, rd = oracle.build_dag(mesh, dirs)
    assert np.array_equal(level, rl) and np.array_equal(order, ro) and np.array_equal(indeg, ri)
    assert np.array_equal(dag.depths()[0], rd)
    dag.close()
