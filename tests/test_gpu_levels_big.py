"""GPU levels, order and in-degrees against the oracle with the counters in the hash table and
some cells of more dependencies than its counts hold (123): a random mesh joined with n cells
that all border each other, whose in-degrees run to n - 1.  Bit-exact."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

import oracle  # noqa: E402
from synth import mesh as M  # noqa: E402
from synth import workloads as W  # noqa: E402
from synth.directions import direction_set  # noqa: E402
from tests.test_gpu_rows import _join  # noqa: E402


@pytest.mark.parametrize("n", [124, 125, 180, 255])
def test_levels_with_many_dependencies(n):
    import paper_2207_12848_amd as sw
    mesh = _join(W.uniform_mesh(2500, np.random.default_rng(n)), M.complete_graph_mesh(n, 5))
    dirs = direction_set(24)[:4]
    dag = sw.build_dag([mesh], dirs, kahn_counters="global")
    level, order, indeg = (dag.split(x)[0] for x in dag.export())
    rl, ro, ri, rd = oracle.build_dag(mesh, dirs)
    assert ri.max() == n - 1
    assert np.array_equal(level, rl) and np.array_equal(order, ro) and np.array_equal(indeg, ri)
    assert np.array_equal(dag.depths()[0], rd)
    dag.close()
