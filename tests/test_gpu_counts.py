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
