"""GPU: calls of different numbers of groups on one DAG, queued on a stream of their own
without waiting in between, give the bits that they give one at a time.  (The tables of the
reductions depend on the number of groups.)"""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

import numpy as np  # noqa: E402
from synth import workloads as W  # noqa: E402


@pytest.mark.parametrize("groups", [(1, 2), (3, 1, 2), (5, 4, 7)])
def test_queued_calls_of_different_groups(groups):
    import paper_2207_12848_amd as sw
    w = W.small_random(20000, 24, seed=5, n_meshes=3)
    C = len(w["kappa"])
    rng = np.random.default_rng(6)
    fields = {G: [torch.tensor(rng.random((C, G), dtype=np.float32), device="cuda") for _ in range(2)] for G in groups}
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        dag = sw.build_dag(w["meshes"], w["dirs"])

        def call(G):
            k, e = fields[G]
            J, A, tot, saved = sw.forward(dag, k, e, save_for_adjoint=True, albedo=0.5, n_scat=3)
            return (J, A, tot) + sw.adjoint(dag, k, e, saved, k, e, albedo=0.5, n_scat=3)
        alone = {}
        for G in groups:
            alone[G] = call(G)
            dag.sync()
        queued = [(G, call(G)) for _ in range(4) for G in groups]
        dag.sync()
    for G, out in queued:
        for x, y in zip(out, alone[G]):
            assert torch.equal(x, y)
    dag.close()
