"""GPU parity of the sweep's slices at their edges, forward and adjoint against the FP64 oracle:

- levels of exactly one slice (64 tasks), one task more, many slices, and levels
  wider than the LDS ring (a lattice swept along an axis has levels of n^2 tasks);
- rows of up to 16 entries (held in registers), a few more (taken from the lanes
  that hold the rest of the slice), more than 64 pairs of rest in a slice (summed
  from memory) and more than 64 entries per row (placed by a second look at the
  faces), on meshes in which every cell borders every other;
- every packing of the groups, odd group counts, and workgroups of 4 to 16 wavefronts.

Tolerances as in test_gpu_parity: J and absorbed within 1e-5 relative per element and
in L1, gradients within 1e-5 in relative L2 and elementwise 1e-4 relative + 1e-6 of the
largest.  Every launch shape gives the same bits."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

import oracle  # noqa: E402
from synth import workloads as W  # noqa: E402
from synth.directions import direction_set  # noqa: E402


def run(w, **kw):
    import paper_2207_12848_amd as sw
    dag = sw.build_dag(w["meshes"], w["dirs"])
    k = torch.tensor(np.asarray(w["kappa"], np.float32), device="cuda")
    e = torch.tensor(np.asarray(w["emission"], np.float32), device="cuda")
    rng = np.random.default_rng(17)
    gJ = torch.tensor(rng.random(k.shape, dtype=np.float32), device="cuda")
    gA = torch.tensor(rng.random(k.shape, dtype=np.float32), device="cuda")
    J, A, tot, saved = sw.forward(dag, k, e, save_for_adjoint=True, check=True, **kw)
    dk, de = sw.adjoint(dag, k, e, saved, gJ, gA, check=True, **kw)
    dag.close()
    return [x.cpu().numpy() for x in (J, A, dk, de)], gJ.cpu().numpy(), gA.cpu().numpy()


def check(w, shapes):
    got, gJ, gA = run(w)
    ref = oracle.forward(w)
    for x, r in ((got[0], ref["J"]), (got[1], ref["absorbed"])):
        big = np.abs(r) >= 1e-20 * np.abs(r).max()
        assert (np.abs(x - r)[big] / np.abs(r[big])).max() <= 1e-5
        assert np.abs(x - r).sum() <= 1e-5 * np.abs(r).sum()
    for x, r in zip(got[2:], oracle.adjoint(w, gJ, gA)):
        assert np.linalg.norm(x - r) <= 1e-5 * np.linalg.norm(r)
        assert (np.abs(x - r) - (1e-4 * np.abs(r) + 1e-6 * np.abs(r).max())).max() <= 0.0
    for kw in shapes:
        for x, y in zip(run(w, **kw)[0], got):
            assert np.array_equal(x, y), kw


@pytest.mark.parametrize("n,G", [(2, 1), (8, 1), (8, 3), (9, 2), (40, 4)])
def test_levels_of_one_and_many_slices(n, G):
    dirs = np.concatenate([np.eye(3), -np.eye(3), direction_set(24)[:5]])
    w = W.lattice_workload(n, dirs, 1.5, [n // 2 + n * (n // 2 + n * (n // 2)), 0], [1.0, 0.5], G=G)
    check(w, [dict(ring=64, block=256), dict(ring=1024, block=512)])


@pytest.mark.parametrize("n,G", [(18, 1), (26, 2), (60, 5), (80, 1), (150, 1)])
def test_long_rows(n, G):
    w = W.many_faces(n, 8, G=G, seed=n)
    check(w, [dict(ring=64, block=256), dict(pack=1), dict(pack=min(G, 3))])


@pytest.mark.parametrize("G,block", [(1, 256), (1, 1024), (2, 256), (4, 512)])
def test_workgroup_sizes(G, block):
    w = W.small_random(5000, 11, G=G, seed=90 + G)
    check(w, [dict(block=block), dict(block=block, ring=256), dict(form="plain"), dict(grid=1)])
