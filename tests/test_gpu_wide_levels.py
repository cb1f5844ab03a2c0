"""GPU parity of levels nearly as wide as the LDS ring, forward and adjoint.

A lattice of 30^3 cells swept along an axis has levels of 900 tasks, 15 slices.  With a
ring of 1024 results and 4 or 8 wavefronts the last slices of a level find their upwind
results in the ring, the first ones load them early and those between read them from
memory once they are stored: the level mixes all three.  Tolerances as in test_gpu_slices,
and the same bits as with the largest ring."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from synth import workloads as W  # noqa: E402
from tests.test_gpu_slices import check  # noqa: E402


@pytest.mark.parametrize("G", [1, 2, 4])
def test_levels_nearly_as_wide_as_the_ring(G):
    n = 30
    dirs = np.concatenate([np.eye(3), -np.eye(3)])
    w = W.lattice_workload(n, dirs, 1.5, [n // 2 + n * (n // 2 + n * (n // 2)), 0], [1.0, 0.5], G=G)
    check(w, [dict(ring=1024, block=512), dict(ring=1024, block=256), dict(ring=1024, block=512, pack=1)])
