"""GPU parity of slices that hold several very long rows, forward and adjoint.

Groups of cells that all border each other, side by side in one mesh: every level has a
task of each group that reaches it, with rows of up to n - 1 entries.  The pairs past a
row's first two or eight are taken 64 at a time, so that columns end at, before and behind
them, down to the longest row alone.  Tolerances as in test_gpu_slices, and the same bits
with a ring of 64 results (older ones from memory) and every packing."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from synth import workloads as W  # noqa: E402
from tests.test_gpu_rows import _join  # noqa: E402
from tests.test_gpu_slices import check  # noqa: E402


@pytest.mark.parametrize("sizes,G", [((61, 61, 61), 1), ((40, 80, 120, 160), 1), ((33, 34, 35, 36, 37, 200), 2),
                                     ((17, 90, 90, 91), 3), ((70,) * 9, 4), ((320, 150), 1), ((161, 18), 5)])
def test_several_long_rows(sizes, G):
    parts = [W.many_faces(n, 6, G=G, seed=300 + k) for k, n in enumerate(sizes)]
    w = parts[0]
    mesh = w["meshes"][0]
    for p in parts[1:]:
        mesh = _join(mesh, p["meshes"][0])
    w = dict(w, meshes=[mesh], **{k: np.concatenate([p[k] for p in parts]) for k in ("kappa", "emission")})
    check(w, [dict(ring=64, block=256), dict(pack=1), dict(pack=min(G, 4), ring=128)])
