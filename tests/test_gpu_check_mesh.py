"""Every condition of the mesh check, violated once somewhere in a valid periodic mesh: the
build is refused with the message that names it; the valid mesh passes, and so does one
whose normals are off by less than the bound."""
import numpy as np
import pytest

pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from synth import workloads as W  # noqa: E402
from synth.directions import direction_set  # noqa: E402


@pytest.fixture(scope="module")
def mesh():
    return W.uniform_mesh(700, np.random.default_rng(3), periodic=True)


def _build(meshes, **kw):
    import paper_2207_12848_amd as sw
    dag = sw.build_dag(meshes, direction_set(8), **kw)
    n = dag.info()["n_cells"]
    dag.close()
    return n


def _broken(mesh, kind):
    m = {k: (v.copy() if isinstance(v, np.ndarray) else v) for k, v in mesh.items()}
    f = 4321  # a face of a cell in the middle
    t = int(m["face_twin"][f])
    shifted = int(np.flatnonzero(m["face_shift"])[17])
    if kind == "ptr start":
        m["face_ptr"][0] = 1
    elif kind == "ptr end":
        m["face_ptr"][-1] -= 1
    elif kind == "ptr order":
        m["face_ptr"][300] = m["face_ptr"][302]
    elif kind == "volume":
        m["cell_volume"][699] = 0.0
    elif kind == "volume nan":
        m["cell_volume"][5] = np.nan
    elif kind == "neighbour":
        m["face_nbr"][f] = 700
    elif kind == "neighbour low":
        m["face_nbr"][f] = -2
    elif kind == "area":
        m["face_area"][f] = -1.0
    elif kind == "area inf":
        m["face_area"][f] = np.inf
    elif kind == "normal":
        m["face_normal"][f] *= 1.0 + 1e-8
    elif kind == "twin range":
        m["face_twin"][f] = len(m["face_nbr"])
    elif kind == "twin":
        m["face_twin"][f] = (t + 1) % len(m["face_nbr"])
    elif kind == "twin area":
        m["face_area"][t] *= 1.0 + 1e-15
    elif kind == "twin normal":
        m["face_normal"][t] = m["face_normal"][f]
    elif kind == "shift":
        m["face_shift"][shifted] *= -1
    elif kind == "wall shift":
        m["face_nbr"][shifted] = -1
    return m


@pytest.mark.parametrize("kind,message", [
    ("ptr start", "face_ptr must run"), ("ptr end", "face_ptr must run"), ("ptr order", "not monotone"),
    ("volume", "volume"), ("volume nan", "volume"), ("neighbour", "out of range"),
    ("neighbour low", "out of range"), ("area", "area"), ("area inf", "area"), ("normal", "not unit"),
    ("twin range", "no consistent twin"), ("twin", "no consistent twin"), ("twin area", "equal areas"),
    ("twin normal", "equal areas"), ("shift", "opposite shifts"), ("wall shift", "periodic shift")])
def test_violations_are_named(mesh, kind, message):
    import paper_2207_12848_amd as sw
    with pytest.raises(sw.SweepError, match="INVALID_ARG.*mesh 1.*" + message):
        _build([mesh, _broken(mesh, kind), _broken(mesh, "volume")])


def test_valid_meshes_pass(mesh):
    near = _broken(mesh, "")
    near["face_normal"] *= 1.0 + 0.95e-9  # between the kernel's bound and the host's
    no_twin = {k: v for k, v in near.items() if k != "face_twin"}
    assert _build([mesh, near, no_twin]) == 2100
    assert _build([mesh], scheme="aligned") == 700
