"""GPU: areas of faces at the edge of what a mesh may hold.

- without the mesh check, an area that is NaN or negative (on one or both sides of a face,
  interior or wall) leaves the cell without a valid A_perp and the sweep reports it, under
  both transport schemes;
- a face of area -0.0 is one of area 0.0: it carries nothing but orders its two cells, so
  levels, in-degrees and results are the same bits."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from synth import workloads as W  # noqa: E402


def _mesh(areas):
    w = W.small_random(600, 24, seed=71)
    m = dict(w["meshes"][0])
    m["face_area"] = m["face_area"].copy()
    for f, a in areas.items():
        m["face_area"][f] = a
    return w, m


def _fields(w):
    return [torch.tensor(np.asarray(w[x], np.float32), device="cuda") for x in ("kappa", "emission")]


def _face(m, wall):
    """A face of the mesh's largest kind: interior, or on the wall."""
    of = np.where((m["face_nbr"] < 0) == wall)[0]
    return int(of[np.argmax(m["face_area"][of])])


@pytest.mark.parametrize("scheme,value,sides", [("area", float("nan"), 2), ("area", float("nan"), 1), ("area", -1.0, 2),
                                                ("area", -1.0, 1), ("area", float("nan"), 0), ("aligned", float("nan"), 2)])
def test_invalid_areas_are_reported(scheme, value, sides):
    import paper_2207_12848_amd as sw
    _, m = _mesh({})
    f = _face(m, wall=sides == 0)
    bad = {f: value}
    if sides == 2:
        bad[int(m["face_twin"][f])] = value
    w, m = _mesh(bad)
    dag = sw.build_dag([m], w["dirs"], validate=False, scheme=scheme)
    with pytest.raises(sw.SweepError, match="Aperp"):
        sw.forward(dag, *_fields(w), check=True)
    dag.close()
    with pytest.raises(sw.SweepError, match="area"):
        sw.build_dag([m], w["dirs"], validate=True, scheme=scheme)


def test_zero_areas_of_either_sign():
    import paper_2207_12848_amd as sw
    _, m = _mesh({})
    faces = np.where(m["face_nbr"] >= 0)[0][::7]
    faces = np.unique(np.concatenate([faces, m["face_twin"][faces]]))
    got = []
    for zero in (0.0, -0.0):
        w, m = _mesh({int(f): zero for f in faces})
        dag = sw.build_dag([m], w["dirs"])
        k, e = _fields(w)
        J, A, tot, saved = sw.forward(dag, k, e, save_for_adjoint=True, check=True)
        got.append(list(dag.export()) + [x.cpu().numpy() for x in (J, A, tot) + sw.adjoint(dag, k, e, saved, k, e, check=True)])
        dag.close()
    for x, y in zip(*got):
        assert np.array_equal(x, y)
