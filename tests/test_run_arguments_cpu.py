"""Argument checks of the native loops that need no GPU: what a run is given is checked
before anything is enqueued.  Only the checks run here, on host tensors."""
import numpy as np
import pytest
import torch

api = pytest.importorskip("paper_2506_02486_amd.api")


class _Device(torch.Tensor):
    """A host tensor that calls itself a device tensor (nothing reads it here)."""
    is_cuda = True


def _device(t):
    return t.as_subclass(_Device)


def _struct(rec_off, traces, plane=None, nt=5):
    g = api.Grid(9, 8, 7)
    vol = [_device(g.zeros("cpu")) for _ in range(4)]
    return api._run_struct(g, *vol, None, nt, None, None, rec_off, traces, None, None, plane, "run")


def test_traces_and_offsets_must_be_on_the_device():
    off, tr = torch.arange(3), torch.zeros((5, 3))
    assert _struct(_device(off), _device(tr))[0].nrec == 3
    for o, t in ((off, _device(tr)), (_device(off), tr), (off, tr)):
        with pytest.raises(TypeError):
            _struct(o, t)


def test_plane_map_must_be_that_of_the_receivers():
    off, tr = _device(torch.arange(3)), _device(torch.zeros((5, 3)))
    m = _device(torch.full((9 * 8,), -1, dtype=torch.int32))
    assert _struct(off, tr, api.ReceiverPlane(m, 2, 3))[0].rec_k == 2
    with pytest.raises(TypeError):
        _struct(off, tr, api.ReceiverPlane(m, 2, 4))


def test_other_receivers_drop_the_plane_map_of_the_old_ones():
    sim = api.Simulation.__new__(api.Simulation)
    sim.rec_off = torch.arange(3)
    sim.rec_plane = api.ReceiverPlane(torch.zeros(1, dtype=torch.int32), 0, 3)
    sim.rec_off = torch.arange(3)
    assert sim.rec_plane is None and sim.nrec == 3


def test_host_side_of_a_step():
    """Addresses of host arrays of every kind, and the faces' checks, made on each call
    against sizes that a grid works out once."""
    w = np.arange(4, dtype=np.float32)
    fixed = w.copy()
    fixed.flags.writeable = False
    for a in (w, w[1:], fixed, np.empty(0, np.float32)):
        assert api._address(a) == a.ctypes.data
    g = api.Grid(9, 8, 7)
    faces = [_device(f) for f in api.face_buffers(g, "cpu")]
    faces[3] = None
    for _ in range(2):
        assert [p for p in api._faces(faces, g)] == [f if f is None else f.data_ptr()
                                                     for f in faces]
    for i in (0, 5):
        bad = list(faces)
        for f in (faces[i][:-1], faces[i].double(), torch.zeros(g.face_elems(i))):
            bad[i] = f
            with pytest.raises(TypeError):
                api._faces(bad, g)
    with pytest.raises(ValueError):
        api._faces(faces[:5], g)


@pytest.mark.gpu
@pytest.mark.parametrize("mode", api.Simulation.MODES)
def test_host_traces_are_refused(mode):
    n = 24
    rec = np.array([[3, 4, 5], [6, 4, 5]], np.int32)
    sim = api.Simulation(np.full((n, n, n), 2000.0, np.float32), exchange="loopback",
                         geom=api.Geometry(src=(9, 9, 9), rec=rec))
    with pytest.raises(TypeError):
        sim.run(4, traces=torch.zeros((4, 2)), mode=mode)
