"""Model preparation at the edges of its launches (fd_cfl_dt, fd_prepare_vdt2(_m)): rows
shorter and longer than a wave, axes shorter than the halo, extremes on the last point."""
import numpy as np
import pytest
import torch

from workloads import random_field

pytestmark = pytest.mark.gpu

api = pytest.importorskip("paper_2506_02486_amd.api")

SHAPES = [(1, 1, 1), (3, 5, 2), (60, 4, 9), (61, 3, 33), (64, 33, 1), (257, 6, 13), (130, 70, 21)]


def _box(v):
    """v on [-4, n+4)^3: face halos from the periodic image, edges and corners 0."""
    nz, ny, nx = v.shape
    out = np.zeros((nz + 8, ny + 8, nx + 8))
    ax = [np.arange(-4, n + 4) for n in v.shape]
    inside = [(a >= 0) & (a < n) for a, n in zip(ax, v.shape)]
    full = v[np.ix_(*[a % n for a, n in zip(ax, v.shape)])]
    outside = ((~inside[0]).astype(int)[:, None, None] + (~inside[1]).astype(int)[None, :, None]
               + (~inside[2]).astype(int)[None, None, :])
    return np.where(outside <= 1, full, out)


@pytest.mark.parametrize("shape", SHAPES)
def test_vdt2_and_max(shape):
    nx, ny, nz = shape
    g = api.Grid(nx, ny, nz)
    v = (3000 + 400 * random_field((nz, ny, nx), 7)).astype(np.float32)
    dt = 7.3e-4
    for corner in (0, -1):  # the largest velocity on the first and on the last point
        v.flat[corner] = 6000.25 + corner
        t, q = g.zeros(), g.zeros()
        g.interior(t).copy_(torch.from_numpy(v))
        assert api.cfl_dt(g, t)[1] == float(v.max())
        api.prepare_vdt2(g, t, q, dt)
        want = _box(((v.astype(np.float64) * dt) ** 2).astype(np.float32)).astype(np.float32)
        assert np.array_equal(g.padded(q).cpu().numpy(), want)
        m = (1.0 / v.astype(np.float64) ** 2).astype(np.float32)
        g.interior(t).copy_(torch.from_numpy(m))
        api.prepare_vdt2_m(g, t, q, dt)
        want = _box((dt * dt / m.astype(np.float64)).astype(np.float32)).astype(np.float32)
        assert np.array_equal(g.padded(q).cpu().numpy(), want)
    v.flat[-1] = -1.0
    g.interior(t).copy_(torch.from_numpy(v))
    with pytest.raises(api.FDError):
        api.cfl_dt(g, t)


# few rows: each shared by several blocks (of several waves in the maximum alone)
@pytest.mark.parametrize("shape", [(70001, 1, 1), (66000, 3, 2), (5003, 9, 4), (260, 5, 6)])
def test_rows_shared_by_blocks(shape):
    nx, ny, nz = shape
    g = api.Grid(nx, ny, nz)
    v = (3000 + 400 * random_field((nz, ny, nx), 7)).astype(np.float32)
    dt = 7.3e-4
    for at in (0, nx // 2 + 1, -1):
        v.flat[at] = 6000.25 + at
        t, q = g.zeros(), g.zeros()
        g.interior(t).copy_(torch.from_numpy(v))
        assert api.cfl_dt(g, t)[1] == float(v.max())
        api.prepare_vdt2(g, t, q, dt)
        want = _box(((v.astype(np.float64) * dt) ** 2).astype(np.float32)).astype(np.float32)
        assert np.array_equal(g.padded(q).cpu().numpy(), want)


def test_shot_with_long_rows_reduces_its_own_maximum():
    """The shot server's vdt2 and max(v) in one pass, several blocks to a row: the sponge is
    designed for the maximum found, on the last point."""
    from paper_2506_02486_amd import serving
    nx, ny, nz = 6000, 9, 10
    v = np.full((nz, ny, nx), 2000.0, np.float32)
    v.flat[-1] = 2600.0
    vd = torch.from_numpy(v).cuda()
    rec = np.array([[nx - 3, 4, 5], [nx // 2, 4, 5]], np.int32)
    shot = serving.Shot(vd, 20, 9e-4, (nx - 5, 4, 5), rec, sponge_width=3)
    with serving.ShotServer(1 << 30, max_slots=2) as srv:
        code, tr, _ = srv.wait(srv.submit(shot))
    assert code == 0
    sim = api.Simulation(vd, dt=9e-4, sponge_width=3, geom=api.Geometry(src=shot.src, rec=rec))
    assert sim.vmax == 2600.0
    assert np.array_equal(tr, sim.run(20).cpu().numpy())


def test_few_long_rows_use_the_whole_device():
    """A model of 4 x 4 long rows is prepared about as fast as a cube of the same padded
    size (38M cells): a row in one wave's hands took 100 times as long."""
    def best(shape, fn):
        g = api.Grid(*shape)
        v, q = g.zeros(), g.zeros()
        g.interior(v).fill_(2500.0)
        times = []
        for _ in range(5):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            fn(g, v, q)
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b))
        return min(times)

    for fn in (lambda g, v, q: api.prepare_vdt2(g, v, q, 1e-3), lambda g, v, q: api.cfl_dt(g, v)):
        assert best((1 << 18, 4, 4), fn) < 5 * best((328, 328, 328), fn)
