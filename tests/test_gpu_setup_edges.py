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
