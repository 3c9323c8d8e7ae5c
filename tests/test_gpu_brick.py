"""The brick kernel (fd_brick.hip), which steps grids of 0.45M to 14.5M points: the same
bits as the other kernels, at the edges of its bricks, and the rule that chooses it."""
import numpy as np
import pytest
import torch

from workloads import random_field, receivers_plane, smooth_velocity
from bitwise import same_bits

api = pytest.importorskip("paper_2506_02486_amd.api")

# one and two planes per brick (up to 2^20 points, above), 8 and 16 lanes; rows whose
# last float4 holds 1, 2, 3 or 4 interior points; whole and ragged bricks on every axis
SHAPES = [(70, 66, 61), (65, 64, 64), (64, 112, 80), (99, 53, 71), (131, 101, 83),
          (128, 96, 90), (190, 83, 77), (96, 113, 97), (132, 100, 81),
          # planes taken in bands: one and two planes per brick, equal bands and a
          # smaller last one; single calls by another kernel (more than 2^22 points)
          (196, 186, 20), (200, 200, 27), (512, 70, 33), (340, 228, 56)]


@pytest.mark.parametrize("shape,faces,want", [
    ((64, 64, 64), False, False), ((64, 80, 80), False, False), ((64, 128, 64), False, True),
    ((64, 128, 64), True, False), ((65, 64, 64), False, True), ((224, 224, 224), True, True),
    ((240, 240, 240), False, True), ((240, 240, 240), True, False),
    ((78, 300, 480), False, True), ((100, 300, 400), False, False),
    ((225, 224, 224), True, False), ((225, 224, 224), False, True),
    ((256, 256, 256), False, False), ((512, 512, 512), True, False),
    ((4, 300, 300), False, False), ((300, 4, 300), False, False), ((640, 640, 2), True, False)])
def test_which_grids_run_as_bricks(shape, faces, want):
    g = api.Grid(*shape)
    assert api.step_bricks(g, faces) is want
    api.set_tiles(3)
    try:
        assert api.step_bricks(g, faces) is False  # only the automatic mode
    finally:
        api.set_tiles(0)


@pytest.mark.parametrize("shape,faces,want", [
    ((64, 64, 64), False, False), ((64, 128, 64), False, True), ((128, 256, 128), False, True),
    ((128, 256, 129), False, False), ((256, 200, 150), False, False),
    ((128, 256, 128), True, True), ((128, 256, 129), True, False), ((256, 136, 72), True, True),
    ((132, 256, 129), True, True), ((260, 200, 150), True, True), ((225, 224, 224), True, False),
    ((130, 130, 130), True, False)])
def test_which_single_calls_run_as_bricks(shape, faces, want):
    g = api.Grid(*shape)
    assert api.step_bricks(g, faces, once=True) is want
    api.set_tiles(1)
    try:
        assert api.step_bricks(g, faces, once=True) is False
    finally:
        api.set_tiles(0)


@pytest.mark.gpu
@pytest.mark.parametrize("shape", SHAPES)
def test_brick_bits_equal_other_kernels(shape):
    """Exchange and fused forward runs with a source and a receiver plane, the scaled
    adjoint step with its residual row and gradient, and the unscaled one's gradient (the
    damped gradient pass): bricks against one thread per point and 64 x 32 marching tiles."""
    nx, ny, nz = shape
    v = smooth_velocity(nx, ny, nz, seed=2, sigma=3.0)
    rec = receivers_plane(nx, ny, nz // 2 + 1)[::3]
    geom = api.Geometry(src=(nx - 2, ny // 2, nz // 2), rec=rec)
    assert api.step_bricks(api.Grid(nx, ny, nz)) is True

    def field(g, seed):
        t = g.zeros()
        g.padded(t).copy_(torch.from_numpy(random_field((nz + 8, ny + 8, nx + 8), seed)))
        return t

    def everything():
        out = []
        for exchange, mode in (("loopback", "native"), (None, "native-fused"), (None, "separate")):
            for width in (0, 6):
                sim = api.Simulation(v, sponge_width=width, exchange=exchange, geom=geom)
                out.append(sim.run(7, mode=mode))
                out += [x.clone() for x in sim.state()]
                if exchange:
                    out += sim.send
        sim = api.Simulation(v, sponge_width=6, geom=geom)
        g = sim.grid
        a, b, u = field(g, 11), field(g, 12), field(g, 13)
        row = torch.from_numpy(random_field((len(rec),), 14)).cuda()
        for sponge in (None, sim.sponge):
            o, acc = g.zeros(), field(g, 15)
            api.adjoint_step_scaled(g, a, b, o, sim.vdt2, sponge, u_n=u, g_b=acc,
                                    src=(geom.src, 0.7), res=(sim.rec_plane, row))
            acc2 = field(g, 16)
            api.adjoint_step(g, a, b, g.zeros(), sim.vdt2, sponge, u_n=u, g_vdt2=acc2,
                             src=(geom.src, 0.7))
            out += [o, acc, acc2]
        return out

    ref = everything()
    assert all(bool(torch.isfinite(t).all()) for t in ref)
    try:
        for tiles in (1, 3):
            api.set_tiles(tiles)
            for i, (x, y) in enumerate(zip(ref, everything())):
                assert same_bits(x, y), (tiles, i)
    finally:
        api.set_tiles(0)


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [(256, 250, 125), (256, 256, 125), (260, 250, 125)])
def test_gradient_pass_on_both_sides_of_its_limit(shape):
    """Rows that fill 128-wide tiles, up to and from 8 million points, and others: the
    gradient pass gives the bits of the 64 x 32 tiles."""
    g = api.Grid(*shape)

    def field(seed):
        t = g.zeros()
        g.padded(t).copy_(torch.from_numpy(random_field((g.nz + 8, g.ny + 8, g.nx + 8), seed)))
        return t

    a, u, q = field(1), field(2), field(3)
    acc = []
    try:
        for tiles in (0, 1):
            api.set_tiles(tiles)
            acc.append(field(4))
            api.adjoint_step(g, None, a, g.zeros(), q, None, u_n=u, g_vdt2=acc[-1],
                             src=((255, 4, 5), 0.7))
    finally:
        api.set_tiles(0)
    assert same_bits(acc[0], acc[1])
