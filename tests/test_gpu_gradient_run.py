"""The gradient's sweeps over several steps (fd_forward_keep, fd_adjoint_run,
fd_grad_accumulate): the bits of the per-step calls they stand for, in each kernel and
at the edges of its tiles, for odd and even numbers of steps."""
import ctypes as C

import numpy as np
import pytest
import torch

from workloads import random_field, receivers_plane, smooth_velocity
from bitwise import same_bits

pytestmark = pytest.mark.gpu

api = pytest.importorskip("paper_2506_02486_amd.api")
from paper_2506_02486_amd import _lib  # noqa: E402


def _random(g, seed):
    t = g.zeros()
    g.interior(t).copy_(torch.from_numpy(random_field((g.nz, g.ny, g.nx), seed)))
    return t


# tile modes 0 (bricks of one and of two planes), 4 and 5 (16-byte lanes in both tile
# shapes); rows whose last float4 holds 1 to 4 interior points
@pytest.mark.parametrize("shape,tiles", [((70, 66, 61), 0), ((131, 101, 83), 0), ((9, 20, 7), 0),
                                         ((70, 37, 29), 4), ((133, 21, 17), 5), ((128, 40, 12), 4),
                                         ((191, 70, 6), 5)])
@pytest.mark.parametrize("nt,plane,sponge", [(5, True, True), (4, False, True), (1, True, False),
                                             (2, True, False)])
def test_runs_equal_per_step_calls(shape, tiles, nt, plane, sponge):
    nx, ny, nz = shape
    sim = api.Simulation(smooth_velocity(nx, ny, nz, seed=2, sigma=3.0), sponge_width=4)
    g, q, sp = sim.grid, sim.vdt2, sim.sponge if sponge else None
    src = (nx - 1, ny // 2, nz // 2)
    rec = receivers_plane(nx, ny, nz // 3)[::2]
    off = torch.from_numpy(g.offsets(rec)).cuda()
    pl = api.receiver_plane(g, rec)
    w = random_field((nt,), 3)
    res = torch.from_numpy(random_field((nt, len(rec)), 4)).cuda()
    w_off = torch.from_numpy(g.offsets(np.array([src], np.int32))).cuda()
    api.set_tiles(tiles)
    try:
        # the forward sweep: states, traces, and the kept sums by way of the gradient
        u = [_random(g, 5), _random(g, 6)] + [g.zeros() for _ in range(nt)]
        tr = torch.zeros((nt, len(rec)), device="cuda")
        for n in range(nt):
            api.step_fused(g, u[n], u[n + 1], u[n + 2], q, sp, (src, float(w[n])))
            api.record_receivers(g, u[n + 2], off, tr[n])
        keep = [torch.full_like(u[0], float("nan")) for _ in range(nt)]
        tr2 = torch.zeros_like(tr)
        up, uc, _ = api.forward_keep(g, u[0].clone(), u[1].clone(), g.zeros(), q, sp, nt, keep,
                                     src=src, wavelet=w, rec_off=off, traces=tr2,
                                     rec_plane=pl if plane else None)
        assert same_bits(tr, tr2)
        assert same_bits(g.interior(up), g.interior(u[nt]))
        assert same_bits(g.interior(uc), g.interior(u[nt + 1]))
        for k in keep:  # nothing outside the interior is written
            assert int(torch.isnan(k).sum()) == g.elems - nx * ny * nz
        # the reverse sweep
        b2, b1, acc = _random(g, 7), _random(g, 8), _random(g, 9)
        c2, c1, acc2 = b2.clone(), b1.clone(), acc.clone()
        w1, w2 = torch.zeros(nt, device="cuda"), torch.zeros(nt, device="cuda")
        for n in range(nt - 1, -1, -1):
            api.record_receivers(g, b1, w_off, w1[n:n + 1])
            api.adjoint_step_scaled(g, b2, b1, b2, q, sp, u_n=u[n + 1], g_b=acc,
                                    src=(src, float(w[n])))
            if n >= 1:
                api.scatter_add_scaled(g, b2, off, res[n - 1], q, sp)
            b2, b1 = b1, b2
        c2, c1 = api.adjoint_run(g, c2, c1, q, sp, nt, keep, acc2, rec_off=off, res=res,
                                 rec_plane=pl if plane else None, w_off=w_off, w_out=w2)
        assert same_bits(w1, w2)
        for x, y in ((b2, c2), (b1, c1), (acc, acc2)):
            assert same_bits(g.interior(x), g.interior(y))
        # the unscaled step's gradient from a kept sum
        a, o, ga = _random(g, 10), g.zeros(), _random(g, 11)
        gb = ga.clone()
        api.adjoint_step(g, None, a, o, q, sp, u_n=u[1], g_vdt2=ga, src=(src, float(w[0])))
        api.grad_accumulate(g, a, keep[0], sp, gb)
        assert same_bits(g.interior(ga), g.interior(gb))
    finally:
        api.set_tiles(0)


# models thin in y or x, one thread per point in the automatic choice, and tile mode 3
@pytest.mark.parametrize("shape,tiles", [((70, 1, 45), 0), ((131, 3, 64), 0), ((8, 70, 33), 0),
                                         ((65, 17, 1), 0), ((2, 3, 1), 0), ((70, 37, 29), 3)])
@pytest.mark.parametrize("nt,plane,sponge", [(5, True, True), (4, False, True), (1, True, False),
                                             (2, True, False)])
def test_runs_of_thin_models_equal_per_step_calls(shape, tiles, nt, plane, sponge):
    test_runs_equal_per_step_calls(shape, tiles, nt, plane, sponge)


def _best(run):
    times = []
    for _ in range(5):
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        a.record()
        run()
        b.record()
        b.synchronize()
        times.append(a.elapsed_time(b))
    return min(times)


def test_kept_sums_of_a_thin_model_cost_what_its_update_does():
    """1000 x 4 x 1000: an update that also writes s_n takes the update's kernel (its floor
    is 20 bytes a point against 16), not tiles that the model leaves mostly empty."""
    g = api.Grid(1000, 4, 1000)
    f = [g.zeros() for _ in range(3)]
    q = g.zeros()
    keep = [g.zeros() for _ in range(8)]
    update = _best(lambda: api.forward_run(g, *f, q, None, 8))
    assert _best(lambda: api.forward_keep(g, *f, q, None, 8, keep)) < 2 * update


@pytest.mark.parametrize("shape", [(64, 17, 3), (65, 16, 2), (66, 5, 4), (71, 33, 2), (3, 18, 5),
                                   (1, 1, 1)])
def test_pointwise_gradient_with_and_without_16_byte_accesses(shape):
    """fd_grad_accumulate on arrays that 16-byte accesses can and cannot take: the same bits,
    rows whose last float4 holds 1 to 4 points, nothing outside the interior written."""
    g = api.Grid(*shape)
    sp = api.Sponge(g, 2, 3000.0, 5e-4)
    out = []
    for off in (0, 1, 2):
        a, s, acc = (torch.from_numpy(random_field((g.elems + off,), seed)).cuda()[off:]
                     for seed in (1, 2, 3))
        for t, seed in ((a, 1), (s, 2), (acc, 3)):
            t.copy_(torch.from_numpy(random_field((g.elems,), seed)))
        for sponge in (None, sp):
            api.grad_accumulate(g, a, s, sponge, acc)
        out.append(acc)
    A, S, G = (g.interior(torch.from_numpy(random_field((g.elems,), i))).double().numpy()
               for i in (1, 2, 3))
    eta = (sp.eta_z.cpu().double().numpy()[:, None, None]
           + sp.eta_y.cpu().double().numpy()[None, :, None]
           + sp.eta_x.cpu().double().numpy()[None, None, :])
    want = G + A * S + A * S / (1 + eta)
    got = g.interior(out[0]).cpu().double().numpy()
    # a few roundings of 2^-24 each, in D (v_rcp_f32: 1 ulp), its products and two sums
    assert np.abs(got - want).max() <= 8 * 2.0 ** -24 * (np.abs(G) + 2 * np.abs(A * S)).max()
    for t in out[1:]:
        assert same_bits(t, out[0])
    inside = torch.zeros(g.elems, dtype=torch.bool)
    g.interior(inside).fill_(True)
    before = torch.from_numpy(random_field((g.elems,), 3))
    assert same_bits(out[0].cpu()[~inside], before[~inside])


def test_pointwise_gradient_of_a_narrow_model_costs_less_than_its_update():
    """4 x 400 x 400: g += D a s_n reads and writes 16 bytes a point and has no neighbours."""
    g = api.Grid(4, 400, 400)
    a, s, acc, out, q = (g.zeros() for _ in range(5))
    step = _best(lambda: [api.adjoint_step(g, a, s, out, q) for _ in range(8)])
    assert _best(lambda: [api.grad_accumulate(g, a, s, None, acc) for _ in range(8)]) < 0.5 * step


def test_states_of_a_kept_forward_run():
    """FWIProblem.states: the wavefields whose stencil sums checkpoint_every = 0 keeps."""
    from paper_2506_02486_amd.fwi import FWIProblem
    nx, ny, nz, nt = 30, 22, 17, 6
    rec = receivers_plane(nx, ny, 3)[::5]
    p = FWIProblem((nx, ny, nz), 5e-4, (9, 8, 7), rec, nt, sponge_width=3, sponge_vmax=2500.0,
                   checkpoint_every=0)
    assert p.states == []
    v = torch.from_numpy(smooth_velocity(nx, ny, nz, seed=2, sigma=3.0)).cuda()
    tr = p.forward(1.0 / v.double().square().float())
    u = p.states
    assert len(u) == nt + 2 and not bool(u[0].any()) and not bool(u[-1].any())
    for n in range(nt):
        row = torch.zeros(len(rec), device="cuda")
        api.record_receivers(p.grid, u[n + 1], p.rec_off, row)
        assert same_bits(row, tr[n])
    assert bool(tr.any())


@pytest.mark.parametrize("scaled", [True, False])
@pytest.mark.parametrize("every,most", [(8, 2 * 3 + 8 + 6), (1, 2 * 31 + 5), (3, 2 * 10 + 3 + 6), (0, 32 + 3), (64, 32 + 6)])
def test_volumes_a_gradient_holds(every, most, scaled):
    """32 steps: a checkpointed gradient holds 2 (S - 1) + C + 6 volumes beside the model's
    two (the zero state of the first segment is no checkpoint), a kept one nt + 3; unscaled
    with C < 2 one more."""
    most += not scaled and every < 2
    from paper_2506_02486_amd.fwi import FWIProblem
    n, nt = 96, 32
    rec = receivers_plane(n, n, 3)[::97]
    p = FWIProblem((n, n, n), 5e-4, (9, 8, 7), rec, nt, sponge_width=3, sponge_vmax=2500.0,
                   checkpoint_every=every)
    m = torch.full((n, n, n), 1 / 2000.0 ** 2, device="cuda")
    res = torch.zeros((nt, len(rec)), device="cuda")
    grads = []
    for _ in range(2):  # a second backward from the same checkpoints
        torch.cuda.synchronize()
        torch.cuda.reset_peak_memory_stats()
        before = torch.cuda.memory_allocated()
        if not grads:
            res += p.forward(m)
        grads.append(p.backward(res, scaled=scaled))
        if len(grads) == 1:
            peak = torch.cuda.max_memory_allocated() - before
            assert peak < (most + 1) * 4 * p.grid.elems  # (the gradient returned: 0.5)
    assert same_bits(*grads) and bool(grads[0].any())


@pytest.mark.parametrize("shape", [(30, 22, 17), (180, 160, 130)])
@pytest.mark.parametrize("plane", [True, False])
def test_gradient_bits_of_every_checkpoint_interval(shape, plane):
    """Segments of 1 step (no recomputation), of 2 to 4 (the last step on the state itself,
    the others step by step or from a copied checkpoint), longer ones and shorter last
    ones: the gradients of the kept run."""
    from paper_2506_02486_amd.fwi import FWIProblem
    nx, ny, nz = shape
    nt = 11
    rec = receivers_plane(nx, ny, 3)[::41]
    if not plane:
        rec[1::2, 2] = 5
    m = 1.0 / torch.from_numpy(smooth_velocity(nx, ny, nz, seed=2, sigma=3.0)).cuda().square()
    res = torch.from_numpy(random_field((nt, len(rec)), 4)).cuda()
    want = {}
    for every in (0, 1, 2, 3, 4, 5, 7, 10, 11, 64):
        p = FWIProblem(shape, 5e-4, (9, 8, 7), rec, nt, sponge_width=3, sponge_vmax=6000.0,
                       checkpoint_every=every)
        p.forward(m)
        for kw in ({"want_grad_w": True}, {"scaled": False, "want_lambda_src": True}):
            got = p.backward(res, **kw)
            for i, t in enumerate(got):
                key = (i, *kw)
                assert bool(t.any())
                assert same_bits(want.setdefault(key, t), t), (every, key)


def test_short_segments_recompute_nothing_that_is_not_needed():
    """256^3, 12 steps: a checkpoint every step needs no recomputation and costs about what
    one every sixth does."""
    from paper_2506_02486_amd.fwi import FWIProblem
    n, nt = 256, 12
    rec = receivers_plane(n, n, 3)[::97]
    m = torch.full((n, n, n), 1 / 2000.0 ** 2, device="cuda")
    res = torch.zeros((nt, len(rec)), device="cuda")
    cost = []
    for every in (1, 6):
        p = FWIProblem((n, n, n), 5e-4, (9, 8, 7), rec, nt, sponge_width=3, sponge_vmax=2500.0,
                       checkpoint_every=every)
        cost.append(_best(lambda: (p.forward(m), p.backward(res))))
        del p
    assert cost[0] < 1.3 * cost[1]


def test_refused_arguments():
    g = api.Grid(40, 20, 10)
    L = api.lib()
    a = [g.zeros() for _ in range(5)]

    def run(keep, **kw):
        r = _lib.fd_reverse()
        r.b_nn, r.b_n1, r.vdt2, r.g_b = (t.data_ptr() for t in a[:4])
        r.nt = 1
        arr = (C.c_void_p * 1)(keep)
        r.keep = C.cast(arr, C.POINTER(C.c_void_p))
        for k, v in kw.items():
            setattr(r, k, v)
        return L.fd_adjoint_run(g.ref, C.byref(r), None)

    ok = a[4].data_ptr()
    assert run(ok, nt=0) == _lib.FD_OK
    for keep, kw in ((None, {}), (a[3].data_ptr(), {}), (ok + 4, {}), (ok, {"nt": -1}),
                     (ok, {"b_nn": None}), (ok, {"g_b": a[0].data_ptr()}), (ok, {"nrec": 3}),
                     (ok, {"w_out": ok})):
        assert run(keep, **kw) == _lib.FD_EINVAL
    r = _lib.fd_run()
    r.u_prev, r.u, r.u_next, r.vdt2 = (t.data_ptr() for t in a[:4])
    r.nt = 1
    for keep in (None, a[1].data_ptr(), ok + 8):
        assert L.fd_forward_keep(g.ref, C.byref(r), (C.c_void_p * 1)(keep), None) == _lib.FD_EINVAL
