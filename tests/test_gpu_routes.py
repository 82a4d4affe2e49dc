"""GPU tests of calls that reach the same result by different kernels: whole
steps against the separate calls, the batch's steps against its substeps."""
import numpy as np
import pytest

from paper_2007_14933_amd import inputs as I
from parity_util import say

pytestmark = pytest.mark.gpu


def jump_net(bias):
    """Bits of a hand-set network: logit = bias - 10 (sum of the six log jumps)."""
    from paper_2007_14933_amd import sensor as SN
    w = np.zeros(1441, dtype=np.float32)
    w[[i * 32 for i in range(4, 10)]] = 1.0  # W1[i][0]
    w[352] = 1.0                             # W2[0][0]
    w[1408] = -10.0                          # w3[0]
    w[1440] = bias                           # b3
    return SN.bf16_bits(w)


def routing_net(prob):
    """The jump_net that calls most interfaces of the problem's state smooth, but
    not all."""
    from paper_2007_14933_amd.solver import Solver
    s = Solver(prob, sensor=1)
    s.apply_bc()
    best = None
    for bias in range(61):
        bits = jump_net(bias)
        s.set_sensor(bits, 0.5)
        s.sensor_update()
        sm, tot = s.sensor_stats()
        if best is None or abs(sm / tot - 0.7) < best[0]:
            best = (abs(sm / tot - 0.7), bits)
    assert best[0] < 0.25
    return best[1]


def step_and_separate(prob, steps, net=None, dilate=1, every=0, **kw):
    """States after whole steps and after the same steps by separate calls."""
    import torch
    from paper_2007_14933_amd.solver import Solver
    a, b = Solver(prob, **kw), Solver(prob, **kw)
    for s in (a, b):
        if net is not None:
            s.set_sensor(net, 0.5, dilate=dilate, every_substage=every)
        s.apply_bc()
    dt = 0.5 * a.compute_dt(0.5)
    for _ in range(steps):
        a.step(dt)
        for k in range(b.nstages):
            b.substep(k, dt)
            b.apply_bc()
    a.check()
    torch.cuda.synchronize()
    if net is not None:
        assert a.sensor_stats() == b.sensor_stats()
    return a, b


@pytest.mark.parametrize("form", [0, 1])
@pytest.mark.parametrize("n", [(60,), (255,), (256,), (31, 6), (32, 7), (33, 8), (70, 64)])
def test_routed_steps_equal_separate_calls(n, form):
    """Learned routing through the one-pass stage, tiles of 255 and of 32 x 7 nodes
    and their edges, every width of the neighbourhood, masks refreshed at every
    step or substage: two steps give the bits of the separate calls."""
    import torch
    prob = I.smooth_random(len(n), n + (1,) * (3 - len(n)), seed=n[0], amp=0.2)
    net = routing_net(prob)
    for dilate, every in ((0, 0), (1, 0), (2, 0), (1, 1)):
        a, b = step_and_separate(prob, 2, net, dilate, every, form=form, sensor=1)
        err = float((a.U - b.U).abs().max())
        say("[gpu routes] routed", n, "form", form, "dilate", dilate, "every", every, "max|diff|", err)
        assert torch.equal(a.U, b.U), err


@pytest.mark.parametrize("form,scheme,sensor", [(0, I.TENO5, 0), (0, I.WENOZ5, 0), (0, I.TENO5, 1), (1, I.TENO5, 1),
                                                (1, I.TENO5, 0)])
def test_batch_steps_substeps_and_solo_calls(form, scheme, sensor):
    """A batch's steps, its substeps (captured or not, whatever their tiles) and the
    problems alone by separate calls: the same bits after six steps."""
    import torch
    from paper_2007_14933_amd.batch import Batch
    from paper_2007_14933_amd.solver import Solver
    rng = np.random.default_rng(11)
    probs = [I.riemann2d(n, rng, t_end=1e9, scheme=scheme) for n in (32, 100, 24, 64, 71)]
    bits = jump_net(3.0)
    kw = dict(weights=bits, threshold=0.5) if sensor else {}
    make = lambda capture: Batch(probs, form=form, sensor=sensor, capture=capture, **kw)  # noqa: E731
    whole, parts = make(True), [make(True)]
    for seg, capture in ((1, False), (8, True), (1024, False)):
        b = make(False)
        b.set_tiles(np.full((len(probs), 2), seg))
        if capture:
            b.capture()
        parts.append(b)
    direct = make(False)
    solo = [Solver(p, form=form, sensor=sensor) for p in probs]
    for s in solo:
        if sensor:
            s.set_sensor(bits, 0.5)
        s.apply_bc()
    for _ in range(6):
        whole.step()
        direct.step()
        for b in parts:
            for k in range(3):
                b.substep(k)
        for s in solo:
            dt = s.compute_dt(0.5)
            for k in range(3):
                s.substep(k, dt)
                s.apply_bc()
    torch.cuda.synchronize()
    if sensor:
        sm, tot = whole.solvers[1].sensor_stats()
        assert 0 < sm < tot
    for p, s in enumerate(solo):
        for b in [whole, direct] + parts:
            assert torch.equal(b.solvers[p].U, s.U), (p, float((b.solvers[p].U - s.U).abs().max()))


def wavy(prob):
    nd = prob.ndim
    X = [np.array(c, dtype=float) for c in prob.coords[:nd]]
    wave = sum(np.sin(2.0 * np.pi * c) for c in X)
    return prob.with_(coords1d=None, coords_full=tuple(c + 0.02 * wave for c in X) + (None,) * (3 - nd))


@pytest.mark.parametrize("scheme", ["WENOZ5", "TENO5"])
@pytest.mark.parametrize("n", [(62, 30), (63, 30), (70, 131), (190, 9), (64, 7, 9), (97, 40, 33)])
def test_precision_form_on_general_meshes(n, scheme):
    """The precision form on wavy meshes around and beyond the width from which the
    FP64 form's x lanes run along x: the launch shape of the x sweep does not
    change a bit, and the residual is the FP64 form's to FP32 rounding (in the mean
    2^-22 of each component's largest value: some four roundings of deviations no
    larger than that; single nodes may flip a cut-off decision)."""
    import torch
    from paper_2007_14933_amd.solver import Solver
    prob = wavy(I.smooth_random(len(n), n + (1,) * (3 - len(n)), seed=n[0], amp=0.2)).with_(scheme=getattr(I, scheme))
    s, ref = Solver(prob, form=1), Solver(prob)
    for q in (s, ref):
        q.apply_bc()
    a = s.residual().clone()
    s.set_sweep_segments([n[0], 0, 0])
    assert torch.equal(s.residual(), a)
    r = ref.residual()
    err = ((a - r).abs() / r.abs().amax(dim=(1, 2, 3), keepdim=True)).mean()
    say("[gpu routes] precision form, general mesh", n, scheme, float(err))
    assert float(err) <= 2.0 ** -22


def central(n, bounded, Re, sutherland=0, **kw):
    bc = tuple((I.EXTRAPOLATE,) * 2 if d in bounded else (I.PERIODIC,) * 2 for d in range(3))
    return I.smooth_random(3, n, seed=n[0], amp=0.05, Re=Re, M=0.5).with_(scheme=I.CENTRAL4, bc=bc,
                                                                         sutherland=sutherland, **kw)


@pytest.mark.parametrize("n,bounded,Re,sutherland", [
    ((66, 18, 130), (2,), 200.0, 0), ((66, 18, 130), (2,), 200.0, 1), ((66, 34, 130), (2,), 0.0, 0),
    ((300, 24, 64), (0,), 200.0, 0), ((321, 40, 40), (0, 1, 2), 200.0, 1), ((70, 97, 40), (1,), 200.0, 0),
    ((96, 40, 33), (0,), 200.0, 0), ((96, 40, 33), (0,), 0.0, 0)])
def test_central_bounded_grids(n, bounded, Re, sutherland):
    """The central residual of bounded 3D grids large enough for the z-marching pass
    with the node passes at the ends (the last two: not), one step against the
    oracle at the run bound 1e-11."""
    from parity_util import gpu_run, normwise_rel, oracle_run
    prob = central(n, bounded, Re, sutherland)
    say("[gpu routes] central", n, bounded, Re, sutherland)
    Ug, tg, _ = gpu_run(prob, 1)
    Uo, to = oracle_run(prob, 1)
    err = normwise_rel(I.interior_view(3, Ug), I.interior_view(3, Uo))
    assert abs(tg - to) <= 1e-12 * to and err.max() <= 1e-11, err


def best_us(f, reps=50, rounds=8):
    """Shortest mean time of f over some rounds, microseconds."""
    import torch
    f()
    best = float("inf")
    for _ in range(rounds):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(reps):
            f()
        b.record()
        b.synchronize()
        best = min(best, 1e3 * a.elapsed_time(b) / reps)
    return best


def test_central_small_bounded_grids_cost_alike():
    """On a small cube the direction that is bounded does not decide the residual's
    time (beside the z-marching pass the node passes at ends in x cost a whole pass
    more: 1.9 times the time of ends in z)."""
    from paper_2007_14933_amd.solver import Solver
    t = []
    for d in (0, 2):
        s = Solver(central((48, 48, 48), (d,), 0.0))
        s.apply_bc()
        R = s.residual()
        t.append(best_us(lambda: s.residual(R=R)))
    say("[gpu routes] central 48^3 bounded in x, z: us", t)
    assert t[0] <= 1.4 * t[1]


def test_central_runs_of_planes_with_sutherlands_law():
    """The z-marching pass holds one block per CU with Sutherland's law and two
    without; its runs of planes are planned for that: on 48^3, one round of blocks
    in either case, the law costs at most a quarter more (one value in seven more
    to stage; runs planned for two blocks per CU take a second round)."""
    from paper_2007_14933_amd.solver import Solver
    t = []
    for law in (1, 0):
        s = Solver(central((48, 48, 48), (), 200.0, law))
        s.apply_bc()
        R = s.residual()
        t.append(best_us(lambda: s.residual(R=R)))
    say("[gpu routes] central 48^3, Sutherland's law and constant viscosity: us", t)
    assert t[0] <= 1.25 * t[1]


@pytest.mark.parametrize("form", [0, 1])
def test_tuner_searches_what_acts(form, tmp_path, monkeypatch):
    """Steps of one pass per stage (FP64) do not depend on the sweeps' tiles: the
    tuner leaves those alone there, and searches them for the unrouted precision
    form; a workgroup count from a cache is not kept where it measures slower (one
    workgroup in place of hundreds), in today's cache or in one written before the
    step took one pass."""
    import json
    import torch
    from paper_2007_14933_amd.batch import Batch
    rng = np.random.default_rng(5)
    probs = [I.riemann2d(n, rng, t_end=1e9) for n in (256, 192, 64)]
    path = tmp_path / "tiles.json"
    monkeypatch.setenv("OSBLI_TILE_CACHE", str(path))
    dev = torch.cuda.get_device_name(0).replace(" ", "_")
    old = {"v2|%s|form%d|sensor0|%dx%d" % (dev, form, p.n[0], p.n[1]): [4, 8] for p in probs}
    old["v2|%s|form%d|sensor0|grid|3" % (dev, form)] = 1
    path.write_text(json.dumps(old))
    tried = []
    set_tiles = Batch.set_tiles
    monkeypatch.setattr(Batch, "set_tiles", lambda self, seg: (tried.append(np.array(seg)), set_tiles(self, seg)))
    b = Batch(probs, form=form)
    default = b.tiles.copy()
    chosen = b.tune(nsteps=2)
    assert b.sweep_blocks != 1
    moved = [t for t in tried if not np.array_equal(np.asarray(t).reshape(default.shape), default)]
    if form == 0:
        assert not moved and np.array_equal(b.tiles, default)
        assert all(tuple(chosen[(p.n[0], p.n[1])]) == tuple(t) for p, t in zip(probs, default))
    else:
        assert moved
    store = json.loads(path.read_text())
    new = [k for k in store if "|grid|" in k and k not in old]
    assert new
    for k in new:
        store[k] = 1
    path.write_text(json.dumps(store))
    c = Batch(probs, form=form)
    c.tune(nsteps=2)
    assert c.sweep_blocks != 1
    assert json.loads(path.read_text())[new[0]] != 1


def test_time_step_beside_idle_contexts():
    """Contexts that never ask for a time step (an ensemble's) do not slow down one
    that does: the reduction returns through pinned words, of which 64 contexts at
    a time have some (else by a copy and a synchronisation, twice the time)."""
    import gc
    import time
    from paper_2007_14933_amd.solver import Solver

    def best(s, reps=200, rounds=8):
        s.compute_dt(0.5)
        out = float("inf")
        for _ in range(rounds):
            t = time.perf_counter()
            for _ in range(reps):
                s.compute_dt(0.5)
            out = min(out, (time.perf_counter() - t) / reps)
        return 1e6 * out
    gc.collect()
    first = Solver(I.sod(100))
    first.apply_bc()
    alone = best(first)
    idle = [Solver(I.sod(20)) for _ in range(70)]
    s = Solver(I.sod(100))
    s.apply_bc()
    beside = best(s)
    say("[gpu routes] time step alone, beside %d contexts: us" % len(idle), alone, beside)
    assert beside <= 1.5 * alone


def test_time_steps_of_more_contexts_than_slots():
    """Every context gets its own right time step, with pinned words or without (70
    at once), in any order, and again once the first ones are gone."""
    import gc
    from paper_2007_14933_amd.solver import Solver
    gc.collect()
    probs = [I.smooth_random(1, (40 + k, 1, 1), seed=k, amp=0.2) for k in range(70)]
    ss = [Solver(p) for p in probs]
    for s in ss:
        s.apply_bc()
    want = []
    for s in ss:
        U = s.interior()[:, 0, 0]
        u = U[1] / U[0]
        a = np.sqrt(1.4 * 0.4 * (U[2] - 0.5 * U[0] * u * u) / U[0])
        want.append(0.5 / ((np.abs(u) + a) * s.prob.n[0]).max())
    for order in (range(70), range(69, -1, -1)):
        for k in order:
            assert abs(ss[k].compute_dt(0.5) - want[k]) <= 1e-12 * want[k], k
    del ss[:40]
    del s
    gc.collect()
    late = Solver(probs[0])
    late.apply_bc()
    assert abs(late.compute_dt(0.5) - want[0]) <= 1e-12 * want[0]
    for k in range(30):
        assert abs(ss[k].compute_dt(0.5) - want[40 + k]) <= 1e-12 * want[40 + k]


def test_solver_dropped_during_a_capture():
    """A solver collected while some other stream captures a graph (the last one: its
    context frees the page of pinned words) leaves the capture valid."""
    import gc
    import torch
    from paper_2007_14933_amd.solver import Solver
    gc.collect()
    s = Solver(I.sod(50))
    s.apply_bc()
    s.compute_dt(0.5)
    x = torch.zeros(1000, device="cuda:0")
    stream, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=stream):
        x.add_(1.0)
        del s
        gc.collect()
        x.add_(1.0)
    for k in range(3):
        graph.replay()
        torch.cuda.synchronize()
        assert float(x.min()) == float(x.max()) == 2.0 * (k + 1)
    t = Solver(I.sod(50))
    t.apply_bc()
    assert t.compute_dt(0.5) > 0.0


@pytest.mark.parametrize("scheme", ["WENOZ5", "TENO5"])
def test_shock_tube_in_large_units(scheme):
    """The shock tube with its unit of time 2^90 times as long (speeds of 1e27, so
    that indicators reach 1e54 and their products 1e162): five steps against the
    oracle at the run bound 1e-11, by whole steps and by separate calls."""
    from parity_util import normwise_rel, oracle_run
    from paper_2007_14933_amd.solver import Solver
    k = 2.0 ** 90
    prob = I.sod(100).with_(scheme=getattr(I, scheme))
    U0 = prob.U0.copy()
    U0[1] *= k
    U0[2] *= k * k
    prob = prob.with_(U0=U0)
    Uo, to = oracle_run(prob, 5)
    assert np.isfinite(Uo).all()
    for whole in (True, False):
        s = Solver(prob)
        s.apply_bc()
        for _ in range(5):
            dt = s.compute_dt(0.5)
            if whole:
                s.step(dt)
            else:
                for st in range(3):
                    s.substep(st, dt)
                    s.apply_bc()
        err = normwise_rel(I.interior_view(1, s.state()), I.interior_view(1, Uo))
        say("[gpu routes] tube in large units", scheme, whole, err)
        assert err.max() <= 1e-11, err


@pytest.mark.parametrize("n", [(40, 40, 40), (128, 130, 128)])
def test_profile_counts_every_sweep(n):
    """The profile of a 3D step accounts for three directions per substage: a launch
    of y and z together (small grids) is a class of its own, counted as two."""
    import sys
    import os
    sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
    import bench
    from paper_2007_14933_amd.solver import Solver
    s = Solver(I.smooth_random(3, n, seed=1, Re=200.0))
    s.apply_bc()
    s.profile()
    s.step(1e-4)
    p = s.profile_read()
    sweeps, ms = bench.sweep_times(p)
    assert sweeps == 9 and ms > 0.0
    together = p["sweep_yz"][0]
    assert together in (0, 3) and (together == 3) == (n[0] == 40)
    assert p["sweep_y"][0] == p["sweep_z"][0] == 3 - together


@pytest.mark.parametrize("form,every", [(0, 0), (1, 0), (0, 1), (1, 1)])
@pytest.mark.parametrize("n", [(33, 31, 40), (70, 40, 37)])
def test_routed_3d_steps(n, form, every):
    """Learned routing in whole 3D steps (y and z sweeps in one launch), FP64 and
    precision form, masks refreshed per step or substage: one step against the
    separate calls.  FP64: 1e-13 of the component's largest value.  Precision form:
    a last bit of the FP64 state moves a deviation by one FP32 rounding, 2^-24 of
    it, which a step weighs by its CFL number: 2^-24 of that value."""
    prob = I.smooth_random(3, n, seed=n[0], amp=0.2, Re=200.0)
    net = routing_net(prob)
    for dilate in (0, 2):
        a, b = step_and_separate(prob, 1, net, dilate, every, form=form, sensor=1)
        scale = b.U.abs().amax(dim=(1, 2, 3), keepdim=True)
        err = float(((a.U - b.U).abs() / scale).max())
        say("[gpu routes] routed 3D", n, "form", form, "every", every, "dilate", dilate, err)
        assert err <= (1e-13 if form == 0 else 2.0 ** -24)


@pytest.mark.parametrize("n", [(40, 33, 20), (50, 61)])
def test_march_segments_on_wavy_meshes(n):
    """Segments of the marching sweeps where the metrics vary (the x sweep's staged
    area vectors among them): every length gives the bits of one segment per line,
    and those are the oracle's residual to the parity bound."""
    import torch
    from oracle import oracle as O
    from paper_2007_14933_amd.solver import Solver
    from parity_util import flux_scale
    prob = wavy(I.smooth_random(len(n), n + (1,) * (3 - len(n)), seed=9, amp=0.2))
    s = Solver(prob)
    s.apply_bc()
    s.set_sweep_segments([200, 200, 200])
    ref = s.residual().clone()
    for seg in (1, 2, 3, 5, 16):
        s.set_sweep_segments([seg, seg, seg])
        assert torch.equal(s.residual(), ref), seg
    U = O.apply_bc(prob, prob.U0.copy())
    S, J = O.metrics(prob)
    err = np.abs(ref.cpu().numpy() - O.residual(prob, S, J, U)).max(axis=(1, 2, 3)) / flux_scale(prob, U, J, S)
    say("[gpu routes] wavy march", n, err)
    assert err.max() <= 1e-13, err
