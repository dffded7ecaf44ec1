"""Solves by resident teams of work-groups against the same solves as a chain of kernels.

`pcg_workgroups` asks for a launch shape of the kernel chain, so the same step with and without it compares
the two: the same recurrence with its dot products grouped otherwise.  Sizes sit at the edges of the team
layout: one member up to 1024 rows, members of 256 rows up to 16384, of 512 above, then one member per compute
unit with several rows per thread; ragged last slices throughout.  Twenty replayed iterations keep the
rounding's growth small: FP64 agrees to 1e-10 (the oracle parity bound), mixed precision to 1e-5 (the bound of
the full-size mixed iteration against the oracle)."""

import ctypes
import threading

import numpy as np
import pytest
import torch  # noqa: F401  (its HIP runtime is the one the library shares)

from paper_2502_10872_amd import inputs as I
from paper_2502_10872_amd import shell as S

pytestmark = pytest.mark.gpu
MAT = I.MATERIAL
BOUND = {S.SHELL_PREC_FP64: 1e-10, S.SHELL_PREC_MIXED: 1e-5}


def rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


def _start(mesh):
    g = I.rng(11)
    n = mesh.meta["n"]
    s, t = np.tile(np.linspace(0, 1, n), n), np.repeat(np.linspace(0, 1, n), n)
    u = 0.002 * mesh.spacing * n * np.sin(2 * np.pi * s) * np.sin(2 * np.pi * t)
    return mesh.X + u[:, None] * g.uniform(0.5, 1.0, 3), 0.1 * np.sin(np.pi * s * t)[:, None] * g.uniform(0.5, 1.0, 3)


def _step(pb, mesh, x, v, wg=0, newton=2, iters=20, **kw):
    S.shell_sim_set_state(pb.sim, x, v, 0)
    counts = np.full((newton, 3), iters, np.int32)
    params, _keep = S.step_params(1 / 60, max_newton=newton, newton_rtol=0.0, replay=counts, pcg_workgroups=wg, **kw)
    rc, st = S.shell_step_implicit(pb.sim, params)
    xo, vo, _ = S.shell_sim_get_state(pb.sim, mesh.nv)
    return xo, vo, st


@pytest.mark.parametrize("precision", [S.SHELL_PREC_FP64, S.SHELL_PREC_MIXED])
@pytest.mark.parametrize("model,n", [("SS", 5), ("EP", 22), ("SS", 23), ("FS", 32), ("ES", 33), ("SS", 127), ("EP", 129),
                                     ("FS", 363), ("SS", 420), ("SS", 600), ("SS", 850)])
def test_team_solves_equal_the_kernel_chain(model, n, precision):
    mesh = I.plate_mesh(n, 1.0, 0.2, 7, model) if model.endswith("P") else I.workload_sphere_cap(n, model)
    x, v = _start(mesh)
    with S.Problem(mesh, MAT, precision=precision) as pb:
        xa, va, sa = _step(pb, mesh, x, v)
        xb, vb, sb = _step(pb, mesh, x, v, wg=512)
    assert np.array_equal(sa["counts"], sb["counts"])
    assert rel(xa - mesh.X, xb - mesh.X) <= BOUND[precision]
    assert rel(va, vb) <= BOUND[precision]


@pytest.mark.parametrize("precision", [S.SHELL_PREC_FP64, S.SHELL_PREC_MIXED])
def test_a_solve_over_several_launches_is_the_same_solve(precision):
    """`chunk` bounds the iterations of one launch: the solve pauses and resumes on the same bits."""
    mesh = I.workload_cylinder(70, "SS")
    x, v = _start(mesh)
    with S.Problem(mesh, MAT, precision=precision) as pb:
        xa, va, _ = _step(pb, mesh, x, v)
        xb, vb, _ = _step(pb, mesh, x, v, chunk=7)
    assert np.array_equal(xa, xb) and np.array_equal(va, vb)


@pytest.mark.parametrize("precision", [S.SHELL_PREC_FP64, S.SHELL_PREC_MIXED])
def test_held_coordinates_and_batches_of_teams(precision):
    """A batch (mixed precision: teams of one launch), one mesh with single coordinates held, against each mesh
    alone through the kernel chain."""
    meshes = [I.workload_cylinder(40, "SS"), I.plate_mesh(21, 1.0, 0.2, 7, "EP"), I.workload_sphere_cap(60, "FS")]
    held = [np.arange(m.nv) % 5 * (np.arange(m.nv) % 7 == 0) if k == 0 else None for k, m in enumerate(meshes)]
    probs = [S.Problem(m, MAT, precision=precision, held=h) for m, h in zip(meshes, held)]
    try:
        starts = [_start(m) for m in meshes]
        chain = [_step(pb, m, x, v, wg=512)[:2] for pb, m, (x, v) in zip(probs, meshes, starts)]
        for pb, (x, v) in zip(probs, starts):
            S.shell_sim_set_state(pb.sim, x, v, 0)
        batch = S.shell_batch_create([pb.sim for pb in probs])
        try:
            params, _keep = S.step_params(1 / 60, max_newton=2, newton_rtol=0.0, replay=np.full((2, 3), 20, np.int32))
            S.shell_batch_step(batch, params, len(probs))
        finally:
            S.shell_destroy_batch(batch)
        for pb, m, (xc, vc) in zip(probs, meshes, chain):
            x, v, _ = S.shell_sim_get_state(pb.sim, m.nv)
            assert rel(x - m.X, xc - m.X) <= BOUND[precision] and rel(v, vc) <= BOUND[precision], m.name
    finally:
        for pb in probs:
            pb.close()


def test_meshes_of_a_batch_whose_solves_end_in_different_launches():
    """Solves to a tolerance end after different numbers of launches; every mesh then takes its own Newton update,
    with the same bits as in one launch, and as each mesh's own step (its team is of the same members)."""
    meshes = [I.plate_mesh(9, 1.0, 0.2, 7, "EP"), I.workload_sphere_cap(40, "SS"), I.workload_cylinder(25, "FS")]
    probs = [S.Problem(m, MAT, precision=S.SHELL_PREC_MIXED) for m in meshes]
    starts = [_start(m) for m in meshes]
    batch = S.shell_batch_create([pb.sim for pb in probs])
    try:
        ends, counts = [], []
        for chunk in (0, 3, 11):
            for pb, (x, v) in zip(probs, starts):
                S.shell_sim_set_state(pb.sim, x, v, 0)
            params, _keep = S.step_params(1 / 60, max_newton=2, newton_rtol=1e-5, pcg_rtol=1e-4, chunk=chunk)
            _, stats = S.shell_batch_step(batch, params, len(probs))
            ends.append([S.shell_sim_get_state(pb.sim, m.nv)[:2] for pb, m in zip(probs, meshes)])
            counts.append([st["counts"] for st in stats])
        assert len({int(np.max(c)) for c in counts[0]}) > 1  # they end apart
        for pb, m, (x, v), end in zip(probs, meshes, starts, ends[0]):
            S.shell_sim_set_state(pb.sim, x, v, 0)
            params, _keep = S.step_params(1 / 60, max_newton=2, newton_rtol=1e-5, pcg_rtol=1e-4)
            S.shell_step_implicit(pb.sim, params)
            alone = S.shell_sim_get_state(pb.sim, m.nv)[:2]
            assert np.array_equal(alone[0], end[0]) and np.array_equal(alone[1], end[1]), m.name
        for end, count in zip(ends[1:], counts[1:]):
            for m, (x, v), (x0, v0) in zip(meshes, end, ends[0]):
                assert np.array_equal(x, x0) and np.array_equal(v, v0), m.name
            assert all(np.array_equal(p, q) for p, q in zip(count, counts[0]))
    finally:
        S.shell_destroy_batch(batch)
        for pb in probs:
            pb.close()


@pytest.mark.parametrize("precision", [S.SHELL_PREC_FP64, S.SHELL_PREC_MIXED])
def test_a_member_that_gives_up_hands_the_solve_to_the_chain(precision):
    """With no time to wait the first unmet meeting ends the launch (every member leaves by itself), and the step
    takes the kernel chain: the same bits as the step that asked for it."""
    mesh = I.workload_cylinder(100, "SS")
    x, v = _start(mesh)
    limit = S.lib().shell_test_team_wait
    limit.argtypes, limit.restype = [ctypes.c_void_p, ctypes.c_uint64], None
    with S.Problem(mesh, MAT, precision=precision) as pb:
        xb, vb, _ = _step(pb, mesh, x, v, wg=512)
        limit(pb.sim, 0)
        xa, va, _ = _step(pb, mesh, x, v)
        limit(pb.sim, 2 ** 64 - 1)
        xc, vc, _ = _step(pb, mesh, x, v)
    assert np.array_equal(xa, xb) and np.array_equal(va, vb)
    assert rel(xc - mesh.X, xb - mesh.X) <= BOUND[precision] and rel(vc, vb) <= BOUND[precision]


def _no_waiting(sim, ticks):
    limit = S.lib().shell_test_team_wait
    limit.argtypes, limit.restype = [ctypes.c_void_p, ctypes.c_uint64], None
    limit(sim, ticks)


@pytest.mark.parametrize("precision", [S.SHELL_PREC_FP64, S.SHELL_PREC_MIXED])
@pytest.mark.parametrize("model,n", [("SS", 5), ("ES", 22), ("SS", 23), ("FS", 33), ("SS", 257), ("ES", 420), ("SS", 600),
                                     ("FS", 850)])
def test_membrane_team_solves_equal_the_kernel_chain(model, n, precision):
    """The coupled solve with the membrane, as a team and (no time to wait; a mesh of one member never waits, so
    its two runs are one) as a chain: one member up to 512 rows, members of 256 rows, then one per compute unit.
    Single coordinates held as well as the ends."""
    mesh = I.workload_cylinder(n, model)
    x, v = _start(mesh)
    counts = np.zeros((2, 3), np.int32)
    counts[:, 0] = 20
    params, _keep = S.step_params(1 / 60, max_newton=2, newton_rtol=0.0, replay=counts)
    out = []
    held = np.arange(mesh.nv) % 5 * (np.arange(mesh.nv) % 11 == 0)
    with S.Problem(mesh, MAT, precision=precision, flags=S.SHELL_FLAG_MEMBRANE, held=held) as pb:
        for ticks in (2 ** 64 - 1, 0):
            _no_waiting(pb.sim, ticks)
            S.shell_sim_set_state(pb.sim, x, v, 0)
            S.shell_step_implicit(pb.sim, params)
            out.append(S.shell_sim_get_state(pb.sim, mesh.nv)[:2])
    (xa, va), (xb, vb) = out
    bound = 1e-10 if precision == S.SHELL_PREC_FP64 else 1e-6
    assert rel(xa - mesh.X, xb - mesh.X) <= bound and rel(va, vb) <= bound


@pytest.mark.parametrize("precision", [S.SHELL_PREC_FP64, S.SHELL_PREC_MIXED])
def test_a_membrane_solve_over_several_launches_is_the_same_solve(precision):
    mesh = I.workload_cylinder(40, "SS")
    x, v = _start(mesh)
    out = []
    with S.Problem(mesh, MAT, precision=precision, flags=S.SHELL_FLAG_MEMBRANE) as pb:
        for chunk in (0, 7):
            params, _keep = S.step_params(1 / 60, max_newton=2, pcg_rtol=1e-8, chunk=chunk)
            S.shell_sim_set_state(pb.sim, x, v, 0)
            rc, st = S.shell_step_implicit(pb.sim, params)
            out.append((st["counts"], *S.shell_sim_get_state(pb.sim, mesh.nv)[:2]))
    assert all(np.array_equal(a, b) for a, b in zip(*out))


def test_a_column_that_goes_non_finite_is_reported_whatever_the_launches():
    """A load that is finite in float64 and overflows float32: its column of the solve is lost in the first iteration,
    while the others iterate on.  The solve ends as non-finite, without a Newton update, in one launch and over
    several."""
    mesh = I.workload_cylinder(40, "SS")
    load = 1e-3 * I.rng(3).standard_normal((mesh.nv, 3))
    load[np.flatnonzero(mesh.pinned == 0)[100], 0] = 1e45
    out = []
    with S.Problem(mesh, MAT, precision=S.SHELL_PREC_MIXED) as pb:
        for chunk in (0, 1, 3):
            S.shell_sim_set_state(pb.sim, mesh.X, np.zeros_like(mesh.X), 0)
            with pytest.raises(S.ShellError, match="NONFINITE"):
                S.shell_solve_static(pb.sim, load, max_newton=2, pcg_rtol=1e-5, chunk=chunk)
            st = S.shell_sim_get_stats(pb.sim)
            assert np.isfinite(st["grad_norm0"])  # the solve was reached
            out.append(st["newton_iters"])
    assert out == [0, 0, 0]


def _membrane_run(mesh, x, v, precision, ticks=2 ** 64 - 1, wg=0, flags=0, step_flags=0, static=False, held=None):
    counts = np.zeros((2, 3), np.int32)
    counts[:, 0] = 20
    with S.Problem(mesh, MAT, precision=precision, flags=S.SHELL_FLAG_MEMBRANE | flags, held=held) as pb:
        _no_waiting(pb.sim, ticks)
        S.shell_sim_set_state(pb.sim, x, v, 0)
        if static:
            load = 1e-6 * I.rng(3).standard_normal((mesh.nv, 3))
            S.shell_solve_static(pb.sim, load, max_newton=2, replay=counts, pcg_workgroups=wg, flags=step_flags)
        else:
            params, _keep = S.step_params(1 / 60, max_newton=2, newton_rtol=0.0, replay=counts, pcg_workgroups=wg,
                                          flags=step_flags)
            S.shell_step_implicit(pb.sim, params)
        return S.shell_sim_get_state(pb.sim, mesh.nv)[:2]


@pytest.mark.parametrize("static", [False, True])
@pytest.mark.parametrize("precision", [S.SHELL_PREC_FP64, S.SHELL_PREC_MIXED])
def test_the_membrane_chain_asked_for_is_the_chain(precision, static):
    """`pcg_workgroups` selects the chain of kernels with the membrane too: the same bits as a team that hands its
    solve over, from captured graphs and launched one by one."""
    mesh = I.workload_cylinder(60, "SS")
    x, v = _start(mesh)
    want = _membrane_run(mesh, x, v, precision, ticks=0, static=static)
    for wg, step_flags in ((1, 0), (512, 0), (512, S.SHELL_STEP_NO_GRAPHS)):
        got = _membrane_run(mesh, x, v, precision, wg=wg, step_flags=step_flags, static=static)
        assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1])


@pytest.mark.parametrize("precision", [S.SHELL_PREC_FP64, S.SHELL_PREC_MIXED])
@pytest.mark.parametrize("model,n", [("SS", 5), ("FS", 8), ("ES", 22), ("SS", 23)])
def test_membrane_solves_of_one_member_equal_the_kernel_chain_and_the_direct_product(model, n, precision):
    """A team of one member never waits and so never hands over (up to 512 vertices; 23 x 23 has three members): the
    chain is asked for.  The direct product's solve of such a mesh is the one of a single work-group over CSR rows (16, 8
    and 4 lanes each; at 23 x 23 its own chain).  Bounds as above."""
    mesh = I.workload_cylinder(n, model)
    x, v = _start(mesh)
    held = np.arange(mesh.nv) % 5 * (np.arange(mesh.nv) % 11 == 0)
    xa, va = _membrane_run(mesh, x, v, precision, held=held)
    bound = 1e-10 if precision == S.SHELL_PREC_FP64 else 1e-6
    for wg, flags in ((512, 0), (0, S.SHELL_FLAG_DIRECT_PRODUCT)):
        xb, vb = _membrane_run(mesh, x, v, precision, wg=wg, flags=flags, held=held)
        assert rel(xa - mesh.X, xb - mesh.X) <= bound and rel(va, vb) <= bound


def _steps_of(kind, torch, out, errors):
    """Three steps of one user on a stream of its own: a mesh whose team takes nearly all compute units, a small mesh,
    a mixed-precision batch, a batch with the membrane."""
    try:
        flags = S.SHELL_FLAG_MEMBRANE if kind == "membrane" else 0
        precision = S.SHELL_PREC_MIXED if kind == "batch" else S.SHELL_PREC_FP64
        meshes = {"large": [I.workload_sphere_cap(400, "SS")], "small": [I.workload_cylinder(70, "FS")],
                  "batch": [I.workload_cylinder(60, "SS"), I.workload_sphere_cap(130, "ES")],
                  "membrane": [I.workload_cylinder(n, "SS") for n in (40, 20, 90)]}[kind]
        probs = [S.Problem(m, MAT, precision=precision, flags=flags) for m in meshes]
        batch = None
        try:
            for pb, m in zip(probs, meshes):
                S.shell_sim_set_state(pb.sim, *_start(m), 0)
            stream = torch.cuda.Stream()
            params, _keep = S.step_params(1 / 60, max_newton=2, newton_rtol=0.0, pcg_rtol=1e-4, max_pcg=400)
            if len(probs) > 1:
                batch = S.shell_batch_create([pb.sim for pb in probs])
            for _ in range(3):
                if batch is not None:
                    S.shell_batch_step(batch, params, len(probs), stream=stream)
                else:
                    S.shell_step_implicit(probs[0].sim, params, stream=stream)
            out[kind] = [S.shell_sim_get_state(pb.sim, pb.nv)[:2] for pb in probs]
        finally:
            if batch is not None:
                S.shell_destroy_batch(batch)
            for pb in probs:
                pb.close()
    except BaseException as e:  # reported by the main thread
        errors.append((kind, e))


def test_teams_of_several_threads_reach_what_each_reaches_alone():
    """Teams share the device's compute units: each launch waits for its members' units, in the order of the requests.
    Four threads at a time, a mesh that needs nearly all units among them, reach their own results bit for bit."""
    kinds = ("large", "small", "batch", "membrane")
    alone, errors = {}, []
    for kind in kinds:
        _steps_of(kind, torch, alone, errors)
    assert not errors, errors
    together = {}
    threads = [threading.Thread(target=_steps_of, args=(kind, torch, together, errors)) for kind in kinds]
    for t in threads:
        t.start()
    for t in threads:
        t.join(timeout=100)
    assert not any(t.is_alive() for t in threads)
    assert not errors, errors
    for kind in kinds:
        for (xa, va), (xt, vt) in zip(alone[kind], together[kind]):
            assert np.isfinite(xa).all() and np.array_equal(xa, xt) and np.array_equal(va, vt), kind


@pytest.mark.parametrize("flags", [0, S.SHELL_FLAG_MEMBRANE])
def test_solves_after_one_that_gave_up_take_the_chain_at_once(flags):
    """Two solves a step: the one that gives up and the 16 after it run as the chain, whatever the wait allowed, and
    then teams again."""
    mesh = I.workload_cylinder(100, "SS")
    x, v = _start(mesh)
    n = [20, 0, 0] if flags else 20  # with the membrane: iterations, halvings
    with S.Problem(mesh, MAT, flags=flags) as pb:
        team = _step(pb, mesh, x, v, iters=n)[:2]
        chain = _step(pb, mesh, x, v, wg=512, iters=n)[:2]
        assert not np.array_equal(team[1], chain[1])
        _no_waiting(pb.sim, 0)
        ends = [_step(pb, mesh, x, v, iters=n)[:2]]
        _no_waiting(pb.sim, 2 ** 64 - 1)
        ends += [_step(pb, mesh, x, v, iters=n)[:2] for _ in range(9)]
    for end in ends[:8]:  # 16 of 17 solves
        assert np.array_equal(end[0], chain[0]) and np.array_equal(end[1], chain[1])
    assert np.array_equal(ends[9][0], team[0]) and np.array_equal(ends[9][1], team[1])
