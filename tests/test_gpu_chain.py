"""The chain of kernels per PCG iteration, which `pcg_workgroups` asks for: captured graphs against direct launches, and
the membrane's staged product against the CSR product.

A step that does not ask for it solves by a team of resident work-groups, which no graph holds, so these comparisons of
the chain's own forms ask for it on every side."""

import numpy as np
import pytest
import torch  # noqa: F401  (its HIP runtime is the one the library shares)

import oracle as O
from paper_2502_10872_amd import inputs as I
from paper_2502_10872_amd import shell as S

pytestmark = pytest.mark.gpu
MAT = I.MATERIAL


def rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


@pytest.mark.parametrize("precision", [S.SHELL_PREC_FP64, S.SHELL_PREC_MIXED])
@pytest.mark.parametrize("model", ["SS", "EP"])
def test_the_chains_graph_replays_equal_direct_launches(model, precision):
    """Four steps that replay the oracle's counts (no powers of two, so that graph pieces and direct remainders mix),
    each graph replayed many times with eager work between; the same bits, and in FP64 the oracle's to 1e-10."""
    mesh = I.workload_cylinder(28, model) if model == "SS" else I.workload_plate32()
    dt, newton = (1 / 30, 2) if model == "SS" else (1 / 60, 1)
    osim = O.Sim(O.Stencils(model, mesh.X, mesh.tris, MAT["young"], MAT["poisson"], MAT["thickness"]), MAT, mesh.pinned)
    steps = [osim.step(dt, max_newton=newton, pcg_rtol=1e-9)[0] for _ in range(4)]
    ends = []
    for flags in (0, S.SHELL_STEP_NO_GRAPHS):
        with S.Problem(mesh, MAT, model=model, precision=precision, block_vertices=128) as pb:
            for counts in steps:
                params, _keep = S.step_params(dt, max_newton=newton, pcg_rtol=1e-9, replay=counts, flags=flags,
                                              pcg_workgroups=512)
                _, st = S.shell_step_implicit(pb.sim, params)
                assert np.array_equal(st["counts"], counts[: st["newton_iters"]])
            ends.append(S.shell_sim_get_state(pb.sim, mesh.nv)[:2])
    (xa, va), (xb, vb) = ends
    assert np.array_equal(xa, xb) and np.array_equal(va, vb)
    if precision == S.SHELL_PREC_FP64:
        assert rel(xa - mesh.X, osim.x - mesh.X) <= 1e-10 and rel(va, osim.v) <= 1e-10


@pytest.mark.parametrize("flags", [0, S.SHELL_FLAG_MEMBRANE])
def test_the_chains_graphs_in_tolerance_mode_equal_direct_launches(flags):
    """Chunks of iterations that double up to a largest, all from graphs after the first; the same counts and bits."""
    mesh = I.cylinder_mesh(32, 0.5, 0.9, 0.8, 0.2, 3, "SS", "ends")
    out = []
    for step_flags in (0, S.SHELL_STEP_NO_GRAPHS):
        with S.Problem(mesh, MAT, flags=flags) as pb:
            params, _ = S.step_params(1 / 60, max_newton=2, pcg_rtol=1e-8, flags=step_flags, pcg_workgroups=512)
            counts = [S.shell_step_implicit(pb.sim, params)[1]["counts"] for _ in range(3)]
            out.append((counts, *S.shell_sim_get_state(pb.sim, mesh.nv)[:2]))
    (ca, xa, va), (cb, xb, vb) = out
    assert all(np.array_equal(a, b) for a, b in zip(ca, cb))
    assert max(int(c.max()) for c in ca) > 48  # several chunks
    assert np.array_equal(xa, xb) and np.array_equal(va, vb)


@pytest.mark.parametrize("precision,bound", [(S.SHELL_PREC_FP64, 1e-12), (S.SHELL_PREC_MIXED, 1e-9)])
@pytest.mark.parametrize("n", [60, 223, 257, 363])
def test_the_membrane_chains_staged_product_agrees_with_the_direct_product(n, precision, bound):
    """The staged product of the chain in row groups of 128 (3600 and 49729 vertices), 256 (66049) and 512 (131769)
    rows, the last of them ragged, against the CSR product (SHELL_FLAG_DIRECT_PRODUCT): one step of two Newton
    iterations with 40 replayed PCG iterations each.  The two sum a row's products in another order, in float64."""
    mesh = I.cylinder_mesh(n, 0.5, 0.9, 0.8, 0.2, 3, "SS", "ends")
    ends = []
    for flags in (0, S.SHELL_FLAG_DIRECT_PRODUCT):
        with S.Problem(mesh, MAT, precision=precision, flags=S.SHELL_FLAG_MEMBRANE | flags) as pb:
            counts = np.array([[40, 0, 0], [40, 0, 0]], np.int32)
            params, _keep = S.step_params(1 / 60, max_newton=2, newton_rtol=1e-12, replay=counts, pcg_workgroups=512)
            _, st = S.shell_step_implicit(pb.sim, params)
            assert st["newton_iters"] == 2 and st["pcg_total"] == 80
            ends.append(S.shell_sim_get_state(pb.sim, mesh.nv)[:2])
    (xa, va), (xb, vb) = ends
    assert np.abs(xa - mesh.X).max() > 0
    assert rel(xa - mesh.X, xb - mesh.X) <= bound and rel(va, vb) <= bound
