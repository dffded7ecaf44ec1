"""The default size of a force work-group's vertex tile against tiles of 2048 vertices set by the caller, and forces
from and into the caller's own arrays.

A stencil's force does not depend on its vertices' internal numbers, and the fixed-point accumulation adds the
same integers per vertex whatever the tile, so the forces agree bit for bit.  The energy
is summed per tile in float64: with E the sum of some 1e5 terms of one sign the two groupings differ by less
than 1e-12 of it."""

import dataclasses

import numpy as np
import pytest
import torch

from paper_2502_10872_amd import inputs as I
from paper_2502_10872_amd import shell as S

pytestmark = pytest.mark.gpu


def eval_forces(mesh, x, model, precision, block, flags):
    with S.Problem(mesh, I.MATERIAL, model=model, precision=precision, block_vertices=block, flags=flags,
                   sim=False) as pb:
        xd = torch.as_tensor(x, device="cuda")
        f = torch.full((mesh.nv, 3), float("nan"), device="cuda",
                       dtype=torch.float32 if precision == S.SHELL_PREC_MIXED else torch.float64)
        e = torch.zeros(1, device="cuda", dtype=torch.float64)
        out = []
        for call in (S.shell_eval_forces, S.shell_eval_forces_noalloc):
            f.fill_(float("nan"))
            call(pb.st, xd, f, e)
            torch.cuda.synchronize()
            out.append((f.cpu().numpy(), float(e.item())))
        return out, pb.info


# one tile; ragged last tiles; either side of each change of size (512 tiles of 64, 128, ...), the second of which
# is the change of the vertex order too
@pytest.mark.parametrize("precision", [S.SHELL_PREC_FP64, S.SHELL_PREC_MIXED])
@pytest.mark.parametrize("model,n,block,flags", [
    ("EP", 5, 64, 0), ("FP", 23, 64, 0), ("SS", 43, 64, S.SHELL_FLAG_MEMBRANE), ("SP", 181, 64, 0),
    ("EP", 182, 128, 0), ("ES", 256, 128, 0), ("FS", 257, 256, S.SHELL_FLAG_MEMBRANE), ("SP", 512, 512, 0),
    ("ES", 700, 1024, S.SHELL_FLAG_MEMBRANE), ("SS", 725, 2048, 0)])
def test_default_tiles_give_the_forces_of_tiles_of_2048(model, n, block, flags, precision):
    mesh = I.plate_mesh(n, 1.0, 0.2, 7, model) if model.endswith("P") else I.workload_sphere_cap(n, model)
    x = mesh.X + 1e-3 * mesh.spacing * I.rng(3).uniform(-1, 1, mesh.X.shape)
    got, info = eval_forces(mesh, x, model, precision, 0, flags)
    want, winfo = eval_forces(mesh, x, model, precision, 2048, flags)
    assert info["block_vertices"] == block and info["nblocks"] == -(-mesh.nv // block)
    assert winfo["block_vertices"] == 2048
    for (f, e), (fw, ew) in zip(got, want):
        assert np.array_equal(f, fw)
        assert abs(e - ew) <= 1e-12 * abs(ew)


# one tile; a whole group of 16 arrivals; one work-group alone in its group; two groups and a remainder
@pytest.mark.parametrize("precision", [S.SHELL_PREC_FP64, S.SHELL_PREC_MIXED])
@pytest.mark.parametrize("model,nv_tiles,flags", [
    ("EP", 1, 0), ("SS", 16, 0), ("ES", 17, S.SHELL_FLAG_MEMBRANE), ("FP", 39, S.SHELL_FLAG_MEMBRANE)])
def test_forces_written_over_the_positions_and_energy_of_all_tiles(model, nv_tiles, flags, precision):
    """Forces into the memory of the positions (gathered first) equal forces into memory of their own (read where
    they lie), call after call, and the energy equals a central difference's: f = -dE/dx along f itself."""
    mesh = I.plate_mesh(int(np.sqrt(64 * nv_tiles)), 1.0, 0.2, 7, model)
    if model.endswith("S"):
        mesh = I.workload_sphere_cap(int(np.sqrt(64 * nv_tiles)), model)
    x = mesh.X + 1e-2 * mesh.spacing * I.rng(3).uniform(-1, 1, mesh.X.shape)
    real = torch.float32 if precision == S.SHELL_PREC_MIXED else torch.float64
    with S.Problem(mesh, I.MATERIAL, model=model, precision=precision, block_vertices=64, flags=flags,
                   sim=False) as pb:
        assert pb.info["nblocks"] == -(-mesh.nv // 64)
        xd = torch.as_tensor(x, device="cuda")
        f = torch.empty(mesh.nv, 3, device="cuda", dtype=real)
        e = torch.zeros(3, device="cuda", dtype=torch.float64)
        for call in (S.shell_eval_forces, S.shell_eval_forces_noalloc):
            for _ in range(3):
                call(pb.st, xd, f, e)
                over = xd.clone()
                call(pb.st, over, over, e[1:])
                torch.cuda.synchronize()
                inside = over.flatten().view(real)[:3 * mesh.nv].view(mesh.nv, 3)
                assert torch.equal(inside, f)
                assert float(e[0]) == float(e[1])
        g = f.double().clone()
        h = 1e-4 * mesh.spacing / float(g.abs().max())
        ends = []
        for sign in (1.0, -1.0):
            S.shell_eval_forces(pb.st, xd + sign * h * g, f, e)
            torch.cuda.synchronize()
            ends.append(float(e[0]))
    # central difference: third-order terms are 1e-8 of the first; the energies' own rounding (float32: 1e-7 of a
    # total some 1e2 to 1e4 times the difference) dominates
    want = -2 * h * float((g * g).sum())
    noise = (1e-6 if precision == S.SHELL_PREC_MIXED else 1e-13) * abs(ends[0])
    assert abs((ends[0] - ends[1]) - want) <= 1e-3 * abs(want) + noise


# one row group and a ragged one; whole groups; the product that isn't staged
@pytest.mark.parametrize("model,n,flags", [("EP", 5, 0), ("SS", 32, 0), ("FP", 45, 0), ("ES", 300, 0),
                                           ("SS", 45, S.SHELL_FLAG_DIRECT_PRODUCT)])
def test_operator_product_over_its_inputs(model, n, flags):
    """q = diag(m) p + dt^2 K p read where p and m lie equals the product over p's and over m's own memory bit
    for bit, and the product without masses plus m p to float64 rounding (1e-13 of the largest value)."""
    mesh = I.plate_mesh(n, 1.0, 0.2, 7, model) if model.endswith("P") else I.workload_sphere_cap(n, model)
    g = I.rng(9)
    p, mass = g.standard_normal((mesh.nv, 3)), g.uniform(0.5, 1.5, mesh.nv)
    with S.Problem(mesh, I.MATERIAL, model=model, flags=flags) as pb:
        pd, md = torch.as_tensor(p, device="cuda"), torch.as_tensor(mass, device="cuda")
        for m in (md, None):
            q = torch.full_like(pd, float("nan"))
            S.shell_hessian_apply(pb.h, m, 0.25, pd, q)
            over = pd.clone()
            S.shell_hessian_apply(pb.h, m, 0.25, over, over)
            one = torch.full_like(pd, float("nan"))
            S.shell_hessian_apply(pb.h, None, 0.25, pd, one)
            torch.cuda.synchronize()
            assert torch.equal(over, q)
            want = one if m is None else one + m[:, None] * pd
            bound = 1e-13 * float(want.abs().max())
            assert float((q - want).abs().max()) <= bound
        both = torch.cat([md, torch.zeros(2 * mesh.nv, device="cuda", dtype=torch.float64)])
        S.shell_hessian_apply(pb.h, both[:mesh.nv], 0.25, pd, both.view(mesh.nv, 3))
        S.shell_hessian_apply(pb.h, md, 0.25, pd, q)
        torch.cuda.synchronize()
        assert torch.equal(both.view(mesh.nv, 3), q)


@pytest.mark.parametrize("model,n,flags", [("SS", 40, 0), ("ES", 90, S.SHELL_FLAG_MEMBRANE)])
def test_captured_forces_and_products_replay(model, n, flags):
    """Replays of a captured evaluation and product on new positions, with eager calls between them, equal the
    eager results bit for bit (the arrival counters are back at zero after every launch)."""
    mesh = I.workload_sphere_cap(n, model)
    with S.Problem(mesh, I.MATERIAL, model=model, flags=flags) as pb:
        x = torch.as_tensor(mesh.X, device="cuda").clone()
        f, q = torch.empty_like(x), torch.empty_like(x)
        e = torch.zeros(1, device="cuda", dtype=torch.float64)

        def run(f, e, q):
            S.shell_eval_forces(pb.st, x, f, e)
            S.shell_hessian_apply(pb.h, None, 0.5, x, q)

        run(f, e, q)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            run(f, e, q)
        f2, q2, e2 = torch.empty_like(f), torch.empty_like(q), torch.empty_like(e)
        for k in range(4):
            x.copy_(torch.as_tensor(mesh.X + 1e-3 * mesh.spacing * I.rng(k).standard_normal(mesh.X.shape)))
            run(f2, e2, q2)
            f.fill_(float("nan"))
            q.fill_(float("nan"))
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(f, f2) and torch.equal(q, q2) and torch.equal(e, e2)


def _same_energy_as_tiles_of_2048(mesh, x, precision, block, reorder):
    out = []
    for T in (block, 2048):
        with S.Problem(mesh, I.MATERIAL, model="EP", precision=precision, block_vertices=T, reorder=reorder,
                       sim=False) as pb:
            xd = torch.as_tensor(x, device="cuda")
            f = torch.empty(mesh.nv, 3, device="cuda",
                            dtype=torch.float32 if precision == S.SHELL_PREC_MIXED else torch.float64)
            e = torch.zeros(2, device="cuda", dtype=torch.float64)
            S.shell_eval_forces(pb.st, xd, f, e)
            S.shell_eval_forces_noalloc(pb.st, xd, f, e[1:])
            torch.cuda.synchronize()
            out.append((f.cpu().numpy(), e.cpu().numpy()))
    (f, e), (fw, ew) = out
    assert np.array_equal(f, fw)
    assert np.all(np.abs(e - ew) <= 1e-12 * np.abs(ew))


# eight threads per vertex of these are no whole number of waves; more tiles than threads in a work-group, so that
# every thread of the last work-group has partials to add
@pytest.mark.parametrize("precision", [S.SHELL_PREC_FP64, S.SHELL_PREC_MIXED])
@pytest.mark.parametrize("block", [65, 90, 100, 127])
def test_energy_of_tiles_of_any_size(block, precision):
    mesh = I.plate_mesh(400, 1.0, 0.2, 7, "EP")
    x = mesh.X + 1e-3 * mesh.spacing * I.rng(3).uniform(-1, 1, mesh.X.shape)
    _same_energy_as_tiles_of_2048(mesh, x, precision, block, 1)


@pytest.mark.parametrize("precision", [S.SHELL_PREC_FP64, S.SHELL_PREC_MIXED])
@pytest.mark.parametrize("block", [65, 100])
def test_energy_of_tiles_with_more_stencils_than_threads(block, precision):
    """Vertices numbered at random: a tile's vertices are no neighbours, and its list holds about twelve stencils
    per vertex, so that every thread of its work-group takes some."""
    mesh = I.plate_mesh(40, 1.0, 0.2, 7, "EP")
    new = I.rng(5).permutation(mesh.nv)
    old = np.argsort(new)
    mesh = dataclasses.replace(mesh, X=mesh.X[old].copy(), tris=new[mesh.tris].astype(mesh.tris.dtype),
                               pinned=mesh.pinned[old].copy())
    x = mesh.X + 1e-3 * mesh.spacing * I.rng(3).uniform(-1, 1, mesh.X.shape)
    _same_energy_as_tiles_of_2048(mesh, x, precision, block, 0)


def test_energies_after_evaluations_that_overlapped():
    """Evaluations of one handle on several streams at a time spoil each other's energies, which the caller is told not
    to do; the handle's later ones are right all the same.  Captured, so that they follow one another closely enough
    to overlap; 32 tiles, so that an evaluation is little more than its arrivals."""
    mesh = I.workload_sphere_cap(45, "SS")
    states = [mesh.X + a * mesh.spacing * I.rng(3).uniform(-1, 1, mesh.X.shape) for a in (1e-3, 2e-3, 3e-3, 4e-3)]
    with S.Problem(mesh, I.MATERIAL, sim=False) as pb:
        xd = torch.as_tensor(states[0], device="cuda").clone()
        f, e = torch.empty_like(xd), torch.zeros(1, device="cuda", dtype=torch.float64)

        def energies():  # at other positions each, so that no partial of an earlier call will do
            out = []
            for x in states:
                xd.copy_(torch.as_tensor(x))
                S.shell_eval_forces(pb.st, xd, f, e)
                torch.cuda.synchronize()
                out.append(float(e))
            return out

        want = energies()
        lanes = []
        for _ in range(4):
            fs, es, graph = torch.empty_like(xd), torch.zeros_like(e), torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph):
                for _ in range(50):
                    S.shell_eval_forces(pb.st, xd, fs, es)
            lanes.append((torch.cuda.Stream(), graph, fs, es))
        for _ in range(40):
            for s, graph, _, _ in lanes:
                with torch.cuda.stream(s):
                    graph.replay()
        torch.cuda.synchronize()
        assert energies() == want
