"""Gram-Schmidt steps of lock-step solves at the sizes where they split: vectors in groups of eight,
systems in groups of four, restarts in between."""
import numpy as np
import pytest

from paper_2103_16073_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F():
    from paper_2103_16073_amd import fmmbem
    fmmbem.lib()
    return fmmbem


@pytest.mark.parametrize("ns", [1, 3, 4, 5, 9])
@pytest.mark.parametrize("restart", [7, 8, 9, 40])
def test_lock_step_solves_vs_single(F, ns, restart):
    """Every system of the batch stops at its tolerance, and at the solution of a solve of its own (the
    operator's condition is far below the 1e3 between the two tolerances)."""
    room = synth.shoebox(3.0, 2.5, 2.0, 0.3)
    ctx = F.Context(0)
    ctx.fmmbem_set_mesh(room.vertices, room.triangles)
    ctx.fmmbem_set_wavenumber(synth.wavenumber(150.0))
    ctx.fmmbem_set_admittance(room.beta)
    rng = np.random.default_rng(3)
    ctx.fmmbem_set_sources(rng.uniform(0.4, 1.6, (ns, 3)))
    kw = dict(tol=1e-8, restart=restart, maxit=400, precond=F.FMMBEM_PC_NEARBLOCK)
    X, reps, rc = ctx.fmmbem_solve_batch(np.arange(ns), **kw)
    assert rc == 0
    for s in range(ns):
        x, rep, rc1 = ctx.fmmbem_solve(s, **kw)
        assert rc1 == 0 and rep.rel_res < 1e-8 and reps[s].rel_res < 1e-8
        assert np.linalg.norm(X[s] - x) < 1e-5 * np.linalg.norm(x), (s, rep.iters, reps[s].iters)
    ctx.close()


# either side of 32 partial sums per vector (N = 8,192), one and two passes
@pytest.mark.parametrize("h", [0.098, 0.094])
@pytest.mark.parametrize("reorth", [0, 1, 2])
def test_partial_sums_vs_both_sides(F, h, reorth):
    """Solves of five sources around the size where the step's kernels stop adding the partial sums
    themselves: each at its tolerance, lock step and alone at one solution."""
    room = synth.shoebox(3.0, 2.5, 2.0, h)
    assert (room.n <= 8192) == (h == 0.098), room.n
    ctx = F.Context(0)
    ctx.fmmbem_set_mesh(room.vertices, room.triangles)
    ctx.fmmbem_set_wavenumber(synth.wavenumber(150.0))
    ctx.fmmbem_set_admittance(room.beta)
    ctx.fmmbem_set_sources(np.random.default_rng(3).uniform(0.4, 1.6, (5, 3)))
    kw = dict(tol=1e-8, restart=60, maxit=400, precond=F.FMMBEM_PC_NEARBLOCK, reorth=reorth)
    X, reps, rc = ctx.fmmbem_solve_batch(np.arange(5), **kw)
    assert rc == 0 and max(r.rel_res for r in reps) < 1e-8
    x, rep, rc1 = ctx.fmmbem_solve(4, **kw)
    assert rc1 == 0 and rep.rel_res < 1e-8
    assert np.linalg.norm(X[4] - x) < 1e-5 * np.linalg.norm(x)
    ctx.close()
