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
