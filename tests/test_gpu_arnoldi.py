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


def fgmres_history(matvec, b, tol, m, reorth, maxit):
    """Residual estimates of restarted GMRES with classical Gram-Schmidt in numpy: one pass (reorth 0), a
    second one where the first removed most of the vector (1), or always (2)."""
    x, hist, bn = np.zeros_like(b), [], np.linalg.norm(b)
    r = b
    while True:
        V, H, g = [r / np.linalg.norm(r)], np.zeros((m + 1, m), complex), np.linalg.norm(r)
        for j in range(m):
            w = matvec(V[j])
            Q, w0 = np.array(V), np.linalg.norm(w)
            h = Q.conj() @ w
            w = w - h @ Q
            if reorth == 2 or (reorth == 1 and not np.linalg.norm(w) > np.sqrt(0.5) * w0):
                d = Q.conj() @ w
                w, h = w - d @ Q, h + d
            H[:j + 1, j], H[j + 1, j] = h, np.linalg.norm(w)
            V.append(w / np.linalg.norm(w))
            e = np.zeros(j + 2, complex)
            e[0] = g
            y = np.linalg.lstsq(H[:j + 2, :j + 1], e, rcond=None)[0]
            hist.append(np.linalg.norm(e - H[:j + 2, :j + 1] @ y) / bn)
            if hist[-1] < tol or len(hist) >= maxit:
                return np.array(hist)
        x = x + y @ np.array(V[:m])
        r = b - matvec(x)


# either side of N = 8,192; one cycle, and restarts on either side of a group of eight vectors
@pytest.mark.parametrize("h", [0.098, 0.094])
@pytest.mark.parametrize("reorth", [0, 1, 2])
@pytest.mark.parametrize("restart", [60, 8, 9])
def test_residual_history_vs_numpy(F, h, reorth, restart):
    """The estimate after every iteration against numpy's on the same operator.  A step's rounding enters
    it as eps over the estimate (with one pass, eps over its square, so that one is held down to 1e-4 only):
    below 1e-7 of it in both; and the lock-step solve's iterations."""
    room = synth.shoebox(3.0, 2.5, 2.0, h)
    ctx = F.Context(0)
    ctx.fmmbem_set_mesh(room.vertices, room.triangles)
    ctx.fmmbem_set_wavenumber(synth.wavenumber(150.0))
    ctx.fmmbem_set_admittance(room.beta)
    ctx.fmmbem_set_sources(np.random.default_rng(3).uniform(0.4, 1.6, (3, 3)))
    tol = 1e-4 if reorth == 0 else 1e-8
    kw = dict(tol=tol, restart=restart, maxit=120, precond=F.FMMBEM_PC_NONE, reorth=reorth)
    ref = fgmres_history(lambda v: ctx.fmmbem_matvec(v)[0], ctx.fmmbem_rhs()[1], tol, restart, reorth, 120)
    x, rep, rc = ctx.fmmbem_solve(1, **kw)
    hist = ctx.fmmbem_solve_history()
    X, reps, rcb = ctx.fmmbem_solve_batch(np.arange(3), **kw)
    ctx.close()
    assert rc == 0 and rcb == 0 and len(hist) == len(ref) == rep.iters and abs(reps[1].iters - rep.iters) <= 1
    assert np.max(np.abs(hist - ref) / ref) < 1e-6, np.abs(hist - ref) / ref
    assert rep.rel_res < tol * (1 + 1e-6) and reps[1].rel_res < tol * (1 + 1e-6)
