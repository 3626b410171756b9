"""P2M and L2P against the library's own all-pairs product (itself checked against the oracle).  P2M:
the edges of its slot blocks (16 rows; 160 and 256 slots, beyond which other kernels take over), its
vectors per pass, the ranges of its Bessel functions.  L2P: few and many leaves, chunks of targets,
expansions in LDS and beyond it."""
import numpy as np
import pytest

from paper_2103_16073_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F():
    from paper_2103_16073_amd import fmmbem
    fmmbem.lib()
    return fmmbem


# p = 16: 153 slots (ten 16-row blocks), 17: 171, 19: 210, 20: 231, 21: 253, 22: the wide kernel;
# leaves of one source up to several groups of sources; k r from below 1e-2 to above 4
@pytest.mark.parametrize("p,f,h,opt", [
    (2, 100.0, 0.3, {}), (5, 100.0, 0.3, {}), (11, 100.0, 0.17, {}),
    (16, 1.0, 0.17, {}), (16, 250.0, 0.34, dict(leaf_max=1)), (16, 250.0, 0.1, {}), (16, 100.0, 0.045, dict(max_depth=2)),
    (17, 250.0, 0.17, {}), (19, 600.0, 0.17, {}), (20, 250.0, 0.1, dict(max_depth=2)), (21, 800.0, 0.17, dict(max_depth=2)),
    (22, 250.0, 0.17, {})])
def test_products_vs_all_pairs(F, p, f, h, opt):
    room = synth.shoebox(3.0, 2.5, 2.0, h)
    ctx = F.Context(0, p_min=p, **opt)
    ctx.fmmbem_set_mesh(room.vertices, room.triangles)
    ctx.fmmbem_set_wavenumber(synth.wavenumber(f))
    ctx.fmmbem_set_admittance(room.beta)
    X = synth.complex_normal(room.n, 5, count=4)
    ref = ctx.fmmbem_matvec(X, exact_far=True)
    # below the default truncation: the ratio of box radius to nearest distance, per degree
    cut = (np.sqrt(0.75) / (2.0 - np.sqrt(0.75))) ** p if p < 16 else 0.0
    for nr in (1, 2, 4):
        for prec, tol in ((F.FMMBEM_FP64, 2e-6), (F.FMMBEM_MIXED, 1e-5)):
            if prec == F.FMMBEM_MIXED and f < 50.0:
                continue  # FP32 does not hold the radial functions of p = 16 at such k times box side
            y = ctx.fmmbem_matvec(X[:nr], precision=prec)
            err = np.linalg.norm(y - ref[:nr], axis=1) / np.linalg.norm(ref[:nr], axis=1)
            assert err.max() < tol + cut, (nr, prec, err, list(ctx.fmmbem_get_info().p)[:4])
    ctx.close()


# four workgroups per leaf and one; leaves of up to 16, 32, 48 and hundreds of targets; four expansions
# per leaf in LDS (p = 16) and beyond its share (p = 28); the unknowns of both sides
@pytest.mark.parametrize("p,f,h,opt", [
    (16, 250.0, 0.34, dict(leaf_max=1)), (16, 250.0, 0.17, {}), (16, 250.0, 0.06, {}), (16, 250.0, 0.045, dict(max_depth=2)),
    (28, 250.0, 0.17, {}), (28, 1500.0, 0.06, {})])
@pytest.mark.parametrize("form", ["bm", "indirect"])
def test_normal_derivatives_vs_all_pairs(F, p, f, h, opt, form):
    room = synth.shoebox(3.0, 2.5, 2.0, h)
    ctx = F.Context(0, p_min=p, **opt)
    ctx.fmmbem_set_mesh(room.vertices, room.triangles)
    ctx.fmmbem_set_wavenumber(synth.wavenumber(f))
    ctx.fmmbem_set_admittance(room.beta)
    ctx.fmmbem_set_formulation(F.FMMBEM_DIRECT_BM if form == "bm" else F.FMMBEM_INDIRECT)
    X = synth.complex_normal(ctx.fmmbem_num_unknowns(), 5)
    ref = ctx.fmmbem_matvec(X, exact_far=True)
    for prec, tol in ((F.FMMBEM_FP64, 2e-6), (F.FMMBEM_MIXED, 1e-4)):
        if prec == F.FMMBEM_MIXED and p > 16:
            continue  # FP32 does not hold the radial functions of p = 28 at this k times box side
        y = ctx.fmmbem_matvec(X, precision=prec)
        assert np.linalg.norm(y - ref) < tol * np.linalg.norm(ref), (prec, np.linalg.norm(y - ref) / np.linalg.norm(ref))
    ctx.close()
