"""Matrix-core translation tiles over truncation numbers at the edges of their row blocks and passes,
against the library's own all-pairs product (itself checked against the oracle)."""
import numpy as np
import pytest

from paper_2103_16073_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F():
    from paper_2103_16073_amd import fmmbem
    fmmbem.lib()
    return fmmbem


# leaf-level p = 16 (the fused tiles) up to 50, parents to 90: degrees of one to six 16-row blocks
@pytest.mark.parametrize("f", [250.0, 700.0, 1000.0, 1530.0, 2500.0, 5000.0])
@pytest.mark.parametrize("opt", [dict(mfma=2, lane_tiles=2), dict(mfma=2, lane_tiles=2, fused=0), {}])
def test_products_over_truncation_numbers(F, f, opt):
    room = synth.shoebox(3.0, 2.5, 2.0, 0.17)
    k = synth.wavenumber(f)
    ctx = F.Context(0, leaf_max=8, max_depth=3, **opt)
    ctx.fmmbem_set_mesh(room.vertices, room.triangles)
    ctx.fmmbem_set_wavenumber(k)
    ctx.fmmbem_set_admittance(room.beta)
    X = synth.complex_normal(room.n, 5, count=4)
    ref = ctx.fmmbem_matvec(X, exact_far=True)
    assert ctx.fmmbem_get_info().depth == 3
    for nr in (1, 2, 4):
        for prec, tol in ((F.FMMBEM_FP64, 2e-6), (F.FMMBEM_MIXED, 1e-5)):
            y = ctx.fmmbem_matvec(X[:nr], precision=prec)
            err = np.linalg.norm(y - ref[:nr], axis=1) / np.linalg.norm(ref[:nr], axis=1)
            assert err.max() < tol, (nr, prec, err, list(ctx.fmmbem_get_info().p)[:4])
    ctx.close()


# classes of a few jobs (octrees of depth 2 and 3 at p = 16): the fused tiles with most of their padding
# skipped against whole-vector tiles; same sums, other order of rounding (a product's own: 1e-14)
@pytest.mark.parametrize("h,depth", [(0.5, 2), (0.2, 2), (0.2, 3)])
def test_small_classes_vs_whole_tiles(F, h, depth):
    room = synth.shoebox(3.0, 2.5, 2.0, h)
    X = synth.complex_normal(room.n, 5, count=4)
    out = []
    for opt in ({}, dict(lane_tiles=0)):
        ctx = F.Context(0, leaf_max=1, max_depth=depth, **opt)
        ctx.fmmbem_set_mesh(room.vertices, room.triangles)
        ctx.fmmbem_set_wavenumber(synth.wavenumber(150.0))
        ctx.fmmbem_set_admittance(room.beta)
        assert ctx.fmmbem_get_info().depth == depth
        out.append([ctx.fmmbem_matvec(X[:nr], precision=prec) for nr in (1, 2, 4)
                    for prec in (F.FMMBEM_FP64, F.FMMBEM_MIXED)])
        ctx.close()
    for i, (a, b) in enumerate(zip(*out)):
        assert np.linalg.norm(a - b) < (1e-12 if i % 2 == 0 else 1e-5) * np.linalg.norm(b), i
