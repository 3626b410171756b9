"""Pair kernels (near field of a product, field at receivers) at the sizes where their split of the
work changes, against the oracle."""
import numpy as np
import pytest

from oracle import bem
from paper_2103_16073_amd import synth
from rc_check import oracle_rc

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F():
    from paper_2103_16073_amd import fmmbem
    fmmbem.lib()
    return fmmbem


def _ctx(F, room, k, **opt):
    ctx = F.Context(0, **opt)
    ctx.fmmbem_set_mesh(room.vertices, room.triangles)
    ctx.fmmbem_set_wavenumber(k)
    ctx.fmmbem_set_admittance(room.beta)
    return ctx


# leaves of a few targets (odd counts, single elements), of about 50, of about 270 (one pass of more
# than 128 lanes) and of more than 512 (several passes); the source list whole or in up to 16 pieces
@pytest.mark.parametrize("h,opt", [(0.5, {}), (0.34, dict(leaf_max=1)), (0.17, {}), (0.07, dict(max_depth=2)),
                                   (0.045, dict(max_depth=2)), (0.045, {})])
@pytest.mark.parametrize("form", ["direct", "bm"])
def test_near_field_leaf_sizes_vs_oracle(F, h, opt, form):
    """The all-pairs product (every pair through the pair kernel) to rounding and the FMM product to
    its truncation, one to four vectors, on sampled rows."""
    room = synth.shoebox(3.0, 2.5, 2.0, h)
    k = synth.wavenumber(250.0)
    ctx = _ctx(F, room, k, **opt)
    if form == "bm":
        ctx.fmmbem_set_formulation(F.FMMBEM_DIRECT_BM)
    rows = np.unique(np.linspace(0, room.n - 1, 40).astype(int))
    X = synth.complex_normal(room.n, 5, count=4)
    rc = oracle_rc(ctx, room)
    rowsf = bem.direct_matvec_rows if form == "direct" else bem.bm_matvec_rows
    ref = np.stack([rowsf(room.vertices, room.triangles, k, room.beta, rc, x, rows) for x in X])
    for nr in ((1, 2, 4) if form == "direct" else (1,)):
        y = ctx.fmmbem_matvec(X[:nr], exact_far=True)[:, rows]
        f = ctx.fmmbem_matvec(X[:nr])[:, rows]
        for q in range(nr):
            s = np.linalg.norm(ref[q])
            assert np.linalg.norm(y[q] - ref[q]) < 1e-12 * s, (nr, q, np.linalg.norm(y[q] - ref[q]) / s)
            assert np.linalg.norm(f[q] - ref[q]) < 2e-6 * s, (nr, q, np.linalg.norm(f[q] - ref[q]) / s)
    ctx.close()


# one to nine points (every points-per-workgroup shape and its remainders), several hundred, and more
# than one launch's worth; the near integrals reaching one cell, or (r_c above the leaf side) several
@pytest.mark.parametrize("h,opt", [(0.34, {}), (0.34, dict(rc=1.7)), (0.1, {})])
def test_field_point_counts_vs_oracle(F, h, opt):
    room = synth.shoebox(3.0, 2.5, 2.0, h)
    k = synth.wavenumber(250.0)
    ctx = _ctx(F, room, k, **opt)
    rs, rec = synth.source_and_receivers(room, 700)
    ctx.fmmbem_set_sources(rs)
    V, T = room.vertices, room.triangles
    c = V[T].mean(axis=1)
    nrm = np.cross(V[T[:, 1]] - V[T[:, 0]], V[T[:, 2]] - V[T[:, 0]])
    nrm /= np.linalg.norm(nrm, axis=1)[:, None]
    sel = np.linspace(0, room.n - 1, 40).astype(int)
    # points in the room, just inside and just outside the walls, and far outside the octree's cube
    pts = np.vstack([rec, c[sel] - 0.03 * nrm[sel], c[sel] + 0.03 * nrm[sel], [[30.0, -4.0, 2.0], [3.5, 2.6, 2.2]]])
    pts = pts[np.random.default_rng(4).permutation(len(pts))]
    x = synth.complex_normal(room.n, 77)
    rc = opt.get("rc") or oracle_rc(ctx, room)
    ref = bem.direct_receivers(V, T, k, room.beta, rs[0], rc, x, pts)
    for nr in (1, 2, 3, 4, 5, 8, 9, len(pts)):
        psi = ctx.fmmbem_eval_field(0, pts[:nr], x)
        assert np.max(np.abs(psi - ref[:nr])) < 1e-10 * np.linalg.norm(ref) / np.sqrt(len(ref)), nr
    if h == 0.34:
        many = np.tile(pts, (66000 // len(pts) + 1, 1))
        psi = ctx.fmmbem_eval_field(0, many, x)
        assert np.max(np.abs(psi - np.tile(ref, len(many) // len(pts)))) < 1e-10 * np.linalg.norm(ref) / np.sqrt(len(ref))
    ctx.close()


@pytest.mark.parametrize("ns", [1, 2, 3, 4, 7])
def test_right_hand_sides_of_many_sources_vs_oracle(F, ns):
    """Sources taken four, two and one per pass: every right-hand side on sampled rows against the
    oracle, amplitudes included, and a product afterwards as before."""
    room, k = synth.config_room(1)
    ctx = _ctx(F, room, k)
    x = synth.complex_normal(room.n, 5)
    before = ctx.fmmbem_matvec(x)
    rs = synth.sample_points(room, ns, 9)
    amp = synth.complex_normal(ns, 6)
    ctx.fmmbem_set_sources(rs, amp)
    b = ctx.fmmbem_rhs()
    rows = np.unique(np.linspace(0, room.n - 1, 60).astype(int))
    rc = oracle_rc(ctx, room)
    for s in range(ns):
        ref = amp[s] * bem.direct_rhs_rows(room.vertices, room.triangles, k, room.beta, rs[s], rc, rows)
        assert np.linalg.norm(b[s, rows] - ref) < 1e-6 * np.linalg.norm(ref), s
    assert np.array_equal(ctx.fmmbem_matvec(x), before)
    ctx.close()
