"""The four near integrals (L, M, L', M') of single triangles against the oracle's adaptive quadrature,
at the points and wavenumbers where their terms are easily lost: on and close to the lines of the
edges, beyond the ends."""
import numpy as np
import pytest

from oracle import bem

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F():
    from paper_2103_16073_amd import fmmbem
    fmmbem.lib()
    return fmmbem


EDGES = [((0, 0, 0), (1, 0, 0)), ((1, 0, 0), (0, 1, 0)), ((0, 1, 0), (0, 0, 0))]


def probes(points, normals):
    """The right triangle of unit legs (element 0), a small triangle centred at every point with the given
    normal, and two far ones that make the octree's leaves larger than r_c and the volume positive."""
    V, T = [np.array(p, float) for p in ((0, 0, 0), (1, 0, 0), (0, 1, 0))], [(0, 1, 2)]
    out = np.full(3, 3 ** -0.5)
    faces = [(x, n, 0.2) for x, n in zip(points, normals)] + [(-9.0 * out, -out, 1.5), (9.0 * out, out, 1.5)]
    for x, n, size in faces:
        a = np.cross(n, [0.3, -0.2, 0.9] if abs(n[2]) < 0.9 else [1.0, 0.0, 0.0])
        a *= size / np.linalg.norm(a)
        b = np.cross(n, a)
        i = len(V)
        V += [x + a, x - 0.5 * a + np.sqrt(0.75) * b, x - 0.5 * a - np.sqrt(0.75) * b]
        T.append((i, i + 1, i + 2))
    return np.array(V), np.array(T)


def unit(rng, n):
    v = rng.normal(size=(n, 3))
    return v / np.linalg.norm(v, axis=1)[:, None]


def near_lines(rng, rhos):
    """Points rho away from the edges' lines, 5 % to 80 % of an edge beyond either end, in and off the
    triangle's plane; normals of all directions and the triangle's own."""
    P, N = [], []
    for a, b in EDGES:
        a, b = np.array(a, float), np.array(b, float)
        for p, q in ((a, b), (b, a)):
            for rho in rhos:
                t = (b - a) / np.linalg.norm(b - a)
                off = np.cross(t, unit(rng, 1)[0]) if len(P) % 2 else np.cross(t, [0.0, 0.0, 1.0])
                P.append(q + rng.uniform(0.05, 0.8) * (q - p) + rho * off / np.linalg.norm(off))
                N.append(np.array([0.0, 0.0, 1.0]) if len(P) % 3 == 0 else unit(rng, 1)[0])
    return P, N


def worst(F, V, T, k):
    """Largest error of the entries of element 0's column, as multiples of 1e-12 of |L| without its
    oscillation (a derivative: times 1 / edge or k)."""
    ctx = F.Context(0, rc=2.4)
    ctx.fmmbem_set_mesh(V, T)
    ctx.fmmbem_set_wavenumber(k)
    ctx.fmmbem_set_admittance(np.full(len(T), 0.5))
    ctx.fmmbem_set_formulation(F.FMMBEM_INDIRECT)
    r, c, L, M = ctx.fmmbem_near_entries()
    Lp, Mp = ctx.fmmbem_near_entries_n()
    ctx.close()
    cen, nrm, area = bem.geometry(V, T)
    w, d = np.zeros(4), max(1.0, k)
    sel = np.nonzero(c == 0)[0]
    assert len(sel) == len(T) - 2
    for e in sel:
        i = r[e]
        ref = bem.pair4(cen[i], nrm[i], V[T[0]], k, self=(i == 0), eta=0.15)
        s = 1e-12 * area[0] / (4 * np.pi * max(0.3, np.linalg.norm(cen[i] - cen[0])))
        w = np.maximum(w, np.abs(np.array([L[e], M[e], Lp[e], Mp[e]]) - ref) / (s * np.array([1.0, d, d, d * d])))
    return w


# k r of the farthest vertices 0.7, 2.5 and 3.9
@pytest.mark.parametrize("k", [0.3, 1.0, 1.6])
def test_on_the_lines_of_edges(F, k):
    V, T = probes(*near_lines(np.random.default_rng(1), [0.0] * 3))
    w = worst(F, V, T, k)
    assert w.max() < 1.0, w


@pytest.mark.parametrize("k", [0.3, 1.0, 1.6])
def test_close_to_the_lines_of_edges(F, k):
    V, T = probes(*near_lines(np.random.default_rng(1), [1e-2, 1e-4, 1e-6, 1e-8, 1e-9, 1e-10, 1e-11, 1e-12, 3e-13, 1e-13]))
    w = worst(F, V, T, k)
    assert w.max() < 1.0, w


def around(rng):
    """Points beside, above and next to the triangle (0.02 to 1 edges off), in its plane, close to its
    edges' lines and on them."""
    P, N = near_lines(rng, [0.0, 1e-10, 1e-6, 1e-3])
    for z in (0.02, 0.1, 0.4, 1.0):
        for x, y in rng.uniform(-0.3, 1.2, (8, 2)):
            P.append(np.array([x, y, z]))
    for phi in rng.uniform(0, 2 * np.pi, 12):
        P.append(np.array([1 / 3, 1 / 3, 0.0]) + rng.uniform(0.95, 1.6) * np.array([np.cos(phi), np.sin(phi), 0.0]))
    N += [np.array([0.0, 0.0, 1.0]) if i % 3 == 0 else unit(rng, 1)[0] for i in range(len(P) - len(N))]
    return P, N


# either side of the largest k r of the series (4; the farthest vertices at 2.5 k) and far beyond
@pytest.mark.parametrize("k", [0.5, 1.5, 1.9, 2.3, 4.0, 6.0, 10.0, 18.0, 28.0])
def test_wavenumbers(F, k):
    V, T = probes(*around(np.random.default_rng(4)))
    w = worst(F, V, T, k)
    assert w.max() < 1.0, w


@pytest.mark.parametrize("form", ["bm", "indirect"])
def test_products_with_a_point_on_an_edges_line(F, form):
    """An element on another surface that lies on the line of an edge: the rows of the product."""
    V, T = probes(*near_lines(np.random.default_rng(2), [0.0]))
    n, k = len(T), 1.0
    ctx = F.Context(0, rc=2.4)
    ctx.fmmbem_set_mesh(V, T)
    ctx.fmmbem_set_wavenumber(k)
    beta = np.linspace(0.2, 0.8, n)
    ctx.fmmbem_set_admittance(beta)
    ctx.fmmbem_set_formulation(F.FMMBEM_DIRECT_BM if form == "bm" else F.FMMBEM_INDIRECT)
    rng = np.random.default_rng(3)
    m = ctx.fmmbem_num_unknowns()
    x = rng.normal(size=m) + 1j * rng.normal(size=m)
    y = ctx.fmmbem_matvec(x, exact_far=True)[0]
    ctx.close()
    rows = np.arange(n)
    if form == "bm":
        ref = bem.bm_matvec_rows(V, T, k, beta, 2.4, x, rows)
    else:
        ref = np.concatenate(bem.indirect_matvec_rows(V, T, k, beta, beta, 2.4, x, rows))
    assert np.abs(y - ref).max() < 1e-12 * np.abs(ref).max(), np.abs(y - ref).max() / np.abs(ref).max()
