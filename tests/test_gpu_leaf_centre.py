"""An element whose centroid is exactly its leaf's centre (k r = 0 in the regular basis), at truncation
numbers on either side of 41, beyond which the spherical Bessel functions take another recurrence."""
import numpy as np
import pytest

from paper_2103_16073_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F():
    from paper_2103_16073_amd import fmmbem
    fmmbem.lib()
    return fmmbem


def with_centred_element(room, ix):
    """The room's mesh and one triangle whose centroid is, to the last bit, the centre of the depth-2
    octree cell ix (of coordinates whose mantissa is below 4/3: every one of them is a third)."""
    lo, hi = room.vertices.min(0), room.vertices.max(0)
    side = float((hi - lo).max()) * (1.0 + 1e-6) + 1e-9
    centre = [float(0.5 * (lo[d] + hi[d]) - 0.5 * side + (ix[d] + 0.5) * (side / 4)) for d in range(3)]
    tri = np.array(centre) + np.array([[0.05, 0.02, 0.0], [-0.03, 0.04, 0.01], [-0.02, -0.06, -0.01]])
    third = [next(t for t in (3.0 * c, np.nextafter(3.0 * c, 0.0), np.nextafter(3.0 * c, 9.0)) if t / 3.0 == c) for c in centre]
    tri[2] = np.array(third) - (tri[0] + tri[1])  # exact: the two differ by less than a factor of 2
    assert ((tri[0] + tri[1] + tri[2]) / 3.0 == centre).all()
    n = len(room.vertices)
    return (np.vstack([room.vertices, tri]), np.vstack([room.triangles, [[n, n + 1, n + 2]]]),
            np.concatenate([room.beta, [0.3]]))


@pytest.mark.parametrize("p", [16, 40, 41, 42, 46, 51])
@pytest.mark.parametrize("form", ["direct", "bm", "indirect"])
def test_product_vs_all_pairs(F, p, form):
    room = synth.shoebox(3.0, 2.5, 2.0, 0.17)
    V, T, beta = with_centred_element(room, (1, 3, 1))
    kd = next(kd for kd in np.arange(1.0, 60.0, 0.05) if int(np.ceil(kd + 4.2 * np.cbrt(kd))) == p)
    ctx = F.Context(0, max_depth=2)
    ctx.fmmbem_set_mesh(V, T)
    ctx.fmmbem_set_wavenumber(kd / (3.0 / 4))
    ctx.fmmbem_set_admittance(beta)
    ctx.fmmbem_set_formulation({"direct": F.FMMBEM_DIRECT, "bm": F.FMMBEM_DIRECT_BM, "indirect": F.FMMBEM_INDIRECT}[form])
    x = synth.complex_normal(ctx.fmmbem_num_unknowns(), 5)
    ref = ctx.fmmbem_matvec(x, exact_far=True)[0]
    y = ctx.fmmbem_matvec(x)[0]
    info = ctx.fmmbem_get_info()
    ctx.close()
    assert info.depth == 2 and info.p[2] == p, (info.depth, info.p[2])
    assert np.isfinite(y).all(), np.nonzero(~np.isfinite(y))[0][:4]
    err = np.linalg.norm(y - ref) / np.linalg.norm(ref)
    at = np.arange(len(T) - 1, len(y), len(T))
    assert err < 2e-6 and np.abs(y[at] - ref[at]).max() < 2e-5 * np.abs(ref).max(), (err, y[at], ref[at])
