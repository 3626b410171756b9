"""Translation tables at the sizes where their kernels' split of the work changes, against the
oracle's projections."""
import numpy as np
import pytest

from oracle import coeffs as OC

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F():
    from paper_2103_16073_amd import fmmbem
    fmmbem.lib()
    return fmmbem


# the smallest tables, and one, two and three strips of 128 diagonal rows with their remainders
@pytest.mark.parametrize("p,ktau", [(1, 2.0), (2, 2.0), (3, 2.0), (4, 2.0), (129, 100.0), (130, 100.0), (131, 100.0),
                                    (132, 100.0), (259, 200.0)])
def test_stabilised_coaxial_table_strip_edges(F, p, ktau):
    blocks = F.fmmbem_coaxial_table(1, ktau, p, method=1)
    scale = np.max(np.abs(blocks[0]))
    for m in sorted({0, 1, 2, p // 2, p - 3, p - 2, p - 1} & set(range(p))):
        rows = sorted({m, m + 1, m + 2, (m + p) // 2, p - 1} & set(range(m, p)))
        ref = OC.coaxial_projection_order("RR", 1.0, ktau, p, m, rows=rows)
        for nn in rows:
            err = np.max(np.abs(blocks[m][nn - m] - ref[nn, m:]))
            assert err < 1e-9 * scale, (m, nn, err / scale)
