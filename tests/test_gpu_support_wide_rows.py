"""Edge support where rows hold hundreds of entries below the 8,192 highest ranks,
as in dense graphs without skew: the lengths at which such a row takes the whole
LDS region or is searched in device memory, with and without entries among the
highest ranks."""
import numpy as np
import pytest

from tests.test_gpu_support_hubs import check_all

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k,joined", [(342, 0), (343, 0), (683, 0), (684, 0), (400, 30), (600, 100), (342, 340), (345, 337)])
def test_long_rows_below_the_hubs(k, joined):
    """K_k below a regular graph of 8,300 vertices of a higher degree, each of
    its vertices joined to `joined` of those: rows of up to k - 1 entries below
    the highest ranks and `joined` among them."""
    rng = np.random.default_rng(1000 * k + joined)
    a, b = np.triu_indices(k, 1)
    n, deg = 8300, k + joined + 40
    ring = np.arange(n)
    s = [a] + [k + ring for j in range(1, deg // 2 + 1)]
    d = [b] + [k + (ring + j) % n for j in range(1, deg // 2 + 1)]
    for v in range(k if joined else 0):
        s.append(np.full(joined, v))
        d.append(k + rng.choice(n, joined, replace=False))
    check_all(k + n, np.concatenate(s).astype(np.int32), np.concatenate(d).astype(np.int32))
