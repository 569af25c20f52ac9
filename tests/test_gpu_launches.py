"""Geometry set-up of grids far larger than the rest of the tests': rays and rows
beyond what one launch takes."""
import numpy as np
import pytest

from paper_2605_04335_amd import workloads as W

pytestmark = pytest.mark.gpu


def slab():
    """4 x 8208 x 8208 cells, the layer x = 1 solid, between two sheets across the box: 67.4 million rays."""
    n, m = 8208, 64
    f = [np.arange(5.0), np.arange(n + 1.0), np.arange(n + 1.0)]
    g = np.linspace(-3.0, n + 3.0, m + 1)
    y, z = np.meshgrid(g, g, indexing="ij")
    v = np.concatenate([np.stack([np.full(y.size, x), y.ravel(), z.ravel()], 1) for x in (1.2, 1.8)])
    q = (np.arange(m)[:, None] * (m + 1) + np.arange(m)).ravel()
    one = np.concatenate([np.stack([q, q + m + 1, q + m + 2], 1), np.stack([q, q + m + 2, q + 1], 1)])
    t = np.concatenate([one, one[:, ::-1] + (m + 1) ** 2]).astype(np.int32)
    return f, [W.Body(v, t, W.KIND_CLOSED)], n


# a closed body across more rays than a launch of a wavefront each takes
def test_classification_of_the_largest_projection():
    import paper_2605_04335_amd as P
    f, bodies, n = slab()
    flags, cst = P.classify(*f, bodies)
    assert (cst["n_solid"], cst["n_ghost"], cst["n_mghost"], cst["pin"]) == (n * n, n * n, 0, 0)
    x = flags.view(n * n, 4)
    assert bool((x[:, 1] == 3).all()) and bool((x[:, 2:] == 0).all()) and bool((x[1:, 0] == 0).all())
    assert int(x[0, 0]) == 8
