"""The neighbour selection's variants at their edges: four lanes a point and
one, 31-bit keys whose distance field overflows on some rows (sparse points)
and the 64-bit selection of graphs that keep every candidate.  Graphs are
compared with the oracle's, exactly."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2401_09721_amd import fgbd  # noqa: E402

from test_gpu_parity import check_graph  # noqa: E402

pytestmark = pytest.mark.gpu


def points(n, seed, spread=1024):
    """n random points, some of them twice, a dense block among them."""
    rng = np.random.default_rng(seed)
    g = rng.integers(0, spread, size=(n, 3))
    g[: n // 4] = rng.integers(500, 512, size=(n // 4, 3))
    return g.astype(np.int32)


@pytest.mark.parametrize("n", [1, 2, 9, 64, 257, 5000])
@pytest.mark.parametrize("L,w,K", [(3, 1, 6), (4, 1, 8), (2, 2, 8), (1, 4, 8), (5, 4, 7), (8, 4, 12), (16, 4, 16),
                                   (8, 1, 8), (6, 2, 3)])
def test_sparse_points(n, L, w, K):
    check_graph(points(n, n + 10 * L), fgbd.default_params(bits=10, num_dirs=L, window=w, k=K))


@pytest.mark.parametrize("n", [81920, 81921])
@pytest.mark.parametrize("L,K", [(8, 8), (3, 16)])
def test_lanes_per_point(n, L, K):
    check_graph(points(n, 3, spread=300), fgbd.default_params(bits=10, num_dirs=L, window=4, k=K))
