"""The polynomial filter at the lines of its variants.  Forward, around the
number of points from which its steps read packed rows (450,000), with groups of 64 points whose gaps all fit a byte, none
do, or some: against the oracle, with the tolerances of this filter's other
tests; and the same results from a graph's first points as from those alone.
Backward, on both sides of each line between in-edges read by rows and through
LDS, and at small sizes, against the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2401_09721_amd import fgbd  # noqa: E402

from gpu_helpers import dev  # noqa: E402
from test_gpu_poly_rows import check  # noqa: E402

pytestmark = pytest.mark.gpu


def _points(n, spread, seed):
    """Points of a dense slab in raster order with, in every `spread`-th run of
    300, one far from the others (0: in none; 1: all far apart)."""
    rng = np.random.default_rng(seed)
    i = np.arange(n)
    g = np.stack([i // 900, i // 30 % 30, i % 30], 1)
    if spread == 1:
        g = rng.integers(0, 1 << 15, size=(n, 3))
    elif spread:
        at = i[(i // 300) % spread == 0][::300]
        g[at] = rng.integers(2000, 1 << 15, size=(len(at), 3))
    return g.astype(np.int32)


@pytest.mark.parametrize("n", [449_999, 450_000, 450_001, 450_063])
@pytest.mark.parametrize("spread,sg", [(0, 1.3), (7, 1.3), (1, 900.0)])
def test_forms_around_the_line(n, spread, sg):
    g = fgbd.build_slg(dev(_points(n, spread, n), torch.int32), fgbd.default_params(bits=15, num_dirs=3))
    check(g, n, 3, sg, n)


@pytest.mark.parametrize("spread", [0, 7, 1])
def test_forms_give_the_same_bits(spread):
    """Rows of the first points, whose neighbours are all among them, in a
    graph past the line and in one of these points alone: every output of the
    forward call has the same bits."""
    n, m = 450_000, 120_000
    prm = fgbd.default_params(bits=15, num_dirs=3)
    part = fgbd.build_slg(dev(_points(m, spread, 5), torch.int32), prm)
    filler = torch.full((n - m, 8), -1, dtype=torch.int32, device="cuda")
    whole = fgbd.SLGraph(torch.cat([part.col, filler]), torch.cat([part.dist2, torch.zeros_like(filler)]),
                         torch.zeros((n, 8), dtype=torch.float32, device="cuda"), None)
    rng = np.random.default_rng(spread)
    x = dev(rng.uniform(0, 255, size=(n, 3)), torch.float32)
    coef = dev([0.3, -0.2, 0.5, 0.4], torch.float32)
    sg = torch.tensor(1.3 if spread != 1 else 900.0, dtype=torch.float64, device="cuda")
    out, saved = fgbd.poly_filter(whole, x, coef, sg)
    pout, psaved = fgbd.poly_filter(part, x[:m].contiguous(), coef, sg)
    torch.cuda.synchronize()
    assert torch.equal(out[:m], pout)
    rows = 2 * 4 - 1  # the iterates, then u_m
    assert torch.equal(saved[:rows * 3 * n].view(rows, n, 3)[:, :m], psaved[:rows * 3 * m].view(rows, m, 3))


@pytest.mark.parametrize("n,k,ncoef", [(200_000, 8, 4), (200_001, 8, 4), (131_072, 12, 4), (131_073, 12, 4), (90_625, 32, 4),
                                       (90_626, 32, 4), (3000, 7, 4), (3000, 6, 4), (3000, 16, 3), (257, 16, 5),
                                       (1, 8, 4)])
def test_adjoint_lines(n, k, ncoef):
    rng = np.random.default_rng(n + k)
    side = max(8, int((4 * n) ** (1 / 3)))
    xyz = rng.integers(0, side, size=(n, 3)).astype(np.int32)
    g = fgbd.build_slg(dev(xyz, torch.int32), fgbd.default_params(bits=10, num_dirs=8, k=k))
    check(g, n, ncoef, 1.5, n)
