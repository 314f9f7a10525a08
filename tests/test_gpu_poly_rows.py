"""The polynomial filter and its adjoint where their rows change form: gaps
below and past a byte (scattered points, a bandwidth that reaches them), rows
with empty slots, blocks of points with more and with fewer in-edges than one
pass holds (a hub, single points), and K other than 8, against the oracle with
the tolerances of the other tests of this filter."""
import math

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle as O  # noqa: E402
from paper_2401_09721_amd import fgbd  # noqa: E402

from gpu_helpers import COLOUR_TOL, dev  # noqa: E402

pytestmark = pytest.mark.gpu


def check(g, n, ncoef, sg, seed):
    rng = np.random.default_rng(seed)
    coef = rng.uniform(-0.5, 1.0, size=ncoef)
    x, go = rng.uniform(0, 255, size=(n, 3)).astype(np.float32), rng.standard_normal((n, 3)).astype(np.float32)
    ct, st = dev(coef, torch.float32), torch.tensor(sg, dtype=torch.float64, device="cuda")
    out, saved = fgbd.poly_filter(g, dev(x, torch.float32), ct, st)
    gx, gc, gs = fgbd.poly_filter_backward(g, saved, ct, st, dev(go, torch.float32))
    torch.cuda.synchronize()
    col, d2 = g.col.cpu().numpy(), g.dist2.cpu().numpy()
    coef32 = coef.astype(np.float32).astype(np.float64)
    assert np.max(np.abs(out.cpu().numpy() - O.poly_filter(col, d2, x, coef32, sg))) <= COLOUR_TOL
    rx, rc, rs = O.poly_filter_grads(col, d2, x, coef32, sg, go)
    assert np.max(np.abs(gx.cpu().numpy() - rx)) <= 1e-3 * max(1.0, np.max(np.abs(rx)))
    assert np.allclose(gc.cpu().numpy(), rc, rtol=1e-3, atol=1e-3 * np.max(np.abs(rc)))
    assert math.isclose(float(gs), rs, rel_tol=1e-3, abs_tol=1e-3 * max(1.0, abs(rs)))


@pytest.mark.parametrize("n", [1, 5, 255, 256, 257, 3000])
@pytest.mark.parametrize("spread,sg", [(20, 1.5), (60, 9.0), (1000, 150.0)])
@pytest.mark.parametrize("k", [8, 6, 16])
def test_gaps_and_empty_slots(n, spread, sg, k):
    rng = np.random.default_rng(n + spread)
    xyz = rng.integers(0, spread, size=(n, 3)).astype(np.int32)
    g = fgbd.build_slg(dev(xyz, torch.int32), fgbd.default_params(bits=10, k=k))
    check(g, n, 4, sg, n)


@pytest.mark.parametrize("n,hubs", [(2048, 1), (5000, 3), (700, 256)])
def test_in_edges_of_a_block(n, hubs):
    """Every point has an edge to each of up to 8 hubs, so a block of points
    holds thousands of in-edges and most blocks none."""
    rng = np.random.default_rng(hubs)
    col = np.full((n, 8), -1, np.int32)
    for k in range(min(hubs, 8)):
        col[:, k] = rng.integers(0, hubs, size=n) if hubs > 8 else k
    col[col == np.arange(n)[:, None]] = n - 1
    d2 = np.where(col >= 0, np.sort(rng.integers(1, 400, size=(n, 8)), axis=1), 0).astype(np.int32)
    c, d = dev(col, torch.int32), dev(d2, torch.int32)
    g = fgbd.SLGraph(c, d, torch.zeros((n, 8), dtype=torch.float32, device="cuda"), None)
    check(g, n, 3, 12.0, n)
