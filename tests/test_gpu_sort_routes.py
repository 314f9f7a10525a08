"""Which route the sort takes, counted by the context's profiling, each case on
a context of its own so that no call before it decides: one top-digit pass and
the local sort, or 8-bit passes.  Graphs are compared with the oracle's,
exactly."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle as O  # noqa: E402
from paper_2401_09721_amd import fgbd  # noqa: E402

from gpu_helpers import dev  # noqa: E402

pytestmark = pytest.mark.gpu


class Sorter:
    """build_slg on one context: the graph's check and the route taken."""

    def __init__(self):
        self.ctx = fgbd.Context("cuda")
        self.ctx.profile(True)

    def route(self):
        kinds = self.ctx.profile_read()
        return kinds["local_sort"][1], kinds["radix_downsweep"][1]

    def __call__(self, xyz, prm, check=True):
        self.ctx.profile_read()
        g = fgbd.build_slg(dev(xyz, torch.int32), prm, ctx=self.ctx)
        torch.cuda.synchronize()  # lets the next call read what this one found
        if check:
            col, d2 = O.slg_graph(xyz, prm.bits, prm.num_dirs, prm.window, prm.k)
            assert np.array_equal(g.col.cpu().numpy(), col)
            assert np.array_equal(g.dist2.cpu().numpy(), np.minimum(d2, (1 << 31) - 1))
        return self.route()

    def __enter__(self):
        return self

    def __exit__(self, *e):
        self.ctx.close()


TOP_DIGIT = (1, 1)


def plane(rng, bits, n):
    """n points of one plane normal to a scan axis: one top digit holds all."""
    flat = rng.choice(1 << (2 * min(bits, 10)), size=n, replace=False)
    return np.stack([flat >> min(bits, 10), flat & ((1 << min(bits, 10)) - 1), np.full(n, 300)], 1).astype(np.int32)


def test_code_widths_do_not_route_each_other():
    rng = np.random.default_rng(1)
    wide, narrow = plane(rng, 11, 40000), rng.integers(0, 1024, size=(5000, 3)).astype(np.int32)
    pw, pn = fgbd.default_params(bits=11), fgbd.default_params(bits=10)
    with Sorter() as s:
        assert s(wide, pw, check=False) == TOP_DIGIT  # its range is found to be very large
        assert s(narrow, pn) == TOP_DIGIT
        assert s(wide, pw) == (0, 5)  # 35-bit codes: five passes of 8 bits
        assert s(narrow, pn) == TOP_DIGIT
    with Sorter() as s:
        crowded = plane(rng, 10, 40000)
        assert s(crowded, pn, check=False) == TOP_DIGIT
        assert s(wide[:5000], pw) == TOP_DIGIT
        assert s(crowded, pn) == (0, 4)
        assert s(wide[:5000], pw) == TOP_DIGIT


def crowded_voxels(rng, bits, voxels, times, others, turn):
    """`voxels` voxels of one scan-line neighbourhood, `times` points each, one
    voxel after the other or in turn, and scattered points."""
    v = rng.integers(0, 1 << bits, size=(1, 3)) // 2 + rng.integers(0, 3, size=(voxels, 3))
    many = np.tile(v, (times, 1)) if turn else np.repeat(v, times, axis=0)
    g = np.concatenate([many, rng.integers(0, 1 << bits, size=(others, 3))])
    return np.minimum(g, (1 << bits) - 1).astype(np.int32)


@pytest.mark.parametrize("turn", [False, True], ids=["runs", "turn"])
@pytest.mark.parametrize("bits,voxels,times,others", [(10, 1, 513, 1), (10, 1, 1024, 0), (10, 3, 700, 1025),
                                                      (10, 8, 1024, 0), (10, 2, 4000, 191), (3, 40, 200, 90),
                                                      (11, 5, 1500, 600), (16, 4, 2000, 3000), (17, 3, 600, 200)])
def test_long_bins(bits, voxels, times, others, turn):
    """Bins past the length that is ranked by counting: the window's keys take
    digit passes in LDS (at 16 and 17 bits also over the code bits below the
    keys), and equal codes keep index order."""
    rng = np.random.default_rng(voxels * times)
    g = crowded_voxels(rng, bits, voxels, times, others, turn)
    with Sorter() as s:
        assert s(g, fgbd.default_params(bits=bits)) == TOP_DIGIT


@pytest.mark.parametrize("n", [1, 65, 1024, 1025, 5000, 8192])
@pytest.mark.parametrize("bits", [1, 2, 3, 10])
def test_one_code(bits, n):
    """Every point in one voxel: no digit differs, index order alone decides."""
    g = np.tile(np.array([[1, 0, 1]], np.int32), (n, 1))
    with Sorter() as s:
        assert s(g, fgbd.default_params(bits=bits)) == TOP_DIGIT
