"""Which route the sort takes, counted by the context's profiling, each case on
a context of its own so that no call before it decides: one top-digit pass and
the local sort, or 8-bit passes.  Graphs are compared with the oracle's,
exactly."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle as O  # noqa: E402
from paper_2401_09721_amd import fgbd  # noqa: E402

from gpu_helpers import compare_denoise, dev  # noqa: E402

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


def planes(rng, bits, n, others, side=None):
    """Planes of n points normal to each scan axis, and scattered points."""
    side = side or min(1 << bits, 1024)
    out = [rng.integers(0, 1 << bits, size=(others, 3))]
    for axis in range(3):
        flat = rng.choice(side * side, size=n, replace=n > side * side)
        out.append(np.insert(np.stack([flat // side, flat % side], 1), axis, (1 << bits) // 3 + axis, axis=1))
    return np.concatenate(out).astype(np.int32)


@pytest.mark.parametrize("order", ["raster", "shuffled"])
@pytest.mark.parametrize("bits,n,others", [(10, 8193, 0), (10, 12288, 4096), (10, 28000, 5000), (10, 70000, 20000),
                                           (7, 16384, 300), (11, 9000, 1), (11, 40000, 9000), (13, 30000, 3000),
                                           (14, 20000, 500), (15, 10000, 2000), (16, 5400, 100)])
def test_large_buckets(bits, n, others, order):
    """One top digit with more points than a block's LDS holds, a first call's
    route: the windows that the bucket reaches share it."""
    rng = np.random.default_rng(n + bits)
    g = planes(rng, bits, n, others)
    g = g[rng.permutation(len(g))] if order == "shuffled" else g[np.lexsort((g[:, 2], g[:, 1], g[:, 0]))]
    with Sorter() as s:
        assert s(g, fgbd.default_params(bits=bits)) == TOP_DIGIT


@pytest.mark.parametrize("order", ["runs", "turn", "shuffled"])
@pytest.mark.parametrize("bits,voxels,times,others", [(10, 1, 8193, 0), (10, 1, 20000, 3000), (10, 3, 9000, 9000),
                                                      (10, 60, 700, 0), (11, 2, 10000, 500), (13, 1, 30000, 30000),
                                                      (16, 1, 9000, 7000)])
def test_large_buckets_of_few_voxels(bits, voxels, times, others, order):
    """Bins of a large bucket that hold more than a range does, down to one code."""
    rng = np.random.default_rng(times + voxels)
    g = crowded_voxels(rng, bits, voxels, times, others, order == "turn")
    g[-others // 2:, 2] = g[0, 2]  # (half of the others in the bucket's plane)
    if order == "shuffled":
        g = g[rng.permutation(len(g))]
    with Sorter() as s:
        assert s(g, fgbd.default_params(bits=bits)) == TOP_DIGIT


@pytest.mark.parametrize("bits,L,n", [(1, 8, 50000), (2, 3, 60000), (3, 8, 60000), (11, 8, 40000)])
def test_large_buckets_of_one_code(bits, L, n):
    """Buckets in which every code is the same, shared as they stand."""
    rng = np.random.default_rng(n)
    g = rng.integers(0, 2, size=(n, 3)).astype(np.int32) * ((1 << min(bits, 3)) - 1)
    with Sorter() as s:
        assert s(g, fgbd.default_params(bits=bits, num_dirs=L)) == TOP_DIGIT


@pytest.mark.parametrize("bits", [10, 11])
def test_large_buckets_of_a_batch(bits):
    prm = fgbd.default_params(bits=bits)
    rng = np.random.default_rng(bits)
    xyz = [planes(rng, bits, n, others) for n, others in ((9000, 100), (30, 20), (13000, 5000), (8200, 0))]
    xyz = [x[np.lexsort((x[:, 2], x[:, 1], x[:, 0]))] for x in xyz]
    rgb = [rng.uniform(0, 255, size=x.shape).astype(np.float32) for x in xyz]
    off = np.concatenate([[0], np.cumsum([len(x) for x in xyz])]).astype(np.int64)
    ctx = fgbd.Context("cuda")
    ctx.profile(True)
    out, res = fgbd.denoise_batched(dev(np.concatenate(xyz), torch.int32), dev(np.concatenate(rgb), torch.float32),
                                    dev(off, torch.int64), prm, ctx=ctx)
    torch.cuda.synchronize()
    assert ctx.profile_read()["local_sort"][1] == 1
    out, recs = out.cpu().numpy(), fgbd.read_results(res)
    for s in range(len(xyz)):
        compare_denoise(out[off[s]:off[s + 1]], recs[s], xyz[s], rgb[s], prm)
    ctx.close()


@pytest.mark.parametrize("bits,passes", [(10, 4), (11, 5)])
def test_calls_ahead_of_the_answer(bits, passes):
    """Calls made one after another, none waited for: once crowded points were
    found, one call in 33 tries the top-digit route again."""
    g = plane(np.random.default_rng(3), bits, 40000)
    prm = fgbd.default_params(bits=bits)
    with Sorter() as s:
        assert s(g, prm, check=False) == TOP_DIGIT
        x = dev(g, torch.int32)
        graphs = [fgbd.build_slg(x, prm, ctx=s.ctx) for _ in range(60)]
        torch.cuda.synchronize()
        assert s.route() == (1, 1 + 59 * passes)
        for other in graphs[1:]:
            assert torch.equal(other.col, graphs[0].col) and torch.equal(other.dist2, graphs[0].dist2)
        assert s(g, prm) == (0, passes)


@pytest.mark.parametrize("bits", [10, 11])
def test_captured_after_a_crowded_call(bits):
    """A captured call takes the route that the eager call before it found; its
    replays give the oracle's graph for crowded and for scattered points."""
    rng = np.random.default_rng(9)
    prm = fgbd.default_params(bits=bits)
    crowded, other = plane(rng, bits, 40000), rng.integers(0, 1 << bits, size=(40000, 3)).astype(np.int32)
    for first in (crowded, other):
        ctx = fgbd.Context("cuda")
        ctx.reserve(prm, len(first))
        x = dev(first, torch.int32)
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            fgbd.build_slg(x, prm, ctx=ctx)
        torch.cuda.synchronize()
        captured = torch.cuda.CUDAGraph()
        with torch.cuda.graph(captured):
            g = fgbd.build_slg(x, prm, ctx=ctx)
        for points in (crowded, other, crowded):
            x.copy_(dev(points, torch.int32))
            captured.replay()
            torch.cuda.synchronize()
            col, d2 = O.slg_graph(points, prm.bits, prm.num_dirs, prm.window, prm.k)
            assert np.array_equal(g.col.cpu().numpy(), col) and np.array_equal(g.dist2.cpu().numpy(), d2)
        ctx.close()
