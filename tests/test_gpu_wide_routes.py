"""Codes above 32 bits at the edges of their routes: the top-digit sort where
the index fits beside the code and the radix passes one point past that, FP64
selection keys and the general selection one point past the bits they hold,
bins and ranges at the local sort's limits, duplicates and batches.  Graphs
are compared with the oracle's, exactly (dist2 saturates at 2^31 - 1)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle as O  # noqa: E402
from paper_2401_09721_amd import fgbd  # noqa: E402

from gpu_helpers import compare_denoise, dev  # noqa: E402

pytestmark = pytest.mark.gpu


def check(xyz, prm):
    g = fgbd.build_slg(dev(xyz, torch.int32), prm)
    torch.cuda.synchronize()
    ocol, od2 = O.slg_graph(xyz, prm.bits, prm.num_dirs, prm.window, prm.k)
    assert np.array_equal(g.col.cpu().numpy(), ocol)
    assert np.array_equal(g.dist2.cpu().numpy(), np.minimum(od2, (1 << 31) - 1))


def points(bits, n, seed):
    """Scattered points, a quarter of them in a block of 12^3 voxels (with
    duplicates), a few at the grid's corners."""
    rng = np.random.default_rng(seed)
    g = rng.integers(0, 1 << bits, size=(n, 3))
    g[: n // 4] = rng.integers(1000, 1012, size=(n // 4, 3))
    g[n // 4: n // 4 + 8] = rng.integers(0, 2, size=g[n // 4: n // 4 + 8].shape) * ((1 << bits) - 1)
    return g[rng.permutation(n)].astype(np.int32)


# largest n whose index fits beside the code, and one more: 50 code bits at
# b = 16 (L = 8), 48 with the axis directions, 53 at b = 17, 62 at b = 20
@pytest.mark.parametrize("bits,L,n", [(16, 8, 16384), (16, 8, 16385), (16, 3, 65536), (16, 3, 65537), (17, 8, 2048),
                                      (17, 8, 2049), (20, 16, 4), (20, 16, 5), (11, 8, 1), (11, 8, 9), (12, 16, 4097),
                                      (15, 16, 20000), (13, 5, 8193)])
@pytest.mark.parametrize("w,K", [(4, 8), (4, 13), (2, 6), (4, 20)])
def test_index_beside_code(bits, L, n, w, K):
    check(points(bits, n, n), fgbd.default_params(bits=bits, num_dirs=L, window=w, k=min(K, 2 * w * L)))


@pytest.mark.parametrize("n", [524288, 524289])
def test_keys_of_63_bits(n):
    check(points(21, n, 1), fgbd.default_params(bits=21, num_dirs=1, window=4, k=5))


def _plane(rng, n):  # one top digit of scan order 0 holds all
    return np.stack([rng.integers(0, 2048, n), rng.integers(0, 2048, n), np.full(n, 700)], 1)


def _lines(rng, length):  # long bins: runs of consecutive x
    x, y = np.meshgrid(np.arange(10, 10 + length), np.arange(300, 1500, 150), indexing="ij")
    line = np.stack([x.ravel(), y.ravel(), np.full(x.size, 1700)], 1)
    return np.concatenate([line, rng.integers(0, 2048, size=(6000, 3))])


def _twice(rng, times):
    v = rng.integers(0, 2048, size=(6, 3))
    return np.concatenate([np.repeat(v, times, axis=0), rng.integers(0, 2048, size=(3000, 3))])


@pytest.mark.parametrize("make", [lambda r: _plane(r, 8192), lambda r: _plane(r, 8193), lambda r: _lines(r, 256),
                                  lambda r: _lines(r, 1200), lambda r: _twice(r, 200), lambda r: _twice(r, 1500)],
                         ids=["plane8192", "plane8193", "lines256", "lines1200", "dups200", "dups1500"])
def test_ranges_and_bins(make):
    rng = np.random.default_rng(8)
    g = make(rng).astype(np.int32)
    check(g[rng.permutation(len(g))], fgbd.default_params(bits=11))


def test_batch():
    prm = fgbd.default_params(bits=12)
    rng = np.random.default_rng(4)
    sizes = (4095, 4097, 1, 0, 8193, 300)
    xyz = [points(12, m, m) for m in sizes]
    rgb = [rng.uniform(0, 255, size=(m, 3)).astype(np.float32) for m in sizes]
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    out, res = fgbd.denoise_batched(dev(np.concatenate(xyz), torch.int32), dev(np.concatenate(rgb), torch.float32),
                                    dev(off, torch.int64), prm)
    torch.cuda.synchronize()
    out, recs = out.cpu().numpy(), fgbd.read_results(res)
    for s in range(len(sizes)):
        if sizes[s]:
            compare_denoise(out[off[s]:off[s + 1]], recs[s], xyz[s], rgb[s], prm)
