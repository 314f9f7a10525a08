"""The local sort of the top-digit route at its edges: ranges of exactly the
LDS capacity and one more, bins at and past the length that is counted in LDS,
duplicates, and batches whose clouds end around window bounds.  Graphs are
compared with the oracle's, exactly."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2401_09721_amd import fgbd, synth  # noqa: E402

from gpu_helpers import compare_denoise, dev  # noqa: E402
from test_gpu_parity import check_graph  # noqa: E402

pytestmark = pytest.mark.gpu


def _bucket(rng, count):
    """`count` points of one top digit of scan order 0 (z = 500) that begin at
    a window's base (4096 points below them), and some above."""
    flat = rng.choice(1 << 20, size=count, replace=False)
    at = np.stack([flat >> 10, flat & 1023, np.full(count, 500)], 1)
    below = np.stack([rng.integers(0, 1024, 4096), rng.integers(0, 1024, 4096), rng.integers(0, 400, 4096)], 1)
    above = np.stack([rng.integers(0, 1024, 900), rng.integers(0, 1024, 900), rng.integers(600, 1024, 900)], 1)
    return np.concatenate([at, below, above])


def _rows(rng, length, rows):
    """`rows` scan lines of `length` consecutive points along x in one plane,
    and scattered points."""
    x, y = np.meshgrid(np.arange(10, 10 + length), np.arange(300, 300 + 7 * rows, 7), indexing="ij")
    line = np.stack([x.ravel(), y.ravel(), np.full(x.size, 700)], 1)
    return np.concatenate([line, rng.integers(0, 1024, size=(6000, 3))])


def _duplicates(rng, voxels, times):
    v = rng.integers(0, 1024, size=(voxels, 3))
    return np.concatenate([np.repeat(v, times, axis=0), rng.integers(0, 1024, size=(3000, 3))])


@pytest.mark.parametrize("make", [
    lambda r: _bucket(r, 8191), lambda r: _bucket(r, 8192), lambda r: _bucket(r, 8193), lambda r: _rows(r, 400, 9),
    lambda r: _rows(r, 512, 3), lambda r: _rows(r, 1000, 4), lambda r: _duplicates(r, 300, 20),
    lambda r: _duplicates(r, 2, 2000), lambda r: r.integers(0, 1024, size=(4097, 3)),
], ids=["bucket8191", "bucket8192", "bucket8193", "rows400", "rows512", "rows1000", "dups20", "dups2000", "random4097"])
def test_ranges_and_bins(make):
    rng = np.random.default_rng(77)
    g = make(rng).astype(np.int32)
    check_graph(g[rng.permutation(len(g))], fgbd.default_params(bits=10, num_dirs=8, window=4, k=8))


@pytest.mark.parametrize("sizes", [(4095, 4096, 4097, 1, 0, 8193), (63, 8192, 2, 12289, 4096), (300,) * 40])
def test_batch_windows(sizes):
    """Each cloud of the batch against the oracle alone."""
    prm = fgbd.default_params(bits=8)
    rng = np.random.default_rng(5)
    shell = synth.random_shapes_cloud(3, bits=8, n_ellipsoids=3, target=16000, sigma=20.0)
    clouds = []
    for m in sizes:
        pick = np.sort(rng.choice(shell.n, size=m, replace=False))
        clouds.append((shell.xyz[pick], shell.noisy[pick]))
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    out, res = fgbd.denoise_batched(dev(np.concatenate([c[0] for c in clouds]), torch.int32),
                                    dev(np.concatenate([c[1] for c in clouds]), torch.float32),
                                    dev(off, torch.int64), prm)
    torch.cuda.synchronize()
    out, recs = out.cpu().numpy(), fgbd.read_results(res)
    for s, (xyz, rgb) in enumerate(clouds):
        if len(xyz):
            compare_denoise(out[off[s]:off[s + 1]], recs[s], xyz, rgb, prm)


@pytest.mark.parametrize("bits", [10, 11])
@pytest.mark.parametrize("voxels,times", [(2, 100), (2, 3000), (3, 1000), (7, 300), (64, 33), (65, 64), (300, 60)])
def test_duplicates_in_turn(bits, voxels, times):
    """A few voxels again and again in turn, so that every 64-point chunk of
    the input has several runs of each top digit: equal codes keep index
    order, in ranges sorted in LDS and in longer ones."""
    rng = np.random.default_rng(voxels)
    v = rng.integers(0, 1 << bits, size=(voxels, 3))
    g = np.concatenate([np.tile(v, (times, 1)), rng.integers(0, 1 << bits, size=(777, 3)), np.tile(v[::-1], (5, 1))])
    check_graph(g.astype(np.int32), fgbd.default_params(bits=bits, num_dirs=8, window=4, k=8))


def _planes(rng, n, extra):
    """Planes of n points normal to each scan axis, in no order, and others."""
    out = [rng.integers(0, 1024, size=(extra, 3))]
    for axis in range(3):
        flat = rng.choice(1 << 20, size=n, replace=False)
        p = np.stack([flat >> 10, flat & 1023], 1)
        out.append(np.insert(p, axis, 300 + 7 * axis, axis=1))
    return np.concatenate(out)


@pytest.mark.parametrize("n", [8193, 9500, 16384, 16385, 24000, 32700, 33000])
def test_planes_past_the_lds(n):
    """Ranges of more than a block's LDS holds, sorted through the two item
    buffers, from one item more to past the flag's length."""
    rng = np.random.default_rng(n)
    g = _planes(rng, n, 5000).astype(np.int32)
    check_graph(g, fgbd.default_params(bits=10, num_dirs=8, window=4, k=8))
