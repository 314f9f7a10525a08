"""Clouds that need more filter sweeps than the default schedule launches on
their own: the first call runs the rest in the looping launch, whose clouds
wait only for their own blocks; later calls on the context launch as many
sweeps as recent calls needed.  Every call gives the same bits."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2401_09721_amd import fgbd  # noqa: E402

from gpu_helpers import compare_denoise, dev  # noqa: E402
from test_gpu_batched import shape_cloud, small_cloud  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("clouds", [1, 5, 64])
def test_more_sweeps_than_the_default_schedule(clouds):
    prm = fgbd.default_params(bits=8)
    # uniform random colours need many sweeps; the shells in between stop early
    parts = [small_cloud(2500 + 311 * (s % 7), 90 + s) if s % 4 == 0 else shape_cloud(40 + s % 5, 3000)
             for s in range(clouds)]
    x = dev(np.concatenate([p[0] for p in parts]), torch.int32)
    c = dev(np.concatenate([p[1] for p in parts]), torch.float32)
    off = np.concatenate([[0], np.cumsum([len(p[0]) for p in parts])]).astype(np.int64)
    ctx = fgbd.Context("cuda")
    ref = None
    for rep in range(5):
        out, res = fgbd.denoise_batched(x, c, dev(off, torch.int64), prm, ctx=ctx)
        torch.cuda.synchronize()  # lets the next call read this call's sweep counts
        got = (out.cpu().numpy(), fgbd.read_results(res))
        if rep == 0:
            ref = got
            assert max(r["sweeps"] for r in got[1]) > ctx.schedule()["sweep_launches"]
            for s, (xyz, rgb) in enumerate(parts[:6]):
                compare_denoise(got[0][off[s]:off[s + 1]], got[1][s], xyz, rgb, prm)
        assert np.array_equal(got[0], ref[0]) and got[1] == ref[1], rep
    ctx.close()


def test_counts_read_back_without_waiting():
    """Calls enqueued one after another, on a context that is closed while
    they run and on one whose counts are read between them, alternating with
    the filter on a stored graph: the bits of a fresh context."""
    prm = fgbd.default_params(bits=8)
    xyz, rgb = shape_cloud(11, 3000)
    x, c = dev(xyz, torch.int32), dev(rgb, torch.float32)
    fresh = fgbd.Context()
    ref, rres = fgbd.denoise(x, c, prm, ctx=fresh)
    torch.cuda.synchronize()
    fresh.close()
    ctx = fgbd.Context()
    g = fgbd.build_slg(x, prm, ctx=ctx)
    noise, spread, _ = fgbd.estimate_noise(g, c, prm, ctx=ctx)
    filtered = None
    for rep in range(12):
        closing = fgbd.Context()
        a, ares = fgbd.denoise(x, c, prm, ctx=closing)
        closing.close()
        b, bres = fgbd.denoise(x, c, prm, ctx=ctx)
        f, fres = fgbd.filter(g, c, prm, noise=noise, spread=spread, ctx=ctx)
        if rep % 3 == 2:
            torch.cuda.synchronize()
        assert torch.equal(a, ref) and torch.equal(b, ref), rep
        assert fgbd.read_result(ares) == fgbd.read_result(bres) == fgbd.read_result(rres), rep
        filtered = f if filtered is None else filtered
        assert torch.equal(f, filtered) and fgbd.read_result(fres)["q"] == fgbd.read_result(rres)["q"], rep
    ctx.close()
