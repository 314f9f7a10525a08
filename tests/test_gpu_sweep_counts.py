"""The number of separate sweep launches, counted by the context's profiling:
it follows what recent calls of the same kind needed, stays with that kind on a
context that makes other calls too, and never passes a schedule that was set."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2401_09721_amd import fgbd  # noqa: E402

from gpu_helpers import dev  # noqa: E402
from test_gpu_batched import shape_cloud, small_cloud  # noqa: E402

pytestmark = pytest.mark.gpu

PRM = dict(bits=8)


def _batch(clouds):
    # uniform random colours need many sweeps; the shells in between stop early
    parts = [small_cloud(2500 + 311 * (s % 7), 90 + s) if s % 4 == 0 else shape_cloud(40 + s % 5, 3000)
             for s in range(clouds)]
    off = np.concatenate([[0], np.cumsum([len(p[0]) for p in parts])]).astype(np.int64)
    return (dev(np.concatenate([p[0] for p in parts]), torch.int32),
            dev(np.concatenate([p[1] for p in parts]), torch.float32), dev(off, torch.int64))


def _launches(ctx, call):
    """Sweep launches of one call (sweeps 1 and 2 are one launch, and the loop
    after the separate ones is one), and the most sweeps a cloud needed."""
    ctx.profile_read()
    _, res = call()
    torch.cuda.synchronize()  # lets the next call read this call's counts
    return ctx.profile_read()["sweep"][1], max(r["sweeps"] for r in fgbd.read_results(res))


def _expected(separate, q_max):
    return separate - 1 + (1 if separate < q_max else 0)


@pytest.mark.parametrize("clouds", [1, 5, 64])
def test_rises_to_what_the_calls_need(clouds):
    prm = fgbd.default_params(**PRM)
    x, c, off = _batch(clouds)
    ctx = fgbd.Context("cuda")
    ctx.profile(True)
    got = [_launches(ctx, lambda: fgbd.denoise_batched(x, c, off, prm, ctx=ctx)) for _ in range(4)]
    needed = got[0][1]
    assert needed > 8
    # the default, one count read (and a spare), counts that agree
    want = [8, min(needed + 1, 64), needed, needed]
    assert [g[0] for g in got] == [_expected(min(w, prm.q_max), prm.q_max) for w in want]
    ctx.close()


def test_other_calls_on_the_context():
    """A batch that needs many sweeps, a frame that needs few and the stored
    graph's filter in turn: each launches what it would alone."""
    prm = fgbd.default_params(**PRM)
    x, c, off = _batch(5)
    xyz, rgb = shape_cloud(41, 3000)
    fx, fc = dev(xyz, torch.int32), dev(rgb, torch.float32)

    def calls(ctx):
        g = fgbd.build_slg(fx, prm, ctx=ctx)
        noise, spread, _ = fgbd.estimate_noise(g, fc, prm, ctx=ctx)
        return {"batch": lambda: fgbd.denoise_batched(x, c, off, prm, ctx=ctx),
                "frame": lambda: fgbd.denoise(fx, fc, prm, ctx=ctx),
                "filter": lambda: fgbd.filter(g, fc, prm, noise=noise, spread=spread, ctx=ctx)}

    alone = {}
    for name in ("batch", "frame", "filter"):
        ctx = fgbd.Context("cuda")
        ctx.profile(True)
        alone[name] = [_launches(ctx, calls(ctx)[name])[0] for _ in range(4)]
        ctx.close()
    assert alone["batch"][-1] > alone["frame"][-1]
    ctx = fgbd.Context("cuda")
    ctx.profile(True)
    mixed = calls(ctx)
    got = {name: [] for name in mixed}
    for _ in range(4):
        for name, call in mixed.items():
            got[name].append(_launches(ctx, call)[0])
    assert got == alone
    ctx.close()


def test_a_set_schedule_bounds_the_count():
    prm = fgbd.default_params(**PRM)
    x, c, off = _batch(5)
    ctx = fgbd.Context("cuda")
    ctx.set_schedule(1024, 1024, 512, 6)
    ctx.profile(True)
    got = [_launches(ctx, lambda: fgbd.denoise_batched(x, c, off, prm, ctx=ctx)) for _ in range(4)]
    assert got[0][1] > 8 and [g[0] for g in got] == [_expected(6, prm.q_max)] * 4
    ctx.close()
