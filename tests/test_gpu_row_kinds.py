"""Rows of every kind that has kernels of its own (K = 6, 8, 16, and any K up
to 8, 16, 32), aligned and not: weights, noise estimate, selection and fixed
sweeps on a stored graph against the oracle, and the whole path."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle as O  # noqa: E402
from paper_2401_09721_amd import fgbd, synth  # noqa: E402

from gpu_helpers import COLOUR_TOL, compare_denoise, dev  # noqa: E402

pytestmark = pytest.mark.gpu


def shifted(t):
    """The same values 4 bytes past a 16-byte boundary."""
    buf = torch.empty(t.numel() + 5, dtype=t.dtype, device=t.device)
    at = (4 - buf.data_ptr() // 4) % 4 + 1
    out = buf[at:at + t.numel()].view(t.shape)
    out.copy_(t)
    assert out.data_ptr() % 16 == 4
    return out


@pytest.mark.parametrize("n", [1, 7, 257, 3001])
@pytest.mark.parametrize("k,patch,aligned", [(6, 0, True), (6, 0, False), (16, 0, True), (16, 0, False), (12, 0, True),
                                             (12, 0, False), (5, 0, True), (1, 0, True), (20, 16, True), (32, 0, True),
                                             (24, 6, False), (16, 12, True), (7, 6, True)])
def test_stored_graph(n, k, patch, aligned):
    prm = fgbd.default_params(bits=8, k=k, patch=patch)
    c = synth.random_shapes_cloud(7, bits=8, n_ellipsoids=3, target=4000, sigma=20.0)
    xyz, rgb = c.xyz[:n], c.noisy[:n]
    P = patch if patch else k
    g = fgbd.build_slg(dev(xyz, torch.int32), prm)
    if not aligned:
        g = fgbd.SLGraph(shifted(g.col), shifted(g.dist2), shifted(g.p), g.result)
    ocol, od2 = O.slg_graph(xyz, 8, 8, 4, k)
    assert np.array_equal(g.col.cpu().numpy(), ocol) and np.array_equal(g.dist2.cpu().numpy(), od2)
    op = O.edge_weights(ocol, od2, O.bandwidth(ocol, od2))
    assert np.allclose(g.p.cpu().numpy(), op, rtol=0, atol=2e-7)
    y = dev(rgb, torch.float32)
    noise, spread, eig3 = fgbd.estimate_noise(g, y, prm, want_eig3=True)
    on = O.estimate_noise(ocol, rgb, P)
    r = fgbd.read_result(noise)
    assert r["n_eff"] == on["n_eff"]
    assert abs(r["sigma_est"] - on["sigma_est"]) <= COLOUR_TOL  # (moments are rounded to 2^-12 per block)
    assert np.allclose(spread.cpu().numpy(), O.patch_spread(ocol, rgb, P), rtol=1e-12, atol=1e-9)
    for q in (0, 1, 3):
        out, _ = fgbd.filter(g, y, prm, q_fixed=q)
        assert np.abs(out.cpu().numpy() - O.filter_power(ocol, op, rgb, q)).max() <= COLOUR_TOL
    out, res = fgbd.filter(g, y, prm, noise=noise, spread=spread)
    out2, res2 = fgbd.denoise(dev(xyz, torch.int32), y, prm)
    torch.cuda.synchronize()
    assert fgbd.read_result(res)["q"] == fgbd.read_result(res2)["q"]
    assert np.abs(out.cpu().numpy() - out2.cpu().numpy()).max() <= 1e-4
    compare_denoise(out2.cpu().numpy(), fgbd.read_result(res2), xyz, rgb, prm)
