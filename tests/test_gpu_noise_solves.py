"""The noise estimate for every patch size up to 18: each form of the moments
and of the eigenvalue solve, at its smallest and largest matrix."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2401_09721_amd import fgbd  # noqa: E402

from gpu_helpers import compare_denoise, dev  # noqa: E402
from test_gpu_batched import shape_cloud  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("patch", range(1, 19))
def test_every_patch_size(patch):
    xyz, rgb = shape_cloud(60 + patch, 2500)
    prm = fgbd.default_params(bits=8, k=18, patch=patch)
    out, res = fgbd.denoise(dev(xyz, torch.int32), dev(rgb, torch.float32), prm)
    torch.cuda.synchronize()
    compare_denoise(out.cpu().numpy(), fgbd.read_result(res), xyz, rgb, prm)
