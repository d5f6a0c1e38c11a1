"""The visibility mask with footprints cut at a small fraction of a standard
deviation: a Gaussian may then be wide enough for its 2D covariance to lose its
determinant to rounding while its footprint stays small, and the mask leaves
such a one to the exact test.  Its bits equal the projection's for every extent."""
import numpy as np
import pytest
import torch

from paper_2510_01767_amd import gsr as C
from paper_2510_01767_amd import scenes
from paper_2510_01767_amd.raster import Rasterizer, camera_tensor, scene_tensors
from tests import parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("eps2d", [0.3, 0.01])
@pytest.mark.parametrize("sigma", [3.0, 1.0, 0.1, 1e-3, 1e-5])
def test_mask_equals_the_projection_at_any_extent(sigma, eps2d):
    C.load(build_if_missing=False)
    print("[gpu-case] cull extent", sigma, eps2d, flush=True)
    n = 4001
    scene = scenes.small_ragged(n=n, sh_degree=0, sizes=((150, 97), (33, 71), (16, 16)))
    rng = np.random.default_rng(n)
    # the widest footprints some 1e4 pixels, whatever the extent
    top = np.log(1.0e4 * 4.0 / (sigma * 100.0))
    scene.log_scales[:] = rng.uniform(-8.0, top + 1.0, scene.log_scales.shape)
    r = Rasterizer(n, 0, [(c["W"], c["H"]) for c in scene.cameras], mode="batched", eps2d=eps2d, sigma_extent=sigma,
                   capacity=1 << 20)
    params, cams = scene_tensors(scene), camera_tensor(scene.cameras)
    bits = r.visibility_mask(params, cams)[0].cpu().numpy()
    r.forward(params, cams)
    torch.cuda.synchronize()
    want = parity.ws_np(r, "view_bits", torch.int32, n)
    assert np.array_equal(bits, want)
    assert np.any(want == 7)  # and most are visible
