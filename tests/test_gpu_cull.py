"""The visibility mask decides most pairs without projecting them: its bits
equal the oracle's away from ambiguous decisions, and those of the projection
for every Gaussian, with footprints from a point to many images, means around
the near plane and the borders, undefined and infinite parameters, and
dilations on both sides of what the accepting test asks for."""
import numpy as np
import pytest
import torch

import oracle
from paper_2510_01767_amd import gsr as C
from paper_2510_01767_amd import scenes
from paper_2510_01767_amd.raster import Rasterizer, camera_tensor, scene_tensors
from tests import parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("project_table", [0, 1])
@pytest.mark.parametrize("eps2d", [0.3, 0.01, 0.009, 0.0])
@pytest.mark.parametrize("n", [1, 257, 3001])
def test_visibility_mask_equals_the_projection(n, eps2d, project_table):
    C.load(build_if_missing=False)
    print("[gpu-case] cull", n, eps2d, project_table, flush=True)
    scene = scenes.small_ragged(n=n, sh_degree=0, sizes=((150, 97), (33, 71), (16, 16)))
    rng = np.random.default_rng(n)
    scene.means[:] = rng.uniform(-5.0, 5.0, scene.means.shape)  # around the cameras, behind them, beside the views
    scene.log_scales[:] = rng.uniform(-12.0, 6.0, scene.log_scales.shape)
    sizes = [(c["W"], c["H"]) for c in scene.cameras]
    clean = oracle.Params.from_scene(scene)
    odd = np.arange(n) % 97 == 5
    for k, v in enumerate((np.nan, np.inf, -np.inf)):
        scene.log_scales[k % 3, odd & (np.arange(n) % 3 == k)] = v
    scene.quats[:, np.arange(n) % 101 == 7] = 0.0
    scene.means[1, np.arange(n) % 103 == 9] = np.nan
    strange = odd | (np.arange(n) % 101 == 7) | (np.arange(n) % 103 == 9)
    r = Rasterizer(n, 0, sizes, mode="batched", eps2d=eps2d, project_table=project_table, capacity=1 << 20)
    params, cams = scene_tensors(scene), camera_tensor(scene.cameras)
    bits = r.visibility_mask(params, cams)[0].cpu().numpy().view(np.uint32)
    r.forward(params, cams)
    torch.cuda.synchronize()
    assert np.array_equal(bits, parity.ws_np(r, "view_bits", torch.int32, n).view(np.uint32))
    opts = oracle.default_opts(eps2d=float(np.float32(eps2d)))
    sure = ~strange
    for c in scene.cameras:
        sure &= ~(oracle.project(clean, c, opts)["margin"] < parity.DELTA)
    want = oracle.visibility_mask(clean, scene.cameras, opts, np.zeros(6, np.float32))[0]
    assert np.array_equal(bits[sure], want[sure])
