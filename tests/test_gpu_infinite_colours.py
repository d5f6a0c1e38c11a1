"""A Gaussian of infinite colour (its SH overflows; the parameter check does not
read SH) shows only where the walk reaches it: a pixel that has stopped in
front of it keeps its colour.  The walk by four entries of launches with few
tiles against the walk by one of the pair counting, bit for bit."""
import pytest
import torch

from paper_2510_01767_amd import gsr as C
from paper_2510_01767_amd import scenes
from paper_2510_01767_amd.raster import Rasterizer, camera_tensor, scene_tensors

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile", [(16, 16), (32, 8), (8, 32)])
@pytest.mark.parametrize("n", [5, 60, 700])
def test_stopped_pixels_keep_their_colour(n, tile):
    C.load(build_if_missing=False)
    print("[gpu-case] infinite colour", n, tile, flush=True)
    scene = scenes.small_ragged(seed=scenes.SEED_BASE + n, n=n, sh_degree=0, sizes=((64, 48), (21, 13)))
    scene.log_scales += 1.0
    r = Rasterizer(n, 0, [(c["W"], c["H"]) for c in scene.cameras], mode="batched", tile=tile, lds_batch=256)
    params, cams = scene_tensors(scene), camera_tensor(scene.cameras)
    params["opacity_logits"] += 4.0
    finite = r.forward(params, cams).clone()
    # one Gaussian of the farther half of the first view
    depth = r.ws_tensor("records", torch.float32, 16 * n).view(n, 16)[:, 14]
    params["sh"][0, torch.argsort(depth)[(3 * n) // 4]] = float("inf")
    got = r.forward(params, cams).clone()
    want = r.images.clone()
    r.pair_counts(params, cams, images=want)
    torch.cuda.synchronize()
    assert torch.equal(got.view(torch.int32), want.view(torch.int32))
    clean = torch.isfinite(got)
    assert torch.equal(got[clean], finite[clean]) and 0 < int(clean.sum()) < got.numel()
