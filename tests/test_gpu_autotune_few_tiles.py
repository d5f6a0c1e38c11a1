"""Where the batch size has no effect (few tiles, recompute, reduction 0) the
autotuner times one and reports the one that runs: 256."""
import pytest
import torch

from paper_2510_01767_amd import gsr as C
from paper_2510_01767_amd import scenes
from paper_2510_01767_amd.raster import Rasterizer, camera_tensor, pack_images, scene_tensors

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [((64, 48),), ((150, 97), (33, 71)), ((256, 256), (96, 96), (64, 40))])
@pytest.mark.parametrize("n", [300, 2000])
def test_the_batch_that_runs_is_reported(n, sizes):
    C.load(build_if_missing=False)
    print("[gpu-case] autotune few tiles", n, sizes, flush=True)
    scene = scenes.small_ragged(n=n, sh_degree=0, sizes=sizes)
    r = Rasterizer(n, 0, [(c["W"], c["H"]) for c in scene.cameras], mode="batched", lds_batch=64)
    args = scene_tensors(scene), camera_tensor(scene.cameras), torch.from_numpy(pack_images(scene.targets)).cuda()
    best, ms = r.autotune(*args, reps=1)
    assert ms > 0.0 and (best.bwd_reduce, best.bwd_variant) in [(q, C.GSR_BWD_RECOMPUTE) for q in (0, 2, 3, 4)]
    assert best.bwd_reduce != 0 or best.lds_batch == 256
    assert r.options.lds_batch == best.lds_batch
