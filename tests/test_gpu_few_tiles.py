"""Launches with few tiles walk four entries at a time and load the next batch
meanwhile: one step and its gradients against the oracle with list lengths
around the groups of four and the 256-entry batches, lists that stop early and
lists that do not, in every form that takes these kernels."""
import numpy as np
import pytest
import torch

import oracle
from paper_2510_01767_amd import gsr as C
from paper_2510_01767_amd import scenes
from paper_2510_01767_amd.raster import Rasterizer, camera_tensor, pack_images, scene_tensors
from tests import parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", ["batched", "plain"])
@pytest.mark.parametrize("opaque", [False, True])
@pytest.mark.parametrize("n", [1, 3, 4, 5, 255, 256, 257, 515])
def test_list_lengths(n, opaque, mode):
    C.load(build_if_missing=False)
    print("[gpu-case] few tiles", n, opaque, mode, flush=True)
    scene = scenes.small_ragged(seed=scenes.SEED_BASE + n, n=n, sh_degree=0, sizes=((16, 16), (21, 13)))
    scene.log_scales += 1.5  # every Gaussian in every tile
    scene.opacity_logits[:] = scene.opacity_logits * 0.3 + (1.0 if opaque else -4.0)
    r = Rasterizer(n, 0, [(c["W"], c["H"]) for c in scene.cameras], mode=mode)
    r.S.zero_()
    r.count.zero_()
    targets = torch.from_numpy(pack_images(scene.targets)).cuda()
    loss, _ = r.step_l1(scene_tensors(scene), camera_tensor(scene.cameras), targets)
    torch.cuda.synchronize()
    assert r.counts().intersections_total >= 2 * n
    ora = oracle.step_l1(oracle.Params.from_scene(scene), scene.cameras, scene.targets, parity.opts_for())
    parity.compare_images(parity.gpu_images(r), ora)
    assert abs(float(loss.item()) - ora["loss"]) <= 1e-5 * abs(ora["loss"])
    ex = parity.excluded_gaussians(ora, n, parity.opts_for(), scene.targets)
    parity.compare_grads(parity.gpu_grad_groups(r.grads), ora["grads"], ex)
