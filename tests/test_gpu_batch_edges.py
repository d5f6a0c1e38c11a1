"""Raster batches hold one entry less than their size, the last place fills up
the shorter sub-block lists, and the reverse pass culls its batches anew (the
fused one keeps the forward's last): one step and its gradients against the
oracle with list lengths around the batch sizes, in every tile shape, batch size and reverse
reduction, on images of few and of many tiles."""
import numpy as np
import pytest
import torch

import oracle
from paper_2510_01767_amd import gsr as C
from paper_2510_01767_amd import scenes
from paper_2510_01767_amd.raster import Rasterizer, camera_tensor, pack_images, scene_tensors
from tests import parity
from tests.test_gpu_fcs import compare_depth, unpack_depth

pytestmark = pytest.mark.gpu

SMALL = ((16, 16), (37, 29))
LARGE = ((1040, 1024),)  # more than 4096 tiles


def check(n, sizes, tile, batch, reduce, opaque, mode, elementwise=True):
    C.load(build_if_missing=False)
    print("[gpu-case] batch edges", n, sizes, tile, batch, reduce, opaque, mode, flush=True)
    scene = scenes.small_ragged(seed=scenes.SEED_BASE + n, n=n, sh_degree=0, sizes=sizes)
    if sizes is SMALL:
        scene.log_scales += 1.2  # nearly every Gaussian in every tile, not in every sub-block
    scene.opacity_logits[:] = scene.opacity_logits * 0.3 + (1.0 if opaque else -4.0)
    r = Rasterizer(n, 0, [(c["W"], c["H"]) for c in scene.cameras], mode=mode, tile=tile, lds_batch=batch,
                   bwd_reduce=reduce)
    r.S.zero_()
    r.count.zero_()
    targets = torch.from_numpy(pack_images(scene.targets)).cuda()
    loss, _ = r.step_l1(scene_tensors(scene), camera_tensor(scene.cameras), targets)
    torch.cuda.synchronize()
    opts = parity.opts_for(tile)
    ora = oracle.step_l1(oracle.Params.from_scene(scene), scene.cameras, scene.targets, opts)
    parity.compare_images(parity.gpu_images(r), ora)
    assert abs(float(loss.item()) - ora["loss"]) <= 1e-5 * abs(ora["loss"])
    ex = parity.excluded_gaussians(ora, n, opts, scene.targets)
    if elementwise:
        parity.compare_grads(parity.gpu_grad_groups(r.grads), ora["grads"], ex)
        return
    gpu, ref = parity.gpu_grad_groups(r.grads), parity.ora_grad_groups(ora["grads"])
    for name in parity.GROUPS:
        a, b = gpu[name][:, ~ex], ref[name][:, ~ex]
        assert np.linalg.norm(a - b) <= parity.GRAD_TOL * np.linalg.norm(b), name


@pytest.mark.parametrize("mode", ["batched", "plain"])
@pytest.mark.parametrize("tile", [(16, 16), (32, 8), (8, 32)])
@pytest.mark.parametrize("batch,reduce,n", [(64, 4, 63), (64, 3, 64), (64, 2, 127), (128, 4, 127), (128, 1, 128),
                                            (128, 4, 255), (256, 4, 255), (256, 3, 256), (256, 4, 511),
                                            (256, 0, 254), (256, 0, 510)])
def test_list_lengths(tile, batch, reduce, n, mode):
    check(n, SMALL, tile, batch, reduce, n % 2 == 0, mode)


@pytest.mark.parametrize("tile", [(16, 16), (32, 8), (8, 32)])
@pytest.mark.parametrize("batch,n", [(64, 130), (128, 300), (256, 700)])
def test_many_tiles(tile, batch, n):
    check(n, LARGE, tile, batch, 0, True, "batched")
    # Faint Gaussians over tens of thousands of pixels whose gradient signs are
    # random: a component whose sum happens to cancel keeps the rounding of the
    # 32-bit atomic additions, which no bound per element relative to the group
    # covers (it varies from run to run with their order); the group's does.
    check(n, LARGE, tile, batch, 0, False, "plain", elementwise=False)


@pytest.mark.parametrize("sizes", [SMALL, LARGE])
@pytest.mark.parametrize("batch,n", [(64, 64), (128, 200), (256, 300)])
def test_depth(sizes, batch, n):
    C.load(build_if_missing=False)
    print("[gpu-case] batch edges depth", n, sizes, batch, flush=True)
    scene = scenes.small_ragged(seed=scenes.SEED_BASE + n, n=n, sh_degree=0, sizes=sizes)
    scene.opacity_logits[:] = scene.opacity_logits * 0.3
    wh = [(c["W"], c["H"]) for c in scene.cameras]
    r = Rasterizer(n, 0, wh, mode="batched", lds_batch=batch)
    _, depth = r.render_depth(scene_tensors(scene), camera_tensor(scene.cameras))
    torch.cuda.synchronize()
    ora = oracle.forward(oracle.Params.from_scene(scene), scene.cameras, parity.opts_for())
    compare_depth(unpack_depth(depth, wh), ora)
