"""The autograd functions leave the gradients in the Rasterizer's own planes too,
where a caller's optimizer step reads them: the same tensors for the
Rasterizer's life, with the last call's values, whichever call it was."""
import pytest
import torch

from paper_2510_01767_amd import gsr as C
from paper_2510_01767_amd import scenes
from paper_2510_01767_amd.raster import (PARAM_NAMES, Rasterizer, camera_tensor, pack_images, render, render_l1,
                                         scene_tensors)

pytestmark = pytest.mark.gpu
RTOL = 1e-5  # the order of float atomics


def near(a, b):
    return float(torch.linalg.norm(a - b)) <= RTOL * float(torch.linalg.norm(b))


@pytest.mark.parametrize("mode", ["batched", "plain"])
@pytest.mark.parametrize("sh", [0, 3])
def test_planes_hold_the_last_gradients(mode, sh):
    C.load(build_if_missing=False)
    scene = scenes.small_ragged(n=500, sh_degree=sh)
    r = Rasterizer(scene.n, sh, [(c["W"], c["H"]) for c in scene.cameras], mode=mode)
    params, cams = scene_tensors(scene), camera_tensor(scene.cameras)
    targets = torch.from_numpy(pack_images(scene.targets)).cuda()
    planes = {k: v for k, v in r.grads.items()}
    r.step_l1(params, cams, targets, stats=False)
    want = {k: v.clone() for k, v in planes.items()}
    leaves = {k: v.clone().requires_grad_(True) for k, v in params.items()}

    def clear():
        for k in PARAM_NAMES:
            planes[k].fill_(float("nan"))
            leaves[k].grad = None

    clear()
    loss, images = render_l1(leaves, r, cams, targets)
    for k in PARAM_NAMES:
        assert r.grads[k] is planes[k] and near(planes[k], want[k]), k
    (2.0 * loss).backward()
    for k in PARAM_NAMES:
        assert near(planes[k], want[k]) and near(leaves[k].grad, 2.0 * want[k]), k

    clear()
    # the L1 loss's own gradient, so that the image form repeats the step
    scale = torch.cat([torch.full((3 * w * h,), 1.0 / (3 * w * h * len(r.sizes)), device="cuda") for w, h in r.sizes])
    out = render(leaves, r, cams)
    out.backward(torch.sign(out.detach() - targets) * scale)
    for k in PARAM_NAMES:
        assert r.grads[k] is planes[k] and near(planes[k], want[k]) and near(leaves[k].grad, want[k]), k
        assert leaves[k].grad.data_ptr() != planes[k].data_ptr()
    # what the planes are used for: an optimizer step on them
    zeros = lambda: {k: torch.zeros_like(v) for k, v in params.items()}
    after, plain = {k: v.clone() for k, v in params.items()}, {k: v.clone() for k, v in params.items()}
    lr = (1e-3,) * 6
    r.adam_step(after, r.grads, zeros(), zeros(), lr, 1, eps=1e-3)
    r.adam_step(plain, want, zeros(), zeros(), lr, 1, eps=1e-3)
    for k in PARAM_NAMES:
        assert near(after[k], plain[k])
