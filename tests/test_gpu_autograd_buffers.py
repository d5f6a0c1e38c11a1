"""The autograd functions hand out gradients in buffers of their own: two
steps' gradients do not share memory, repeat the plain call's values, scale
with the incoming gradient under both forms of the reverse function, and a
plan that accumulates still returns its running sums."""
import pytest
import torch

from paper_2510_01767_amd import gsr as C
from paper_2510_01767_amd import scenes
from paper_2510_01767_amd.raster import (PARAM_NAMES, Rasterizer, camera_tensor, pack_images, render, render_l1,
                                         scene_tensors)

pytestmark = pytest.mark.gpu
RTOL = 1e-5  # the order of float atomics


def setup(**kw):
    C.load(build_if_missing=False)
    scene = scenes.small_ragged(n=500, sh_degree=1)
    r = Rasterizer(scene.n, 1, [(c["W"], c["H"]) for c in scene.cameras], mode="batched", **kw)
    return r, scene_tensors(scene), camera_tensor(scene.cameras), torch.from_numpy(pack_images(scene.targets)).cuda()


def leaves(params):
    return {k: v.clone().requires_grad_(True) for k, v in params.items()}


def near(a, b):
    return float(torch.linalg.norm(a - b)) <= RTOL * float(torch.linalg.norm(b))


@pytest.mark.parametrize("create_graph", [False, True])
def test_steps_do_not_share_gradients(create_graph):
    r, params, cams, targets = setup()
    r.step_l1(params, cams, targets, stats=False)
    want = {k: v.clone() for k, v in r.grads.items()}
    la, lb = leaves(params), leaves(params)
    a, _ = render_l1(la, r, cams, targets)
    b, _ = render_l1(lb, r, cams, targets)
    ga = torch.autograd.grad(3.0 * a, [la[k] for k in PARAM_NAMES], create_graph=create_graph)
    gb = torch.autograd.grad(b, [lb[k] for k in PARAM_NAMES])
    for k, x, y in zip(PARAM_NAMES, ga, gb):
        assert near(x.detach(), 3.0 * want[k]) and near(y, want[k])
        assert len({x.data_ptr(), y.data_ptr(), r.grads[k].data_ptr()}) == 3
    g = (torch.rand_like(targets) - 0.5)
    lc = leaves(params)
    first = torch.autograd.grad(render(lc, r, cams), [lc[k] for k in PARAM_NAMES], g)
    second = torch.autograd.grad(render(lc, r, cams), [lc[k] for k in PARAM_NAMES], 2.0 * g)
    for x, y in zip(first, second):
        assert near(y, 2.0 * x) and x.data_ptr() != y.data_ptr()


def test_accumulating_plans_return_their_sums():
    r, params, cams, targets = setup(accumulate_grads=1)
    total = []
    for _ in range(2):
        p = leaves(params)
        loss, _ = render_l1(p, r, cams, targets)
        total.append(torch.autograd.grad(loss, [p[k] for k in PARAM_NAMES]))
    for k, x, y in zip(PARAM_NAMES, *total):
        assert near(y, 2.0 * x) and near(r.grads[k], y)
