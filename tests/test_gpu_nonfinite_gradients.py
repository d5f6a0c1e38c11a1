"""An image gradient with a NaN and an infinity in it, as a caller's own loss can
give: only Gaussians that the pixel's tile lists take part in that pixel, so
every other gradient equals the run in which those pixels have none, with
sub-block lists of unequal lengths, on images of few and of many tiles.  An
entry that no pixel of a wavefront's step blends is left out of the reverse
walk, whichever walk that is."""
import numpy as np
import pytest
import torch

from paper_2510_01767_amd import gsr as C
from paper_2510_01767_amd import scenes
from paper_2510_01767_amd.raster import Rasterizer, camera_tensor, scene_tensors
from tests import parity

pytestmark = pytest.mark.gpu

FEW = ((70, 61), (93, 64))
MANY = ((70, 61), (1040, 1024))  # more than 4096 tiles
RTOL = 1e-5  # the order of float atomics


def build(n, sizes, tile, reduce, **kw):
    C.load(build_if_missing=False)
    scene = scenes.small_ragged(seed=scenes.SEED_BASE + n, n=n, sh_degree=1, sizes=sizes)
    if sizes is MANY:
        scene.log_scales += 1.5
    r = Rasterizer(n, 1, [(c["W"], c["H"]) for c in scene.cameras], mode="batched", tile=tile, bwd_reduce=reduce,
                   capacity=1 << 21, **kw)
    return scene, r, scene_tensors(scene), camera_tensor(scene.cameras)


def gradients(r, params, cams, g):
    r.forward(params, cams)
    r.backward(params, cams, g, stats=False)
    torch.cuda.synchronize()
    return {k: v.clone() for k, v in r.grads.items()}


def odd_pixels(r, g, view, every):
    """g with a NaN or an infinity at some pixels of the view, g with zeros there, and the pixels."""
    base, (W, H) = 3 * sum(w * h for w, h in r.sizes[:view]), r.sizes[view]
    ys, xs = (a.ravel() for a in np.meshgrid(np.arange(5, H, every), np.arange(3, W, every), indexing="ij"))
    at = torch.from_numpy(ys * W + xs).cuda()
    bad, none = g.clone(), g.clone()
    for ch in range(3):
        none[base + ch * W * H + at] = 0.0
    bad[base + at[0::2]] = float("nan")
    bad[base + W * H + at[1::2]] = float("inf")
    return bad, none, np.stack([xs, ys], 1)


def listed_at(r, view, pix, tile):
    """The Gaussians whose tile rectangle in the view holds one of the pixels' tiles."""
    rect = np.ascontiguousarray(parity.gpu_records(r)[view * r.n:(view + 1) * r.n, 12:14]).view(np.uint32)
    tx, ty = (pix // np.array(tile)).T[:, :, None]
    hit = ((rect[:, 0] & 0xffff) <= tx) & (tx <= (rect[:, 1] & 0xffff)) & ((rect[:, 0] >> 16) <= ty) & \
          (ty <= (rect[:, 1] >> 16))
    return hit.any(0) & visible_in(r, view)


def visible_in(r, view):
    return (parity.ws_np(r, "view_bits", torch.int32, r.n).view(np.uint32) >> view) & 1 == 1


@pytest.mark.parametrize("reduce", [0, 1, 2, 3, 4])
@pytest.mark.parametrize("tile", [(16, 16), (32, 8), (8, 32)])
@pytest.mark.parametrize("sizes", [FEW, MANY])
def test_only_listed_gaussians_take_part(sizes, tile, reduce):
    n, view = 600, 1
    print("[gpu-case] non-finite image gradient", sizes, tile, reduce, flush=True)
    scene, r, params, cams = build(n, sizes, tile, reduce)
    g = torch.from_numpy(np.random.default_rng(n).uniform(-1.0, 1.0, 3 * r.pixels).astype(np.float32)).cuda()
    bad, none, pix = odd_pixels(r, g, view, 29 if sizes is FEW else 331)
    # the first Gaussian of the first view lies elsewhere
    r.forward(params, cams)
    k = int(np.nonzero(~listed_at(r, view, pix, tile) & visible_in(r, 0))[0][0])
    for v in params.values():
        v[..., [0, k]] = v[..., [k, 0]]
    got, want = gradients(r, params, cams, bad), gradients(r, params, cams, none)
    listed = listed_at(r, view, pix, tile)
    assert 0 < listed.sum() < n and not listed[0] and visible_in(r, 0)[0]
    free = torch.from_numpy(~listed).cuda()
    for k, w in want.items():
        a, b = got[k][..., free], w[..., free]
        assert bool(torch.isfinite(a).all()), k
        assert float(torch.linalg.norm(a - b)) <= RTOL * float(torch.linalg.norm(b)), k
    assert not bool(torch.isfinite(got["sh"]).all())  # those that the pixels blend carry it


@pytest.mark.parametrize("what", ["image gradient", "colour"])
@pytest.mark.parametrize("tile", [(16, 16), (32, 8), (8, 32)])
@pytest.mark.parametrize("n", [150, 900])
def test_few_tiles_touch_what_many_tiles_do(n, tile, what):
    """The walk by four entries (reduction 0, few tiles) adds a non-finite term to no Gaussian that the walk by one
    (reduction 4) leaves out: an entry that no pixel of its step blends.  For an image gradient they are the same."""
    print("[gpu-case] non-finite", what, n, tile, flush=True)
    touched = []
    for reduce in (0, 4):
        scene, r, params, cams = build(n, FEW, tile, reduce, lds_batch=256)
        params["opacity_logits"] += 2.0  # many pixels stop before their list's end
        g = torch.from_numpy(np.random.default_rng(n).uniform(-1.0, 1.0, 3 * r.pixels).astype(np.float32)).cuda()
        if what == "colour":
            params["sh"][0, ::50] = float("inf")
        else:
            g = odd_pixels(r, g, 1, 17)[0]
        touched.append({k: ~torch.isfinite(v) for k, v in gradients(r, params, cams, g).items()})
    assert 0 < int(touched[1]["opacity_logits"].sum()) < n
    for k in touched[0]:
        assert not bool((touched[0][k] & ~touched[1][k]).any()), k
        assert what == "colour" or torch.equal(touched[0][k], touched[1][k]), k
