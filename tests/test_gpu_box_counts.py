"""Coverage counts around the box table's group size, on boxes that overlap,
repeat, touch, hold nothing or have infinite or undefined bounds, and depths
that back-project to infinite or undefined points: equal to comparing every
stored point with every box."""
import numpy as np
import pytest
import torch

from paper_2510_01767_amd import gsr as C
from paper_2510_01767_amd import scenes
from paper_2510_01767_amd.raster import Rasterizer, camera_tensor

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_blocks", [1, 2, 31, 32, 62, 63, 64, 127, 1024])
@pytest.mark.parametrize("sizes", [((1, 1),), ((150, 97), (33, 71)), ((1031, 517),)])
def test_counts_equal_brute_force(n_blocks, sizes):
    C.load(build_if_missing=False)
    print("[gpu-case] box counts", n_blocks, sizes, flush=True)
    scene = scenes.small_ragged(n=10, sh_degree=0, sizes=sizes)
    r = Rasterizer(10, 0, sizes, mode="batched")
    cams = camera_tensor(scene.cameras)
    rng = np.random.default_rng(n_blocks)
    depth = rng.uniform(0.0, 8.0, r.pixels).astype(np.float32)
    depth[::97], depth[5::97], depth[11::97], depth[17::97] = 0.0, np.nan, np.inf, 4.0
    depth = torch.from_numpy(depth).cuda()
    points = r.back_project(cams, depth).cpu().numpy()
    lo = rng.uniform(-4.0, 3.0, (n_blocks, 3))
    boxes = np.concatenate([lo, lo + rng.uniform(0.0, 4.0, (n_blocks, 3))], 1).astype(np.float32)
    k = np.arange(n_blocks)
    boxes[k % 11 == 3] = boxes[0]                                 # repeats
    boxes[k % 13 == 4, 0] = boxes[0, 3]                           # touch another box's face
    boxes[k % 17 == 5, :3], boxes[k % 17 == 5, 3:] = -np.inf, np.inf
    boxes[k % 19 == 6, 4] = boxes[k % 19 == 6, 1]                 # empty
    boxes[k % 23 == 7, 5] = np.nan
    boxes[k % 29 == 8, 0] = np.nan
    finite = points[:, np.isfinite(points).all(0)]
    if n_blocks > 2 and finite.shape[1]:
        boxes[2, :3] = finite[:, finite.shape[1] // 2]            # a point exactly on a corner
        boxes[2, 3:] = boxes[2, :3] + 1.0
    counts, ratio, selected = r.camera_coverage(cams, depth, torch.from_numpy(boxes).cuda(), tau=0.05)
    at = 0
    for v, (W, H) in enumerate(sizes):
        p = points[:, at:at + W * H]
        at += W * H
        want = np.array([((p >= b[:3, None]) & (p < b[3:, None])).all(0).sum() for b in boxes])
        assert np.array_equal(counts[v].cpu().numpy(), want)
        assert np.array_equal(ratio[v].cpu().numpy(), (want / (W * H)).astype(np.float32))
