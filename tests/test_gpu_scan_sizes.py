"""The tile scan by one workgroup and by three launches, around the tile
counts where the choice changes and with views of very different sizes: list
starts, per-view counts and the schedule against the records' rectangles."""
import numpy as np
import pytest
import torch

from paper_2510_01767_amd import gsr as C
from paper_2510_01767_amd import scenes
from paper_2510_01767_amd.raster import Rasterizer, camera_tensor, pack_images, scene_tensors
from tests import parity

pytestmark = pytest.mark.gpu

SIZES = {
    "1 tile": ((16, 16),),
    "4095 tiles": ((16 * 1023, 64), (48, 16)),
    "4096 tiles": ((16 * 1024, 64),),
    "4097 tiles": ((16, 16), (16 * 1024, 64)),
    "12288 tiles": ((16 * 1024, 192),),
    "12289 tiles": ((16 * 1024, 192), (3, 2)),
    "16 views": tuple((16 * 60 + 7 * k, 16 * 15 + k) for k in range(16)),
}


@pytest.mark.parametrize("mode", ["batched", "plain"])
@pytest.mark.parametrize("name", SIZES)
def test_scan_starts_counts_and_schedule(name, mode):
    C.load(build_if_missing=False)
    print("[gpu-case] scan", name, mode, flush=True)
    scene = scenes.small_ragged(n=700, sh_degree=0, sizes=SIZES[name])
    V, n = scene.n_views, scene.n
    r = Rasterizer(n, 0, [(c["W"], c["H"]) for c in scene.cameras], mode=mode, capacity=1 << 22)
    targets = torch.from_numpy(pack_images(scene.targets)).cuda()
    loss, images = r.step_l1(scene_tensors(scene), camera_tensor(scene.cameras), targets)
    torch.cuda.synchronize()
    rec, bits = parity.gpu_records(r), parity.ws_np(r, "view_bits", torch.int32, n).view(np.uint32)
    rect = np.ascontiguousarray(rec[:, 12:14]).view(np.uint32)
    counts, per_view = [], []
    for v, (W, H) in enumerate(r.sizes):
        tx, ty = (W + 15) // 16, (H + 15) // 16
        c = np.zeros((ty, tx), np.int64)
        for i in np.nonzero((bits >> v) & 1)[0]:
            a, b = (int(x) for x in rect[v * n + i])
            c[a >> 16:(b >> 16) + 1, a & 0xffff:(b & 0xffff) + 1] += 1
        counts.append(c.ravel())
        per_view.append(int(c.sum()))
    counts = np.concatenate(counts)
    tiles = r.layout.tiles_total
    starts = parity.ws_np(r, "tile_start", torch.int32, tiles + 1).view(np.uint32).astype(np.int64)
    assert np.array_equal(starts, np.concatenate([[0], np.cumsum(counts)]))
    q = r.counts()
    assert list(q.intersections[:V]) == per_view and q.overflow == 0
    want = np.mean([np.abs(a - b).mean(dtype=np.float64) for a, b in
                    zip(parity.gpu_images(r), [np.asarray(t) for t in scene.targets])])
    assert abs(float(loss.item()) - want) <= 1e-6 * want
    if mode == "batched":
        order = r.ws_tensor("tile_order", torch.int32, tiles).cpu().numpy()
        assert np.array_equal(np.sort(order), np.arange(tiles))
        assert np.all(np.diff(np.minimum(counts[order] // 4, 1023)) <= 0)
