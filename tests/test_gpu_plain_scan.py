"""The plain form scans and sorts view by view: the three-launch scan of a view
whose chunk sums lie behind another view's pixels at an odd place, with starts
that go on from the view before, and lists of every length class in more than
one view, against the batched form's."""
import numpy as np
import pytest
import torch

from paper_2510_01767_amd import gsr as C
from paper_2510_01767_amd import scenes
from paper_2510_01767_amd.raster import Rasterizer, camera_tensor, scene_tensors
from tests import parity
from tests import test_gpu_scan_sizes as scan
from tests.test_gpu_sort_long import CLASSES

pytestmark = pytest.mark.gpu

# views of up to 12 288 tiles are scanned by one workgroup
SIZES = {
    "odd place": ((3, 3), (16 * 1024, 208), (37, 29)),
    "first and last": ((16 * 1024, 193), (5, 7), (16 * 1000, 208)),
}


@pytest.mark.parametrize("mode", ["plain", "batched"])
@pytest.mark.parametrize("name", SIZES)
def test_scan_of_a_large_view_among_others(name, mode, monkeypatch):
    monkeypatch.setitem(scan.SIZES, name, SIZES[name])
    scan.test_scan_starts_counts_and_schedule(name, mode)


def test_long_lists_in_every_view():
    C.load(build_if_missing=False)
    scene = scenes.dense_cloud(sizes=((256, 256), (250, 240)))
    n, sizes = scene.n, [(c["W"], c["H"]) for c in scene.cameras]
    params, cams = scene_tensors(scene), camera_tensor(scene.cameras)
    found = {}
    for mode in ("plain", "batched"):
        print("[gpu-case] long lists", mode, flush=True)
        r = Rasterizer(n, scene.sh_degree, sizes, mode=mode, capacity=12_000_000)
        r.forward(params, cams)
        torch.cuda.synchronize()
        assert r.counts().overflow == 0
        starts = parity.ws_np(r, "tile_start", torch.int32, r.layout.tiles_total + 1).view(np.uint32).astype(np.int64)
        found[mode] = starts, parity.ws_np(r, "keys", torch.int64, int(starts[-1])), list(r.counts().intersections[:2])
        del r
    (s, k, c), (s2, k2, c2) = found["plain"], found["batched"]
    assert np.array_equal(s, s2) and np.array_equal(k, k2) and c == c2
    lens, first = np.diff(s), 256  # tiles of the first view
    for view in (lens[:first], lens[first:]):
        for lo, hi, path in CLASSES:
            assert ((view >= lo) & (view <= hi)).any(), path
