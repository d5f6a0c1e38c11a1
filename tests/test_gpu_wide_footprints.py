"""Records that cover many tiles: their entries past the fourth are placed by
the whole wavefront.  Every tile's list is compared with the oracle's binning,
record for record, for counts around a wavefront and a workgroup, with and
without the projection's tile table."""
import numpy as np
import pytest
import torch

import oracle
from paper_2510_01767_amd import gsr as C
from paper_2510_01767_amd import scenes
from paper_2510_01767_amd.raster import Rasterizer, camera_tensor, pack_images, scene_tensors
from tests import parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("project_table", [0, 1])
@pytest.mark.parametrize("n", [1, 63, 64, 65, 300])
def test_wide_footprints_are_binned_like_the_oracle(n, project_table):
    C.load(build_if_missing=False)
    scene = scenes.small_ragged(n=n, sh_degree=0, sizes=((190, 129), (70, 33)))
    # every fifth Gaussian large: up to the whole grid of tiles
    scene.log_scales[:, ::5] += np.linspace(1.0, 4.0, scene.log_scales[:, ::5].shape[1], dtype=np.float32)
    print("[gpu-case] wide footprints", n, project_table, flush=True)
    sizes = [(c["W"], c["H"]) for c in scene.cameras]
    r = Rasterizer(n, 0, sizes, mode="batched", project_table=project_table)
    r.step_l1(scene_tensors(scene), camera_tensor(scene.cameras), torch.from_numpy(pack_images(scene.targets)).cuda())
    torch.cuda.synchronize()
    ora = oracle.step_l1(oracle.Params.from_scene(scene), scene.cameras, scene.targets, parity.opts_for())
    ob, tiles = ora["bins"], r.layout.tiles_total
    starts = parity.ws_np(r, "tile_start", torch.int32, tiles + 1).view(np.uint32).astype(np.int64)
    keys = parity.ws_np(r, "keys", torch.int64, int(starts[-1])).view(np.uint64)
    assert parity.unambiguous_tiles(ora).all()  # (a property of this seeded scene)
    assert starts[-1] == ob["count"] == r.counts().intersections_total
    assert np.array_equal(np.diff(starts), ob["ranges"][:, 1] - ob["ranges"][:, 0])
    assert np.array_equal((keys & 0xffffffff).astype(np.int64), np.concatenate(
        [ob["values"][a:b] for a, b in ob["ranges"]]).astype(np.int64))
    per = np.bincount((keys & 0xffffffff).astype(np.int64))
    assert per.max() > 64 or n == 1  # some record has more tiles than a wavefront has lanes
