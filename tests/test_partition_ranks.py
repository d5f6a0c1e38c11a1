"""The partition's order statistics by histogram and by selection, around the
centre and rank counts where the choice changes and on values that fill the
histogram unevenly: the library's host partition equals the oracle's, bit for
bit.  No GPU is needed."""
import numpy as np
import pytest

from oracle import partition as op
from paper_2510_01767_amd import gsr as C
from paper_2510_01767_amd import scenes


@pytest.mark.parametrize("values", ["city", "rounded", "equal", "tiny", "unbounded box", "huge box"])
@pytest.mark.parametrize("steps", [1, 3, 7])
@pytest.mark.parametrize("n", [16383, 16384, 40001])
def test_partition_equals_the_oracle(n, steps, values):
    pi = scenes.partition_input(seed=n + steps, n=n, n_views=9, pixels=(40, 80))
    box, c = pi.aabb.copy(), pi.centers.copy()
    if values == "rounded":
        c[:2] = np.floor(c[:2] / 7.0) * 7.0
        box[:2] = -105.0
    elif values == "equal":
        c[:2] = np.float32(3.25)
    elif values == "tiny":
        c[:2] *= np.float32(1e-35)
    elif values == "unbounded box":
        box[:3], box[3:] = -np.inf, np.inf
    elif values == "huge box":
        box[:3], box[3:] = -3.0e38, 3.0e38
    want = op.kd_partition(box, c, pi.points, pi.offsets, 6, steps=steps)
    blocks, assign, load = C.gsr_partition_blocks(box, c, pi.points, pi.offsets, 6, 0.1, steps, 0.1, 0.9)
    for b, (w, cams) in enumerate(want):
        assert np.array_equal(blocks[b], w) and list(np.nonzero(assign[b])[0]) == list(cams) and load[b] == len(cams)
