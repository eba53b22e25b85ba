"""The ways a patch or a box is counted: a wave each (small patches, boxes that
are many), workgroups of two or four waves (few boxes, larger unaligned
patches), one pixel or four a thread.  Bins equal the oracle's exactly."""
import numpy as np
import pytest

from paper_1812_07607_amd import ops

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bins", [4, 8, 16])
@pytest.mark.parametrize("n,h,w", [(3000, 1, 1), (2500, 3, 3), (5001, 5, 7), (300, 8, 8), (2049, 5, 13), (70, 31, 33),
                                   (2100, 25, 41), (9, 25, 41), (41001, 3, 11)])
def test_unaligned_patches(orc, n, h, w, bins):
    """pixels from one to past a wave's, patches either side of a route's counts"""
    from gpu_util import dev, host
    px = np.random.default_rng(n).integers(0, 256, size=(n + 1, h, w, 3), dtype=np.uint8)
    d = dev(px.reshape(-1))[3 * h * w:].reshape(n, h, w, 3)  # (unaligned for every odd size)
    assert np.array_equal(host(ops.featurize_rgb8(d, bins)), orc.hist_rgb8(px[1:], bins))


@pytest.mark.parametrize("n", [7, 2048, 2049, 40960, 40961])
def test_boxes_by_number(orc, n):
    """mostly small boxes (one pixel to 64 and past), some of a whole frame"""
    from gpu_util import dev, host
    rng = np.random.default_rng(n)
    H, W = 60, 81
    frames = rng.integers(0, 256, size=(3, H, W, 3), dtype=np.uint8)
    side = rng.integers(1, 11, size=(n, 2))
    side[rng.integers(0, n, size=max(1, n // 100))] = (W, H)
    x0 = (rng.random(n) * (W - side[:, 0] + 1)).astype(int)
    y0 = (rng.random(n) * (H - side[:, 1] + 1)).astype(int)
    box = np.stack([rng.integers(0, 3, size=n), x0, y0, x0 + side[:, 0], y0 + side[:, 1]], 1).astype(np.int32)
    got = host(ops.featurize_crops_rgb8(dev(frames), dev(box), 8))
    for b, g in zip(box, got):
        px = np.ascontiguousarray(frames[b[0], b[2]:b[4], b[1]:b[3]])
        assert np.array_equal(g, orc.hist_rgb8(px[None], 8)[0])


def test_bad_box_among_many():
    """a box outside its frame is refused in the wave-per-box route too"""
    from gpu_util import dev
    from paper_1812_07607_amd import _lib
    frames = np.zeros((1, 20, 20, 3), np.uint8)
    box = np.tile(np.array([0, 1, 1, 5, 5], np.int32), (41000, 1))
    box[40999, 3] = 21
    with pytest.raises(_lib.DLError):
        ops.featurize_crops_rgb8(dev(frames), dev(box), 8)
