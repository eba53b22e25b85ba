"""Pixel runs of every small width (single pixels, a partial group of four,
whole groups with a remainder), boxes in the last corner of the last frame
and patches that no 16-byte load fits: counts equal numpy's exactly."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def hist(px, bins):
    q = px.reshape(-1, 3).astype(np.int64) // (256 // bins)
    n = np.bincount((q[:, 0] * bins + q[:, 1]) * bins + q[:, 2], minlength=bins ** 3)
    return n.astype(np.float32) / np.float32(len(q))


@pytest.mark.parametrize("bins", [1, 2, 8, 16])
def test_boxes(bins):
    from paper_1812_07607_amd import ops
    rng = np.random.default_rng(bins)
    H, W = 37, 53
    frames = rng.integers(0, 256, size=(3, H, W, 3), dtype=np.uint8)
    frames[1] = frames[1, 0, 0]  # one colour: every neighbour equal
    boxes = [(f, W - w, H - h, W, H) for f in (0, 1, 2) for w in list(range(1, 14)) + [31, 52, 53] for h in (1, 2, 5, 37)]
    boxes += [(2, x, 3, x + w, 20) for x in range(5) for w in (3, 4, 6, 17)]
    got = ops.featurize_crops_rgb8(torch.tensor(frames, device="cuda"),
                                   torch.tensor(boxes, dtype=torch.int32, device="cuda"), bins).cpu().numpy()
    for b, (f, x0, y0, x1, y1) in enumerate(boxes):
        assert np.array_equal(got[b], hist(frames[f, y0:y1, x0:x1], bins)), boxes[b]


@pytest.mark.parametrize("h,w", [(1, 1), (1, 2), (1, 3), (1, 4), (1, 5), (3, 3), (5, 7), (31, 33), (20, 21)])
def test_patches(h, w):
    from paper_1812_07607_amd import ops
    rng = np.random.default_rng(h * 100 + w)
    px = rng.integers(0, 256, size=(37, h, w, 3), dtype=np.uint8)
    got = ops.featurize_rgb8(torch.tensor(px, device="cuda"), 8).cpu().numpy()
    for p in range(len(px)):
        assert np.array_equal(got[p], hist(px[p], 8)), p
