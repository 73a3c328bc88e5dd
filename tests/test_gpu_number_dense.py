"""Numbering of dense detections in batches that one workgroup numbers (up to
96 tiles) and one tile more: isolated pixels, up to a quarter of all, and
structures across many tiles, in frames whose pixel counts are no multiples of
the words of a bitmap.  Label maps, boxes and counts against a labelling of the
mask in raster order of the first pixels."""
import numpy as np
import pytest
import torch
from scipy import ndimage

import paper_2502_10783_amd as ipp

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.fixture(scope="module")
def ctx():
    c = ipp.Context(0)
    c.reserve(128 << 20)         # room for a record of every second pixel
    yield c
    c.close()


def _mask(kind, h, w, rng):
    m = np.zeros((h, w), bool)
    if kind == "pixels":
        m[::2, ::2] = True
    elif kind == "some":
        m[::2, ::2] = rng.random(m[::2, ::2].shape) < 0.3
    elif kind == "lines":
        m[:, ::2] = rng.random((h, -(-w // 2))) < 0.9
    elif kind == "noise":
        m = rng.random((h, w)) < 0.16
    return m


def _labels(mask, min_area, conn):
    lab, n = ndimage.label(mask, np.ones((3, 3)) if conn == 8 else None)
    if n == 0:
        return lab, 0
    first = ndimage.minimum(np.arange(mask.size).reshape(mask.shape), lab,
                            np.arange(1, n + 1)).astype(np.int64)
    area = np.bincount(lab.ravel(), minlength=n + 1)[1:]
    new = np.zeros(n + 1, np.int64)
    keep = np.flatnonzero(area >= min_area)
    new[keep[np.argsort(first[keep])] + 1] = np.arange(1, keep.size + 1)
    return new[lab], keep.size


# 96 tiles of 64 x 64 in one frame and in several, one tile, and 97
@pytest.mark.parametrize("shapes", [
    [(512, 768)], [(511, 509), (129, 255), (63, 31), (1, 1), (200, 61)],
    [(64, 64)], [(512, 768), (5, 5)]])
@pytest.mark.parametrize("kind", ["pixels", "some", "lines", "noise"])
@pytest.mark.parametrize("min_area,conn", [(1, 8), (3, 4)])
def test_dense_numbering(ctx, shapes, kind, min_area, conn):
    rng = np.random.default_rng(sum(h * 7 + w for h, w in shapes))
    masks = [_mask(kind, h, w, rng) for h, w in shapes]
    frames = [torch.from_numpy(m.astype(np.float32)).to(DEV) for m in masks]
    zeros = [torch.zeros_like(f) for f in frames]
    half = [torch.full_like(f, 0.5) for f in frames]
    p = ipp.Params(det_nsigma=1.0, min_area=min_area, connectivity=conn)
    out = ctx.detect(frames, zeros, half, p,
                     capacity=sum(m.size for m in masks) // 2 + 64)
    torch.cuda.synchronize()
    assert int(out["diag"][2]) == 0
    t = out["table"].rows()
    off = out["table"].frame_offsets.cpu().numpy()
    for f, m in enumerate(masks):
        lab, n = _labels(m, min_area, conn)
        assert np.array_equal(out["labels"][f].cpu().numpy(), lab)
        assert off[f + 1] - off[f] == n
        rows = slice(off[f], off[f + 1])
        assert np.array_equal(t["frame"][rows], np.full(n, f))
        assert np.array_equal(t["label"][rows], np.arange(1, n + 1))
        if n == 0:
            continue
        assert np.array_equal(t["npix"][rows],
                              np.bincount(lab.ravel(), minlength=n + 1)[1:])
        for k, box in enumerate(ndimage.find_objects(lab)[:500]):
            assert (t["ymin"][rows][k], t["ymax"][rows][k] + 1,
                    t["xmin"][rows][k], t["xmax"][rows][k] + 1) == (
                box[0].start, box[0].stop, box[1].start, box[1].stop)
