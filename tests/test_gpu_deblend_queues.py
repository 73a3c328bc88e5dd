"""Deblending of the same candidates in tables of different capacity, at both
sides of the lengths from which rows are taken from several counters (256) and
each class of candidates has a kernel of its own (2048): the same maps, objects
and counts."""
import numpy as np
import pytest
import torch

import paper_2502_10783_amd as ipp

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def test_any_capacity_gives_the_same_objects():
    rng = np.random.default_rng(12)
    h, w = 700, 900
    yy, xx = np.mgrid[-12:13, -12:13].astype(np.float64)
    img = rng.normal(0.0, 1.0, (h, w))
    # pairs that blend, and singles
    for k in range(230):
        cy, cx = 20 + 45 * (k // 19) + 4, 20 + 45 * (k % 19) + 4
        img[cy - 12:cy + 13, cx - 12:cx + 13] += 300.0 * np.exp(
            -(yy ** 2 + xx ** 2) / 4.0)
        if k % 2:
            img[cy - 12:cy + 13, cx - 12:cx + 13] += 250.0 * np.exp(
                -((yy - 1) ** 2 + (xx - 6) ** 2) / 4.0)
    img = torch.from_numpy(img.astype(np.float32)).to(DEV)
    bkg, rms = torch.zeros_like(img), torch.ones_like(img)
    p = ipp.Params(det_nsigma=5.0)
    ctx = ipp.Context(0)
    first = None
    for capacity in (230, 254, 255, 256, 2047, 2048, 4096):
        det = ctx.detect([img], [bkg], [rms], p, capacity=capacity)
        d = ctx.deblend([img], [bkg], [rms], det["labels"], det["table"], p,
                        ipp.DeblendParams(mincont=0.001), capacity=1024)
        torch.cuda.synchronize()
        assert det["table"].count() == 230
        assert d["diag"].cpu().tolist()[2:] == [0, 345]
        got = [d["objects"][0].cpu().numpy(), d["parent"][:345].cpu().numpy(),
               d["table"].rows()]
        if first is None:
            first = got
        assert np.array_equal(got[0], first[0])
        assert np.array_equal(got[1], first[1])
        for k, v in got[2].items():
            assert np.array_equal(v, first[2][k], equal_nan=True), k
    ctx.close()


# scale 1e6: sums of more than 64 bits, every candidate in the pool's scratch;
# 1e12: every weight clamped to 2^62 - 1, so that nothing splits
@pytest.mark.parametrize("scale", [1.0, 1e6, 1e12])
@pytest.mark.parametrize("conn", [4, 8])
def test_every_class_in_one_kernel_and_in_three(scale, conn):
    rng = np.random.default_rng(8)
    img = np.zeros((260, 420))
    # boxes of about 100 to 12,000 pixels (a wavefront up to 512, a workgroup
    # up to 2048, in LDS up to 6144), several peaks in each
    for x0, side in ((10, 8), (30, 14), (60, 22), (95, 30), (140, 44),
                     (200, 72), (290, 110)):
        img[20:20 + side, x0:x0 + side] = 200.0
        yy, xx = np.mgrid[0:260, 0:420]
        for _ in range(3 + side // 12):
            cy, cx = 20 + rng.uniform(2, side - 2), x0 + rng.uniform(2, side - 2)
            img += 4000.0 * np.exp(-((yy - cy) ** 2 + (xx - cx) ** 2) / 4.0) * (
                (yy >= 20) & (yy < 20 + side) & (xx >= x0) & (xx < x0 + side))
    img[200:202, ::3] = 900.0 * rng.random((2, 140))      # and tiny ones
    img = torch.from_numpy((img * scale).astype(np.float32)).to(DEV)
    bkg, rms = torch.zeros_like(img), torch.full_like(img, 20.0 * scale)
    p = ipp.Params(det_nsigma=2.0, connectivity=conn)
    ctx = ipp.Context(0)
    first = None
    for capacity in (100, 2047, 2048):
        det = ctx.detect([img], [bkg], [rms], p, capacity=capacity)
        d = ctx.deblend([img], [bkg], [rms], det["labels"], det["table"], p,
                        ipp.DeblendParams(mincont=0.002), capacity=1024)
        torch.cuda.synchronize()
        assert d["diag"].cpu().tolist()[2] == 0
        n = d["table"].count()
        if scale < 1e12:
            assert n > det["table"].count() + 6
        else:
            assert n == det["table"].count()
        got = [d["objects"][0].cpu().numpy(), d["parent"][:n].cpu().numpy(),
               d["table"].rows()]
        if first is None:
            first = got
        assert np.array_equal(got[0], first[0])
        assert np.array_equal(got[1], first[1])
        for k, v in got[2].items():
            assert np.array_equal(v, first[2][k], equal_nan=True), k
    ctx.close()
