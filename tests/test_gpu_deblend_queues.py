"""Deblending of the same candidates in tables of different capacity, at both
sides of the length from which the one-wavefront kernel takes its rows from
several counters (256 rows and one): the same maps, objects and counts."""
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
    for capacity in (230, 254, 255, 256, 4096):
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
