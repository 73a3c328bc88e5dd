"""Regions whose rows are not whole groups of four columns, at both sides of
the sizes where the statistics change from a wavefront's 16 to its 64 values a
lane and to the workgroup's, against the oracle: every pixel of a region counts
(a row of mesh_w pixels takes ceil(mesh_w / 4) groups).  Medians are exact;
the deviation holds the bar of the region statistics' own tests (1e-11)."""
import numpy as np
import pytest
import torch

import oracle
from oracle import background as obg

import paper_2502_10783_amd as ipp

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.fixture(scope="module")
def ctx():
    c = ipp.Context(0)
    yield c
    c.close()


# groups of four a region: up to 256, up to 1024 and more, with at most 1024
# or 4096 pixels on the far side of each line
@pytest.mark.parametrize("mesh", [
    (28, 33), (28, 34), (30, 34), (60, 17), (51, 17), (32, 32), (64, 63),
    (62, 66), (65, 63), (124, 33), (113, 33), (60, 66), (64, 64), (128, 29)])
@pytest.mark.parametrize("masked", [False, True])
def test_every_pixel_of_a_region_counts(ctx, mesh, masked):
    mh, mw = mesh
    rng = np.random.default_rng(100 * mh + mw)
    h, w = 2 * mh + mh // 2, 2 * mw + mw - 3
    img = rng.normal(900.0, 7.0, (h, w)).astype(np.float32)
    # a gradient along the rows, so that a row left out moves the median
    img += np.linspace(0.0, 400.0, h, dtype=np.float32)[:, None]
    mask = rng.random((h, w)) < 0.1 if masked else None
    kw = dict(mesh_h=mh, mesh_w=mw)
    p, op = ipp.Params(**kw), oracle.Params(**kw)
    masks = None
    if masked:
        masks = [torch.from_numpy(mask.astype(np.uint8)).to(DEV)]
    out = ctx.background([torch.from_numpy(img).to(DEV)], p, masks=masks,
                         mesh=True)
    torch.cuda.synchronize()
    braw, rraw, n, _, _ = obg.mesh_stats(img, op, mask)
    assert np.array_equal(out["n_used"][0].cpu().numpy(), n)
    np.testing.assert_allclose(out["bkg_raw"][0].cpu().numpy(), braw,
                               rtol=1e-12, atol=0)
    np.testing.assert_allclose(out["rms_raw"][0].cpu().numpy(), rraw,
                               rtol=1e-11, atol=0)
