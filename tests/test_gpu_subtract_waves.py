"""Stamp subtraction at the stamp counts where the wavefronts of a workgroup
and the stamps of a wavefront change (512 and 1024 stamps a wavefront), with
four, three and two wavefronts' slices of LDS and both tile widths: sampled
pixels and the last stamps against the oracle, within the bar of the other
cases (1e-5 of the convolution's condition scale)."""
import math

import numpy as np
import pytest
import torch

from oracle import subtract as osb

import paper_2502_10783_amd as ipp

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.fixture(scope="module")
def ctx():
    c = ipp.Context(0)
    yield c
    c.close()


def _side(stamps, stamp):
    """A frame of so many stamps, the last column and row of them ragged."""
    rows = 1
    while stamps // (rows + 1) * stamp > 1400 and rows < 64:
        rows += 1
    while stamps % rows:
        rows -= 1
    return rows * stamp - 1, stamps // rows * stamp - 2


SMALL = ((0.9, 2.0), (3, 1))
LARGE = ((0.8, 1.2, 2.0, 3.0), (7, 7, 7, 7))


# stamp, half-width, basis; wavefronts whose slices fit a workgroup's LDS
@pytest.mark.parametrize("stamp,hw,basis,nw", [
    (5, 1, SMALL, 4), (21, 10, SMALL, 4), (24, 13, SMALL, 3),
    (32, 15, LARGE, 2)])
@pytest.mark.parametrize("per_wave,off", [(256, -1), (256, 0), (512, -1),
                                          (512, 0), (1024, -1), (1024, 0)])
def test_stamp_counts(ctx, stamp, hw, basis, nw, per_wave, off):
    stamps = per_wave * nw + off
    h, w = _side(stamps, stamp)
    assert -(-h // stamp) * -(-w // stamp) == stamps and w <= 32767
    rng = np.random.default_rng(1000 * stamp + stamps)
    sp = ipp.SubtractParams(half_width=hw, stamp=stamp, sigmas=basis[0],
                            orders=basis[1], spatial_order=1, bkg_order=1)
    R = rng.normal(500, 50, (h, w)).astype(np.float32)
    I = rng.normal(300, 30, (h, w)).astype(np.float32)
    ns = osb.n_poly(sp.spatial_order)
    a = [(rng.normal(0, 1, ns) / (s ** (i + j) * math.factorial(i + j)))
         .tolist() for s, i, j in osb.basis_terms(sp.sigmas, sp.orders)]
    b = rng.normal(0, 5, osb.n_poly(sp.bkg_order)).tolist()
    coef = np.concatenate([np.ravel(a), b])[None]
    D = ctx.subtract([torch.from_numpy(I).to(DEV)],
                     [torch.from_numpy(R).to(DEV)], sp,
                     torch.from_numpy(coef).to(DEV))[0].cpu().numpy()
    pix = sorted({(int(x), int(y)) for x, y in
                  zip(rng.integers(0, w, 25), rng.integers(0, h, 25))} |
                 {(0, 0), (w - 1, 0), (0, h - 1), (w - 1, h - 1),
                  (w - stamp, h - 1), (w // 2, h - 1)})
    want = osb.subtract(I, R, sp.sigmas, sp.orders, hw, a, sp.spatial_order,
                        b, sp.bkg_order, stamp=stamp, pixels=pix)
    Kb = osb.basis(sp.sigmas, sp.orders, hw)
    for x, y in pix:
        xs = [s for s in osb.stamps(w, stamp) if s[0] <= x < s[1]][0]
        ys = [s for s in osb.stamps(h, stamp) if s[0] <= y < s[1]][0]
        K = osb.stamp_kernel(Kb, a, sp.spatial_order, w, h, xs[2], ys[2])
        B = osb.poly(b, sp.bkg_order, osb.norm_coord(xs[2], w),
                     osb.norm_coord(ys[2], h))
        scale = osb.condition_scale(R, K, x, y, hw) + abs(I[y, x]) + abs(B)
        assert abs(float(D[y, x]) - want[y, x]) <= 1e-5 * scale, (x, y)
    # and nothing is left out or depends on which wavefront came first
    D2 = ctx.subtract([torch.from_numpy(I).to(DEV)],
                      [torch.from_numpy(R).to(DEV)], sp,
                      torch.from_numpy(coef).to(DEV))[0].cpu().numpy()
    assert np.array_equal(D, D2) and np.isfinite(D).all()
