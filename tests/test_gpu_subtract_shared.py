"""Stamps that a workgroup shares, at the lines of the rule that splits them:
stamps of 22, 28, 29 and 32 pixels (two to four wavefronts; seven and four
outputs a thread), half-widths 5 to 8, and 1023 to 8192 stamps.  Every pixel of
a frame equals the same pixel of a frame of few of these stamps (the sums do not
depend on the split), and those are the oracle's within the bar of the other
cases."""
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


@pytest.mark.parametrize("stamp", [22, 28, 29, 32])
@pytest.mark.parametrize("hw", [1, 5, 6, 8, 15])
def test_the_split_does_not_change_a_pixel(ctx, stamp, hw):
    rng = np.random.default_rng(100 * stamp + hw)
    # constant over the frame: the kernel of every stamp is the same
    sp = ipp.SubtractParams(half_width=hw, stamp=stamp, sigmas=(0.9, 2.0),
                            orders=(3, 1), spatial_order=0, bkg_order=0)
    a = [(rng.normal(0, 1, 1) / (s ** (i + j) * math.factorial(i + j)))
         .tolist() for s, i, j in osb.basis_terms(sp.sigmas, sp.orders)]
    b = [3.5]
    coef = torch.tensor(np.concatenate([np.ravel(a), b])[None], device=DEV)

    def run(I, R):
        return ctx.subtract([torch.from_numpy(I).to(DEV)],
                            [torch.from_numpy(R).to(DEV)], sp,
                            coef)[0].cpu().numpy()

    # a strip of 2 x 4 stamps, the last ones ragged, against the oracle
    h, w = 2 * stamp - 3, 4 * stamp - 5
    R = rng.normal(500, 50, (h, w)).astype(np.float32)
    I = rng.normal(300, 30, (h, w)).astype(np.float32)
    D = run(I, R)
    pix = [(x, y) for y in range(h) for x in range(w)][::37] + \
        [(0, 0), (w - 1, 0), (0, h - 1), (w - 1, h - 1)]
    want = osb.subtract(I, R, sp.sigmas, sp.orders, hw, a, 0, b, 0,
                        stamp=stamp, pixels=pix)
    Kb = osb.basis(sp.sigmas, sp.orders, hw)
    K = osb.stamp_kernel(Kb, a, 0, w, h, w / 2.0, h / 2.0)
    for x, y in pix:
        scale = osb.condition_scale(R, K, x, y, hw) + abs(I[y, x]) + 3.5
        assert abs(float(D[y, x]) - want[y, x]) <= 1e-5 * scale, (x, y)

    # the strip repeated down a frame, a gap of zeros between the copies so
    # that every copy sees the zeros that the strip's edge sees
    pitch = -(-(h + 2 * hw) // stamp) * stamp
    for rows in (255, 256, 511, 512, 2047, 2048):     # four stamps a row
        # (frames side by side where one would be taller than 32767)
        parts = -(-rows * stamp // 32000)
        each = rows // parts * stamp
        n = (each - h) // pitch + 1
        big_R = np.zeros((each, w), np.float32)
        big_I = np.zeros((each, w), np.float32)
        for k in range(n):
            big_R[k * pitch:k * pitch + h] = R
            big_I[k * pitch:k * pitch + h] = I
        rest = (rows - rows // parts * parts) * stamp
        sizes = [each + rest] + [each] * (parts - 1)
        Is = [torch.zeros((s, w), device=DEV) for s in sizes]
        Rs = [torch.zeros((s, w), device=DEV) for s in sizes]
        for x, y in zip(Is, Rs):
            x[:each].copy_(torch.from_numpy(big_I))
            y[:each].copy_(torch.from_numpy(big_R))
        out = ctx.subtract(Is, Rs, sp, coef.repeat(parts, 1).contiguous())
        for o in out:
            big = o.cpu().numpy()
            for k in range(n):
                assert np.array_equal(big[k * pitch:k * pitch + h], D), (rows,
                                                                         k)
