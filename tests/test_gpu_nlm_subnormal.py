"""Bhattacharyya weights in FP32 where the determinant of a pair's sum is
subnormal for some pairs and normal for others (one wave meets both): the
logarithm of the former takes another path than that of the latter."""
import numpy as np
import pytest
import torch

from oracle import nlm
from paper_1807_08084_amd import ops as O
from paper_1807_08084_amd import synth

pytestmark = pytest.mark.gpu
W8 = np.array([1, 1, 1, 2, 2, 2, 2, 2, 2], dtype=np.float64)[:, None]


def _det(z):
    a, d, f, br, bi, cr, ci, er, ei = z
    return (a * (d * f - er * er - ei * ei) - f * (br * br + bi * bi) - d * (cr * cr + ci * ci)
            + 2.0 * (br * (er * cr + ei * ci) + bi * (er * ci - ei * cr)))


# Twenty roundings of at most 2^-150 against sums of 2^-128 and more: 5e-6 in
# the determinant, a quarter of that in a weight (n_looks / h), and FP32's own
# rounding beside it: below the 1e-4 of images of ordinary scale.
@pytest.mark.parametrize("H,W,r", [(30, 70, 2), (9, 64, 16), (520, 600, 1)])
def test_subnormal_determinants(H, W, r):
    img = synth.make_image(H, W, 16, (1, 1), (0.5, 1.0), 11).planes
    img = img * 2.0 ** np.round((-131.0 - np.log2(_det(img.reshape(9, -1)).min())) / 3.0)
    z32 = img.astype(np.float32)
    ref_in = z32.astype(np.float64).reshape(9, -1)
    det = _det(ref_in)
    tiny = 2.0 ** -126
    assert (8.0 * det < tiny).any() and (8.0 * det > tiny).any()
    out, _ = O.nlm_wishart(torch.from_numpy(z32).cuda(), torch.from_numpy(det.astype(np.float32).reshape(H, W)).cuda(),
                           4.0, r, 16.0, "bhattacharyya")
    out = out.cpu().numpy().astype(np.float64).reshape(9, -1)
    y = min(H, 24)  # rows compared, with their halo
    hi = min(H, y + r)
    ref, _ = nlm.nlm_wishart(np.ascontiguousarray(ref_in.reshape(9, H, W)[:, :hi]).reshape(9, -1), hi, W, r, 4.0, 16.0,
                             "bhattacharyya")
    got, ref = out.reshape(9, H, W)[:, :y].reshape(9, -1), ref.reshape(9, hi, W)[:, :y].reshape(9, -1)
    scale = 1.0 / np.abs(ref).max()
    e = np.sqrt((W8 * ((got - ref) * scale) ** 2).sum(0) / (W8 * (ref * scale) ** 2).sum(0))
    assert e.max() <= 1e-4, e.max()
