"""Boxcar where the way a row is walked and stored changes: one or two columns
a lane, one to eight waves a block, streaming or cached stores.  A pixel's
result depends on its window alone, so a large image's outputs have the bits of
a small crop's (of the same column parity) away from the crop's sides, and are
the same with and without Z."""
import pytest
import torch

from paper_1807_08084_amd import ops as O

pytestmark = pytest.mark.gpu


def _bits(a):
    return a.contiguous().view(torch.int64 if a.dtype == torch.float64 else torch.int32)


# widths at the edges of 64- and 128-column tiles and of blocks of 4 and 8 of
# them; the last three write more than 256 MB with Z
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("H,W", [(9, 1), (40, 63), (41, 65), (60, 127), (37, 129), (33, 191), (50, 193), (21, 257),
                                 (70, 511), (35, 513), (90, 1025), (1200, 3073), (2000, 2017), (37000, 100)])
@pytest.mark.parametrize("r", [1, 2, 3])
def test_crops_and_outputs_agree(dtype, H, W, r):
    g = torch.Generator("cuda").manual_seed(H * W + r)
    s = torch.randn((6, H, W), generator=g, device="cuda", dtype=dtype)
    z, inv, det, st = O.boxcar_inv_det(s, r, want_z=True, status=True)
    _, inv1, det1, _ = O.boxcar_inv_det(s, r)
    assert torch.equal(_bits(inv), _bits(inv1)) and torch.equal(_bits(det), _bits(det1))
    spots = [(0, 0), (H // 2, W // 2 // 2 * 2), (max(0, H - 24), max(0, W - 70) // 2 * 2), (0, max(0, W - 70) // 2 * 2)]
    for y0, x0 in spots:
        y1, x1 = min(H, y0 + 24), min(W, x0 + 72)
        cz, ci, cd, cs = O.boxcar_inv_det(s[:, y0:y1, x0:x1].contiguous(), r, want_z=True, status=True)
        # the image's own sides clip the crop's windows alike
        t, b = (0 if y0 == 0 else r), (0 if y1 == H else r)
        lf, rt = (0 if x0 == 0 else r), (0 if x1 == W else r)
        ys, xs = slice(t, y1 - y0 - b), slice(lf, x1 - x0 - rt)
        Y, X = slice(y0 + t, y1 - b), slice(x0 + lf, x1 - rt)
        assert torch.equal(_bits(cz[:, ys, xs]), _bits(z[:, Y, X]))
        assert torch.equal(_bits(ci[:, ys, xs]), _bits(inv[:, Y, X]))
        assert torch.equal(_bits(cd[ys, xs]), _bits(det[Y, X])) and torch.equal(cs[ys, xs], st[Y, X])
