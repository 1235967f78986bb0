"""A NaN or infinite single-look pixel reaches the boxcar outputs whose window
holds it and no others: two columns of a lane share their windows' inner
columns, and a strip's running sums pass the pixel's row."""
import pytest
import torch

from paper_1807_08084_amd import ops as O

pytestmark = pytest.mark.gpu


def _bits(a):
    return a.contiguous().view(torch.int64 if a.dtype == torch.float64 else torch.int32)


# columns of either parity, at the seams of 64- and 128-column tiles and at the sides
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("value", [float("nan"), float("inf")])
@pytest.mark.parametrize("r", [1, 2, 3])
@pytest.mark.parametrize("H,W", [(41, 256), (41, 301)])
def test_non_finite_pixel_stays_in_its_windows(dtype, value, r, H, W):
    g = torch.Generator("cuda").manual_seed(5)
    s = torch.randn((6, H, W), generator=g, device="cuda", dtype=dtype)
    clean = O.boxcar_inv_det(s, r, want_z=True, status=True)
    for y, x in ((20, 64), (20, 65), (7, 127), (7, 128), (0, 0), (H - 1, W - 1), (33, 200), (16, 191)):
        t = s.clone()
        t[2, y, x] = value
        z, inv, det, st = O.boxcar_inv_det(t, r, want_z=True, status=True)
        inside = torch.zeros((H, W), dtype=torch.bool, device="cuda")
        inside[max(0, y - r):y + r + 1, max(0, x - r):x + r + 1] = True
        for got, ref in ((z, clean[0]), (inv, clean[1]), (det[None], clean[2][None])):
            assert torch.equal(_bits(got[:, ~inside]), _bits(ref[:, ~inside]))
        assert torch.equal(st[~inside], clean[3][~inside])
        assert not torch.isfinite(z[1][inside]).any() and not torch.isfinite(det[inside]).any()
        assert (st[inside] == 3).all()
