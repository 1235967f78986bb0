"""Nonlocal means at the sizes where its tilings change: the waves per tile
and the rows per lane by the number of two-row tiles, windows that cover no
more than a tile, ragged last tiles, and non-finite pixels (which reach the
outputs whose window holds them and no others)."""
import numpy as np
import pytest
import torch

from oracle import nlm
from paper_1807_08084_amd import synth

pytestmark = pytest.mark.gpu
W8 = np.array([1, 1, 1, 2, 2, 2, 2, 2, 2], dtype=np.float64)[:, None]


@pytest.fixture(scope="module")
def ops():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1807_08084_amd import ops as o
    o.compute_units()
    return o


def _aux(ops, z, distance):
    inv, det, _ = ops.inv_det(z, "adjugate", "compensated")
    return inv if distance == "kl" else det.contiguous()


# two-row tiles: 1 (eight waves each), 1023, 1024 (four), 9215, 9216 (one wave)
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("distance", ["kl", "bhattacharyya"])
@pytest.mark.parametrize("H,W,r", [(1, 1, 16), (2, 64, 1), (2045, 60, 2), (2047, 63, 1), (3686, 320, 1),
                                   (3686, 319, 2), (18431, 5, 1), (6143, 129, 3)])
def test_tilings(ops, dtype, distance, H, W, r):
    n_looks, h = 4.0, 16.0
    img = synth.make_image(H, W, 4, (1, 1), (1e-2, 1.0), 7).planes
    if dtype == torch.float32:
        img = img.astype(np.float32).astype(np.float64)
    z = torch.from_numpy(np.ascontiguousarray(img)).to("cuda", dtype)
    out, ws = ops.nlm_wishart(z, _aux(ops, z, distance), n_looks, r, h, distance, want_wsum=True)
    out, ws = out.cpu().numpy().astype(np.float64), ws.cpu().numpy()
    tol = 1e-10 if dtype == torch.float64 else 1e-4
    # bands of rows: the first, the last and one inside, with their halos
    for y0 in sorted({0, max(0, H // 2 - 3), max(0, H - 7)}):
        lo, hi = max(0, y0 - r), min(H, y0 + 7 + r)
        ref, ref_ws = nlm.nlm_wishart(np.ascontiguousarray(img[:, lo:hi]).reshape(9, -1), hi - lo, W, r, n_looks, h,
                                      distance)
        y1 = min(H, y0 + 7)
        ref = ref.reshape(9, hi - lo, W)[:, y0 - lo:y1 - lo].reshape(9, -1)
        got = out[:, y0:y1].reshape(9, -1)
        e = np.sqrt((W8 * (got - ref) ** 2).sum(0) / (W8 * ref ** 2).sum(0))
        assert e.max() <= tol, (y0, e.max())
        assert np.allclose(ws[y0:y1].reshape(-1), ref_ws.reshape(hi - lo, W)[y0 - lo:y1 - lo].reshape(-1),
                           rtol=100 * tol)


@pytest.mark.parametrize("distance", ["kl", "bhattacharyya"])
@pytest.mark.parametrize("value", [np.nan, np.inf])
@pytest.mark.parametrize("H,W", [(40, 150), (1500, 900)])  # shared tiles, single-wave tiles
def test_non_finite_pixels_stay_in_their_windows(ops, distance, value, H, W):
    r = 3
    img = synth.make_image(H, W, 4, (2, 2), (1e-2, 1.0), 7).planes.astype(np.float32)
    z = torch.from_numpy(np.ascontiguousarray(img)).to("cuda")
    clean, _ = ops.nlm_wishart(z, _aux(ops, z, distance), 4.0, r, 16.0, distance)
    y, x = 21, 66
    z[0, y, x] = value
    out, _ = ops.nlm_wishart(z, _aux(ops, z, distance), 4.0, r, 16.0, distance)
    touched = torch.zeros((H, W), dtype=torch.bool, device="cuda")
    touched[y - r:y + r + 1, x - r:x + r + 1] = True
    assert torch.equal(out[:, ~touched], clean[:, ~touched])
    assert torch.isnan(out[0][touched]).all()
