"""FP64 nonlocal means at sizes that take each of its shapes (one or two output
rows a lane; one, four or eight waves a tile), with ragged last tiles and
windows of fewer rows than waves, against the FP64 oracle."""
import numpy as np
import pytest
import torch

from oracle import nlm
from paper_1807_08084_amd import ops as O
from paper_1807_08084_amd import synth

pytestmark = pytest.mark.gpu
W8 = np.array([1, 1, 1, 2, 2, 2, 2, 2, 2], dtype=np.float64)[:, None]


# one row a lane and one wave a tile at the small radii, four waves at 129x127 and 173x585; two rows and one, four or
# eight waves among the rest
@pytest.mark.parametrize("distance", ["kl", "bhattacharyya"])
@pytest.mark.parametrize("H,W,r", [(551, 173, 1), (401, 399, 2), (680, 190, 0), (129, 127, 5), (173, 585, 5), (257, 255, 5),
                                   (33, 70, 16), (133, 101, 16), (799, 123, 3), (1501, 700, 1), (3, 500, 2), (700, 3, 4)])
def test_against_the_oracle(distance, H, W, r):
    img = synth.make_image(H, W, 4, (1, 1), (1e-2, 1.0), 9).planes
    z = torch.from_numpy(np.ascontiguousarray(img)).to("cuda")
    inv, det, _ = O.inv_det(z, "adjugate", "compensated")
    out, ws = O.nlm_wishart(z, inv if distance == "kl" else det.contiguous(), 4.0, r, 4.0, distance, want_wsum=True)
    out, ws = out.cpu().numpy(), ws.cpu().numpy()
    # bands of rows: the first, the last and one inside, with their halos
    for y0 in sorted({0, max(0, H // 2 - 3), max(0, H - 7)}):
        lo, hi, y1 = max(0, y0 - r), min(H, y0 + 7 + r), min(H, y0 + 7)
        ref, ref_ws = nlm.nlm_wishart(np.ascontiguousarray(img[:, lo:hi]).reshape(9, -1), hi - lo, W, r, 4.0, 4.0, distance)
        ref = ref.reshape(9, hi - lo, W)[:, y0 - lo:y1 - lo].reshape(9, -1)
        got = out[:, y0:y1].reshape(9, -1)
        e = np.sqrt((W8 * (got - ref) ** 2).sum(0) / (W8 * ref ** 2).sum(0))
        assert e.max() <= 1e-10, (y0, e.max())
        assert np.allclose(ws[y0:y1].reshape(-1), ref_ws.reshape(hi - lo, W)[y0 - lo:y1 - lo].reshape(-1), rtol=1e-10)
