"""Boxcar at the sizes where its strips and stores change: every strip height
(by the number of blocks), heights that end inside a strip or its halo, and
rows that do and do not start on a 128-byte line; Z against the __float128
oracle at the strips' edges, the inverse bitwise that of the stored Z."""
import numpy as np
import pytest
import torch

from oracle import boxcar
from paper_1807_08084_amd import ops as O
from paper_1807_08084_amd import synth
from _helpers import U32, U64, to_np

pytestmark = pytest.mark.gpu


def _bits(a):
    return a.contiguous().view(torch.int64 if a.dtype == torch.float64 else torch.int32)


# short and tall strips, one and several rounds of them (256 compute units)
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("H,W,r", [(300, 64, 1), (303, 96, 2), (1025, 1024, 3), (1500, 2049, 1), (2050, 2048, 2),
                                   (3001, 2944, 3), (4100, 3000, 1), (5000, 4096, 1)])
def test_strips(dtype, H, W, r):
    g = np.random.default_rng(H + W)
    one = synth.make_image(64, 64, 1, (2, 2), (1e-2, 1.0), 5, with_looks=True).looks
    reps = (1, -(-H // 64), -(-W // 64))
    s_np = np.ascontiguousarray(np.tile(one, reps)[:, :H, :W] * g.uniform(0.5, 2.0, (1, H, 1)))
    if dtype == torch.float32:
        s_np = s_np.astype(np.float32).astype(np.float64)
    s = O.upload_planes(s_np, dtype)
    z, inv, det, st = O.boxcar_inv_det(s, r, want_z=True, status=True)
    inv2, det2, st2 = O.inv_det(z, status=True)
    assert torch.equal(_bits(inv), _bits(inv2)) and torch.equal(_bits(det), _bits(det2)) and torch.equal(st, st2)
    z3, inv3, det3, _ = O.boxcar_inv_det(s, r)
    assert z3 is None and torch.equal(_bits(inv3), _bits(inv)) and torch.equal(_bits(det3), _bits(det))
    ys = sorted({y for e in (4, 8, 16, 24, 32, 64, 192, H) for y in (e - 1, e) if y < H} | {0, H - 1})
    pix = np.array([y * W + x for y in ys for x in (0, min(63, W - 1), W // 2, W - 1)])
    (zh, zl), mag = boxcar.boxcar128(s_np.reshape(6, -1), H, W, r, pixels=pix)
    u = U32 if dtype == torch.float32 else U64
    err = np.abs((to_np(z).reshape(9, -1)[:, pix] - zh) - zl)
    assert np.all(err <= u * np.abs(zh) + (4 * (2 * r + 1) ** 2 + 4) * U64 * mag), err.max()
