"""Which accesses stream is chosen by the input's size and the gradient's
alignment: on either side of both lines the bits are those of a launch without
streaming accesses."""
import pytest
import torch

from paper_1807_08084_amd import ops as O

pytestmark = pytest.mark.gpu


def _bits(a):
    return a.contiguous().view(torch.int64 if a.dtype == torch.float64 else torch.int32)


def _planes(n, dtype, seed):
    g = torch.Generator("cuda").manual_seed(seed)
    z = torch.randn((9, n), generator=g, device="cuda", dtype=dtype) * 0.2
    z[:3] = 1.0 + z[:3].abs()
    return z


# nine planes of 192 MB hold 5592405.3 FP32 and 2796202.7 FP64 pixels, eighteen half of that; of 48 MB, a quarter
@pytest.mark.parametrize("dtype,n", [(torch.float32, 5592405), (torch.float32, 5592406), (torch.float32, 2796202),
                                     (torch.float32, 2796203), (torch.float64, 2796202), (torch.float64, 2796203),
                                     (torch.float64, 1398101), (torch.float64, 1398102), (torch.float32, 1001),
                                     (torch.float32, 1398101), (torch.float32, 1398102)])
def test_streaming_or_not_the_same_bits(dtype, n):
    z, s = _planes(n, dtype, 1), _planes(n, dtype, 2)
    plain, padded = torch.empty_like(z), O.empty_planes(9, (n,), dtype)
    g = torch.tensor(1.5, dtype=torch.float64, device="cuda")

    def all_outputs():
        inv, det, st = O.inv_det(z, status=True)
        loss, grad, _ = O.wishart_loglik(s, z, 4.0, forward=True, backward=True, grad_loss=g, grad=plain)
        _, back, _ = O.wishart_loglik(s, z, 4.0, forward=False, backward=True, grad_loss=g, grad=padded)
        return [x.clone() for x in (inv, det, grad, back)], st, loss

    a = all_outputs()
    keys = [(O.inv_det_launch_op(n), "compensated"), (O.wishart_launch_op(n), "plain")]
    keep = [O.get_launch(op, dtype, "adjugate", p) for op, p in keys]
    try:
        for (op, p), k in zip(keys, keep):
            assert k["nontemporal"] == 1
            O.set_launch(op, dtype, "adjugate", p, dict(k, nontemporal=0))
        b = all_outputs()
    finally:
        for (op, p), k in zip(keys, keep):
            O.set_launch(op, dtype, "adjugate", p, k)
    torch.cuda.synchronize()
    assert all(torch.equal(_bits(x), _bits(y)) for x, y in zip(a[0], b[0]))
    assert torch.equal(a[1], b[1]) and torch.equal(_bits(a[2]), _bits(b[2]))  # (the loss may be NaN: some are not PD)
    assert torch.equal(_bits(a[0][2]), _bits(a[0][3]))


@pytest.mark.parametrize("dtype,n", [(torch.float32, 2796203), (torch.float64, 1398101), (torch.float32, 70001)])
def test_finite_loss_has_the_same_bits(dtype, n):
    z, s = _planes(n, dtype, 3), _planes(n, dtype, 4)
    z[3:] *= 0.1
    s[3:] *= 0.1
    op = O.wishart_launch_op(n)
    keep = O.get_launch(op, dtype, "adjugate", "plain")
    losses = []
    try:
        for nt in (1, 0):
            O.set_launch(op, dtype, "adjugate", "plain", dict(keep, nontemporal=nt))
            for kw in ({}, {"backward": True}, {"backward": True, "grad": torch.empty_like(z)}):
                losses.append(O.wishart_loglik(s, z, 4.0, **kw)[0])
    finally:
        O.set_launch(op, dtype, "adjugate", "plain", keep)
    torch.cuda.synchronize()
    assert torch.isfinite(losses[0]).item() and all(torch.equal(x, losses[0]) for x in losses)


# eighteen planes of 80 MB hold 1165084.4 FP32 and 582542.2 FP64 pixels, of 176 MB 2563185.8 and 1281592.9
@pytest.mark.parametrize("dtype,n", [(torch.float32, 1165084), (torch.float32, 1165085), (torch.float32, 2563185),
                                     (torch.float32, 2563186), (torch.float64, 582543), (torch.float64, 1281593),
                                     (torch.float32, 1165088), (torch.float32, 8388611)])
def test_the_same_bits_around_the_gradients_lines(dtype, n):
    test_streaming_or_not_the_same_bits(dtype, n)
