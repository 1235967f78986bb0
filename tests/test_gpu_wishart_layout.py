"""The layout of the gradient that autograd is handed: contiguous for a leaf,
which autograd then keeps without a copy; padded planes for a large computed
Sigma, whose gradient nobody keeps; the same bits either way."""
import pytest
import torch

from paper_1807_08084_amd import ops as O

pytestmark = pytest.mark.gpu


def _planes(n, dtype, seed):
    g = torch.Generator("cuda").manual_seed(seed)
    z = torch.randn((9, n), generator=g, device="cuda", dtype=dtype) * 0.05
    z[:3] = 1.0 + z[:3].abs()
    return z


# eighteen planes of 176 MB hold 2563185.8 FP32 and 1281592.9 FP64 pixels
@pytest.mark.parametrize("dtype,n,padded", [(torch.float32, 1001, False), (torch.float32, 2563185, False),
                                            (torch.float32, 2563186, True), (torch.float64, 1281592, False),
                                            (torch.float64, 1281593, True), (torch.float32, 4194304, True)])
def test_layout(dtype, n, padded):
    z = _planes(n, dtype, 1)
    leaf = _planes(n, dtype, 2).requires_grad_(True)
    O.wishart_nll(leaf, z, 4.0).backward()
    assert leaf.grad.is_contiguous()

    theta = leaf.detach().requires_grad_(True)
    sigma = theta * 1.0
    seen = []
    sigma.register_hook(lambda g: seen.append((g.stride(), g.clone())))
    O.wishart_nll(sigma, z, 4.0).backward()
    pitch = O.recommended_pitch(dtype, n) if padded else n
    assert seen[0][0] == (pitch, 1)
    assert torch.equal(seen[0][1], leaf.grad) and torch.equal(theta.grad, leaf.grad)
