"""A forward pass of the Wishart likelihood runs with more resident blocks than
the pass that also writes the gradient: its loss and per-pixel terms have the
same bits, in both launch entries, with and without a cap in the table and with
the largest one the table takes."""
import pytest
import torch

from paper_1807_08084_amd import ops as O
from paper_1807_08084_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("n", [1, 127, 128 * 300 + 5, (1 << 23) + 3])
@pytest.mark.parametrize("cap", [None, 0, 64])
def test_forward_alone_is_the_fused_loss(dtype, n, cap):
    one = torch.from_numpy(synth.make_image(64, 64, 8, (2, 2), (1e-2, 1.0), 7).planes.reshape(9, -1)).to("cuda", dtype)
    z = one.repeat(1, -(-n // one.shape[1]))[:, :n].contiguous()
    s = (z * 1.25).contiguous()
    op = O.wishart_launch_op(n)
    keep = O.get_launch(op, dtype, "adjugate", "plain")
    try:
        if cap is not None:
            O.set_launch(op, dtype, "adjugate", "plain", dict(keep, blocks_per_cu=cap))
        fused, _, ell = O.wishart_loglik(s, z, 8.0, forward=True, backward=True, ell=True)
        loss, _, ell1 = O.wishart_loglik(s, z, 8.0, forward=True, ell=True)
        torch.cuda.synchronize()
    finally:
        O.set_launch(op, dtype, "adjugate", "plain", keep)
    assert torch.isfinite(loss).item()
    assert torch.equal(loss, fused) and torch.equal(ell1, ell)
