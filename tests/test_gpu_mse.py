"""The MSE kernel where its threads take one ray, several, or a remainder, against FP64 torch on the CPU."""
import pytest
import torch

from paper_2307_15333_amd import core

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("gather", [True, False])
@pytest.mark.parametrize("n", [1, 1023, 262144, 262145, 4 * 262144 + 3])
def test_every_ray_once(n, gather):
    """The residual is exact in FP64 and the gradient one rounding of a product, so it is equal bit for bit; the loss
    is an FP64 sum of 3 n non-negative terms, off by at most 3 n 2^-53 of itself."""
    rng = torch.Generator().manual_seed(n)
    pred = torch.rand((n, 3), generator=rng)
    rows = n + 7 if gather else n
    target = torch.rand((rows, 3), generator=rng)
    idx = torch.randint(0, rows, (n,), generator=rng) if gather else None
    loss, grad = core.mse_loss(pred.cuda(), target.cuda(), idx.cuda() if gather else None)
    e = pred.double() - (target[idx] if gather else target).double()
    want = (2.0 / (3.0 * n)) * e
    assert torch.equal(grad.cpu(), want.float())
    ref = float((e * e).sum() / (3.0 * n))
    assert abs(float(loss) - ref) <= 3 * n * 2.0 ** -53 * ref * 2
