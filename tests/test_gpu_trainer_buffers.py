"""A trainer's buffers given to its network by the caller."""
import numpy as np
import pytest
import torch

from paper_1711_04471_amd import surrogate as S

pytestmark = pytest.mark.gpu


def test_the_trainers_loss_gradient_can_be_passed_to_backward():
    """It has 4 channels per pixel; a network that took it for 32 would read past its end."""
    dev = torch.device("cuda")
    n, ny, nx = 3, 37, 45
    gen = torch.Generator(device=dev).manual_seed(1)
    fields = lambda: torch.randn(3, n, ny, nx, device=dev, generator=gen)
    ds = S.Dataset(fields(), fields(), np.zeros(n, int), torch.rand(1, ny, nx, device=dev, generator=gen) + 1,
                   torch.ones(1, ny, nx, dtype=torch.uint8, device=dev))
    ds.stats = S.compute_stats(ds)
    net = S.ConvNet(seed=1)
    trainer = S.Trainer(net, ds, batch=n)
    trainer.step(np.arange(n))
    want = net.grad.clone()
    assert want.abs().max() > 0
    for d_out in (trainer.dout, torch.nn.functional.pad(trainer.dout, (0, 28))):
        net.grad.zero_()
        net.backward(trainer.x16, d_out, n, ny, nx, trainer.work)
        # the last layer takes both widths in the same order of sums
        assert torch.equal(net.grad, want)
