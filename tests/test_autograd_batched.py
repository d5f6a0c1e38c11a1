"""The L1 step's reverse function scales the step's gradients by the incoming one
in every form that autograd calls it in: alone, for a batch of incoming
gradients at once, and with a graph of its own (CPU: the forward is a stand-in
that saves five tensors as the step does)."""
import pytest
import torch

from paper_2510_01767_amd.raster import PARAM_NAMES, RasterizeL1Fn

SHAPES = dict(means=(3, 7), log_scales=(3, 7), quats=(4, 7), opacity_logits=(7,), sh=(12, 7))


class StandIn(torch.autograd.Function):
    """sum of the parameters' squares over two, and an image; saves the gradients like RasterizeL1Fn."""

    @staticmethod
    def forward(ctx, *args):
        params = args[:5]
        ctx.save_for_backward(*[p.detach().clone() for p in params])
        images = torch.zeros(2)
        ctx.mark_non_differentiable(images)
        return sum((p * p).sum() / 2 for p in params), images

    backward = staticmethod(RasterizeL1Fn.backward)


def loss_of(seed=0):
    g = torch.Generator().manual_seed(seed)
    leaves = [torch.randn(SHAPES[k], generator=g, requires_grad=True) for k in PARAM_NAMES]
    return leaves, StandIn.apply(*leaves, None, None, None)[0]


@pytest.mark.parametrize("create_graph", [False, True])
def test_scales_by_the_incoming_gradient(create_graph):
    leaves, loss = loss_of()
    scale = torch.tensor(3.0, requires_grad=True)
    got = torch.autograd.grad(loss, leaves, scale, create_graph=create_graph)
    for x, p in zip(got, leaves):
        assert torch.equal(x.detach(), 3.0 * p.detach())
    if create_graph:
        (d,) = torch.autograd.grad(sum(x.sum() for x in got), scale)
        assert torch.allclose(d, sum(p.detach().sum() for p in leaves))


def test_a_batch_of_incoming_gradients():
    leaves, loss = loss_of()
    scales = torch.tensor([1.0, -2.0, 0.5, 0.0])
    got = torch.autograd.grad(loss, leaves, scales, is_grads_batched=True)
    for x, p in zip(got, leaves):
        want = torch.stack([s * p.detach() for s in scales])
        assert x.shape == want.shape and torch.equal(x, want)
