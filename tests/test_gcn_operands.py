"""Which tensors the layer's own dense kernels may take (no GPU)."""
import torch

from paper_2603_08734_amd import gcn


def test_a_batched_gradient_is_told_from_a_matrix_with_memory():
    seen = []

    class Identity(torch.autograd.Function):
        @staticmethod
        def forward(ctx, x):
            return x.clone()

        @staticmethod
        def backward(ctx, g):
            # to the other checks it is a contiguous matrix
            seen.append((type(g) is torch.Tensor and g.dim() == 2 and g.is_contiguous(), gcn._has_memory(g)))
            return g

    x = torch.ones(3, 4, requires_grad=True)
    torch.autograd.grad(Identity.apply(x), x, torch.ones(5, 3, 4), is_grads_batched=True)
    torch.autograd.grad(Identity.apply(x), x, torch.ones(3, 4))
    assert seen == [(True, False), (True, True)]
