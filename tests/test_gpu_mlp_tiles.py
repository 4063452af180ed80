"""The proposal network at the edges of its tiles (32 rows, 64 columns,
fragments of 16 along the sums): one layer and several, widths and batches of
one, below, at and above each edge, a smaller batch after a larger one, against
the same arithmetic in FP64 with operands rounded to BF16 per product.  An FP32
sum that rounds to the other BF16 neighbour moves one activation by at most
2^-8, so the bar is 5e-3; a wrong index is of order one."""
import numpy as np
import pytest

from oracle import mlp as OM

pytestmark = pytest.mark.gpu


def _rel(a, b):
    return np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-30)


@pytest.mark.parametrize("dims", [[1, 1], [5, 64], [16, 33, 2], [65, 31, 32, 17], [64, 100, 128, 96, 7]])
def test_edges_of_tiles(dims):
    import torch
    from paper_2505_05940_amd.mlp import MLP
    rng = np.random.default_rng(len(dims))
    net = MLP(dims, max_batch=70)
    net.init_params(seed=3)
    for B in (70, 1, 31, 32, 33, 65):
        theta = net.params().astype(float)
        x = rng.normal(size=(B, dims[0])).astype(np.float32)
        dy = rng.normal(size=(B, dims[-1])).astype(np.float32)
        y = net.forward(torch.tensor(x, device="cuda")).cpu().numpy()
        net.backward(torch.tensor(dy, device="cuda"))
        acts = OM.forward_bf16_operands(theta, dims, x.astype(float))
        assert _rel(y, acts[-1]) < 5e-3, B
        assert _rel(net.grads(), OM.backward_bf16_operands(theta, dims, acts, dy.astype(float))) < 5e-3, B
        net.adam_step(1e-3)
    net.close()


@pytest.mark.parametrize("dims,B", [([7, 1], 3), ([33, 65, 5], 33), ([64, 32, 64, 4], 32)])
def test_training_leaves_operands_and_batch(dims, B):
    """After single steps and recorded epochs of one, two and three batches,
    replayed: the products' copies of the weights are those of the parameters
    (a fresh network on them answers the same, bit for bit), and a backward
    pass sees the last batch."""
    import torch
    from paper_2505_05940_amd.mlp import MLP
    g = torch.Generator(device="cpu").manual_seed(5)
    X, Z = torch.randn(200, dims[0], generator=g).cuda(), torch.randn(200, dims[-1], generator=g).cuda()
    dy = torch.randn(B, dims[-1], generator=g).cuda()
    net, other = MLP(dims, max_batch=B + 40), MLP(dims, max_batch=B)
    net.init_params(seed=6)
    for steps in (0, 1, 2, 3, 3):
        order = torch.randperm(200, generator=g)[:B * max(steps, 1)].cuda()
        if steps:
            net.train_epoch(X, Z, order, B, 1e-3)
        else:
            net.train_step(X, Z, order, 1e-3)
        other.set_params(net.params())
        last = X[order[-B:]]
        other.forward(last)
        other.backward(dy)
        net.backward(dy)
        if len(dims) == 2:  # no ReLU decisions of older weights
            assert np.array_equal(net.grads(), other.grads()), steps
        assert np.array_equal(net.forward(last).cpu().numpy(), other.forward(last).cpu().numpy()), steps
        net.backward(dy)
        assert np.array_equal(net.grads(), other.grads()), steps
    net.close()
    other.close()
