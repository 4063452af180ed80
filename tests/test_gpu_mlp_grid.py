"""Phases of more workgroups than one row of a grid holds (2^15): the
conversion of a wide input of many rows, forward and in a training step, against
torch on operands rounded to BF16.  FP32 sums of 4096 and 20000 products: 1e-5
covers their order, a row or column that is missing is of order one (bars as
for single products elsewhere, 5e-3)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
DIMS, B = [4096, 8], 20000  # 625 x 64 tiles of the input


def test_wide_input_of_many_rows():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2505_05940_amd.mlp import MLP
    gen = torch.Generator(device="cuda").manual_seed(1)
    x = torch.randn(B, DIMS[0], generator=gen, device="cuda")
    z = torch.randn(B, DIMS[1], generator=gen, device="cuda")
    net = MLP(DIMS, max_batch=B)
    net.init_params(seed=2)
    theta = torch.tensor(net.params(), device="cuda")
    W, b = theta[:DIMS[0] * DIMS[1]].reshape(DIMS[1], DIMS[0]), theta[DIMS[0] * DIMS[1]:]
    xr, Wr = x.bfloat16().float(), W.bfloat16().float()
    ref = xr @ Wr.t() + b
    y = net.forward(x)
    assert (y - ref).norm() < 5e-3 * ref.norm()
    assert ((y - ref).norm(dim=1) < 5e-2 * ref.norm(dim=1)).all()  # every row
    order = torch.randperm(B, generator=gen, device="cuda")
    loss = torch.zeros(1, device="cuda")
    net.train_step(x, z, order, 1e-3, loss_acc=loss)
    e = ref - z
    assert abs(loss.item() - (e * e).mean().item()) < 5e-3 * (e * e).mean().item()
    g = (2.0 / (B * DIMS[1]) * e).bfloat16().float()
    gW = g.t() @ xr
    got = torch.tensor(net.grads(), device="cuda")[:DIMS[0] * DIMS[1]].reshape(DIMS[1], DIMS[0])
    assert (got - gW).norm() < 5e-3 * gW.norm()
    net.close()
