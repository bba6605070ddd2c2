"""The training gradient's sums over positions: what is added up in FP32 does not grow with the batch.

Constant fields through centre taps make every term of a gradient sum the same number, short enough that FP32 adds
up the positions of one partial sum (256 in the output layer's backward, 16 n in the weight gradients) without
rounding, in any order: what remains are the roundings of a partial sum's row and of the gradient, 2^-24 each.
A longer FP32 sum drops the same bits of every term, about 1e-4 in all at 2^28 positions."""
import pytest
import torch

pytestmark = pytest.mark.gpu


# 128^3: 4 and 512 tiles of 512 positions per 1,024 blocks; 16^3: partial sums of half a tile
@pytest.mark.parametrize("m,batch", [(16, 3), (32, 64), (128, 1), (128, 128)])
def test_gradient_of_constant_fields_is_exact(gpu_lib, m, batch):
    from paper_1504_02591_amd import native
    dev = torch.device("cuda", 0)
    cells = batch * m ** 3
    plan = native.Plan(m, 200.0, (37.0, -60.0, 110.0), 2.0, 0.7, 0.0, batch=batch, randoms=False, cnn=True)
    w1, w2, w3 = torch.zeros(16, 27, 8), torch.zeros(16, 27, 16), torch.zeros(27, 16)
    w1[:, 13, 0] = 1.0                                     # a1 = delta
    w2[:, 13, :] = torch.eye(16)                           # a2 = a1
    w3[13, :] = 0.25                                       # y = 4 a2 + b3
    a, y = 21.0 / 16, 1461.0 / 256                         # 5 and 11 bits
    b3 = y - 4 * a
    th = torch.cat([w1.flatten(), torch.zeros(16), w2.flatten(), torch.zeros(16), w3.flatten(), torch.tensor([b3])])
    delta = torch.full((batch, m, m, m), a, device=dev)
    up = torch.full_like(delta, 13.125)                    # 0.1 u_p rounds to 21/16
    grad = torch.zeros(native.CNN_PARAMS, dtype=torch.float32, device=dev)
    loss = plan.cnn_train_step(th.to(dev), None, None, 0, 0.0, delta, up, torch.zeros_like(delta), grad_out=grad)
    plan.close()
    inv = float(torch.tensor(2.0, dtype=torch.float32) / torch.tensor(float(cells), dtype=torch.float32))
    dy = float(torch.tensor(inv * y, dtype=torch.float32))
    d2 = float(torch.tensor(0.25 * dy).to(torch.bfloat16))
    assert abs(loss - y * y) <= 1e-12 * y * y
    g = grad.double().cpu()
    g1, gb1, g2, gb2, g3, gb3 = torch.split(g, [16 * 27 * 8, 16, 16 * 27 * 16, 16, 27 * 16, 1])
    worst = {}
    for name, got, want in (("W1", g1.view(16, 27, 8)[:, :, :2], cells * d2 * a), ("b1", gb1, cells * d2),
                            ("W2", g2, cells * d2 * a), ("b2", gb2, cells * d2), ("W3", g3, cells * dy * a),
                            ("b3", gb3, cells * dy)):
        worst[name] = float((got - want).abs().max()) / want
    print(m, batch, {k: f"{v:.1e}" for k, v in worst.items()}, flush=True)
    assert max(worst.values()) <= 2 * 2.0 ** -24, worst
