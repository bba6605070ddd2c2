"""The sums over cells that a non-gradient start's first eps is formed from (S2 = sum Delta^2)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def eps1(native, n, c, passes):
    """eps_1 of the start Delta = c everywhere on an empty field, with a network of zeros and an output bias."""
    dev = torch.device("cuda", 0)
    # beta = 1, so that no start is rejected; the observer far away, so that Psi_0 = c r is nearly uniform and
    # eps_1^2 = 1 + (S2 - 2 S3) / ||Psi_1||^2 is nearly S2 / ||Psi_1||^2
    plan = native.Plan(n, 10.0 * n, (-50.0 * n, 4.0 * n, 7.0 * n), 1.0, 1.0, 10.0, randoms=False, keep_delta=True,
                       start_buffers=True, cnn=True, cnn_quarter=True)
    net = torch.zeros(native.CNN_PARAMS, device=dev)
    net[-1] = float(np.float32(c / 10))
    m = plan.cnn_n
    zero = torch.zeros((1, m, m, m), device=dev)
    du = plan.cnn_forward(net, zero, zero)
    assert float(du.min()) == c == float(du.max())
    plan.set_delta(torch.zeros((n, n, n), device=dev))
    plan.solve(native.START_LEARNED, net)
    _, _, eps = plan.iterate(passes, 0.0)
    assert plan.restarts() == [0]
    plan.close()
    return eps[0][0]


@pytest.mark.parametrize("n", [128, 256, 512])
@pytest.mark.parametrize("passes", [1, 2])
def test_first_eps_does_not_depend_on_the_scale_of_the_start(gpu_lib, n, passes):
    # eps_1 is a ratio of lengths: the same for every c.  c = 3.5 squares to 6 bits and sums exactly; c = 995/256
    # squares to 20 bits (990025 = 1 mod 8), of which FP32 adds up 16 exactly and loses one unit in each of the next
    # 16: a thread's sum of 32 terms would be 16 / (32 * 990025) = 5e-7 too small and eps_1 half of that.  The
    # other roundings are random and average out over 2^21 cells or more; a fifth of the effect is allowed.
    from paper_1504_02591_amd import native
    a, b = eps1(native, n, 3.5, passes), eps1(native, n, 995.0 / 256, passes)
    print(n, passes, a, b, b / a - 1.0, flush=True)
    assert a > 5.0 and abs(b / a - 1.0) <= 5e-8
