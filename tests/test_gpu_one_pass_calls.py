"""A call that is sure to stop after its first pass launches what a call of one pass does, and no more."""
import pytest
import torch

pytestmark = pytest.mark.gpu


# growth, tolerance: no growth (eps_1 = 0), and tolerances above what the first pass can give, beta / (1 - beta)
@pytest.mark.parametrize("n,batch", [(32, 1), (64, 40), (128, 1), (256, 1)])
@pytest.mark.parametrize("growth,tol,relaxed", [(0.0, 1e-3, False), (0.0, 1e-3, True), (0.6, 3.0, False), (0.6, 3.0, True)])
def test_no_launch_for_a_second_pass(gpu_lib, n, batch, growth, tol, relaxed):
    from paper_1504_02591_amd import native
    dev = torch.device("cuda", 0)
    g = torch.Generator(device=dev).manual_seed(n)
    d = torch.randn((batch, n, n, n), generator=g, device=dev)
    plan = native.Plan(n, 10.0 * n, (-300.0, 4.0 * n, 7.0 * n), 1.0, growth, 10.0, randoms=False, batch=batch,
                       relaxed=relaxed)
    out = []
    for passes, t in ((1, 0.0), (30, tol)):
        plan.set_delta(d)
        plan.solve()
        plan.profile_start()
        _, iters, eps = plan.iterate(passes, t)
        launches = {k: v[0] for k, v in plan.profile_stop().items()}
        out.append((launches, iters, eps, plan.psi()))
    plan.close()
    assert set(out[0][1]) == {1}
    assert out[0][:3] == out[1][:3]
    same = torch.equal(out[0][3], out[1][3])
    assert same
