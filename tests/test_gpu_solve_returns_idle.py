"""recon_solve is a synchronisation point: with a plain start, and when it refuses, nothing of it is left queued."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,batch,randoms", [(64, 1, True), (256, 4, True), (256, 8, False), (512, 1, True)])
def test_solve_leaves_its_stream_idle(gpu_lib, n, batch, randoms):
    from paper_1504_02591_amd import native
    dev = torch.device("cuda", 0)
    g = torch.Generator(device=dev).manual_seed(n)
    m = 1000 * batch
    gal, ran = (torch.rand((m, 3), generator=g, device=dev) * (10.0 * n) for _ in range(2))
    off = None if batch == 1 else torch.arange(0, m + 1, m // batch, device=dev)
    plan = native.Plan(n, 10.0 * n, (-300.0, 4.0 * n, 7.0 * n), 1.5, 0.8, 10.0, batch=batch, randoms=randoms)
    bad = gal.clone()
    bad[7, 1] = float("nan")
    for pos, refused in ((gal, False), (bad, True), (gal, False)):
        plan.paint(native.GAL, pos, None, off)
        if randoms:
            plan.paint(native.RAN, ran, None, off)
        if refused:
            with pytest.raises(native.ReconError) as e:
                plan.solve()
            idle = plan.stream.query()
            assert e.value.code == native.RECON_EINVAL
        else:
            plan.solve()
            idle = plan.stream.query()
        assert idle
    plan.close()
