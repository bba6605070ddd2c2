"""A plan on a stream of a device that is not the current one (needs two GPUs)."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def test_plan_on_a_stream_of_another_device(gpu_lib):
    if torch.cuda.device_count() < 2:
        pytest.skip("needs two GPUs")
    from paper_1504_02591_amd import native
    n, out = 64, []
    d = torch.randn((n, n, n), generator=torch.Generator().manual_seed(3))
    for dev, current in ((0, 0), (1, 0), (0, 1)):
        torch.cuda.set_device(current)
        with torch.cuda.device(dev):
            stream = torch.cuda.Stream()
            field = d.to(f"cuda:{dev}")
            torch.cuda.synchronize()
        torch.cuda.set_device(current)
        with torch.cuda.stream(stream):
            torch.cuda.set_device(current)
            plan = native.Plan(n, 640.0, (-300.0, 256.0, 448.0), 1.5, 0.8, 10.0, randoms=False, device=f"cuda:{dev}")
            assert torch.cuda.current_device() == current
            plan.set_delta(field)
            plan.solve()
            plan.iterate(8, 1e-3)
            out.append(plan.psi()[0].cpu())
            plan.close()
    torch.cuda.set_device(0)
    assert torch.equal(out[0], out[1]) and torch.equal(out[0], out[2])
