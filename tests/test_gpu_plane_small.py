"""The plane kernels at 8^3, where a transform has no barrier of its own."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch", [1, 300, 2049])
@pytest.mark.parametrize("start,relaxed", [(0, False), (2, True)])
def test_passes_of_a_batch_are_those_of_each_realisation(gpu_lib, batch, start, relaxed):
    # 300 realisations: two z tiles per block (8 tiles each, 1,024 blocks kept); 2,049: eight; alone: one
    from paper_1504_02591_amd import native
    n, dev = 8, torch.device("cuda", 0)
    g = torch.Generator(device=dev).manual_seed(batch)
    d = torch.randn((batch, n, n, n), generator=g, device=dev)
    kw = dict(box_len=80.0, observer=(-300.0, 32.0, 56.0), bias=1.5, growth=0.8, smooth_r=10.0, randoms=False,
              start_buffers=start != 0, relaxed=relaxed)
    many, one = native.Plan(n, batch=batch, **kw), native.Plan(n, **kw)
    many.set_delta(d)
    many.solve(start)
    _, iters, eps = many.iterate(12, 0.01)
    psi = many.psi()
    for b in sorted({0, 1 % batch, batch // 3, batch // 2, batch - 1}):
        one.set_delta(d[b].contiguous())
        one.solve(start)
        _, i1, e1 = one.iterate(12, 0.01)
        same = torch.equal(one.psi()[0], psi[b])
        assert same and i1[0] == iters[b] and e1[0] == eps[b]
    many.close()
    one.close()
