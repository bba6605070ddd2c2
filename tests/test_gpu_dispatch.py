"""Launch-shape rules: a result must not depend on which launch shape a size, count or batch selects."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def dev():
    return torch.device("cuda", 0)


def field(n, seed):
    rng = np.random.default_rng(seed)
    f = rng.standard_normal((n, n, n)).astype(np.float32)
    return torch.from_numpy(f - f.mean()).to(dev())


@pytest.mark.parametrize("n,batch", [(8, 40), (32, 64), (64, 20), (128, 9)])
def test_z_tiles_per_block_do_not_change_the_result(gpu_lib, n, batch):
    # alone, a realisation's z step runs one tile per block; in the batch, several: the same bits
    from paper_1504_02591_amd import native
    kw = dict(box_len=10.0 * n, observer=(-300.0, 4.0 * n, 7.0 * n), bias=1.5, growth=0.8, smooth_r=10.0, randoms=False)
    fields = [field(n, 100 + b) for b in range(batch)]
    many = native.Plan(n, batch=batch, **kw)
    many.set_delta(torch.stack(fields))
    many.solve()
    _, _, eps = many.iterate(3, 0.0)
    psi = many.psi()
    one = native.Plan(n, **kw)
    for b in (0, batch // 2, batch - 1):
        one.set_delta(fields[b])
        one.solve()
        _, _, e1 = one.iterate(3, 0.0)
        assert torch.equal(one.psi()[0], psi[b])
        np.testing.assert_allclose(e1[0], eps[b], rtol=1e-12)
    many.close()
    one.close()
