"""Which nearest-grid-point deposits go through the bricks, and that the grid is the same either way."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def catalogue(n, m, batch, seed):
    """Positions over the box and beyond it, a third in one cell, a fifth half-way between nodes or a hair off,
    some on the box's corners; weights; ragged offsets."""
    dev = torch.device("cuda", 0)
    rng = np.random.default_rng(seed)
    pos = (rng.random((m, 3)) * 11.0 * n - 0.5 * n).astype(np.float32)
    third, k = m // 3, m // 5
    pos[third:2 * third] = ((rng.random((third, 3)) * 0.9 + n // 2 + 0.05) * 10.0).astype(np.float32)
    pos[:k] = (np.floor(pos[:k] / 10.0) + 0.5) * 10.0
    pos[:k // 3, 0] = np.nextafter(pos[:k // 3, 0], np.float32(0))
    pos[k // 3:k // 2, 1] = -1e-9
    corners = np.array([[i & 1, (i >> 1) & 1, i >> 2] for i in range(8)], dtype=np.float32) * np.float32(10.0 * n)
    pos[m - 8:] = corners[:m]
    off = None
    if batch > 1:
        cuts = np.sort(rng.integers(0, m + 1, batch - 1))
        off = torch.tensor(np.concatenate([[0], cuts, [m]]), device=dev)
    w = torch.from_numpy((rng.random(m) * 3).astype(np.float32)).to(dev)
    return torch.from_numpy(pos).to(dev), w, off


@pytest.mark.parametrize("n,batch,m,randoms,through", [(64, 1, 20011, True, False), (128, 1, 20011, False, False),
                                                       (128, 1, 20011, True, True), (128, 1, 9, True, True),
                                                       (128, 9, 30011, True, True), (256, 1, 70001, False, False),
                                                       (256, 1, 70001, True, True)])
def test_route_of_a_deposit(gpu_lib, n, batch, m, randoms, through):
    from paper_1504_02591_amd import native
    kw = dict(box_len=10.0 * n, observer=(-300.0, 4.0 * n, 7.0 * n), bias=1.5, growth=0.8, smooth_r=10.0,
              randoms=randoms, batch=batch)
    direct, plan = native.Plan(n, **kw), native.Plan(n, max_objects=m, **kw)
    for which in (native.GAL, native.RAN) if randoms else (native.GAL,):
        pos, w, off = catalogue(n, m, batch, n + which)
        for weights, add in ((w, False), (None, True), (None, False)):
            direct.paint(which, pos, weights, off, ngp=True, accumulate=add)
            plan.profile_start()
            plan.paint(which, pos, weights, off, ngp=True, accumulate=add)
            used = plan.profile_stop()
            assert ("bin" in used) == through, used
            same = torch.equal(direct.grid(which), plan.grid(which))
            assert same
    direct.close()
    plan.close()


@pytest.mark.parametrize("n,batch,m", [(128, 1, 20011), (128, 9, 30011)])
def test_nearest_grid_point_over_and_under_cloud_in_cell(gpu_lib, n, batch, m):
    from paper_1504_02591_amd import native
    pos, w, off = catalogue(n, m, batch, n)
    kw = dict(box_len=10.0 * n, observer=(-300.0, 4.0 * n, 7.0 * n), bias=1.5, growth=0.8, smooth_r=10.0, batch=batch)
    direct, plan = native.Plan(n, **kw), native.Plan(n, max_objects=m, **kw)
    for steps in ([(w, False), (w, True)], [(None, True), (w, False)], [(w, True), (None, True)]):
        for p in (direct, plan):
            for i, (weights, ngp) in enumerate(steps):
                p.paint(native.GAL, pos, weights, off, accumulate=i > 0, ngp=ngp)
        same = torch.equal(direct.grid(native.GAL), plan.grid(native.GAL))
        assert same
    direct.close()
    plan.close()
