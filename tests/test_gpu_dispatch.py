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


@pytest.mark.parametrize("m,batch", [(16, 1), (16, 3), (64, 1), (128, 1)])
def test_training_gradient_against_64_bits(gpu_lib, m, batch):
    # one tile per backward block (16^3), several blocks and several tiles per block (128^3), and tiles that
    # cross from one realisation to the next; the reference is the network in FP64 with bf16 rounding at
    # the kernels' points.  Tolerance: a bf16 rounding that falls the other way is one part in 2^8 of one
    # term, so sums of 4096 terms or more agree to better than 5e-3, as the existing gradient test takes.
    from paper_1504_02591_amd import native
    from oracle import cnn_oracle as C
    rng = np.random.default_rng(m + batch)
    box, obs = 200.0, (37.0, -60.0, 110.0)
    shape = (batch, m, m, m)
    d, u = (rng.standard_normal(shape).astype(np.float32) for _ in range(2))
    u *= 20
    t = (-0.15 * u + 0.2 * rng.standard_normal(shape)).astype(np.float32)
    th = C.init_params(5).astype(np.float32)
    plan = native.Plan(m, box, obs, 2.0, 0.7, 0.0, batch=batch, randoms=False, cnn=True)
    grad = torch.zeros(native.CNN_PARAMS, dtype=torch.float32, device=dev())
    up = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).to(dev())  # noqa: E731
    loss = plan.cnn_train_step(up(th), None, None, 0, 0.0, up(d), up(u), up(t), grad_out=grad)
    plan.close()
    p = {k: torch.from_numpy(v).to(dev()) for k, v in C.unpack(th).items()}

    def bf(x):
        return x + (x.to(torch.float32).to(torch.bfloat16).double() - x).detach()

    w = {k: (bf(v) if k[0] == "W" else v).detach().requires_grad_(True) for k, v in p.items()}

    def conv(x, W):
        y = 0
        for k, (dx, dy, dz) in enumerate(C.TAPS):
            y = y + torch.matmul(torch.roll(x, (-dz, -dy, -dx), (0, 1, 2)), W[:, k].t().contiguous())
        return y

    i = torch.arange(m, device=dev(), dtype=torch.float64) * (box / m)
    r = torch.stack([(i - obs[0]).view(1, 1, m).expand(m, m, m), (i - obs[1]).view(1, m, 1).expand(m, m, m),
                     (i - obs[2]).view(m, 1, 1).expand(m, m, m)], -1)
    r = r / r.norm(dim=-1, keepdim=True)
    total = 0.0
    for b in range(batch):
        x = torch.cat([up(d[b]).double()[..., None], C.S_U * up(u[b]).double()[..., None], r,
                       torch.zeros((m, m, m, 3), dtype=torch.float64, device=dev())], -1)
        a1 = bf(torch.relu(conv(bf(x), w["W1"]) + w["b1"]))
        a2 = bf(torch.relu(conv(a1, w["W2"]) + w["b2"]))
        y = (conv(a2, w["W3"]) + w["b3"])[..., 0]
        part = ((y - C.S_U * up(t[b]).double()) ** 2).sum() / (batch * m ** 3)
        part.backward()
        total += float(part.detach())
    assert abs(loss - total) <= 1e-4 * total
    g, off = grad.double(), 0
    for name, shp in C.SHAPES:
        size = int(np.prod(shp))
        ref = w[name].grad.reshape(-1)
        e = float((g[off:off + size] - ref).norm() / ref.norm())
        print(f"m={m} batch={batch} grad {name}: rel L2 {e:.2e}", flush=True)
        assert e < 5e-3, name
        off += size
