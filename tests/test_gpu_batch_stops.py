"""Realisations of a batch that stop at different passes end as each does alone, bit for bit, on every engine.

What is run ahead for the realisations that go on differs from what a single one gets, so the displacement of one
that stops comes from other launches: state X rebuilt from D_n, or kept; a full, combined or recombined state Y."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def fields(n, batch, seed):
    """Fields from rough to smooth, which converge at different rates."""
    dev = torch.device("cuda", 0)
    g = torch.Generator(device=dev).manual_seed(seed)
    k = torch.fft.fftfreq(n, device=dev) * n
    k2 = k.view(-1, 1, 1) ** 2 + k.view(1, -1, 1) ** 2 + k[:n // 2 + 1].view(1, 1, -1) ** 2
    out = []
    for i in range(batch):
        f = torch.fft.rfftn(torch.randn((n, n, n), generator=g, device=dev))
        f[0, 0, 0] = 0
        out.append(torch.fft.irfftn(f * torch.exp(-k2 * (0.02 * (i % 7))), s=(n, n, n)).float().contiguous())
    return out


@pytest.mark.parametrize("n,batch", [(16, 5), (64, 8), (128, 4), (128, 9), (256, 1), (256, 5), (512, 3)])
@pytest.mark.parametrize("start,relaxed,graphs", [(0, False, False), (0, True, True), (2, False, False), (2, True, False)])
def test_a_stopped_realisation_is_as_alone(gpu_lib, n, batch, start, relaxed, graphs):
    from paper_1504_02591_amd import native
    kw = dict(box_len=10.0 * n, observer=(4.0 * n, -2.0 * n, 3.0 * n), bias=1.1, growth=0.9, smooth_r=0.0, randoms=False,
              start_buffers=start != 0, relaxed=relaxed)
    fs = fields(n, batch, 300 + n)
    many, one = native.Plan(n, batch=batch, graphs=graphs, **kw), native.Plan(n, **kw)
    for tol in (0.1, 0.01):
        many.set_delta(torch.stack(fs))
        many.solve(start)
        _, iters, eps = many.iterate(14, tol)
        psi = many.psi()
        for i in range(0, batch, max(1, batch // 5)):
            one.set_delta(fs[i])
            one.solve(start)
            _, i1, e1 = one.iterate(14, tol)
            assert i1[0] == iters[i] and e1[0] == eps[i]
            same = torch.equal(one.psi()[0], psi[i])
            # and as a fixed number of passes gives it
            one.set_delta(fs[i])
            one.solve(start)
            one.iterate(i1[0], 0.0)
            assert same and torch.equal(one.psi()[0], psi[i])
        print(n, batch, start, relaxed, graphs, tol, list(iters), flush=True)
    many.close()
    one.close()


@pytest.mark.parametrize("n,levels", [(32, 0), (64, 0), (64, 1), (128, 1), (256, 2)])
@pytest.mark.parametrize("relaxed", [False, True])
def test_rejected_and_accepted_learned_starts_in_one_batch(gpu_lib, n, levels, relaxed):
    # a network of zeros with an output bias adds the same radial displacement everywhere: harmless against a large
    # field, worse than the plain start against a small one, which is rejected and starts over while others go on
    from paper_1504_02591_amd import native
    dev = torch.device("cuda", 0)
    batch = 4
    kw = dict(box_len=10.0 * n, observer=(4.0 * n, -2.0 * n, 3.0 * n), bias=1.8, growth=0.8, smooth_r=0.0, randoms=False,
              start_buffers=True, keep_delta=True, cnn=True, cnn_half=levels == 1, cnn_quarter=levels == 2, relaxed=relaxed)
    fs = [f * s for f, s in zip(fields(n, batch, n), (1.0, 1e-4, 1.0, 1e-5))]
    net = torch.zeros(native.CNN_PARAMS, device=dev)
    net[-1] = 0.002
    many, one = native.Plan(n, batch=batch, **kw), native.Plan(n, **kw)
    for tol in (0.05, 0.002):
        many.set_delta(torch.stack(fs))
        many.solve(native.START_LEARNED, net)
        rc, iters, eps = many.iterate(20, tol)
        psi, restarts = many.psi(), many.restarts()
        assert sorted(set(restarts)) == [0, 1], restarts
        for i in range(batch):
            one.set_delta(fs[i])
            one.solve(native.START_LEARNED, net)
            _, i1, e1 = one.iterate(20, tol)
            assert one.restarts()[0] == restarts[i]
            same = torch.equal(one.psi()[0], psi[i])
            print(n, levels, relaxed, tol, i, iters[i], i1[0], restarts[i], same, flush=True)
            assert i1[0] == iters[i] and e1[0] == eps[i] and same
    many.close()
    one.close()
