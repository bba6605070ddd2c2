"""The debug build (device bounds checks) on the transform engines: plane kernels, radix-8 and column engine.

On valid inputs it must count no out-of-bounds index, and give the release build's results: grids bit for bit,
fields to 1e-6 in rel L2 (the checks change the code around the transforms, so FP32 contractions may differ: some
6e-8 a rounding, a few dozen roundings deep).  The fields of the lognormal option are not compared: in voids, at
its floor of 1e-3, the logarithm magnifies those roundings a thousandfold."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def run(native, lib, n, randoms, start, kw):
    dev = torch.device("cuda", 0)
    g = torch.Generator(device=dev).manual_seed(n + start)
    m, box = 200000, 10.0 * n
    gal = torch.rand((m, 3), generator=g, device=dev) * box
    gal[:m // 2] = 0.3 * box + 0.4 * gal[:m // 2]
    ran = (torch.rand((m, 3), generator=g, device=dev) * 0.6 + 0.2) * box
    net = None
    if start == native.START_LEARNED:
        net = 0.02 * torch.randn(native.CNN_PARAMS, generator=g, device=dev)
    plan = native.Plan(n, box, (-0.4 * box, 0.3 * box, 0.6 * box), 1.5, 0.7, 30.0, randoms=randoms, keep_delta=True,
                       start_buffers=start != 0, max_objects=m, lib=lib, **kw)
    ngp = kw.get("graphs", False)
    plan.paint(native.GAL, gal, ngp=ngp)
    if randoms:
        plan.paint(native.RAN, ran, ngp=ngp)
    plan.solve(start, net)
    _, _, eps = plan.iterate(3, 0.0)
    out = [plan.grid(native.GAL), plan.delta(), plan.psi(), plan.radial(), plan.shift(native.GAL, gal),
           torch.tensor(eps[0], dtype=torch.float64)]
    plan.close()
    return out


@pytest.mark.parametrize("n,randoms,start,kw", [
    (8, False, 0, dict(graphs=True)), (16, True, 2, {}), (64, True, 0, dict(graphs=True)),
    (128, True, 2, {}), (256, True, 3, dict(cnn=True, cnn_quarter=True)), (256, False, 0, dict(lognormal=True)),
    (256, True, 2, dict(graphs=True, relaxed=True)), (512, True, 2, {}), (512, False, 0, dict(lognormal=True))])
def test_no_index_outside_on_any_engine(gpu_lib, n, randoms, start, kw):
    from paper_1504_02591_amd import native
    dbg = native.load(native.debug_lib_path())
    assert dbg.recon_debug_violations(1) >= 0
    got = run(native, dbg, n, randoms, start, kw)
    assert dbg.recon_debug_violations(0) == 0
    ref = run(native, None, n, randoms, start, kw)
    assert torch.equal(got[0], ref[0])
    for a, b in zip(got[1:], ref[1:]):
        assert torch.isfinite(a).all() and torch.isfinite(b).all()
        if kw.get("lognormal"):
            continue
        off, size = float((a.double() - b.double()).norm()), float(b.double().norm())
        assert off <= 1e-6 * size
