"""Which catalogues the shift puts into brick order first, and that the result is the same either way.

Binning pays for a catalogue in no spatial order and costs one that is in order, so the route follows what the
nearest-grid-point deposit of that catalogue found."""
import pytest
import torch

pytestmark = pytest.mark.gpu
LEAST = 2 ** 17 + 42 * 16 ** 3                             # objects over all of 256^3 from which they are binned


def catalogue(n, m, order, seed):
    dev = torch.device("cuda", 0)
    g = torch.Generator(device=dev).manual_seed(seed)
    box = 10.0 * n
    pos = torch.rand((m, 3), generator=g, device=dev) * box
    if order in ("x", "y", "z"):                           # sorted along one axis: no neighbours in space
        a = "xyz".index(order)
        pos = pos[torch.argsort(pos[:, a])]
    elif order == "lattice":
        k = round(m ** (1 / 3))
        i = torch.arange(k, device=dev, dtype=torch.float32) * (box / k)
        z, y, x = torch.meshgrid(i, i, i, indexing="ij")
        q = torch.stack([x.reshape(-1), y.reshape(-1), z.reshape(-1)], 1)
        pos[:q.shape[0]] = (q + pos[:q.shape[0]] / k)[:m]
    elif order == "clump":
        pos = pos * 0.02 + 0.31 * box
    elif order == "eighth":                                # in no order over 8^3 of the 16^3 bricks
        pos = pos * 0.4999
    return pos.contiguous()


@pytest.mark.parametrize("order,m,bins", [("random", LEAST - 1, False), ("random", LEAST, True),
                                          ("random", 500000, True), ("x", 500000, True), ("y", 500000, True),
                                          ("z", 500000, True), ("lattice", 512000, False), ("clump", 400000, False),
                                          ("eighth", 2 ** 17 + 14 * 4096 + 28 * 512 - 1, False),
                                          ("eighth", 2 ** 17 + 14 * 4096 + 28 * 512, True)])
def test_route_follows_the_order_of_the_catalogue(gpu_lib, order, m, bins):
    from paper_1504_02591_amd import native
    n = 256
    kw = dict(box_len=10.0 * n, observer=(-300.0, 4.0 * n, 7.0 * n), bias=1.5, growth=0.8, smooth_r=10.0)
    gal, ran = catalogue(n, m, order, 5), catalogue(n, LEAST + m + 17, "random", 6)
    direct, plan = native.Plan(n, **kw), native.Plan(n, max_objects=LEAST + m + 17, **kw)
    for p in (direct, plan):
        p.paint(native.GAL, gal, ngp=True)
        p.paint(native.RAN, ran, ngp=True)
        p.solve()
        p.iterate(1, 0.0)

    def shift(which, pos):
        plan.profile_start()
        got = plan.shift(which, pos, want_pos=True)
        used = plan.profile_stop()
        want = direct.shift(which, pos, want_pos=True)
        same = torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
        assert same
        return "bin" in used

    assert shift(native.GAL, gal) == bins
    assert shift(native.RAN, ran)
    assert not shift(native.GAL, ran)                      # not a catalogue of the length that was deposited
    if bins:
        assert shift(native.GAL, gal.clone())
    # a cloud-in-cell deposit's copy is in the way, and a new deposit's order is not known before the solve
    plan.paint(native.RAN, ran)
    plan.solve()
    plan.iterate(1, 0.0)
    direct.paint(native.RAN, ran)
    direct.solve()
    direct.iterate(1, 0.0)
    assert not shift(native.GAL, gal)
    direct.close()
    plan.close()


def test_route_without_a_deposit_and_without_randoms(gpu_lib):
    from paper_1504_02591_amd import native
    n, m = 256, 500000
    pos = catalogue(n, m, "random", 7)
    dev = torch.device("cuda", 0)
    delta = torch.randn((n, n, n), generator=torch.Generator(device=dev).manual_seed(8), device=dev)
    for randoms in (True, False):
        kw = dict(box_len=10.0 * n, observer=(-300.0, 4.0 * n, 7.0 * n), bias=1.5, growth=0.8, smooth_r=10.0, randoms=randoms)
        plan = native.Plan(n, max_objects=m, **kw)
        if randoms:
            plan.set_delta(delta)
        else:
            plan.paint(native.GAL, pos, ngp=True)
        plan.solve()
        plan.iterate(1, 0.0)
        plan.profile_start()
        plan.shift(native.GAL, pos)
        assert "bin" not in plan.profile_stop()
        plan.close()


def test_batch_in_no_order_is_binned(gpu_lib):
    from paper_1504_02591_amd import native
    n, batch, m = 256, 2, 2 * LEAST + 1001                 # (twice the bricks, 14 and 28 for each)
    pos = catalogue(n, m, "random", 9)
    off = torch.tensor([0, 300007, m], device=pos.device)
    kw = dict(box_len=10.0 * n, observer=(-300.0, 4.0 * n, 7.0 * n), bias=1.5, growth=0.8, smooth_r=10.0, batch=batch)
    out = []
    for mo in (0, m):
        plan = native.Plan(n, max_objects=mo, **kw)
        plan.paint(native.GAL, pos, None, off, ngp=True)
        plan.paint(native.RAN, pos, None, off, ngp=True)
        plan.solve()
        plan.iterate(1, 0.0)
        plan.profile_start()
        out.append(plan.shift(native.RAN, pos, off))
        assert ("bin" in plan.profile_stop()) == (mo > 0)
        plan.close()
    same = torch.equal(out[0], out[1])
    assert same
