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


def clumped(n, box, m, seed):
    """Positions over the box and beyond it, a third of them inside one cell, some on nodes and faces."""
    rng = np.random.default_rng(seed)
    pos = (rng.random((m, 3)) * 1.1 * box - 0.05 * box).astype(np.float32)
    k = m // 3
    pos[:k] = ((rng.random((k, 3)) * 0.9 + n // 2 + 0.05) * (box / n)).astype(np.float32)
    faces = np.array([[i & 1, (i >> 1) & 1, i >> 2] for i in range(8)], dtype=np.float32) * np.float32(box)
    pos[k:k + 8] = faces[:m - k]
    return pos, (rng.random(m) * 3).astype(np.float32)


# histogram sizes (512, 4096, 32768 bins; more: windows), one or several binning blocks, bricks split into
# parts (32^3 to 256^3) or not, scans with and without run totals (more than 65,536 bricks)
@pytest.mark.parametrize("n,batch,m", [(8, 1, 5000), (16, 3, 1023), (32, 1, 1), (32, 1, 2049), (32, 1, 60001),
                                       (32, 65, 40000), (64, 1, 100003), (128, 1, 4097), (128, 9, 30011),
                                       (256, 1, 70001), (256, 17, 50021)])
def test_binned_deposit_and_shift_match_the_direct_ones(gpu_lib, n, batch, m):
    from paper_1504_02591_amd import native
    box = 10.0 * n
    pos, w = clumped(n, box, m, 7 * n + batch)
    rng = np.random.default_rng(3)
    cuts = np.sort(rng.integers(0, m + 1, batch - 1))
    off = None if batch == 1 else torch.tensor(np.concatenate([[0], cuts, [m]]), device=dev())
    pos, w = torch.from_numpy(pos).to(dev()), torch.from_numpy(w).to(dev())
    kw = dict(box_len=box, observer=(-300.0, 4.0 * n, 7.0 * n), bias=1.5, growth=0.8, smooth_r=10.0, randoms=False,
              batch=batch)
    direct, binned = native.Plan(n, **kw), native.Plan(n, max_objects=m, **kw)
    for weights in (w, None):
        for plan in (direct, binned):
            plan.paint(native.GAL, pos, weights, off)
        assert torch.equal(direct.grid(native.GAL), binned.grid(native.GAL))
    for plan in (direct, binned):                      # a second deposit on top
        plan.paint(native.GAL, pos, w, off, accumulate=True)
    assert torch.equal(direct.grid(native.GAL), binned.grid(native.GAL))
    if batch * n ** 3 <= 16 * 128 ** 3:                # the shift of the brick-ordered copy, any displacement
        psi = field(n, 1).repeat(batch, 1, 1, 1)
        for plan in (direct, binned):
            plan.set_delta(psi)
            plan.solve()
            plan.iterate(1, 0.0)
        assert torch.equal(direct.shift(native.GAL, pos, off), binned.shift(native.GAL, pos, off))
    direct.close()
    binned.close()


def test_invalid_objects_are_counted_per_grid(gpu_lib):
    # an invalid object makes solve refuse until its grid is painted anew; an accumulating deposit keeps
    # the refusal, and a valid one on top does not lift it
    from paper_1504_02591_amd import native
    n, m = 32, 5000
    pos, _ = clumped(n, 320.0, m, 5)
    good = torch.from_numpy(pos).to(dev())
    bad = good.clone()
    bad[m - 1, 1] = float("nan")
    plan = native.Plan(n, 320.0, (-300.0, 0.0, 0.0), 1.0, 0.5, 20.0, randoms=False, max_objects=m)

    def refused():
        try:
            plan.solve()
        except native.ReconError as e:
            assert e.code == native.RECON_EINVAL and "1 objects" in str(e)
            return True
        return False

    plan.paint(native.GAL, bad)
    assert refused() and refused()
    plan.paint(native.GAL, good, accumulate=True)
    assert refused()
    plan.paint(native.GAL, good)
    assert not refused()
    plan.paint(native.GAL, good)
    plan.paint(native.GAL, bad, accumulate=True)
    assert refused()
    plan.paint(native.GAL, good[:0])
    plan.paint(native.GAL, good, accumulate=True)
    assert not refused()
    plan.close()


# nearest-grid-point deposits: through the bricks from 128^3 on (weights, ragged batches, on top of and
# under cloud-in-cell deposits), per-object atomics below
@pytest.mark.parametrize("n,batch,m", [(64, 1, 3001), (128, 1, 1), (128, 1, 20011), (128, 9, 30011), (256, 1, 70001)])
def test_ngp_deposit_through_the_bricks_matches_the_direct_one(gpu_lib, n, batch, m):
    from paper_1504_02591_amd import native
    box = 10.0 * n
    pos, w = clumped(n, box, m, n + batch)
    k = m // 5                                           # exactly half-way, a hair below and above, and t = 1
    pos[:k] = (np.floor(pos[:k] / 10.0) + 0.5) * 10.0
    pos[:k // 3, 0] = np.nextafter(pos[:k // 3, 0], np.float32(0))
    pos[k // 3:k // 2, 1] = -1e-9
    rng = np.random.default_rng(3)
    cuts = np.sort(rng.integers(0, m + 1, batch - 1))
    off = None if batch == 1 else torch.tensor(np.concatenate([[0], cuts, [m]]), device=dev())
    pos, w = torch.from_numpy(pos).to(dev()), torch.from_numpy(w).to(dev())
    kw = dict(box_len=box, observer=(-300.0, 4.0 * n, 7.0 * n), bias=1.5, growth=0.8, smooth_r=10.0, randoms=False,
              batch=batch)
    direct, binned = native.Plan(n, **kw), native.Plan(n, max_objects=m, **kw)
    for steps in ([(w, True)], [(None, True)], [(w, True), (None, True)], [(w, False), (w, True)],
                  [(None, True), (w, False)]):
        for plan in (direct, binned):
            for i, (weights, ngp) in enumerate(steps):
                plan.paint(native.GAL, pos, weights, off, accumulate=i > 0, ngp=ngp)
        assert torch.equal(direct.grid(native.GAL), binned.grid(native.GAL))
    direct.close()
    binned.close()


@pytest.mark.parametrize("m", [(1 << 18) - 1, 1 << 18, 300007])
def test_shift_in_brick_order_without_a_deposited_copy(gpu_lib, m):
    # 256^3, enough objects per brick: the shift bins the catalogue itself; the same bits as object by object
    from paper_1504_02591_amd import native
    n = 256
    box = 10.0 * n
    pos, _ = clumped(n, box, m, 11)
    pos[m // 2] = np.inf
    pos = torch.from_numpy(pos).to(dev())
    kw = dict(box_len=box, observer=(-300.0, 4.0 * n, 7.0 * n), bias=1.5, growth=0.8, smooth_r=10.0, randoms=False)
    direct, binned = native.Plan(n, **kw), native.Plan(n, max_objects=m, **kw)
    d = field(n, 4)
    out = []
    for plan in (direct, binned):
        plan.set_delta(d)
        plan.solve()
        plan.iterate(1, 0.0)
        out.append((plan.shift(native.GAL, pos, want_pos=True), plan.shift(native.RAN, pos)))
    (a, b) = out
    ok = torch.isfinite(pos).all(1)
    assert torch.equal(a[0][0], b[0][0]) and torch.equal(a[1], b[1])
    assert torch.equal(a[0][1][ok], b[0][1][ok]) and not ok.all() and a[1][~ok].abs().max() == 0
    # a deposited copy stays what it was: the shift of another catalogue leaves it alone
    binned.paint(native.GAL, pos[:m // 2])
    first = pos[:m // 2]
    binned.paint(native.GAL, first)
    binned.solve()
    binned.iterate(1, 0.0)
    want = binned.shift(native.GAL, first.clone())
    binned.shift(native.GAL, pos)
    assert torch.equal(binned.shift(native.GAL, first), want)
    direct.close()
    binned.close()


def test_ngp_deposit_keeps_the_cic_copy_a_shift_may_name(gpu_lib):
    import ctypes
    from paper_1504_02591_amd import native
    n, m = 128, 5000
    pos, _ = clumped(n, 1280.0, m, 6)
    ran = torch.from_numpy(pos).to(dev())
    gal = torch.from_numpy(clumped(n, 1280.0, m, 8)[0]).to(dev())
    plan = native.Plan(n, 1280.0, (-300.0, 0.0, 0.0), 1.0, 0.5, 20.0, max_objects=m)
    plan.paint(native.RAN, ran)
    plan.paint(native.GAL, gal, ngp=True)
    plan.solve()
    plan.iterate(1, 0.0)
    want, got = plan.shift(native.RAN, ran.clone()), torch.empty_like(ran)

    def named(which, t):
        return plan.lib.recon_shift(plan.handle, which | native.SHIFT_AS_PAINTED, ctypes.c_void_p(t.data_ptr()), m,
                                    None, ctypes.c_void_p(got.data_ptr()), None)

    assert named(native.RAN, ran) == native.RECON_OK
    torch.cuda.synchronize()
    assert torch.equal(got, want)
    assert named(native.GAL, gal) == native.RECON_EINVAL   # an NGP deposit's copy is not one to name
    plan.close()


@pytest.mark.parametrize("start,relaxed,graphs", [("PLAIN", False, False), ("PLAIN", True, True), ("FFTA2", False, True)])
def test_work_queued_ahead_of_the_convergence_test_changes_nothing(gpu_lib, start, relaxed, graphs):
    # tolerances on either side of every pass's eps (so that the expected next eps is right, wrong and
    # undecided in turn), in one call, in calls of one pass, and resumed after the end: the same passes and the
    # same bits as a fixed number of passes; two realisations that stop at different passes, too
    from paper_1504_02591_amd import native
    n, total = 32, 7
    s = getattr(native, "START_" + start)
    kw = dict(box_len=320.0, observer=(-300.0, 128.0, 224.0), bias=1.0, growth=0.7, smooth_r=10.0, randoms=False,
              start_buffers=start != "PLAIN", relaxed=relaxed, graphs=graphs)
    d = field(n, 21)
    plan = native.Plan(n, **kw)

    def run(pieces, tol):
        plan.set_delta(d)
        plan.solve(s)
        for k in pieces:
            rc, passes, eps = plan.iterate(k, tol)
        return rc, passes[0], eps[0], plan.psi()

    fixed = {k: run([k], 0.0) for k in range(1, total + 1)}
    eps = fixed[total][2]
    for k in range(1, total):
        for f in (1.0 - 1e-6, 1.0 + 1e-6, 0.8, 1.25):
            tol = eps[k - 1] * f
            stop = next((i + 1 for i, e in enumerate(eps) if e <= tol), None)
            if stop is None:
                continue
            rc, passes, _, psi = run([total], tol)
            assert passes == stop and rc == native.RECON_OK and torch.equal(psi, fixed[stop][3])
            rc, passes, _, psi = run([1] * stop, tol)
            assert passes == stop and rc == native.RECON_OK and torch.equal(psi, fixed[stop][3])
    for pieces in ([2, 1, 3], [1, 0, 4], [0, 5]):        # resumed, also straight after a displacement was formed
        assert torch.equal(run(pieces, 0.0)[3], fixed[sum(pieces)][3])
    plan.close()
    smooth = torch.fft.irfftn(torch.fft.rfftn(d.cpu()) * (torch.arange(n // 2 + 1) < 2), s=(n, n, n)).to(dev())
    both = native.Plan(n, batch=2, **kw)
    tol = eps[3]
    both.set_delta(torch.stack([d, smooth.contiguous()]))
    both.solve(s)
    _, passes, _ = both.iterate(total, tol)
    psi = both.psi()
    one = native.Plan(n, **kw)
    for b, f in enumerate((d, smooth.contiguous())):
        one.set_delta(f)
        one.solve(s)
        _, p, _ = one.iterate(total, tol)
        assert p[0] == passes[b] and torch.equal(one.psi()[0], psi[b])
    one.close()
    both.close()


def field_reference(delta, box, obs, b, f, passes, start, relax):
    """The pass iteration in 64 bits with torch's transforms; yields the three components of Psi."""
    n = delta.shape[-1]
    m = torch.arange(n, device=delta.device, dtype=torch.float64)
    k = torch.where(m < n // 2, m, m - n) * (2 * np.pi / box)
    dk = torch.where(m == n // 2, torch.zeros_like(k), k)
    kv = (k.view(n, 1, 1), k.view(1, n, 1), k[:n // 2 + 1].abs().view(1, 1, -1))
    d = (dk[:n // 2 + 1].view(1, 1, -1), dk.view(1, n, 1), dk.view(n, 1, 1))          # x, y, z
    k2 = kv[0] ** 2 + kv[1] ** 2 + kv[2] ** 2
    k2[0, 0, 0] = 1.0
    x = m * (box / n)
    r = [(x - obs[0]).view(1, 1, n), (x - obs[1]).view(1, n, 1), (x - obs[2]).view(n, 1, 1)]
    dist = torch.sqrt(r[0] ** 2 + r[1] ** 2 + r[2] ** 2)
    spec = lambda a: torch.fft.rfftn(a)                                               # noqa: E731
    comp = lambda s, j: torch.fft.irfftn(1j * d[j] * s / (b * k2), s=(n, n, n))       # noqa: E731
    ds = spec(delta.double())
    ds[0, 0, 0] = 0
    cur = ds

    def along(s):
        u = torch.zeros_like(dist)
        for j in range(3):
            u += comp(s, j) * (r[j] / dist)
        return u

    for p in range(passes):
        u = along(cur)
        if p == 0 and start == 2:                                                    # FFTA-2: u (1 - c)
            u *= 1.0 - 3.0 * (f / b) / (7.0 + 3.0 * (f / b))
        new = ds.clone()
        for j in range(3):
            new += f * 1j * d[j] * spec(u * (r[j] / dist))
        new[0, 0, 0] = 0
        w = 1.0 if relax is None or (p == 0 and start != 0) else relax
        cur = w * new + (1.0 - w) * cur
        del new, u
    for j in range(3):
        yield comp(cur, j)


@pytest.mark.parametrize("n,start,relaxed", [(128, 0, False), (256, 0, False), (256, 0, True), (256, 2, False),
                                             (512, 0, False), (512, 2, True), (1024, 0, False)])
def test_passes_of_a_white_field_against_64_bits(gpu_lib, n, start, relaxed):
    # every mode up to the Nyquist planes through both transform engines (below and from 256) and each form
    # of the z step.  Tolerance: a transform of 2^30 points in FP32 is off by about 6e-8 sqrt(30) = 3e-7,
    # two passes are five of them in a row, and the line of sight adds its own rounding: 1e-5 with a margin
    # as the plane-wave test at 1024 takes.
    from paper_1504_02591_amd import native
    box, obs, b, f = 10.0 * n, (-3.0 * n, 4.0 * n + 3.0, 7.0 * n), 1.8, 0.8
    g = torch.Generator(device=dev()).manual_seed(n + start)
    delta = torch.randn((n, n, n), generator=g, device=dev(), dtype=torch.float32)
    delta -= delta.mean()
    plan = native.Plan(n, box, obs, b, f, 0.0, randoms=False, relaxed=relaxed,
                       start_buffers=start != 0)
    plan.set_delta(delta)
    plan.solve(start)
    plan.iterate(2, 0.0)
    psi = plan.psi()[0]
    plan.close()
    num = den = 0.0
    w = 2.0 / (2.0 + f / b) if relaxed else None
    for j, want in enumerate(field_reference(delta, box, obs, b, f, 2, start, w)):
        num += float(((psi[j].double() - want) ** 2).sum())
        den += float((want ** 2).sum())
    print(f"{n}^3 start {start} relaxed {relaxed}: rel L2 {(num / den) ** 0.5:.2e}", flush=True)
    assert num <= 1e-10 * den


@pytest.mark.parametrize("n", [16, 128, 256])
def test_grid_cells_round_once_to_floats(gpu_lib, n):
    # one object on a node of the 16^3-brick lattice per brick, weights over the whole range a cell can hold
    # (below and above 2^53 units of 2^-32): without smoothing delta_s + 1 is the grid over its mean, to the
    # transforms' rounding, 1e-6 of the largest cell
    from paper_1504_02591_amd import native
    m = (n // 16) ** 3
    rng = np.random.default_rng(n)
    cell = np.stack(np.meshgrid(*[np.arange(n // 16)] * 3, indexing="ij"), -1).reshape(m, 3) * 16 + 5
    w = (2.0 ** rng.uniform(-2, 5.9, m)).astype(np.float32)
    heavy = np.repeat(np.arange(min(m, 8)), 40000)               # 40,000 objects of weight 63 on one node each
    for more in (heavy[:0], heavy):
        pos = np.concatenate([cell, cell[more]]).astype(np.float32)
        wt = np.concatenate([w, np.full(len(more), 63, np.float32)])
        plan = native.Plan(n, float(n), (-3.0 * n, 0.0, 0.0), 1.0, 0.5, 0.0, randoms=False, keep_delta=True)
        plan.paint(native.GAL, torch.from_numpy(pos).to(dev()), torch.from_numpy(wt).to(dev()))
        plan.solve()
        d = plan.delta()[0].double()
        g = plan.grid(native.GAL)[0].double()
        plan.close()
        want = g / g.mean() - 1.0
        assert float((d - want).abs().max()) <= 1e-6 * float(want.abs().max())


@pytest.mark.parametrize("n", [8, 16, 32, 64])
@pytest.mark.parametrize("start,relaxed", [(0, False), (0, True), (2, False)])
def test_plane_passes_against_64_bits(gpu_lib, n, start, relaxed):
    # the sizes whose y and x steps run per plane; tolerance as in the white-field test above
    from paper_1504_02591_amd import native
    box, obs, b, f = 10.0 * n, (-3.0 * n, 4.0 * n + 3.0, 7.0 * n), 1.8, 0.8
    g = torch.Generator(device=dev()).manual_seed(n + start)
    delta = torch.randn((n, n, n), generator=g, device=dev(), dtype=torch.float32)
    delta -= delta.mean()
    w = 2.0 / (2.0 + f / b) if relaxed else None
    want = torch.stack(list(field_reference(delta, box, obs, b, f, 3, start, w)))
    for graphs in (False, True):
        plan = native.Plan(n, box, obs, b, f, 0.0, randoms=False, relaxed=relaxed, start_buffers=start != 0,
                           graphs=graphs)
        plan.set_delta(delta)
        plan.solve(start)
        plan.iterate(2, 0.0)
        plan.iterate(1, 0.0)
        psi = plan.psi()[0].double()
        plan.close()
        assert float((psi - want).norm()) <= 1e-5 * float(want.norm())


@pytest.mark.parametrize("n,batch", [(16, 5), (32, 70), (64, 4), (64, 33)])
def test_plane_passes_of_a_batch_that_stops_at_different_passes(gpu_lib, n, batch):
    # work queued ahead for realisations that go on, and taken back for one that stops: each ends as it does
    # alone, bit for bit, also where the sums of a batch go through the reduction kernel
    from paper_1504_02591_amd import native
    kw = dict(box_len=10.0 * n, observer=(4.0 * n, -2.0 * n, 3.0 * n), bias=1.1, growth=0.9, smooth_r=0.0, randoms=False)
    # smooth and rough fields converge at different rates
    fields = []
    for i in range(batch):
        f = torch.fft.rfftn(field(n, 300 + i))
        k = torch.fft.fftfreq(n, device=dev()) * n
        k2 = k.view(-1, 1, 1) ** 2 + k.view(1, -1, 1) ** 2 + k[:n // 2 + 1].view(1, 1, -1) ** 2
        fields.append(torch.fft.irfftn(f * torch.exp(-k2 * (0.02 * (i % 7))), s=(n, n, n)).float().contiguous())
    many = native.Plan(n, batch=batch, **kw)
    many.set_delta(torch.stack(fields))
    many.solve()
    _, iters, eps = many.iterate(12, 0.02)
    psi = many.psi()
    many.close()
    one = native.Plan(n, **kw)
    seen = set()
    for i in range(0, batch, max(1, batch // 8)):
        one.set_delta(fields[i])
        one.solve()
        _, it1, e1 = one.iterate(12, 0.02)
        seen.add(int(it1[0]))
        assert it1[0] == iters[i]
        assert torch.equal(one.psi()[0], psi[i])
        assert e1[0] == eps[i]
    one.close()
    print(n, batch, sorted(seen), flush=True)


@pytest.mark.parametrize("n,batch", [(128, 2), (256, 2)])
def test_non_temporal_choice_does_not_change_the_result(gpu_lib, n, batch):
    # one of 128^3 and two of 256^3 run hinted, two of 128^3 and one of 256^3 plain: the same bits
    test_z_tiles_per_block_do_not_change_the_result(gpu_lib, n, batch)
