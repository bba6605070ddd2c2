"""The shift of a catalogue with objects it rejects (a position that is not finite, or out of reach of the box)."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,m,painted", [(32, 1000, None), (32, 1000, "cic"), (128, 4097, "ngp"), (256, 600000, None),
                                         (256, 600000, "ngp"), (256, 600000, "cic")])
def test_every_row_of_both_outputs_is_written(gpu_lib, n, m, painted):
    # object by object and in brick order alike: a rejected object moves by 0 and is written where it was
    from paper_1504_02591_amd import native
    dev = torch.device("cuda", 0)
    g = torch.Generator(device=dev).manual_seed(n)
    box = 10.0 * n
    pos = torch.rand((m, 3), generator=g, device=dev) * box
    nan, inf = float("nan"), float("inf")
    bad = {3: (nan, 1.0, 2.0), 64: (inf, 5.0, nan), 500: (1.0, -inf, 2.0), 777: (1.0, 2.0, 3e10), m - 1: (-4e12, 0.0, 0.0)}
    for i, p in bad.items():
        pos[i] = torch.tensor(p, device=dev)
    good = torch.ones(m, dtype=torch.bool, device=dev)
    good[list(bad)] = False
    clean = pos.clone()
    clean[~good] = 5.0
    plan = native.Plan(n, box, (-300.0, 4.0 * n, 7.0 * n), 1.5, 0.8, 10.0, max_objects=m)
    paint = dict(ngp=painted == "ngp")
    if painted:
        plan.paint(native.GAL, clean, **paint)
        plan.paint(native.RAN, clean, **paint)
        plan.solve()
    else:
        plan.set_delta(torch.randn((n, n, n), generator=g, device=dev))
        plan.solve()
    plan.iterate(1, 0.0)
    for which in (native.GAL, native.RAN):
        disp, out = torch.full_like(pos, 123.0), torch.full_like(pos, 321.0)
        plan.shift(which, pos, want_pos=True, out_disp=disp, out_pos=out)
        assert float(disp[~good].abs().max()) == 0.0
        assert torch.isfinite(disp).all() and float(disp[good].abs().max()) < 123.0
        want = pos + disp
        assert torch.equal(torch.isnan(out), torch.isnan(pos))
        assert torch.equal(torch.nan_to_num(out, nan=0.5), torch.nan_to_num(want, nan=0.5))
    plan.close()
