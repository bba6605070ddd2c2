"""Workloads of the reconstruction library, for timing and for comparing outputs.

Every case goes through the public binding (paper_1504_02591_amd.native.Plan) the way a user's program
does: the plan, the catalogues and the network parameters are in hand on the GPU, and one pass is one
reconstruction (deposit, solve, correction passes, shift), one streamed deposit, or one training step of
the learned start.  Inputs are synthetic and made on the GPU from the seed: a Gaussian linear field
with the generators' power spectrum, objects clustered by it, and redshift-space positions.

    listed()             the named cases
    draw(rng)            one more case of the same ranges
    prepare(case, seed)  plan and inputs
    run(state)           one pass, and its outputs
    work(case)           bytes and operations one pass cannot do without
    exact(case, seed)    the same outputs in 64 bits, with plain torch
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1504_02591_amd import learned, native

START = {"plain": native.START_PLAIN, "ffta1": native.START_FFTA1, "ffta2": native.START_FFTA2,
         "learned": native.START_LEARNED}

# Geometry of a periodic lattice box (the N-body stand-in) and of a survey cone (the mock catalogues'
# stand-in) as the generators have them: a cell of 3500/512 Mpc/h and a shell of 1100 to 1800 Mpc/h
# in a box of 3500, both shrunk with the grid.
BOX = dict(kind="box", batch=1, cell=15.625, bias=1.0, growth=0.7, smooth=10.0, far=1.0, npart=32, ran=0,
           weights=False, lognormal=False, relaxed=False, start="plain", tol=1e-3, passes=30, graphs=False,
           ngp=False, spread=1.0, want_pos=False)
SURVEY = dict(kind="survey", batch=1, cell=3500.0 / 512, bias=2.0, growth=0.74, smooth=15.0, gal=11000, ran=50,
              weights=False, lognormal=False, relaxed=False, start="plain", tol=1e-3, passes=30, graphs=False,
              ngp=False, spread=1.0, want_pos=False)


def listed():
    return [
        # the smallest call: the 32^3 lattice box of the smoke check, four fixed passes; launches and
        # read-backs, not bytes, are what it costs
        dict(BOX, name="box32", n=32, npart=32, ran=2, smooth=20.0, tol=0.0, passes=4),
        # the oracle-sized periodic box (64^3 over 1000 Mpc/h, 5x randoms) with weighted objects and the
        # start of eq. (approx2): a test-sized box in a parameter study
        dict(BOX, name="box64_ffta2", n=64, npart=64, ran=5, weights=True, start="ffta2"),
        # a small survey with completeness/FKP-like weights, positions wanted as well as displacements:
        # the interactive size
        dict(SURVEY, name="survey128_weighted", n=128, gal=10900, weights=True, want_pos=True),
        # a set of small mocks through one plan, as for a covariance matrix: 16 realisations of 128^3 with
        # ragged counts, the steady pass replayed as a graph
        dict(SURVEY, name="mocks128x16", n=128, batch=16, gal=11000, spread=2.0, graphs=True),
        # the paper's own binning (nearest grid point) on a 256^3 survey
        dict(SURVEY, name="survey256_ngp", n=256, gal=86800, ngp=True),
        # a periodic 256^3 box without randoms (mean density), the lognormal overdensity, beta = 0.76: no
        # empty bricks anywhere and many passes
        dict(BOX, name="box256_lognormal", n=256, cell=2000.0 / 256, npart=256, growth=0.76, far=2.0, lognormal=True),
        # the benchmark's survey: 512^3 over 3500 Mpc/h, 694,771 galaxies, 50x randoms, plain start
        dict(SURVEY, name="survey512", n=512, gal=694771),
        # the same from the learned start (committed network on the 128^3 grid), the headline's other leg
        dict(SURVEY, name="survey512_learned", n=512, gal=694771, start="learned"),
        # the batched workload: realisations of 256^3 with log-uniform counts and the relaxed pass
        dict(SURVEY, name="batch256x8_relaxed", n=256, cell=1500.0 / 256, batch=8, gal=316000, spread=10.0,
             relaxed=True),
        # the largest grid: the precision study's box (1024^3 over 2000 Mpc/h, observer 5000 Mpc/h from the
        # centre), 384^3 particles, relaxed passes
        dict(BOX, name="box1024_relaxed", n=1024, cell=2000.0 / 1024, npart=384, growth=0.76, far=2.0, relaxed=True),
        # a catalogue too large for one call, deposited in pieces that add to the grid, and the grid itself
        dict(kind="stream", name="stream256", n=256, cell=3500.0 / 512, objects=8000003, pieces=4, weights=True,
             ngp=False, batch=1),
        # one training step of the learned start on its committed configuration (128^3 network grid of a
        # 512^3 plan): forward, backward, Adam
        dict(kind="train", name="train128", n=512, levels=2, batch=1),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("box", "box", "survey", "survey", "survey", "mocks", "mocks", "stream", "train"))
    if kind == "box":
        n = rng.choice((32, 64, 64, 128, 128, 256, 256, 512, 1024))
        npart = min(384, max(16, int(n * rng.uniform(0.4, 1.1))))
        ran = rng.choice((0, 2, 5)) if n <= 256 and 2 * npart >= n and npart <= 200 else 0
        tol = rng.choice((0.0, 1e-3))
        relaxed = n == 1024 or rng.random() < 0.4
        passes = rng.randint(1, 5) if tol == 0.0 else 30
        return dict(BOX, n=n, cell=round(rng.uniform(3.0, 8.0), 3), npart=npart, ran=ran,
                    growth=round(rng.uniform(0.4, 0.8), 3),
                    smooth=round(rng.uniform(10.0, 20.0), 2), far=rng.choice((1.0, 2.0)), weights=rng.random() < 0.3,
                    lognormal=ran == 0 and rng.random() < 0.3, relaxed=relaxed, tol=tol, passes=passes,
                    start=rng.choice(("plain", "ffta1", "ffta2")) if n <= 512 else "plain",
                    graphs=rng.random() < 0.2, ngp=n <= 256 and rng.random() < 0.2, want_pos=rng.random() < 0.3)
    if kind == "survey":
        n = rng.choice((64, 128, 256, 256, 512))
        full = 694771 * (n / 512.0) ** 3
        return dict(SURVEY, n=n, gal=_logint(rng, max(1500, 0.2 * full), 1.05 * full + 2000),
                    ran=rng.choice((10, 20, 50)), growth=round(rng.uniform(0.5, 0.9), 3), smooth=round(rng.uniform(10.0, 20.0), 2),
                    weights=rng.random() < 0.4, relaxed=rng.random() < 0.4, ngp=rng.random() < 0.25,
                    start=rng.choice(("plain", "plain", "ffta1", "ffta2", "learned")),
                    tol=rng.choice((1e-3, 1e-3, 0.0)), passes=rng.randint(5, 8), want_pos=rng.random() < 0.3)
    if kind == "mocks":
        n = rng.choice((32, 64, 128, 256))
        batch = rng.randint(2, {32: 24, 64: 20, 128: 14, 256: 6}[n])
        full = 694771 * (n / 512.0) ** 3
        return dict(SURVEY, n=n, batch=batch, gal=_logint(rng, max(900, 0.4 * full), 3.0 * full + 900),
                    spread=round(rng.uniform(1.0, 6.0), 2), ran=rng.choice((10, 20, 50)), relaxed=rng.random() < 0.5,
                    weights=rng.random() < 0.3, graphs=rng.random() < 0.5, tol=rng.choice((1e-3, 0.0)),
                    passes=rng.randint(6, 9), start=rng.choice(("plain", "plain", "ffta2")))
    if kind == "stream":
        return dict(kind="stream", n=rng.choice((64, 128, 256, 512)), cell=3500.0 / 512, batch=1,
                    objects=_logint(rng, 3e4, 2e7), pieces=rng.randint(1, 7), weights=rng.random() < 0.5,
                    ngp=rng.random() < 0.2)
    levels = rng.choice((0, 1, 2))
    m = rng.choice((16, 32, 64, 64, 128))
    return dict(kind="train", n=m << levels, levels=levels, batch=rng.randint(1, 3))


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------
def _dev():
    return torch.device("cuda", torch.cuda.current_device())


def _linear(m, box, gen):
    """Gaussian linear field with P(k) = A k / (1 + (k/0.02)^3), sigma_8 = 0.8, on m^3 and its displacement."""
    dev = gen.device
    fk = torch.fft.rfftn(torch.randn((m, m, m), generator=gen, device=dev))
    kf = 2.0 * math.pi / box
    k1 = torch.fft.fftfreq(m, d=1.0 / m, device=dev) * kf
    kh = torch.arange(m // 2 + 1, device=dev, dtype=torch.float32) * kf
    kz, ky, kx = k1.view(m, 1, 1), k1.view(1, m, 1), kh.view(1, 1, -1)
    k2 = kx * kx + ky * ky + kz * kz
    kk = k2.sqrt()
    fk *= torch.sqrt(7.455e6 * kk / (1.0 + (kk / 0.02) ** 3) * (m ** 3 / box ** 3))
    delta = torch.fft.irfftn(fk, s=(m, m, m))
    k2[0, 0, 0] = 1.0
    fk /= k2
    ny = m // 2
    out = []
    for ax, k in ((2, kx), (1, ky), (0, kz)):
        d = k.clone()
        d.select(ax, ny).zero_()
        out.append(torch.fft.irfftn(fk * (1j * d), s=(m, m, m)))
    return delta, torch.stack(out)


def _at(field, pos, box):
    """Nearest-node values of [..., m, m, m] fields at positions."""
    m = field.shape[-1]
    i = torch.remainder(torch.round(pos * (m / box)).long(), m)
    flat = (i[:, 2] * m + i[:, 1]) * m + i[:, 0]
    return field.reshape(*field.shape[:-3], -1)[..., flat]


def _to_redshift(x, p, obs, growth):
    rel = x - obs
    r = rel / rel.norm(dim=1, keepdim=True).clamp_min(1e-6)
    return x + growth * (p * r).sum(1, keepdim=True) * r


def _wrap(x, box):
    x = torch.remainder(x, box)
    return torch.where(x >= box, torch.zeros_like(x), x).contiguous()


def _box_catalogue(case, gen):
    dev, m = gen.device, case["npart"]
    box = case["cell"] * case["n"]
    g = min(256, 1 << max(4, (m - 1).bit_length()))
    _, psi = _linear(g, box, gen)
    h = box / m
    i = torch.arange(m, device=dev, dtype=torch.float32) * h
    obs = torch.tensor(_observer(case), device=dev, dtype=torch.float32)
    parts = []
    step = max(1, (1 << 24) // (m * m))
    for z0 in range(0, m, step):                       # slabs of the lattice, plane by plane in memory
        qz, qy, qx = torch.meshgrid(i[z0:z0 + step], i, i, indexing="ij")
        q = torch.stack([qx.reshape(-1), qy.reshape(-1), qz.reshape(-1)], 1)
        p = _at(psi, q, box).t()
        parts.append(_wrap(_to_redshift(q + p, p, obs, case["growth"]), box))
    gal = torch.cat(parts)
    ran = None
    if case["ran"]:
        ran = _wrap(torch.rand((case["ran"] * m ** 3, 3), generator=gen, device=dev) * box, box)
    return gal, ran


def _cone(count, box, gen, keep=None):
    """count points uniform in the survey's cone shell (times the acceptance keep(points)), in random order."""
    dev = gen.device
    r0, r1 = box * (1100.0 / 3500.0), box * (1800.0 / 3500.0)
    cmax = 1.0 - 2.5 / (2.0 * math.pi)
    a = torch.full((3,), 1.0 / math.sqrt(3.0), device=dev)
    e1 = torch.tensor([1.0, -1.0, 0.0], device=dev) / math.sqrt(2.0)
    e2 = torch.linalg.cross(a, e1)
    parts, have = [], 0
    while have < count:
        m = min(1 << 24, int((count - have) * (1.3 if keep is None else 6.0)) + 4096)
        u = torch.rand((4, m), generator=gen, device=dev)
        r = (r0 ** 3 + u[0] * (r1 ** 3 - r0 ** 3)) ** (1.0 / 3.0)
        ct = 1.0 - u[1] * (1.0 - cmax)
        st = torch.sqrt((1.0 - ct * ct).clamp_min(0.0))
        ph = 2.0 * math.pi * u[2]
        x = box / 2 + r[:, None] * ((st * torch.cos(ph))[:, None] * e1 + (st * torch.sin(ph))[:, None] * e2
                                    + ct[:, None] * a)
        ok = ((x >= 0) & (x < box)).all(1)
        if keep is not None:
            ok &= u[3] < keep(x)
        parts.append(x[ok][:count - have])
        have += parts[-1].shape[0]
    return torch.cat(parts)


def _survey_catalogue(case, count, gen):
    box = case["cell"] * case["n"]
    delta, psi = _linear(min(256, max(32, case["n"])), box, gen)
    obs = torch.tensor(_observer(case), device=gen.device, dtype=torch.float32)
    top = 1.0 + case["bias"] * 3.0 * float(delta.std())
    x = _cone(count, box, gen, lambda p: (1.0 + case["bias"] * _at(delta, p, box)) / top)
    p = _at(psi, x, box).t()
    gal = _wrap(_to_redshift(x, p, obs, case["growth"]), box)
    return gal, _wrap(_cone(case["ran"] * count, box, gen), box)


def _counts(case):
    """Galaxies of each realisation: log-uniform over a factor `spread` around case["gal"]."""
    b = case["batch"]
    if b == 1:
        return [case["gal"]]
    lo = case["gal"] / math.sqrt(case["spread"])
    return [int(lo * case["spread"] ** (((7 * i + 3) % b) / (b - 1))) | 1 for i in range(b)]


def _observer(case):
    box = case["cell"] * case["n"]
    if case["kind"] == "box":
        return (-case["far"] * box, box / 2, box / 2)
    return (box / 2, box / 2, box / 2)


def _generator(seed):
    gen = torch.Generator(device=_dev())
    gen.manual_seed(int(seed))
    return gen


def _inputs(case, seed):
    """gal, gal_w, gal_off, ran, ran_w, ran_off of a reconstruction case."""
    gen = _generator(seed)
    if case["kind"] == "box":
        gal, ran = _box_catalogue(case, gen)
        goff = roff = None
    else:
        got = [_survey_catalogue(case, c, gen) for c in _counts(case)]
        gal, ran = torch.cat([g for g, _ in got]), torch.cat([r for _, r in got])
        goff = roff = None
        if case["batch"] > 1:
            goff = torch.tensor(np.cumsum([0] + [g.shape[0] for g, _ in got]), device=gen.device)
            roff = torch.tensor(np.cumsum([0] + [r.shape[0] for _, r in got]), device=gen.device)
    gw = rw = None
    if case["weights"]:
        gw = 0.5 + torch.rand(gal.shape[0], generator=gen, device=gen.device)
        if ran is not None:
            rw = 0.5 + torch.rand(ran.shape[0], generator=gen, device=gen.device)
    return gal, gw, goff, ran, rw, roff


def _network():
    with np.load(learned.WEIGHTS, allow_pickle=False) as z:
        return torch.from_numpy(z["params"].astype(np.float32)).to(_dev())


def _stream_inputs(case, seed):
    gen = _generator(seed)
    pos = _wrap(_cone(case["objects"], case["cell"] * case["n"], gen), case["cell"] * case["n"])
    w = 0.5 + torch.rand(pos.shape[0], generator=gen, device=gen.device) if case["weights"] else None
    cuts = np.linspace(0, pos.shape[0], case["pieces"] + 1).astype(int)
    return [(pos[a:b].clone(), None if w is None else w[a:b].clone()) for a, b in zip(cuts[:-1], cuts[1:]) if b > a]


TRAIN_GEOMETRY = dict(box_len=3500.0, observer=(1750.0,) * 3, bias=2.0, growth=0.74, smooth_r=15.0)


def _train_inputs(case, seed):
    """A smoothed overdensity, its radial displacement and a target correction on the network grid, and
    parameters with moments as some way into a run."""
    gen = _generator(seed)
    m = case["n"] >> case["levels"]
    box = TRAIN_GEOMETRY["box_len"]
    fields = []
    for _ in range(case["batch"]):
        delta, psi = _linear(m, box, gen)
        i = (torch.arange(m, device=gen.device, dtype=torch.float32) + 0.25) * (box / m) - box / 2
        z, y, x = torch.meshgrid(i, i, i, indexing="ij")
        u = (psi[0] * x + psi[1] * y + psi[2] * z) / torch.sqrt(x * x + y * y + z * z)
        fields.append((0.3 * delta, u, -0.2 * u + 0.5 * torch.randn((m, m, m), generator=gen, device=gen.device)))
    d, u, t = (torch.stack([f[k] for f in fields]).contiguous() for k in range(3))
    th = torch.from_numpy(learned.init_params(int(seed) % 1000)).to(gen.device)
    mom = 1e-3 * torch.randn(th.shape[0], generator=gen, device=gen.device)
    return th, mom, mom * mom + 1e-6, d, u, t


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------
def prepare(case, seed):
    n = case["n"]
    if case["kind"] == "train":
        g = TRAIN_GEOMETRY
        plan = native.Plan(n, g["box_len"], g["observer"], g["bias"], g["growth"], g["smooth_r"], randoms=False,
                           batch=case["batch"], cnn=True, cnn_half=case["levels"] == 1,
                           cnn_quarter=case["levels"] == 2)
        th, m, v, d, u, t = _train_inputs(case, seed)
        return dict(case=case, plan=plan, th=th, m=m, v=v, d=d, u=u, t=t, grad=torch.empty_like(th))
    box = case["cell"] * n
    if case["kind"] == "stream":
        parts = _stream_inputs(case, seed)
        plan = native.Plan(n, box, (box / 2,) * 3, 2.0, 0.74, 15.0, randoms=False,
                           max_objects=0 if case["ngp"] else max(p.shape[0] for p, _ in parts))
        return dict(case=case, plan=plan, parts=parts)
    gal, gw, goff, ran, rw, roff = _inputs(case, seed)
    start = START[case["start"]]
    lrn = case["start"] == "learned"
    plan = native.Plan(n, box, _observer(case), case["bias"], case["growth"], case["smooth"], batch=case["batch"],
                       randoms=ran is not None, keep_delta=lrn, start_buffers=case["start"] != "plain", cnn=lrn,
                       cnn_quarter=lrn, graphs=case["graphs"], lognormal=case["lognormal"], relaxed=case["relaxed"],
                       max_objects=max(gal.shape[0], 0 if ran is None else ran.shape[0]))
    return dict(case=case, plan=plan, gal=gal, gw=gw, goff=goff, ran=ran, rw=rw, roff=roff, start=start,
                net=_network() if lrn else None)


# Step and rate of the training case: its moments are made up, so the step's bias correction is near 1.
TRAIN_STEP, TRAIN_LR = 900, 1e-4


def _history(case, rows, dtype):
    """The eps of every pass, [batch][passes allowed], 0 after the last."""
    out = np.zeros((case["batch"], case["passes"]), dtype=dtype)
    for b, row in enumerate(rows):
        out[b, :len(row)] = row
    return out


def run(state):
    case, plan = state["case"], state["plan"]
    if case["kind"] == "train":
        loss = plan.cnn_train_step(state["th"], state["m"], state["v"], TRAIN_STEP, TRAIN_LR, state["d"], state["u"],
                                   state["t"], state["grad"])
        return {"loss": loss, "grad": state["grad"], "params": state["th"], "m": state["m"], "v": state["v"]}
    if case["kind"] == "stream":
        for k, (pos, w) in enumerate(state["parts"]):
            plan.paint(native.GAL, pos, w, accumulate=k > 0, ngp=case["ngp"])
        return {"grid": plan.grid(native.GAL)}
    plan.paint(native.GAL, state["gal"], state["gw"], state["goff"], ngp=case["ngp"])
    if state["ran"] is not None:
        plan.paint(native.RAN, state["ran"], state["rw"], state["roff"], ngp=case["ngp"])
    plan.solve(state["start"], state["net"])
    _, passes, eps = plan.iterate(case["passes"], case["tol"])
    out = {"passes": np.asarray(passes), "eps": _history(case, eps, np.float32)}
    got = plan.shift(native.GAL, state["gal"], state["goff"], want_pos=case["want_pos"])
    out["gal"] = got
    if state["ran"] is not None:
        out["ran"] = plan.shift(native.RAN, state["ran"], state["roff"])
    return out


# ---------------------------------------------------------------------------
# Floors
# ---------------------------------------------------------------------------
def _usual_passes(case):
    """Passes counted by work(): the fixed number, or about what the tolerance takes (the error shrinks
    by about beta, or beta / (2 + beta) for the relaxed pass, and the radial part of it less)."""
    if case["tol"] == 0.0:
        return case["passes"]
    beta = case["growth"] / case["bias"]
    rate = 0.6 * beta / (2.0 + beta) if case["relaxed"] else 0.9 * beta
    return min(case["passes"], max(2, math.ceil(math.log(1e-3) / math.log(rate))))


def work(case):
    n, b = case["n"], case["batch"]
    if case["kind"] == "train":
        cells = b * (n >> case["levels"]) ** 3
        macs = 27 * (8 * 16 + 16 * 16 + 16)
        # forward, input gradients (layers 2 and 3) and weight gradients; three input fields in, and the
        # bf16 activations and their gradients (2 x 16 channels each) out and in once
        flops = 2.0 * cells * (2 * macs + 27 * (16 * 16 + 16))
        return {"bytes": cells * (12.0 + 4 * 2 * 32), "flops": flops}
    if case["kind"] == "stream":
        obj = case["objects"]
        return {"bytes": obj * (16.0 if case["weights"] else 12.0) + 8.0 * n ** 3, "flops": 60.0 * obj}
    if case["kind"] == "box":
        gal, ran = case["npart"] ** 3, case["ran"] * case["npart"] ** 3
    else:
        gal = sum(_counts(case))
        ran = case["ran"] * gal
    passes = _usual_passes(case)
    per = 16.0 if case["weights"] else 12.0
    obj = (gal + ran) * (per + 12.0 + 12.0)                 # deposit in, shift in and out
    spec = (n // 2 + 1) * n * n * 8.0 * b
    grids = 2 if ran else 1
    real = n ** 3 * 4.0 * b
    # a three-axis transform of n^3 reads and writes the field at least twice (the rows of one axis do
    # not fit the chip beside the planes of the other two): 4 spectra a pass for the inverse and the
    # forward of the two carried fields, and D_s, D_n in and D_n out; the setup smooths each grid and
    # transforms the overdensity; the displacement is written and gathered
    nbytes = obj + spec * (7.0 * passes + 6.0 * grids + 4.0) + 3.0 * real * 2 + 8.0 * n ** 3 * b * grids
    fft = 2.5 * n ** 3 * math.log2(n ** 3) * b              # one real transform
    return {"bytes": nbytes, "flops": fft * (5.0 * passes + 2.0 * grids + 4.0)}


# ---------------------------------------------------------------------------
# The same outputs in 64 bits
# ---------------------------------------------------------------------------
def _coords(pos, n, box):
    """Cell, 16-bit fraction and FP32 fraction of every object: the library's deposit frame."""
    s = torch.tensor(np.float32(n / box), device=pos.device)
    u = pos * s
    fl = torch.floor(u)
    t = u - fl
    return torch.remainder(fl.long(), n), torch.floor(t.double() * 65536.0).long(), t


def _chunks(m, step=1 << 24):
    return [(a, min(m, a + step)) for a in range(0, m, step)]


def _deposit64(pos, w, n, box, ngp, grid=None):
    """The integer deposit by its definition (units of 2^-32 weight)."""
    if grid is None:
        grid = torch.zeros(n ** 3, dtype=torch.int64, device=pos.device)
    for a, b in _chunks(pos.shape[0]):
        i, tau, t = _coords(pos[a:b], n, box)
        wq = torch.full((b - a,), 1 << 32, dtype=torch.int64, device=pos.device) if w is None else \
            torch.round(w[a:b].double() * 4294967296.0).long()
        if ngp:
            j = torch.remainder(i + (t >= 0.5).long(), n)
            grid.index_add_(0, (j[:, 2] * n + j[:, 1]) * n + j[:, 0], wq)
            continue
        rest = wq.clone()
        for k in range(8):
            d = (k & 1, (k >> 1) & 1, k >> 2)
            j = [torch.remainder(i[:, ax] + d[ax], n) for ax in range(3)]
            cell = (j[2] * n + j[1]) * n + j[0]
            if k == 7:
                part = rest
            else:
                c = 1
                for ax in range(3):
                    c = c * (tau[:, ax] if d[ax] else 65536 - tau[:, ax])
                part = (wq * (c >> 24) + ((wq * (c & 0xFFFFFF)) >> 24)) >> 24
                rest = rest - part
            grid.index_add_(0, cell, part)
    return grid


class _Modes:
    """Wavenumbers of rfftn over [z][y][x] and the line of sight, in 64 bits."""

    def __init__(self, n, box, obs, dev):
        kf = 2.0 * math.pi / box
        m = torch.fft.fftfreq(n, d=1.0 / n, device=dev, dtype=torch.float64)
        h = torch.arange(n // 2 + 1, device=dev, dtype=torch.float64)
        md, hd = m.clone(), h.clone()
        md[n // 2] = 0.0
        hd[n // 2] = 0.0
        self.n = n
        self.k = (h.view(1, 1, -1) * kf, m.view(1, n, 1) * kf, m.view(n, 1, 1) * kf)
        self.d = (hd.view(1, 1, -1) * kf, md.view(1, n, 1) * kf, md.view(n, 1, 1) * kf)
        i = torch.arange(n, device=dev, dtype=torch.float64) * (box / n)
        self.r = ((i - obs[0]).view(1, 1, n), (i - obs[1]).view(1, n, 1), (i - obs[2]).view(n, 1, 1))

    def k2(self):
        return self.k[0] ** 2 + self.k[1] ** 2 + self.k[2] ** 2

    def inverse_r(self):
        r = torch.sqrt(self.r[0] ** 2 + self.r[1] ** 2 + self.r[2] ** 2)
        return torch.where(r > 0, 1.0 / r, torch.zeros_like(r))


def _smooth64(grid, M, radius):
    n = M.n
    f = torch.fft.rfftn(grid.view(n, n, n).double() * 2.0 ** -32)
    f *= torch.exp(-0.5 * radius * radius * M.k2())
    return torch.fft.irfftn(f, s=(n, n, n))


def _overdensity64(gg, gr, M, radius, tau=0.1):
    n = M.n
    wg = int(gg.sum())
    g = _smooth64(gg, M, radius)
    if gr is None:
        return g / (wg * 2.0 ** -32 / n ** 3) - 1.0
    wr, occ = int(gr.sum()), int((gr != 0).sum())
    s = gr.view(n, n, n)
    for ax in range(3):
        s = s + torch.roll(s, 1, ax) + torch.roll(s, -1, ax)
    mask = s > math.floor(tau * 27.0 * wr / occ)
    ar = _smooth64(gr, M, radius) * (wg / wr)
    mask &= ar > 0
    return torch.where(mask, (g - ar) / torch.where(mask, ar, torch.ones_like(ar)), torch.zeros_like(g))


def _psi64(D, M, bias):
    """Components of i k' D / (b k^2), one at a time."""
    n = M.n
    k2 = M.k2()
    k2[0, 0, 0] = 1.0
    P = D / (bias * k2)
    P[0, 0, 0] = 0.0
    return [torch.fft.irfftn(P * (1j * d), s=(n, n, n)) for d in M.d]


def _network64(net, delta, u, box, obs):
    """The learned start's radial correction in 64 bits (no rounding of weights or activations)."""
    p = net.double()
    m = delta.shape[-1]
    M = _Modes(m, box, obs, delta.device)
    ir = M.inverse_r()
    x = torch.stack([delta, 0.1 * u] + [(r * ir).expand(m, m, m) for r in M.r] + [torch.zeros_like(delta)] * 3, -1)
    at = 0
    for cin, cout, last in ((8, 16, False), (16, 16, False), (16, 1, True)):
        W = p[at:at + cout * 27 * cin].view(cout, 27, cin)
        at += W.numel()
        bias = p[at:at + cout]
        at += cout
        x = _conv64(x, W) + bias
        if not last:
            x = torch.relu(x)
    return x[..., 0] / 0.1


def _conv64(x, W):
    """Periodic 3^3 cross-correlation of [z][y][x][c], taps ordered (dz, dy, dx)."""
    y = 0
    for t in range(27):
        dx, dy, dz = t % 3 - 1, (t // 3) % 3 - 1, t // 9 - 1
        y = y + torch.matmul(torch.roll(x, (-dz, -dy, -dx), (0, 1, 2)), W[:, t].t().contiguous())
    return y


def _restrict64(f):
    for ax in range(3):
        f = 0.5 * f + 0.25 * (torch.roll(f, 1, ax) + torch.roll(f, -1, ax))
        f = f.index_select(ax, torch.arange(0, f.shape[ax], 2, device=f.device))
    return f


def _prolong64(c):
    for ax in range(3):
        mid = 0.5 * (c + torch.roll(c, -1, ax))
        c = torch.stack([c, mid], ax + 1).flatten(ax, ax + 1)
    return c


def _iterate64(delta, M, case, box, obs, net):
    bias, f = case["bias"], case["growth"]
    beta = f / bias
    ir = M.inverse_r()
    D_s = torch.fft.rfftn(delta)
    psi = _psi64(D_s, M, bias)
    if case["start"] != "plain":
        u = sum(p * r for p, r in zip(psi, M.r)) * ir
        if case["start"] == "learned":
            c = _network64(net, _restrict64(_restrict64(delta)), _restrict64(_restrict64(u)), box, obs)
            add = _prolong64(_prolong64(c))
        else:
            add = -u * (beta / (1.0 + beta) if case["start"] == "ffta1" else 3.0 * beta / (7.0 + 3.0 * beta))
        add *= ir
        psi = [p + add * r for p, r in zip(psi, M.r)]
        del u, add
    w = 2.0 / (2.0 + beta) if case["relaxed"] else 1.0
    D, eps = D_s, []
    for k in range(case["passes"]):
        q = sum(p * r for p, r in zip(psi, M.r)) * ir * ir
        new = D_s.clone()
        for r, d in zip(M.r, M.d):
            new += torch.fft.rfftn(q * r) * (1j * f * d)
        D = new if w == 1.0 or (k == 0 and case["start"] != "plain") else (1.0 - w) * D + w * new
        del new, q
        nxt = _psi64(D, M, bias)
        num = sum(float((a - b).square().sum()) for a, b in zip(nxt, psi))
        den = sum(float(a.square().sum()) for a in nxt)
        psi = nxt
        eps.append(math.sqrt(num / den))
        if case["tol"] > 0.0 and eps[-1] <= case["tol"]:
            break
    return psi, eps


def _shift64(psi, pos, n, box, obs, growth):
    out = torch.empty(pos.shape, dtype=torch.float64, device=pos.device)
    for a, b in _chunks(pos.shape[0]):
        i, _, t = _coords(pos[a:b], n, box)
        t = t.double()
        p = torch.zeros((b - a, 3), dtype=torch.float64, device=pos.device)
        for k in range(8):
            d = (k & 1, (k >> 1) & 1, k >> 2)
            wgt = 1.0
            for ax in range(3):
                wgt = wgt * (t[:, ax] if d[ax] else 1.0 - t[:, ax])
            j = [torch.remainder(i[:, ax] + d[ax], n) for ax in range(3)]
            cell = (j[2] * n + j[1]) * n + j[0]
            for c in range(3):
                p[:, c] += wgt * psi[c].reshape(-1)[cell]
        o = -p
        if growth:
            rel = pos[a:b].double() - torch.tensor(obs, dtype=torch.float64, device=pos.device)
            r = rel / rel.norm(dim=1, keepdim=True).clamp_min(1e-300)
            o -= growth * (p * r).sum(1, keepdim=True) * r
        out[a:b] = o
    return out


def _train64(case, seed):
    th, m, v, d, u, t = _train_inputs(case, seed)
    box, obs = TRAIN_GEOMETRY["box_len"], TRAIN_GEOMETRY["observer"]
    p = th.double().requires_grad_(True)
    cells = d.numel()
    loss = 0.0
    for k in range(case["batch"]):
        y = 0.1 * _network64(p, d[k].double(), u[k].double(), box, obs)
        part = ((y - 0.1 * t[k].double()) ** 2).sum() / cells
        part.backward()
        loss += float(part)
    g = p.grad
    m = 0.9 * m.double() + 0.1 * g
    v = 0.999 * v.double() + 0.001 * g * g
    p = th.double() - TRAIN_LR * (m / (1.0 - 0.9 ** TRAIN_STEP)) / (torch.sqrt(v / (1.0 - 0.999 ** TRAIN_STEP)) + 1e-8)
    return {"loss": loss, "grad": g, "params": p, "m": m, "v": v}


def exact(case, seed):
    if case["kind"] == "train":
        return _train64(case, seed)
    n = case["n"]
    box = case["cell"] * n
    if case["kind"] == "stream":
        return None                                   # whole numbers only
    gal, gw, goff, ran, rw, roff = _inputs(case, seed)
    obs = _observer(case)
    net = _network() if case["start"] == "learned" else None
    B = case["batch"]
    go = [0, gal.shape[0]] if goff is None else goff.tolist()
    ro = None if ran is None else ([0, ran.shape[0]] if roff is None else roff.tolist())
    out = {"passes": None, "eps": [], "gal": [], "ran": []}
    M = _Modes(n, box, obs, gal.device)
    for b in range(B):
        g = gal[go[b]:go[b + 1]]
        gg = _deposit64(g, None if gw is None else gw[go[b]:go[b + 1]], n, box, case["ngp"])
        gr = None
        if ran is not None:
            r = ran[ro[b]:ro[b + 1]]
            gr = _deposit64(r, None if rw is None else rw[ro[b]:ro[b + 1]], n, box, case["ngp"])
        delta = _overdensity64(gg, gr, M, case["smooth"])
        del gg, gr
        if case["lognormal"]:
            delta = torch.log(delta.add_(1.0).clamp_min_(1e-3))
            delta -= delta.mean()
        psi, eps = _iterate64(delta, M, case, box, obs, net)
        del delta
        out["eps"].append(eps)
        out["gal"].append(_shift64(psi, g, n, box, obs, case["growth"]))
        if ran is not None:
            out["ran"].append(_shift64(psi, r, n, box, obs, 0.0))
        del psi
    disp = torch.cat(out["gal"])
    out["gal"] = (disp, gal.double() + disp) if case["want_pos"] else disp
    out["eps"] = _history(case, out["eps"], np.float64)
    if ran is None:
        del out["ran"]
    else:
        out["ran"] = torch.cat(out["ran"])
    return out
