"""Workloads that the estimator is timed on, through its public entry points.

Each case is what a user's program does in one pass: particles already on the
GPU and a handle that the program keeps go in, spectra, shell statistics or
gradients come out.  ``listed()`` holds the named workloads, ``draw()`` gives
further ones over the same ranges, ``prepare()`` makes the inputs from a seed,
``run()`` is one pass, ``work()`` what a pass cannot do without, and
``exact()`` the same outputs in 64 bits from plain torch.

Kinds of case:

* ``power``: ``Estimator.power`` of one set or a batch of sets;
* ``replay``: the same pass of a batch, captured once as a HIP graph;
* ``grad``: a chi^2 loss of P(k) and its gradient with respect to the positions;
* ``bispectrum``: P(k) and the bispectrum of every closed triangle;
* ``direct``: the direct sum, the estimator's own modes and their auto and
  cross spectra (the aliasing comparison).
"""

import math
import random

import numpy as np
import torch

DEVICE = "cuda"


# ---------------------------------------------------------------- the cases
def _case(name, kind, n_grid, n, **kw):
    c = {"name": name, "kind": kind, "n_grid": n_grid, "n": n, "box": 1000.0, "order": 4, "interlace": 1,
         "dtype": "f32", "dist": "za", "masses": False, "batch": 1, "n_dk": 1, "n_bins": n_grid // 2, "shot": False}
    c.update(kw)
    return c


def listed():
    return [
        # a quick look at a small catalogue: launches and latency are all there is
        _case("power_32_small", "power", 32, 5000, dist="uniform", box=500.0),
        # the paper's comparison grid, N_G = 100 (mixed radix, ragged tiles), on
        # float64 positions of a galaxy catalogue, shot noise subtracted
        _case("power_100_tsc_f64", "power", 100, 100003, order=3, dtype="f64", dist="halos", shot=True),
        # an ordinary simulation output: one particle per cell
        _case("power_256", "power", 256, 256 ** 3),
        # the paper's Zel'dovich runs: 360^3 particles on N_G = 480
        _case("power_480_paper", "power", 480, 360 ** 3, box=2400.0),
        # the largest single grid: 512^3 particles on 1024^3
        _case("power_1024", "power", 1024, 512 ** 3, box=2000.0),
        # CIC without interlacing, the estimator most catalogues were measured
        # with so far: clustered float64 positions, wide shells
        _case("power_512_cic_f64", "power", 512, 16 * 1024 * 1024, order=2, interlace=0, dtype="f64", dist="halos", n_dk=2,
              n_bins=128),
        # halo catalogue with masses, eight interlaced grids
        _case("power_256_eight_masses", "power", 256, 2000000, interlace=3, masses=True, dist="halos"),
        # covariance from mocks: 64 uneven sets on 128^3, replayed as one graph
        _case("replay_64_mocks", "replay", 128, 72000000, batch=64, box=500.0, dist="mocks"),
        # a step of field-level inference: 128^3 particles, 256^3 grid
        _case("grad_256", "grad", 256, 128 ** 3),
        # a step of a sampler on a small problem
        _case("grad_64_small", "grad", 64, 32 ** 3, box=500.0),
        # P(k) and all closed triangles of 32 shells
        _case("bispectrum_256", "bispectrum", 256, 256 ** 3, n_dk=2, n_bins=32),
        # aliasing measured against direct summation on every mode
        _case("direct_64", "direct", 64, 64 ** 3, box=500.0, n_bins=32),
    ]


def _smooth(v):
    for p in (2, 3, 5):
        while v % p == 0:
            v //= p
    return v == 1


GRIDS = [v for v in range(32, 1025, 4) if _smooth(v)]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _grid(rng, lo, hi):
    v = _log(rng, lo, hi)
    return min((g for g in GRIDS if lo <= g <= hi), key=lambda g: abs(math.log(g / v)))


def _cost(c):
    """Rough time of a pass, in units of one grid cell through one stage."""
    ng = 2 ** c["interlace"]
    part = c["n"] * (4.0 + ng * (1.0 + c["order"] ** 3 / 32.0)) * (1.5 if c["masses"] else 1.0)
    cells = 3.0 * c["batch"] * ng * float(c["n_grid"]) ** 3
    return (part + cells) * (3.0 if c["kind"] == "grad" else 1.0)


def draw(rng):
    kind = rng.choice(["power", "power", "power", "power", "replay", "grad", "grad", "bispectrum", "direct"])
    top = _cost(listed()[4])
    while True:
        if kind == "power":
            g = _grid(rng, 32, 1024)
            n = int(min(2.0 ** 27, max(1000.0, float(g) ** 3 * _log(rng, 1 / 64, 2.0))))
            batch = 1
            if g <= 128 and rng.random() < 0.3:
                batch = rng.randint(2, 16)
                n = max(n, 2000 * batch)
            dk = rng.choice([1, 1, 2, 4])
            c = _case("", kind, g, n, order=rng.choice([1, 2, 3, 4, 4, 4, 5, 6]), interlace=rng.choice([0, 1, 1, 1, 1, 2, 3]),
                      dtype=rng.choice(["f32", "f32", "f64"]), dist=rng.choice(["uniform", "za", "halos"]),
                      masses=rng.random() < 0.25, batch=batch, n_dk=dk, n_bins=max(1, int(g // (2 * dk) * rng.choice([1.0, 1.0, 0.5]))),
                      shot=rng.random() < 0.5, box=rng.choice([500.0, 1000.0, 2400.0]))
        elif kind == "replay":
            g = _grid(rng, 32, 160)
            batch = rng.randint(2, 64)
            n = int(batch * _log(rng, 5000.0, 2.0e6))
            c = _case("", kind, g, n, order=rng.choice([2, 3, 4, 4]), interlace=rng.choice([0, 1, 1]), batch=batch, dist="mocks", box=500.0)
        elif kind == "grad":
            g = _grid(rng, 32, 384)
            n = int(min(4.0e6, max(1000.0, float(g) ** 3 * _log(rng, 1 / 32, 1.0))))
            c = _case("", kind, g, n, order=rng.choice([2, 3, 4, 4, 5]), interlace=rng.choice([0, 1, 1, 1, 2]),
                      dist=rng.choice(["za", "uniform", "halos"]), masses=rng.random() < 0.2,
                      n_bins=max(1, int(g // 2 * rng.choice([1.0, 0.75, 0.5]))))
        elif kind == "bispectrum":
            g = _grid(rng, 48, 288)
            dk = rng.choice([1, 2, 3, 4])
            most = max(b for b in range(0, 41) if 3 * (2 * b + 1) * dk < 2 * g and _alias_free(b, dk) <= g)
            c = _case("", kind, g, int(min(1.6e7, max(2000.0, float(g) ** 3 * _log(rng, 1 / 32, 1.0)))), n_dk=dk,
                      n_bins=rng.randint(max(1, most // 2), max(1, most)), interlace=rng.choice([0, 1, 1]), order=rng.choice([2, 3, 4]),
                      dist=rng.choice(["za", "halos"]))
        else:
            g = _grid(rng, 32, 64)
            c = _case("", kind, g, int(_log(rng, 2000.0, 262144.0)), dtype=rng.choice(["f32", "f64"]), masses=rng.random() < 0.3,
                      dist=rng.choice(["za", "halos"]), box=500.0)
        if c["dist"] == "za":  # a whole lattice
            side = max(s for s in _SIDES if s ** 3 <= max(c["n"], 10 ** 3))
            c["n"] = side ** 3
        if _cost(c) <= top:
            del c["name"]
            return c


_SIDES = [s for s in range(8, 513, 2) if _smooth(s)]


def _alias_free(n_bins, n_dk):
    v = 3 * (((2 * n_bins + 1) * n_dk - 1) // 2) + 1
    while not _smooth(v):
        v += 1
    return v


# ---------------------------------------------------------------- inputs
def _gen(seed):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(seed)
    return g


def _uniform(n, box, g, dtype):
    return torch.rand((n, 3), generator=g, device=DEVICE, dtype=dtype) * box


def _halos(n, box, g, dtype):
    """Half of the particles uniform, half in Gaussian clumps of about 100."""
    half = n // 2
    centres = _uniform(max(1, half // 100), box, g, dtype)
    at = torch.randint(0, centres.shape[0], (half,), generator=g, device=DEVICE)
    clumped = centres[at] + torch.randn((half, 3), generator=g, device=DEVICE, dtype=dtype) * (box / 400.0)
    out = torch.cat([_uniform(n - half, box, g, dtype), torch.remainder(clumped, box)])
    return out[torch.randperm(n, generator=g, device=DEVICE)].contiguous()


def _zeldovich(side, box, g, dtype):
    """Cubic lattice displaced by a Gaussian field of power k^-1.5, with an rms of 0.3 spacings per axis."""
    white = torch.fft.rfftn(torch.randn((side,) * 3, generator=g, device=DEVICE))
    f = torch.fft.fftfreq(side, 1.0 / side, device=DEVICE)
    m = [f[:, None, None], f[None, :, None], torch.arange(side // 2 + 1, device=DEVICE, dtype=torch.float32)[None, None, :]]
    m2 = m[0] ** 2 + m[1] ** 2 + m[2] ** 2
    m2[0, 0, 0] = 1.0
    white *= m2 ** (-0.75 / 2 - 1.0)
    white[0, 0, 0] = 0
    del m2
    for a in range(3):  # no lattice Nyquist modes
        white.select(a, side // 2).zero_()
    out = torch.empty((side, side, side, 3), device=DEVICE, dtype=dtype)
    for a in range(3):
        psi = torch.fft.irfftn(1j * m[a] * white, s=(side,) * 3)
        shape = [1, 1, 1]
        shape[a] = side
        q = torch.arange(side, device=DEVICE, dtype=dtype).reshape(shape)
        out[..., a] = torch.remainder((q + psi * (0.3 / psi.std())) * (box / side), box)
        del psi
    return out.reshape(-1, 3)


def _counts(case):
    """Particles per set of a batch: log-uniform around the mean, fixed by the case (not by the seed)."""
    if case["batch"] == 1:
        return [case["n"]]
    r = random.Random(case["batch"])
    raw = [math.exp(r.uniform(0.0, math.log(40.0))) for _ in range(case["batch"])]
    return [max(100, int(case["n"] * v / sum(raw))) for v in raw]


def _positions(case, seed):
    g = _gen(seed)
    dtype = torch.float64 if case["dtype"] == "f64" else torch.float32
    parts = []
    for i, n in enumerate(_counts(case)):
        dist = case["dist"]
        if dist == "mocks":  # uniform and clustered sets in turn
            dist = "halos" if i % 2 else "uniform"
        if dist == "za":
            side = round(n ** (1 / 3))
            if side ** 3 != n:
                side = max(s for s in _SIDES if s ** 3 <= n)
            p = _zeldovich(side, case["box"], g, dtype)
            if p.shape[0] < n:
                p = torch.cat([p, _uniform(n - p.shape[0], case["box"], g, dtype)])
        else:
            p = (_uniform if dist == "uniform" else _halos)(n, case["box"], g, dtype)
        parts.append(p)
    pos = parts[0] if len(parts) == 1 else torch.cat(parts)
    w = None
    if case["masses"]:
        w = torch.empty(pos.shape[0], device=DEVICE).exponential_(1.0, generator=g)
    return pos.contiguous(), w


def _target(case):
    """Fiducial spectrum and variance of the chi^2 loss, per shell."""
    n_b, k = _shells(case["n_grid"], case["n_dk"], case["n_bins"], case["box"])
    vol = case["box"] ** 3
    t = vol / case["n"] * (1.0 + 20.0 * (k / k[0]) ** -1.5)
    return t, 2.0 * t ** 2 / n_b.double()


def _triangles(n_bins):
    return np.array([(a, b, c) for a in range(1, n_bins + 1) for b in range(1, a + 1) for c in range(max(1, a - b), b + 1)], dtype=np.int32)


def prepare(case, seed):
    from paper_1512_07295_amd.estimator import Estimator

    pos, w = _positions(case, seed)
    n = pos.shape[0]
    est = Estimator(case["n_grid"], case["box"], case["order"], case["interlace"], case["batch"], n, weighted=case["masses"])
    if w is not None:
        est.set_weights(w)
    s = {"case": case, "est": est, "pos": pos, "w": w, "offsets": None}
    if case["batch"] > 1:
        s["offsets"] = torch.tensor(np.concatenate([[0], np.cumsum(_counts(case))]), dtype=torch.int64, device=DEVICE)
    if case["kind"] == "replay":
        est.capture(pos, s["offsets"], case["n_dk"], case["n_bins"], case["shot"])
    elif case["kind"] == "grad":
        s["target"], s["sigma2"] = _target(case)
    elif case["kind"] == "bispectrum":
        s["triangles"] = _triangles(case["n_bins"])
    return s


# ---------------------------------------------------------------- one pass
def run(s):
    case, est, pos = s["case"], s["est"], s["pos"]
    dk, nb = case["n_dk"], case["n_bins"]
    if case["kind"] == "power":
        return dict(zip(("k", "p", "modes"), est.power(pos, s["offsets"], dk, nb, case["shot"])))
    if case["kind"] == "replay":
        return dict(zip(("k", "p", "modes"), est.replay()))
    if case["kind"] == "grad":
        from paper_1512_07295_amd.estimator import PowerSpectrumFn

        x = pos.detach().requires_grad_(True)
        p = PowerSpectrumFn.apply(x, est, dk, nb, None)
        loss = ((p - s["target"]) ** 2 / s["sigma2"]).sum()
        loss.backward()
        return {"p": p.detach(), "loss": loss.detach(), "grad": x.grad}
    if case["kind"] == "bispectrum":
        k, p, modes = est.power(pos, None, dk, nb)
        b, n_tri = est.bispectrum(s["triangles"], dk, nb)
        return {"k": k, "p": p, "modes": modes, "b": b, "n_tri": n_tri}
    ds = est.direct_delta(pos)
    est.deposit(pos)
    est.transform()
    dg = est.export_delta()
    k, p_ds, modes = est.spectrum_power(ds, None, dk, nb)
    _, p_x, _ = est.spectrum_power(dg, ds, dk, nb)
    return {"delta_ds": ds, "delta_g": dg, "k": k, "p_ds": p_ds, "p_x": p_x, "modes": modes}


def work(case):
    """Positions and masses in, results out; stencil sums, transforms and mode sums as arithmetic."""
    n, g, ng = float(case["n"]), float(case["n_grid"]), 2 ** case["interlace"]
    sets, nb = case["batch"], case["n_bins"]
    b = n * (12 if case["dtype"] == "f32" else 24) + (4 * n if case["masses"] else 0) + 24 * sets * nb
    fft = sets * ng * 2.5 * g ** 3 * 3 * math.log2(g)
    stencil = 2.0 * n * ng * case["order"] ** 3
    f = stencil + fft + 8 * sets * g ** 3
    if case["kind"] == "grad":
        b += n * 12
        f = 2 * (stencil + fft + 8 * g ** 3) + fft + 3 * stencil
    elif case["kind"] == "bispectrum":
        tri, m = len(_triangles(nb)), float(_alias_free(nb, case["n_dk"]))
        b += 16 * tri
        f += nb * 2.5 * m ** 3 * 3 * math.log2(m) + 2.0 * tri * m ** 3
    elif case["kind"] == "direct":
        modes = g * g * (g / 2 + 1)
        b += 2 * 16 * modes
        f += 8 * n * modes
    return {"bytes": b, "flops": f}


# ---------------------------------------------------------------- 64 bits
_MASKS = {0: (0,), 1: (0, 7), 2: (0, 3, 5, 6), 3: tuple(range(8))}


def _signed(n):
    i = torch.arange(n, device=DEVICE)
    return torch.where(i <= n // 2, i, i - n)


def _bins_of(n, n_dk, n_bins):
    """Shell of every |m|^2 (0: none)."""
    v = 4 * torch.arange(3 * (n // 2) ** 2 + 1, device=DEVICE)
    edges = torch.tensor([((2 * b + 1) * n_dk) ** 2 for b in range(n_bins + 1)], device=DEVICE)
    b = torch.bucketize(v, edges, right=True)
    return torch.where(b > n_bins, torch.zeros_like(b), b)


def _planes(n, step):
    """(x0, x1, |m|^2, half-spectrum weight) of x planes of the half spectrum."""
    m = _signed(n)
    mz = torch.arange(n // 2 + 1, device=DEVICE)
    w = torch.full((n // 2 + 1,), 2.0, device=DEVICE, dtype=torch.float64)
    w[0] = w[n // 2] = 1.0
    for x0 in range(0, n, step):
        x1 = min(n, x0 + step)
        m2 = m[x0:x1, None, None] ** 2 + m[None, :, None] ** 2 + mz[None, None, :] ** 2
        yield x0, x1, m2, w.expand(m2.shape)


def _step(n):
    return max(1, min(n, (1 << 23) // (n * (n // 2 + 1))))


def _shell_sums(n, n_dk, n_bins, values):
    """Sum over the modes of each shell of weight * values(x0, x1, |m|^2)."""
    table = _bins_of(n, n_dk, n_bins)
    total = torch.zeros(n_bins + 1, device=DEVICE, dtype=torch.float64)
    for x0, x1, m2, w in _planes(n, _step(n)):
        b = table[m2]
        total += torch.bincount(b.reshape(-1), (w * values(x0, x1, m2)).reshape(-1), minlength=n_bins + 1)
    return total[1:]


def _shells(n, n_dk, n_bins, box):
    """(modes, mean |k|) per shell."""
    n_b = _shell_sums(n, n_dk, n_bins, lambda x0, x1, m2: torch.ones(m2.shape, device=DEVICE, dtype=torch.float64))
    k = _shell_sums(n, n_dk, n_bins, lambda x0, x1, m2: m2.double().sqrt())
    return n_b.round().long(), 2 * math.pi / box * k / n_b


def _stencil(order, u):
    """First cell, the B-spline weights and their derivatives with respect to u."""
    t = u if order % 2 == 0 else u + 0.5
    cell = torch.floor(t)
    f = t - cell
    w = [torch.ones_like(f)]
    low = w
    for q in range(2, order + 1):
        low = w
        zero = torch.zeros_like(f)
        prev = [zero] + w + [zero]
        w = [((f + (q - 1 - k)) * prev[k] + (1 + k - f) * prev[k + 1]) / (q - 1) for k in range(q)]
    zero = torch.zeros_like(f)
    ends = [zero] + low + [zero]
    d = [ends[k] - ends[k + 1] for k in range(order)] if order > 1 else [zero]
    first = cell.long() - ((order // 2 - 1) if order % 2 == 0 else (order - 1) // 2)
    return first, w, d


def _wrapped(case, pos):
    x = torch.remainder(pos.double(), case["box"])
    return x * (case["n_grid"] / case["box"])


def _deposit(case, pos, w, mask):
    n = case["n_grid"]
    rho = torch.zeros(n ** 3, device=DEVICE, dtype=torch.float64)
    for j0 in range(0, pos.shape[0], 1 << 24):
        u = _wrapped(case, pos[j0:j0 + (1 << 24)])
        ax = [_stencil(case["order"], u[:, a] + (0.5 if mask >> a & 1 else 0.0)) for a in range(3)]
        mass = 1.0 if w is None else w[j0:j0 + (1 << 24)].double()
        for a in range(case["order"]):
            ia, wa = torch.remainder(ax[0][0] + a, n) * n, ax[0][1][a] * mass
            for b in range(case["order"]):
                iab, wab = (ia + torch.remainder(ax[1][0] + b, n)) * n, wa * ax[1][1][b]
                for c in range(case["order"]):
                    rho.index_add_(0, iab + torch.remainder(ax[2][0] + c, n), wab * ax[2][1][c])
    return rho.reshape(n, n, n)


def _phase(n, mask, x0, x1, sign=1.0):
    m = _signed(n).double()
    mz = torch.arange(n // 2 + 1, device=DEVICE, dtype=torch.float64)
    s = 0.0
    if mask & 1:
        s = s + m[x0:x1, None, None]
    if mask & 2:
        s = s + m[None, :, None]
    if mask & 4:
        s = s + mz[None, None, :]
    return torch.exp(1j * math.pi * sign / n * s) if mask else 1.0


def _spectrum(case, pos, w):
    """The combined modes C(m) on the half spectrum."""
    n, masks = case["n_grid"], _MASKS[case["interlace"]]
    c = None
    for mask in masks:
        f = torch.fft.rfftn(_deposit(case, pos, w, mask))
        if mask:
            for x in range(0, n, _step(n)):
                f[x:x + _step(n)] *= _phase(n, mask, x, min(n, x + _step(n)))
        c = f if c is None else c.add_(f)
        del f
    return c.div_(len(masks))


def _window(case):
    x = torch.sinc(_signed(case["n_grid"]).double() / case["n_grid"]) ** case["order"]
    return x[:, None, None], x[None, :, None], x[None, None, :case["n_grid"] // 2 + 1]


def _power(case, pos, w):
    n, dk, nb, vol = case["n_grid"], case["n_dk"], case["n_bins"], case["box"] ** 3
    c, (wx, wy, wz) = _spectrum(case, pos, w), _window(case)
    total = float(pos.shape[0]) if w is None else float(w.double().sum())
    squares = float(pos.shape[0]) if w is None else float(w.double().square().sum())
    n_b, k = _shells(n, dk, nb, case["box"])
    s = _shell_sums(n, dk, nb, lambda x0, x1, m2: (c[x0:x1].abs() / (wx[x0:x1] * wy * wz)) ** 2)
    p = vol * s / total ** 2 / n_b
    return k, p, n_b, c, total, p - vol * squares / total ** 2


def _exact_power(case, seed):
    pos, w = _positions(case, seed)
    out, at = [], 0
    for n in _counts(case):
        k, p, n_b, _, _, sub = _power(case, pos[at:at + n], None if w is None else w[at:at + n])
        out.append((k, sub if case["shot"] else p, n_b))
        at += n
    return {name: torch.stack([o[i] for o in out]) for i, name in enumerate(("k", "p", "modes"))}


def _exact_grad(case, seed):
    pos, w = _positions(case, seed)
    n, dk, nb, vol = case["n_grid"], case["n_dk"], case["n_bins"], case["box"] ** 3
    _, p, n_b, c, total, _ = _power(case, pos, w)
    t, s2 = _target(case)
    coef = torch.zeros(nb + 1, device=DEVICE, dtype=torch.float64)
    coef[1:] = 2 * (p - t) / s2 * vol / total ** 2 / n_b
    table, (wx, wy, wz) = _bins_of(n, dk, nb), _window(case)
    for x0, x1, m2, _ in _planes(n, _step(n)):
        c[x0:x1] *= coef[table[m2]] / (wx[x0:x1] * wy * wz) ** 2
    grad = torch.zeros(pos.shape, device=DEVICE, dtype=torch.float64)
    masks = _MASKS[case["interlace"]]
    for mask in masks:
        f = torch.fft.ifftn(c * _phase(n, mask, 0, n, -1.0), dim=(0, 1))
        f[..., 0].imag.zero_()
        f[..., n // 2].imag.zero_()
        gamma = (torch.fft.irfft(f, n=n, dim=2) * (2.0 * n ** 3 / len(masks))).reshape(-1)
        del f
        u = _wrapped(case, pos)
        ax = [_stencil(case["order"], u[:, a] + (0.5 if mask >> a & 1 else 0.0)) for a in range(3)]
        for a in range(case["order"]):
            for b in range(case["order"]):
                row = (torch.remainder(ax[0][0] + a, n) * n + torch.remainder(ax[1][0] + b, n)) * n
                for d in range(case["order"]):
                    v = gamma[row + torch.remainder(ax[2][0] + d, n)]
                    (x, dx), (y, dy), (z, dz) = ((ax[i][1][q], ax[i][2][q]) for i, q in enumerate((a, b, d)))
                    grad[:, 0] += v * dx * y * z
                    grad[:, 1] += v * x * dy * z
                    grad[:, 2] += v * x * y * dz
    grad *= n / case["box"]
    if w is not None:
        grad *= w.double()[:, None]
    return {"p": p[None], "loss": ((p - t) ** 2 / s2).sum(), "grad": grad}


def _exact_bispectrum(case, seed):
    pos, w = _positions(case, seed)
    n, dk, nb = case["n_grid"], case["n_dk"], case["n_bins"]
    k, p, n_b, c, total, _ = _power(case, pos, w)
    wx, wy, wz = _window(case)
    c /= total * wx * wy * wz
    shell = torch.cat([_bins_of(n, dk, nb)[m2] for _, _, m2, _ in _planes(n, _step(n))])
    sums = []
    for data in (True, False):
        fields = torch.empty((nb, n ** 3), device=DEVICE, dtype=torch.float64)
        for b in range(nb):
            modes = torch.where(shell == b + 1, c if data else 1.0, 0.0).to(torch.complex128)
            fields[b] = (torch.fft.irfftn(modes, s=(n, n, n)) * n ** 3).reshape(-1)
        t = torch.zeros((nb, nb, nb), device=DEVICE, dtype=torch.float64)
        for at in range(0, n ** 3, 1 << 21):
            part = fields[:, at:at + (1 << 21)]
            right = part.T.contiguous()
            for b in range(nb):
                t[b, :b + 1] += (part[:b + 1] * part[b]) @ right
        sums.append(t)
    tri = torch.as_tensor(_triangles(nb), device=DEVICE).long() - 1
    i, j = (t[tri[:, 0], tri[:, 1], tri[:, 2]] for t in sums)
    bk = torch.where(j > 0.5, case["box"] ** 6 * i / j, torch.full_like(i, float("nan")))
    return {"k": k[None], "p": p[None], "modes": n_b[None], "b": bk, "n_tri": (j / n ** 3).round()}


def _exact_direct(case, seed):
    pos, w = _positions(case, seed)
    n, dk, nb, vol = case["n_grid"], case["n_dk"], case["n_bins"], case["box"] ** 3
    half = n // 2 + 1
    ds = torch.zeros((n * n, half), device=DEVICE, dtype=torch.complex128)
    m = _signed(n).double()
    for j0 in range(0, pos.shape[0], 4096):
        x = torch.remainder(pos[j0:j0 + 4096].double(), case["box"]) / case["box"]
        ex, ey = (torch.exp(-2j * math.pi * m[:, None] * x[None, :, a]) for a in (0, 1))
        ez = torch.exp(-2j * math.pi * torch.arange(half, device=DEVICE, dtype=torch.float64)[None, :] * x[:, 2, None])
        if w is not None:
            ez = ez * w[j0:j0 + 4096].double()[:, None]
        ds += (ex[:, None, :] * ey[None, :, :]).reshape(n * n, -1) @ ez
    _, _, n_b, c, total, _ = _power(case, pos, w)
    ds = (ds / total).reshape(n, n, half)
    wx, wy, wz = _window(case)
    dg = c / (total * wx * wy * wz)
    _, k = _shells(n, dk, nb, case["box"])
    p_ds = vol * _shell_sums(n, dk, nb, lambda x0, x1, m2: ds[x0:x1].abs() ** 2) / n_b
    p_x = vol * _shell_sums(n, dk, nb, lambda x0, x1, m2: (dg[x0:x1] * ds[x0:x1].conj()).real) / n_b
    return {"delta_ds": torch.view_as_real(ds), "delta_g": torch.view_as_real(dg), "k": k, "p_ds": p_ds, "p_x": p_x, "modes": n_b}


def exact(case, seed):
    if case["n"] * 2.0 ** case["interlace"] * case["order"] ** 3 > 2.0e10:
        return None
    return {"power": _exact_power, "replay": _exact_power, "grad": _exact_grad, "bispectrum": _exact_bispectrum,
            "direct": _exact_direct}[case["kind"]](case, seed)
