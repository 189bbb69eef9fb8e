"""The work that a user of this framework has it do, as cases that can be timed and compared.

A case is a dict of plain values.  `prepare` makes its inputs on the GPU from a seed, `run` is one pass through the
public entry points, `work` what a pass cannot do without, and `exact` the same results in 64 bits from the method's
definitions alone (plain torch, nothing of this package).

Fields are Gaussian with two correlation lengths blended across the grid; masks are cloud-like blobs topped up by
single pixels, or single pixels only, as in the configurations of `paper_2212_01317_amd.synth`; values under a gap are
NaN.  Temperatures that a case hands over itself are log-uniform in the range that calibration finds on such fields.
"""
from __future__ import annotations

import math

import torch

import paper_2212_01317_amd as mpr

DEV = "cuda"


def listed():
    return [
        # The smallest problem: plain MPR on 128 x 128, one global temperature, 10 chains, 100 + 100 sweeps.
        dict(name="predict_128", kind="plane", call="predict", form="block", H=128, W=128, p=0.33, blobs=0.0, R=10,
             lb_h=128, lb_w=128, start="mean", stop="fixed", n_eq=100, n_max=100, n_samp=100),
        # One prediction of the validation procedure on the smallest map (256 x 256, 30 % removed, automatic stop).
        dict(name="predict_256_auto", kind="plane", call="predict", form="block", H=256, W=256, p=0.3, blobs=0.0, R=10,
             lb_h=32, lb_w=32, start="mean", stop="auto", n_eq=0, n_max=200, n_samp=1),
        # A map of odd sides with site-specific temperatures.
        dict(name="predict_sst_517x389", kind="plane", call="predict", form="site", H=517, W=389, p=0.5, blobs=0.5, R=16,
             lb_h=16, lb_w=16, start="mean", stop="auto", n_eq=0, n_max=60, n_samp=2),
        # The chains of a map of 1024 x 1024 with 100 realizations, 16 x 16 blocks, automatic stop.
        dict(name="simulate_1024_r100", kind="plane", call="simulate", form="block", H=1024, W=1024, p=0.5, blobs=0.5,
             R=100, lb_h=16, lb_w=16, start="mean", stop="auto", n_eq=0, n_max=30, n_samp=1),
        # Few chains on a large map: the validation procedure at 2048 x 2048 from the uniform start of plain MPR.
        dict(name="simulate_2048_r10", kind="plane", call="simulate", form="block", H=2048, W=2048, p=0.5, blobs=0.0,
             R=10, lb_h=32, lb_w=32, start="random", stop="fixed", n_eq=40, n_max=40, n_samp=1),
        # The largest plane: 4096 x 4096, 60 % gaps, mostly blobs, 32 x 32 blocks, 128 realizations.
        dict(name="simulate_4096_r128", kind="plane", call="simulate", form="block", H=4096, W=4096, p=0.6, blobs=0.8,
             R=128, lb_h=32, lb_w=32, start="mean", stop="fixed", n_eq=24, n_max=24, n_samp=1),
        # One temperature per bond direction, odd sides.
        dict(name="directional_701x903_r64", kind="plane", call="simulate", form="directional", H=701, W=903, p=0.4,
             blobs=0.0, R=64, lb_h=32, lb_w=32, start="mean", stop="fixed", n_eq=30, n_max=30, n_samp=1),
        # Many scenes of different sizes and gap fractions in one call, 64 realizations each, automatic stop.
        dict(name="batch_48_r64", kind="batch", n=48, side_lo=64, side_hi=1024, R=64, lb=16, n_max=60, n_samp=1),
        # Forward and backward through the temperatures: 512 x 512, 1024 realizations.
        dict(name="gradient_512_r1024", kind="gradient", H=512, W=512, p=0.5, blobs=0.5, R=1024, lb=32, n_eq=30),
        # The cubic lattice.
        dict(name="cube_160_r128", kind="cube", D=160, H=160, W=160, p=0.6, R=128, lb=32, stop="fixed", n_eq=15,
             n_max=15, n_samp=1),
        # The matching curve that each new q needs once: 121 temperatures on 128 x 128.
        dict(name="curve_121x128", kind="curve", dim=2, nT=121, L=128, n_therm=150, n_meas=300),
        # The steps around the chains on a large map: angles, block temperatures, their smoothing, prediction, errors.
        dict(name="steps_4096", kind="steps", H=4096, W=4096, p=0.6, blobs=0.8, lb_h=32, lb_w=32, r_s=1, n_s=5),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["plane", "plane", "plane", "plane", "sweep", "batch", "gradient", "cube", "curve", "steps"])
    p, blobs = round(rng.uniform(0.1, 0.9), 3), rng.choice([0.0, 0.5, 0.8])
    if kind == "plane":
        form = rng.choice(["block", "block", "block", "site", "dc", "directional"])
        H, W = _log(rng, 64, 2048), _log(rng, 64, 2048)
        R = max(2, min(_log(rng, 4, 256), int(4e8 / (H * W))))
        lb = rng.choice([8, 12, 16, 24, 32, 33, 64])
        n_eq = rng.randint(10, 60)
        return dict(kind="plane", call=rng.choice(["predict", "simulate"]), form=form, H=H, W=W, p=p, blobs=blobs, R=R,
                    lb_h=lb, lb_w=rng.choice([lb, 16]), start=rng.choice(["mean", "mean", "random"]),
                    stop=rng.choice(["fixed", "auto"]), n_eq=n_eq, n_max=max(n_eq, 25), n_samp=rng.randint(1, 4))
    if kind == "sweep":
        H, W = _log(rng, 64, 2048), _log(rng, 64, 2048)
        return dict(kind="sweep", H=H, W=W, p=p, blobs=blobs, R=max(1, min(_log(rng, 2, 128), int(2e8 / (H * W)))),
                    lb=rng.choice([8, 16, 32]), first=rng.randint(1, 500), n=rng.randint(1, 40),
                    energy=rng.choice([True, False]))
    if kind == "batch":
        lo = _log(rng, 48, 128)
        return dict(kind="batch", n=_log(rng, 4, 48), side_lo=lo, side_hi=rng.choice([256, 512, 1024]),
                    R=rng.choice([8, 10, 32, 64, 100]), lb=rng.choice([8, 16, 32]), n_max=rng.randint(25, 60),
                    n_samp=rng.randint(1, 2))
    if kind == "gradient":
        H, W = _log(rng, 64, 512), _log(rng, 64, 512)
        return dict(kind="gradient", H=H, W=W, p=p, blobs=blobs, R=_log(rng, 32, 1024), lb=rng.choice([16, 32]),
                    n_eq=rng.randint(10, 30))
    if kind == "cube":
        D, H, W = (_log(rng, 16, 160) for _ in range(3))
        n_eq = rng.randint(5, 15)
        return dict(kind="cube", D=D, H=H, W=W, p=p, R=_log(rng, 16, 128), lb=rng.choice([8, 16, 32]),
                    stop=rng.choice(["fixed", "auto"]), n_eq=n_eq, n_max=max(n_eq, 25), n_samp=1)
    if kind == "curve":
        dim = rng.choice([2, 2, 3])
        L = 2 * _log(rng, 8, 64) if dim == 2 else 2 * _log(rng, 4, 16)
        return dict(kind="curve", dim=dim, nT=_log(rng, 16, 121), L=L, n_therm=rng.randint(30, 150),
                    n_meas=rng.randint(30, 300))
    return dict(kind="steps", H=_log(rng, 128, 4096), W=_log(rng, 128, 4096), p=p, blobs=blobs,
                lb_h=rng.choice([8, 16, 32, 50]), lb_w=rng.choice([8, 16, 32, 50]), r_s=rng.choice([1, 2]),
                n_s=rng.randint(1, 5))


# ---- inputs ----

def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _gauss(shape, xi, g):
    """Standardised Gaussian field whose spectrum is that of the covariance exp(-r / xi), cut from a periodic one whose
    sides are powers of two."""
    k2, torus = 0.0, [1 << max(4, (n - 1).bit_length()) for n in shape]
    for d, n in enumerate(torus):
        f = 2 * math.pi * torch.fft.fftfreq(n, device=DEV)
        k2 = k2 + f.reshape([-1 if i == d else 1 for i in range(len(shape))]) ** 2
    amp = (1.0 + xi * xi * k2) ** (-(len(shape) + 1) / 4)
    f = torch.fft.ifftn(torch.fft.fftn(torch.randn(torus, device=DEV, generator=g)) * amp).real
    f = f[tuple(slice(0, n) for n in shape)]
    return ((f - f.mean()) / f.std()).contiguous()


def _map(shape, p, blobs, g):
    """(field with NaN under the gaps, the full field, mask: 1 = sample)."""
    w = torch.linspace(0, 1, shape[-1], device=DEV)
    full = ((1 - w) * _gauss(shape, 3.0, g) + w * _gauss(shape, 16.0, g)).float().contiguous()
    n = full.numel()
    gap = torch.zeros(n, dtype=torch.bool, device=DEV)
    total, cloud = int(round(p * n)), int(round(p * blobs * n))
    if cloud:
        gap[_gauss(shape, 24.0, g).reshape(-1).argsort()[:cloud]] = True
    rank = torch.rand(n, device=DEV, generator=g)
    rank[gap] = -1.0
    gap[rank.argsort()[:total]] = True
    mask = (~gap).to(torch.uint8).reshape(shape).contiguous()
    z = full.clone()
    z[gap.reshape(shape)] = math.nan
    return z, full, mask


def _temps(count, g):
    lo, hi = math.log(0.015), math.log(0.3)
    return torch.exp(lo + (hi - lo) * torch.rand(count, device=DEV, generator=g))


def _curve():
    """A monotone matching curve: the energy per bond of the planar rotator chain, 121 temperatures in [1e-3, 1e2]."""
    T = 10.0 ** (torch.arange(121, device=DEV, dtype=torch.float64) / 24 - 3)
    return T, -torch.special.i1e(1 / T) / torch.special.i0e(1 / T)


def _angles(z, mask):
    v = torch.where(mask > 0, z.double(), torch.zeros((), dtype=torch.float64, device=DEV))
    lo, hi = (z[mask > 0].min().double(), z[mask > 0].max().double())
    t = torch.where(mask > 0, (v - lo) / (hi - lo), torch.zeros_like(v))
    return t.float().contiguous(), torch.stack([lo, hi])


def _nb(n, lb):
    return -(-n // lb)


def _sides(case):
    """(H, W, gap fraction, share of blobs) of the scenes of a batch: the same for every seed."""
    r = torch.rand((case["n"], 4), generator=torch.Generator().manual_seed(case["n"]), dtype=torch.float64).tolist()
    side = lambda u: int(round(case["side_lo"] * (case["side_hi"] / case["side_lo"]) ** u))
    return [(side(a), side(b), 0.1 + 0.8 * c, 0.0 if d < 0.5 else 1.0) for a, b, c, d in r]


def _config(case, seed, **kw):
    auto = case.get("stop", "auto") == "auto"
    form = case.get("form", "block")
    base = dict(n_real=case["R"], seed=int(seed) * 7919 + 17, scene_id=5,
                stop_mode=mpr.STOP_AUTO if auto else mpr.STOP_FIXED, n_eq=case.get("n_eq", 0),
                n_max=case.get("n_max", 1), n_samp=case.get("n_samp", 1),
                init_mode=mpr.INIT_RANDOM if case.get("start") == "random" else mpr.INIT_BLOCK_MEAN,
                t_mode=mpr.T_SITE if form == "site" else mpr.T_BLOCK,
                order=mpr.ORDER_DC if form == "dc" else mpr.ORDER_SC,
                coupling=mpr.COUPLING_DIRECTIONAL if form == "directional" else mpr.COUPLING_ISOTROPIC)
    return {**base, **kw}


def prepare(case, seed):
    g, kind = _gen(seed), case["kind"]
    s = dict(case=case, seed=seed)
    if kind == "curve":
        s["T"] = torch.exp(torch.linspace(math.log(1e-3), math.log(1e2), case["nT"], device=DEV)).float().contiguous()
        return s
    if kind == "batch":
        scenes = []
        for i, (H, W, p, blobs) in enumerate(_sides(case)):
            z, _, mask = _map((H, W), p, blobs, g)
            T = _temps(_nb(H, case["lb"]) * _nb(W, case["lb"]), g)
            scenes.append(dict(t=_angles(z, mask)[0], mask=mask, T_blocks=T, block=(case["lb"], case["lb"]), scene_id=i))
        s.update(scenes=scenes, cfg=_config(case, seed, scene_id=0))
        return s
    shape = (case["D"], case["H"], case["W"]) if kind == "cube" else (case["H"], case["W"])
    z, full, mask = _map(shape, case["p"], case.get("blobs", 0.0), g)
    s.update(z=z, full=full, mask=mask, curve=_curve(), ev=(1 - mask).contiguous())
    s["t"], s["range"] = _angles(z, mask)
    lb = [case.get("lb_h", case.get("lb")), case.get("lb_w", case.get("lb"))]
    if kind == "cube":
        lb = [case["lb"]] + lb
    B = math.prod(_nb(n, b) for n, b in zip(shape, lb))
    form = case.get("form", "block")
    s["lb"] = lb
    s["Tb"] = _temps(z.numel() if form == "site" else 2 * B if form == "directional" else B, g)
    if kind == "gradient":
        s["Tb"] = s["Tb"].reshape(_nb(shape[0], lb[0]), _nb(shape[1], lb[1])).requires_grad_()
        s["gz"] = torch.randn(shape, device=DEV, generator=g)
    if kind == "sweep":
        r = (torch.rand((case["R"],) + shape, device=DEV, generator=g) * 16777216).floor().clamp(max=16777215) / 16777216
        s["state"] = torch.where(mask > 0, s["t"], r).contiguous()
        s["alt"] = s["state"].clone()
    if kind == "steps":
        s["acc"] = torch.where(mask > 0, 0.0, 40 * torch.rand(shape, device=DEV, generator=g, dtype=torch.float64))
    if kind in ("plane", "cube", "sweep", "gradient"):
        s["cfg"] = _config(case, seed)
        if kind == "gradient":
            s["cfg"].update(stop_mode=mpr.STOP_FIXED)
    return s


# ---- one pass ----

def _sim(o, s):
    """The energy series only after a fixed number of sweeps: under the automatic stop its length is `sweeps` + 1."""
    fixed = s["cfg"]["stop_mode"] == mpr.STOP_FIXED
    return dict(state=o.state, acc=o.acc, sweeps=o.sweeps, **({"energy": o.energy} if fixed else {}))


def run(s):
    c, kind = s["case"], s["case"]["kind"]
    if kind == "plane" and c["call"] == "predict":
        k = {x: s["cfg"][x] for x in ("init_mode", "stop_mode", "n_eq", "n_samp", "n_max", "seed", "scene_id", "order")}
        o = mpr.predict(s["z"], s["mask"], tuple(s["lb"]), c["R"], curve=s["curve"],
                        sst=(1, 5) if c["form"] == "site" else None, directional=c["form"] == "directional", **k)
        return dict(zhat=o.zhat, T=o.T, **_sim(o.sim, s))
    if kind == "plane":
        return _sim(mpr.mpr_simulate(s["t"], s["mask"], s["Tb"], *s["lb"], mpr.SimConfig(**s["cfg"])), s)
    if kind == "sweep":
        # the chains go on in a copy, so that the saved state can be resumed again
        st = s["state"].clone()
        e = mpr.mpr_sweep(st, s["mask"], s["Tb"], *s["lb"], mpr.SimConfig(**s["cfg"]), c["first"], c["n"],
                          want_energy=c["energy"], state_alt=s["alt"])
        return dict(state=st, energy=e)
    if kind == "batch":
        o = mpr.mpr_simulate_batched(s["scenes"], mpr.SimConfig(**s["cfg"]), want_energy=False)
        return dict(acc=torch.cat([x.acc.reshape(-1) for x in o.outputs]),
                    state=torch.cat([x.state.reshape(-1) for x in o.outputs]), sweeps=[float(x.sweeps) for x in o.outputs])
    if kind == "gradient":
        s["Tb"].grad = None
        zhat = mpr.MPRFunction.apply(s["Tb"], s["t"], s["mask"], s["full"], s["range"], tuple(s["lb"]),
                                     mpr.SimConfig(**s["cfg"]))
        zhat.backward(s["gz"])
        return dict(zhat=zhat, grad=s["Tb"].grad)
    if kind == "cube":
        return _sim(mpr.mpr_simulate3d(s["t"], s["mask"], s["Tb"], *s["lb"], mpr.SimConfig(**s["cfg"])), s)
    if kind == "curve":
        f = mpr.mpr_reference_curve if c["dim"] == 2 else mpr.mpr_reference_curve3d
        return dict(e=f(s["T"], L=c["L"], n_therm=c["n_therm"], n_meas=c["n_meas"], seed=int(s["seed"]) + 3))
    t, rng = mpr.mpr_map_angles(s["z"], s["mask"])
    T, e, nb = mpr.mpr_calibrate_temperature(t, s["mask"], *s["lb"], *s["curve"])
    Ts = mpr.mpr_sst_temperatures(T, c["H"], c["W"], *s["lb"], c["r_s"], c["n_s"])
    zhat = mpr.mpr_predict(s["acc"], s["z"], s["mask"], 40, rng)
    return dict(t=t, range=rng, T=T, e=e, n=nb, Ts=Ts, zhat=zhat, err=mpr.mpr_validate(zhat, s["full"], s["ev"]))


def work(case):
    """An update takes about 55 operations (half a Philox block, two uniforms, cos and sin of the proposal, the field
    of the neighbours, the Boltzmann test), a site of a chain 10 a sweep; an automatic stop runs 25 sweeps at least."""
    kind = case["kind"]
    if kind == "steps":
        n = case["H"] * case["W"]
        return dict(bytes=n * (4 + 1 + 4 + 8 + 4 + 4 + 4 + 1), flops=n * (40 + 9 * case["n_s"]))
    if kind == "curve":
        n = case["nT"] * case["L"] ** case["dim"]
        return dict(bytes=12 * case["nT"], flops=n * (65 * (case["n_therm"] + case["n_meas"]) + 8 * case["n_meas"]))
    if kind == "batch":
        u = math.log(case["side_hi"] / case["side_lo"])
        n, p = case["n"] * ((case["side_hi"] - case["side_lo"]) / u) ** 2, 0.5
        sweeps = 25 + case["n_samp"]
    else:
        n, p = case.get("D", 1) * case["H"] * case["W"], case["p"]
        sweeps = (case["n"] if kind == "sweep" else
                  (25 if case.get("stop") == "auto" else case["n_eq"]) + case.get("n_samp", 1))
    R = case["R"]
    out = 4 * R if kind != "gradient" else 4
    read = 4 * R if kind == "sweep" else 5
    return dict(bytes=n * (out + read + 8), flops=n * R * sweeps * (55 * p + 10))


# ---- the same in 64 bits, from the definitions ----

_M0, _M1, _LOW = 0xD2511F53, 0xCD9E8D57, 0xFFFFFFFF


def _philox(c0, c1, c2, c3, seed):
    k0, k1 = seed & _LOW, (seed >> 32) & _LOW
    for _ in range(10):
        a, b = c0 * _M0, c2 * _M1          # modulo 2^64: both halves of the product
        c0, c1, c2, c3 = ((b >> 32) & _LOW) ^ c1 ^ k0, b & _LOW, ((a >> 32) & _LOW) ^ c3 ^ k1, a & _LOW
        k0, k1 = (k0 + 0x9E3779B9) & _LOW, (k1 + 0xBB67AE85) & _LOW
    return c0, c1, c2, c3


class _Lattice:
    """Chains on a grid of two or three dimensions in float64: the single and the double checkerboard order."""

    def __init__(self, shape, R, seed, scene, tag=0, q=0.5, periodic=False, offset=0):
        self.shape, self.R, self.seed, self.w3, self.q, self.periodic = shape, R, seed, scene << 4, q, periodic
        ix = [torch.arange(n, device=DEV).reshape([-1 if i == d else 1 for i in range(len(shape))])
              for d, n in enumerate(shape)]
        self.col = sum(ix) % 2 + torch.zeros(shape, dtype=torch.int64, device=DEV)
        rows = ix[0] if len(shape) == 2 else ix[0] * shape[1] + ix[1]
        Mw = -(-shape[-1] // 4)
        self.pair = (rows * Mw + torch.arange(Mw, device=DEV)).unsqueeze(0)
        self.real = (offset + torch.arange(R, device=DEV)).reshape([-1] + [1] * len(shape))
        self.second = ((ix[-1] >> 1) & 1).bool().unsqueeze(0)
        self.bonds = [(d, n) for d, n in enumerate(shape)]
        self.tag = tag

    def uniforms(self, sweep, colour):
        w = _philox(self.pair + 0 * self.real, torch.full_like(self.pair, sweep), self.real + 0 * self.pair,
                    torch.full_like(self.pair, self.w3 | self.tag << 1 | colour), self.seed)
        W = self.shape[-1]
        up = [torch.repeat_interleave(x >> 8, 4, dim=-1)[..., :W] for x in w]
        return tuple(torch.where(self.second, up[i + 2], up[i]).double() * 2.0 ** -24 for i in (0, 1))

    def neighbours(self, st):
        for d, n in self.bonds:
            for sh in (1, -1):
                nb = torch.roll(st, sh, d + 1)
                if self.periodic:
                    yield d, nb, 1.0
                    continue
                ok = torch.ones(n, device=DEV, dtype=torch.float64)
                ok[0 if sh == 1 else -1] = 0
                yield d, nb, ok.reshape([1] + [-1 if i == d else 1 for i in range(len(self.shape))])

    def phase(self, st, sweep, colour, where, T):
        """One colour; T: one temperature for all bonds, or (vertical, horizontal)."""
        u1, u2 = self.uniforms(sweep, colour)
        a = [0.0, 0.0]
        for d, nb, ok in self.neighbours(st):
            k = 2 * math.pi * self.q
            i = 1 if isinstance(T, tuple) and d == 1 else 0
            a[i] = a[i] + ok * (torch.cos(k * (u1 - nb)) - torch.cos(k * (st - nb)))
        if isinstance(T, tuple):
            take = u2 < torch.exp(a[0] / T[0] + a[1] / T[1])
        else:
            a = a[0]
            take = torch.where(T > 0, u2 < torch.exp(a / torch.where(T > 0, T, 1.0)), a >= 0)
        return torch.where(take & where & (self.col == colour), u1, st)

    def sweep(self, st, k, free, T, parity=None):
        for half in (None,) if parity is None else (0, 1):
            for colour in (0, 1):
                st = self.phase(st, k, colour, free if half is None else free & (parity == half), T)
        return st

    def energy(self, st):
        """Mean energy per bond of each chain."""
        tot, count = 0.0, 0
        for d, n in self.bonds:
            e = -torch.cos(2 * math.pi * self.q * (st - torch.roll(st, -1, d + 1)))
            e = e if self.periodic else e.narrow(d + 1, 0, n - 1)
            tot, count = tot + e.flatten(1).sum(1), count + e[0].numel()
        return tot / count


def _block_of(shape, lb):
    b = 0
    for d, (n, l) in enumerate(zip(shape, lb)):
        b = b * _nb(n, l) + (torch.arange(n, device=DEV) // l).reshape([-1 if i == d else 1 for i in range(len(shape))])
    return b + torch.zeros(shape, dtype=torch.int64, device=DEV)


def _sum_by(block, v, count):
    return torch.zeros(count, dtype=torch.float64, device=DEV).index_add_(0, block.reshape(-1), v.double().reshape(-1))


def _stats(t, mask, lb, dims):
    """(sum of the bond energies of samples, their number) per block, over the bonds along `dims`; owner: lower index."""
    block, t, m = _block_of(t.shape, lb), t.double(), mask > 0
    count = math.prod(_nb(n, l) for n, l in zip(t.shape, lb))
    S = N = 0.0
    for d in dims:
        ok = m & torch.roll(m, -1, d)
        ok.narrow(d, t.shape[d] - 1, 1).zero_()
        S = S + _sum_by(block, torch.where(ok, -torch.cos(math.pi * (t - torch.roll(t, -1, d))), 0.0), count)
        N = N + _sum_by(block, ok, count)
    return S, N


def _match(S, N, curve):
    """Block temperatures from the matching curve, blocks without bonds take the median."""
    cT, ce = curve
    e = torch.where(N > 0, S / N.clamp(min=1), 0.0)
    up = torch.cummax(ce, 0).values
    i = torch.searchsorted(up, e).clamp(max=len(up))
    j = i.clamp(1, len(up) - 1)
    lam = (e - up[j - 1]) / (up[j] - up[j - 1])
    T = torch.exp((1 - lam) * torch.log(cT[j - 1]) + lam * torch.log(cT[j]))
    T = torch.where(i == 0, cT[0] * (e + 1) / (ce[0] + 1), torch.where(i == len(up), cT[-1], T))
    T = torch.where(e <= -1, 0.0, T).float()
    have = T[N > 0].sort().values
    mid = (have[(len(have) - 1) // 2].double() + have[len(have) // 2].double()) * 0.5
    return torch.where(N > 0, T, mid.float()), e


def _smooth(T, shape, lb, r, passes):
    a = T.double().reshape(-1)[_block_of(shape, lb)]
    pad = lambda x: torch.nn.functional.pad(x, (r, r, r, r))
    for _ in range(passes):
        b, n, s, m = pad(a), pad(torch.ones_like(a)), 0.0, 0.0
        for dy in range(2 * r + 1):
            for dx in range(2 * r + 1):
                s = s + b[dy:dy + shape[0], dx:dx + shape[1]]
                m = m + n[dy:dy + shape[0], dx:dx + shape[1]]
        a = s / m
    return a.float()


def _start(t, mask, lb, R, random, lat):
    if random:
        lat.tag = 1
        u = [lat.uniforms(0, c)[0] for c in (0, 1)]
        lat.tag = 0
        g = torch.where(lat.col == 0, u[0], u[1])
    else:
        block = _block_of(t.shape, lb)
        count = math.prod(_nb(n, l) for n, l in zip(t.shape, lb))
        S, N = _sum_by(block, t * (mask > 0), count), _sum_by(block, mask, count)
        g = torch.where(N > 0, S / N.clamp(min=1), S.sum() / N.sum()).float().double()[block].unsqueeze(0)
    return torch.where(mask > 0, t.double(), g).expand((R,) + t.shape)


def _chains(t, mask, lb, T, cfg, parity=None):
    """Start, sweeps up to the stop, sampling: dict(state, acc, energy, sweeps)."""
    R, free = cfg["n_real"], mask == 0
    lat = _Lattice(tuple(t.shape), R, cfg["seed"], cfg["scene_id"])
    st = _start(t, mask, lb, R, cfg["init_mode"] == mpr.INIT_RANDOM, lat)
    auto = cfg["stop_mode"] == mpr.STOP_AUTO
    e, k = [float(lat.energy(st).mean())], 0
    while k < (cfg["n_max"] if auto else cfg["n_eq"]):
        k += 1
        st = lat.sweep(st, k, free, T, parity)
        e.append(float(lat.energy(st).mean()))
        if auto and k >= 25 and k % 5 == 0:
            x = torch.arange(20, dtype=torch.float64) - 9.5
            slope = float((x * torch.tensor(e[-20:], dtype=torch.float64)).sum())
            if slope * (e[-1] - e[0]) <= 0:
                break
    acc = torch.zeros(t.shape, dtype=torch.float64, device=DEV)
    for i in range(cfg["n_samp"]):
        st = lat.sweep(st, k + 1 + i, free, T, parity)
        acc = acc + torch.where(free, st.sum(0), 0.0)
    return dict(state=st, acc=acc, sweeps=None, **({} if auto else {"energy": torch.tensor(e, dtype=torch.float64)}))


def exact(case, seed):
    kind = case["kind"]
    n = case.get("D", 1) * case.get("H", 1) * case.get("W", 1)
    cost = n * case.get("R", 0) * (max(case.get("n_eq", 0), case.get("n_max", 0)) + case.get("n_samp", 1))
    if kind == "batch":
        cost = sum(h * w for h, w, _, _ in _sides(case)) * case["R"] * (case["n_max"] + case["n_samp"])
    if kind == "sweep":
        cost = n * case["R"] * case["n"]
    if cost > 3e9 or (kind == "batch" and case["n"] > 12):
        return None
    with torch.no_grad():
        return _exact(prepare(case, seed))


def _exact(s):
    c, kind = s["case"], s["case"]["kind"]
    if kind == "curve":
        lat = _Lattice((c["L"],) * c["dim"], c["nT"], int(s["seed"]) + 3, 0, tag=2, periodic=True)
        T = s["T"].double().reshape([-1] + [1] * c["dim"])
        st = torch.full((c["nT"],) + lat.shape, 0.5, dtype=torch.float64, device=DEV)
        free, e = torch.ones(lat.shape, dtype=torch.bool, device=DEV), 0.0
        for k in range(1, c["n_therm"] + c["n_meas"] + 1):
            st = lat.sweep(st, k, free, T)
            if k > c["n_therm"]:
                e = e + lat.energy(st)
        return dict(e=e / c["n_meas"])
    if kind == "batch":
        got = [_chains(x["t"], x["mask"], x["block"], x["T_blocks"].double()[_block_of(x["t"].shape, x["block"])],
                       {**s["cfg"], "scene_id": x["scene_id"]}) for x in s["scenes"]]
        return dict(acc=torch.cat([x["acc"].reshape(-1) for x in got]),
                    state=torch.cat([x["state"].reshape(-1) for x in got]), sweeps=[None] * len(got))
    shape, lb, t, mask = tuple(s["mask"].shape), s["lb"], s["t"], s["mask"]
    block = _block_of(shape, lb)
    if kind == "steps":
        T, e = _match(*_stats(t, mask, lb, (0, 1)), s["curve"])
        zhat = torch.where(mask > 0, s["z"].double(), s["range"][0] + (s["range"][1] - s["range"][0]) * s["acc"] / 40)
        d = (s["full"].double() - zhat.float().double())[mask == 0]
        v = torch.where(mask > 0, s["z"].double(), s["range"][0])
        nby = (_nb(shape[0], lb[0]), _nb(shape[1], lb[1]))
        return dict(t=(v - s["range"][0]) / (s["range"][1] - s["range"][0]), range=s["range"], T=T.double().reshape(nby),
                    e=e.reshape(nby), n=None, Ts=_smooth(T, shape, lb, c["r_s"], c["n_s"]).double(), zhat=zhat,
                    err=torch.stack([d.abs().mean(), d.square().mean().sqrt()]) if len(d) else torch.zeros(2))
    form, Tb = c.get("form", "block"), s["Tb"].detach()
    out, parity = {}, None
    if kind == "plane" and c["call"] == "predict":
        if form == "directional":
            Tb = torch.stack([_match(*_stats(t, mask, lb, (d,)), s["curve"])[0] for d in (1, 0)]).clamp(min=1e-3)
        else:
            Tb = _match(*_stats(t, mask, lb, (0, 1)), s["curve"])[0]
        if form == "site":
            Tb = _smooth(Tb, shape, lb, 1, 5)
        nby = (_nb(shape[0], lb[0]), _nb(shape[1], lb[1]))
        out["T"] = Tb.double().reshape(shape if form == "site" else (2,) + nby if form == "directional" else nby)
    if form == "directional":
        Tx, Ty = Tb.double().reshape(2, -1).clamp(min=float(torch.tensor(1e-3))).unbind()
        T = (Ty[block], Tx[block])
    else:
        T = Tb.double().reshape(shape) if form == "site" else Tb.double().reshape(-1)[block]
    if form == "dc":
        parity = (torch.arange(shape[0], device=DEV)[:, None] // lb[0] + torch.arange(shape[1], device=DEV) // lb[1]) % 2
    if kind == "sweep":
        lat, st, e = _Lattice(shape, c["R"], s["cfg"]["seed"], s["cfg"]["scene_id"]), s["state"].double(), []
        for k in range(c["first"], c["first"] + c["n"]):
            st = lat.sweep(st, k, mask == 0, T)
            e.append(float(lat.energy(st).mean()))
        return dict(state=st, energy=torch.tensor(e, dtype=torch.float64) if c["energy"] else None)
    got = _chains(t, mask, lb, T, s["cfg"], parity)
    if kind == "cube" or (kind == "plane" and c["call"] == "simulate"):
        return got
    lo, span = s["range"][0], s["range"][1] - s["range"][0]
    mean = got["acc"] / (c["R"] * s["cfg"]["n_samp"])
    zhat = torch.where(mask > 0, s["full"].double(), lo + span * mean)
    if kind == "plane":
        return dict(zhat=zhat, **out, **got)
    # the gradient: covariance over the chains of sum(gz dz/dt t) and each block's energy, over T^2
    st, free = got["state"], mask == 0
    f = (torch.where(free, s["gz"].double() * span, 0.0) * st).flatten(1).sum(1)
    site = torch.zeros_like(st)
    lat = _Lattice(shape, c["R"], 0, 0)
    fz = free.double().unsqueeze(0)
    for (d, nb, ok), (_, other, _) in zip(lat.neighbours(st), lat.neighbours(fz)):
        site = site - ok * (1 - 0.5 * other) * torch.cos(math.pi * (st - nb))
    site = torch.where(free, site, 0.0).flatten(1)
    B = s["Tb"].numel()
    Hb = torch.zeros((c["R"], B), dtype=torch.float64, device=DEV).index_add_(1, block.reshape(-1), site)
    cov = ((f - f.mean())[:, None] * (Hb - Hb.mean(0))).sum(0) / (c["R"] - 1)
    return dict(zhat=zhat, grad=(cov / s["Tb"].detach().double().reshape(-1) ** 2).reshape(s["Tb"].shape))
