"""Performance cases of the QED step: what a particle-in-cell or Monte Carlo program has it do.

Each case is one pass of such a program's time loop, or one call of the batched functions, over
the sizes the library is used at: tiles of a thousand particles (where latency and launches
count), the 65,536 electrons of the paper-like run, and 2^24 + 2^24 particles; FP64 and MIXED,
optical-depth and local decisions, fields as arrays, as a plane wave or uniform, with and
without the fused push, beyond-LCFA leptons, plans replayed from a graph, and the batched chi,
rate and sampling calls.  Particles live in one structure of arrays per program, tiles are
slices of it (so a tile starts wherever the previous one ended).

exact() gives the same results from quadrature in 64 bits, written here from the formulas of
the paper (arXiv:2301.07684) with plain torch.
"""
import math
import random

import numpy as np
import torch

DEV = torch.device("cuda", 0) if torch.cuda.is_available() else torch.device("cpu")
F8 = dict(dtype=torch.float64, device=DEV)

# laser wavelength 0.8 um, time step 0.01 fs, CODATA 2018
OMEGA_R = 2.0 * math.pi * 299792458.0 / 0.8e-6
LAMBDA_R = 299792458.0 / OMEGA_R
DT = 1e-17 * OMEGA_R
LC = 3.8615926796e-13 / LAMBDA_R
K_RATE = 7.2973525693e-3 / (math.sqrt(3.0) * math.pi) / LC
GAMMA_10GEV = 1.0e4 / 0.51099895

ELECTRON, POSITRON, PHOTON = 0, 1, 2
UID0 = 1 << 40
MADE, MADE_ARRAYS = ("photons", "electrons", "positrons"), ("px", "py", "pz", "tau", "uid", "parent")

# fractions of the leptons that emit and of the photons that convert in a first step
EVENTS = {"wave": (0.042, 0.0033), "wave_fields": (0.042, 0.0033), "skew": (0.17, 0.088),
          "static": (0.13, 0.03), "uniform": (0.003, 0.0)}


def _step(name, electrons, photons, geometry, precision="fp64", decision="depth", push=False,
          trunc=False, entry="step", products=False):
    return dict(name=name, kind="step", electrons=electrons, photons=photons, geometry=geometry,
                precision=precision, decision=decision, push=push, trunc=trunc, entry=entry,
                products=products)


def listed():
    return [
        # the smallest tile of a particle-in-cell code, stepped by itself: latency and launches
        _step("step_1k", 1003, 997, "static"),
        # 65,536 electrons in a static field, the paper-like run
        _step("step_64k", 65536, 0, "static"),
        # a mid-sized step whose program merges the products in a reproducible order (by parent)
        _step("step_merge_500k", 262144, 240001, "wave", decision="local", products=True),
        # the large FP64 step: 2^24 electrons meeting a plane wave, and as many photons
        _step("step_32m", 1 << 24, 1 << 24, "wave"),
        # the MIXED form where chi spreads over seven decades and emitters are dense; ragged
        _step("step_skew_4m", 2000003, 2000003, "skew", precision="mixed"),
        # fields given as the wave they come from, electrons pushed inside the step
        _step("step_push_wave_6m", 3000017, 3000000, "wave_fields", push=True),
        # validation set-up: 10 GeV electrons in a constant, uniform field, pushed in the step
        _step("step_uniform_16m", 1 << 24, 0, "uniform", push=True),
        # 64 uneven tiles of all species, MIXED, one graph replay per step
        dict(name="tiles_64", kind="tiles", tiles=64, smallest=1000, largest=1000000, layout=104,
             precision="mixed"),
        # one batch of a serving loop: beyond-LCFA electrons and photons of several simulations
        dict(name="served_6", kind="served", sims=6, smallest=200000, largest=2000000, layout=7,
             precision="mixed"),
        # particle loading and diagnostics through the batched calls
        dict(name="load_3m", kind="load", n=3000017, species=PHOTON, precision="fp64"),
        # energies for a program that makes its own decisions
        dict(name="photons_1m", kind="photons", n=1000003, precision="fp64", chi_lo=1e-3,
             chi_hi=1e2),
        dict(name="pairs_250k", kind="pairs", n=250007, precision="mixed", chi_lo=0.05,
             chi_hi=1e3),
    ]


def _size(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step"] * 6 + ["tiles", "served", "load", "photons", "pairs"])
    precision = rng.choice(["fp64", "mixed"])
    if kind == "step":
        geometry = rng.choice(["wave", "wave", "wave_fields", "skew", "static", "uniform"])
        electrons = _size(rng, 1000, 1 << 23)
        photons = 0 if geometry == "uniform" or rng.random() < 0.3 else _size(rng, 1000, 1 << 22)
        push = geometry in ("uniform", "wave_fields") or rng.random() < 0.3
        c = _step("", electrons, photons, geometry, precision,
                  rng.choice(["depth", "depth", "local"]), push, rng.random() < 0.15,
                  rng.choice(["step", "step", "step", "plan", "noalloc"]),
                  electrons + photons < 1000000 and rng.random() < 0.2)
        del c["name"]
        return c
    if kind == "tiles":
        return dict(kind=kind, tiles=rng.randint(2, 96), smallest=1000,
                    largest=_size(rng, 4000, 1000000), layout=rng.randint(1, 999),
                    precision=precision)
    if kind == "served":
        return dict(kind=kind, sims=rng.randint(1, 8), smallest=10000,
                    largest=_size(rng, 20000, 2000000), layout=rng.randint(1, 999),
                    precision=precision)
    if kind == "load":
        return dict(kind=kind, n=_size(rng, 1000, 6000000),
                    species=rng.choice([ELECTRON, POSITRON, PHOTON]), precision=precision)
    lo, hi = rng.choice([(1e-3, 1e2), (1e-4, 1e3)]) if kind == "photons" else (0.05, 1e3)
    return dict(kind=kind, n=_size(rng, 1000, 3000000), precision=precision, chi_lo=lo, chi_hi=hi)


# ---- inputs ---------------------------------------------------------------------------------------
class _Draws:
    """Uniform variates of one seed, on the device."""

    def __init__(self, seed):
        self.g = torch.Generator(device=DEV)
        self.g.manual_seed(int(seed))

    def u(self, n):
        return torch.rand(n, generator=self.g, **F8).clamp_(2.0 ** -53, 1.0 - 2.0 ** -53)

    def log_uniform(self, n, lo, hi):
        return torch.exp(math.log(lo) + math.log(hi / lo) * self.u(n))


def _layout(case):
    """[(species, n), ...]: the tiles of a case, in the order they lie in the arrays."""
    if case["kind"] == "step":
        tiles = [(ELECTRON, case["electrons"]), (PHOTON, case["photons"])]
        return [t for t in tiles if t[1] > 0]
    r = random.Random(case["layout"])
    if case["kind"] == "tiles":
        return [((ELECTRON, POSITRON, PHOTON)[k % 3],
                 _size(r, case["smallest"], case["largest"])) for k in range(case["tiles"])]
    out = []
    for _ in range(case["sims"]):
        n = _size(r, case["smallest"], case["largest"])
        out += [(ELECTRON, n // 2), (PHOTON, n - n // 2)]
    return out


def _geometry(case):
    return case["geometry"] if case["kind"] == "step" else \
        {"tiles": "static", "served": "wave_fields"}[case["kind"]]


def _particles(case, seed):
    """Momenta, fields, ids and species of a case's particles, as arrays over all its tiles."""
    tiles = _layout(case)
    n = sum(m for _, m in tiles)
    d = _Draws(seed)
    photon = torch.cat([torch.full((m,), sp == PHOTON, dtype=torch.bool, device=DEV)
                        for sp, m in tiles])
    z = torch.zeros(n, **F8)
    geometry = _geometry(case)
    if geometry == "uniform":
        gamma = torch.full((n,), GAMMA_10GEV, **F8)
    else:
        gamma = d.log_uniform(n, 1e2, 1e5)
    pm = torch.where(photon, gamma, torch.sqrt((gamma - 1.0) * (gamma + 1.0)))
    s = dict(tiles=tiles, n=n, photon=photon, wave=None,
             uid=torch.arange(UID0, UID0 + n, dtype=torch.int64, device=DEV))
    if geometry == "uniform":
        s["p"] = [pm, z.clone(), z.clone()]
        one = lambda v: torch.full((1,), v, **F8)
        b = 1.0 / (float(pm[0]) * LC)   # chi = 1
        s["E"], s["B"] = [one(0.0), one(0.0), one(0.0)], [one(0.0), one(0.0), one(b)]
        return s
    if geometry == "static":
        ct, ph = 2.0 * d.u(n) - 1.0, 2.0 * math.pi * d.u(n)
        st = torch.sqrt(1.0 - ct * ct)
        cp, sp = torch.cos(ph), torch.sin(ph)
        b = d.log_uniform(n, 1e-3, 1e2) / (pm * LC)
        az = 2.0 * math.pi * d.u(n)
        ca, sa = torch.cos(az), torch.sin(az)
        s["p"] = [pm * st * cp, pm * st * sp, pm * ct]
        # B along cos(az) e_theta + sin(az) e_phi, perpendicular to p
        s["E"] = [z.clone(), z.clone(), z.clone()]
        s["B"] = [b * (ca * ct * cp - sa * sp), b * (ca * ct * sp + sa * cp), -b * ca * st]
        return s
    s["p"] = [-pm, z.clone(), z.clone()]
    if geometry == "skew":
        amp = d.log_uniform(n, 1e-4, 1e3) / ((gamma + pm) * LC)
        amp = torch.where(d.u(n) < 0.5, -amp, amp)
    else:
        a, phase = 10.0 + 490.0 * d.u(n), 2.0 * math.pi * d.u(n)
        if geometry == "wave_fields":
            s["wave"] = (a, phase)
        amp = a * torch.cos(phase)
    s["E"], s["B"] = [z.clone(), amp, z.clone()], [z.clone(), z.clone(), amp.clone()]
    return s


def _capacities(s):
    photons = sum(m for sp, m in s["tiles"] if sp == PHOTON)
    pairs = photons // 3 + 64
    return dict(photons=(s["n"] - photons) // 2 + 64, electrons=pairs, positrons=pairs)


# ---- prepare and run ------------------------------------------------------------------------------
def _handle(sfq, case, **kw):
    return sfq.Handle(ref_length=LAMBDA_R, dt=DT,
                      precision=sfq.MIXED if case["precision"] == "mixed" else sfq.FP64, **kw)


def _prepare_step(sfq, case, seed):
    s = _particles(case, seed)
    local = case.get("decision") == "local"
    h = _handle(sfq, case, decision=sfq.LOCAL if local else sfq.OPTICAL_DEPTH,
                approx=sfq.APPROX_TRUNCATED if case.get("trunc") else sfq.APPROX_FULL)
    tau = None if local else h.init_optical_depth(s["uid"], seed=seed)
    alive = torch.ones(s["n"], dtype=torch.uint8, device=DEV)
    uniform, wave = _geometry(case) == "uniform", s["wave"]
    tiles, at = [], 0
    for species, m in s["tiles"]:
        cut = slice(at, at + m)
        kw = dict(tau=None if local else tau[cut], uid=s["uid"][cut],
                  alive=alive[cut] if species == PHOTON else None)
        if wave:
            kw.update(field_mode=sfq.FIELDS_PLANE_WAVE, wave_amp=wave[0][cut],
                      wave_phase=wave[1][cut], wave_k=(1.0, 0.0, 0.0), wave_pol=(0.0, 1.0, 0.0))
            fields = [None] * 6
        elif uniform:
            kw.update(field_mode=sfq.FIELDS_UNIFORM)
            fields = s["E"] + s["B"]
        else:
            fields = [f[cut] for f in s["E"] + s["B"]]
        tiles.append(sfq.TileArrays(species, *[p[cut] for p in s["p"]], *fields, **kw))
        at += m
    n = _capacities(s)
    prods = sfq.ProductBuffers.empty(n["photons"], n["electrons"], DEV)
    cnt = sfq.Counters(DEV)
    state = dict(case=case, h=h, tiles=tiles, prods=prods, cnt=cnt, seed=seed, step=0)
    if case["kind"] == "tiles" or case["entry"] == "plan":
        state["plan"] = h.plan(tiles, seed=seed, step=1, products=prods, counters=cnt,
                               push=bool(case.get("push")))
        state["plan"].capture(1)
    # all counters but the last, which says how the work was scheduled
    state["out"] = dict(px=s["p"][0], py=s["p"][1], pz=s["p"][2], alive=alive,
                        counts=prods.counts, counters=cnt.t[:7])
    if not local:
        state["out"]["tau"] = tau
    if case.get("products"):
        state["out"]["products"] = {
            name: {f: torch.zeros_like(getattr(getattr(prods, name), f)) for f in MADE_ARRAYS}
            for name in MADE}
    return state


def _prepare_served(sfq, case, seed):
    s = _particles(case, seed)
    h = _handle(sfq, case, decision=sfq.LOCAL, blcfa=True)
    alive = torch.ones(s["n"], dtype=torch.uint8, device=DEV)
    created = torch.ones(s["n"], dtype=torch.uint8, device=DEV)
    fperp, dfperp = torch.zeros(3 * s["n"], **F8), torch.zeros(3 * s["n"], **F8)
    counts = torch.zeros((case["sims"], 3), dtype=torch.int64, device=DEV)
    tiles, sets, at = [], [], 0
    for k, (species, m) in enumerate(s["tiles"]):
        cut, cut3 = slice(at, at + m), slice(3 * at, 3 * (at + m))
        kw = dict(uid=s["uid"][cut], product_set=k // 2, field_mode=sfq.FIELDS_PLANE_WAVE,
                  wave_amp=s["wave"][0][cut], wave_phase=s["wave"][1][cut],
                  wave_k=(1.0, 0.0, 0.0), wave_pol=(0.0, 1.0, 0.0))
        if species == PHOTON:
            kw.update(alive=alive[cut])
        else:
            kw.update(fperp=fperp[cut3], dfperp=dfperp[cut3], just_created=created[cut])
            sets.append(sfq.ProductBuffers.empty(m // 3 + 256, m // 4 + 256, DEV))
            sets[-1].counts = counts[len(sets) - 1]
        tiles.append(sfq.TileArrays(species, *[p[cut] for p in s["p"]], **kw))
        at += m
    cnt = sfq.Counters(DEV)
    state = dict(case=case, h=h, tiles=tiles, sets=sets, cnt=cnt, seed=seed, step=0,
                 out=dict(px=s["p"][0], py=s["p"][1], pz=s["p"][2], alive=alive, fperp=fperp,
                          dfperp=dfperp, created=created, counts=counts, counters=cnt.t[:7]))
    for _ in range(3):   # an electron's first steps only record its force
        _run_served(state)
    return state


def prepare(case, seed):
    from paper_2301_07684_amd import sfq

    if case["kind"] in ("step", "tiles"):
        return _prepare_step(sfq, case, seed)
    if case["kind"] == "served":
        return _prepare_served(sfq, case, seed)
    state = _call_inputs(case, seed)
    state.update(case=case, h=_handle(sfq, case), seed=seed)
    return state


def _call_inputs(case, seed):
    n = case["n"]
    if case["kind"] == "load":
        s = _particles(dict(kind="step", geometry="static", layout=0,
                            electrons=0 if case["species"] == PHOTON else n,
                            photons=n if case["species"] == PHOTON else 0), seed)
        return dict(p=s["p"], E=s["E"], B=s["B"], uid=s["uid"])
    d = _Draws(seed)
    return dict(gamma=d.log_uniform(n, 1e2, 1e5),
                chi=d.log_uniform(n, case["chi_lo"], case["chi_hi"]), r=d.u(n))


def _run_served(s):
    for t in s["tiles"]:
        t.step_offset = s["step"]
        t.wave_phase0 = 2.0 * DT * s["step"]
    s["h"].step(s["tiles"], seed=s["seed"], step=0, counters=s["cnt"], product_sets=s["sets"],
                push=True, zero_product_counts=True)
    s["step"] += 1
    return s["out"]


def _run_step(s):
    case = s["case"]
    if "plan" in s:
        s["plan"].replay()
    else:
        s["step"] += 1
        call = s["h"].step_noalloc if case["entry"] == "noalloc" else s["h"].step
        call(s["tiles"], seed=s["seed"], step=s["step"], products=s["prods"], counters=s["cnt"],
             push=case["push"], zero_product_counts=True)
    if not case.get("products"):
        return s["out"]
    # the products' order in their buffers is not defined: the program puts them into its own
    # arrays by parent
    for name, n in zip(MADE, s["prods"].host_counts()):
        b = getattr(s["prods"], name)
        order = torch.argsort(b.parent[:n])
        for f, dst in s["out"]["products"][name].items():
            torch.index_select(getattr(b, f)[:n], 0, order, out=dst[:n])
    return s["out"]


def run(state):
    kind = state["case"]["kind"]
    if kind in ("step", "tiles"):
        return _run_step(state)
    if kind == "served":
        return _run_served(state)
    h = state["h"]
    if kind == "load":
        species = state["case"]["species"]
        tau = h.init_optical_depth(state["uid"], seed=state["seed"])
        gamma, chi = h.chi(species, state["p"], state["E"], state["B"])
        return dict(tau=tau, gamma=gamma, chi=chi, rate=h.rates(species, gamma, chi))
    sample = h.sample_photon if kind == "photons" else h.sample_pair
    first, second = sample(state["gamma"], state["chi"], state["r"])
    return dict(first=first, second=second)


# ---- work -----------------------------------------------------------------------------------------
def work(case):
    """Bytes of the inputs read and the outputs written, and FP64 or FP32 operations."""
    n = case.get("n", 0)
    if case["kind"] == "load":       # uid, p, E, B; tau, gamma, chi, rate
        return dict(bytes=n * (8 + 72 + 32), flops=n * 220)
    if case["kind"] in ("photons", "pairs"):
        return dict(bytes=n * 40, flops=n * 260)
    geometry = _geometry(case)
    fields = {"wave_fields": 16, "uniform": 0}.get(geometry, 48)
    local = case["kind"] == "served" or case.get("decision") == "local"
    push = case["kind"] == "served" or case.get("push")
    emit, convert = EVENTS[geometry]
    total = flops = 0.0
    for species, m in _layout(case):
        lepton = species != PHOTON
        per = 24 + fields + (8 if local else 16) + (0 if lepton else 1)
        per += 24 if lepton and push else 0
        if lepton and case["kind"] == "served":
            per += 2 * 48 + 1        # the stored force and its difference, read and written
        per += (88 * emit if lepton else 105 * convert)
        total += m * per
        flops += m * (200 + (60 if lepton and push else 0) + (60 if geometry == "wave_fields" else 0))
    return dict(bytes=total, flops=flops)


# ---- the same from quadrature ---------------------------------------------------------------------
def _philox(seed, uid, step, purpose):
    """Philox4x32-10: the words x0:x1 and x2:x3 as int64 bit patterns."""
    m = 0xFFFFFFFF
    x = [uid & m, (uid >> 32) & m, torch.full_like(uid, step & m), torch.full_like(uid, purpose)]
    k0, k1 = seed & m, (seed >> 32) & m
    for _ in range(10):
        p0, p1 = x[0] * 0xD2511F53, x[2] * 0xCD9E8D57
        x = [((p1 >> 32) & m) ^ x[1] ^ k0, p1 & m, ((p0 >> 32) & m) ^ x[3] ^ k1, p0 & m]
        k0, k1 = (k0 + 0x9E3779B9) & m, (k1 + 0xBB67AE85) & m
    return (x[0] << 32) | x[1], (x[2] << 32) | x[3]


def _uniform(word):
    return (((word >> 12) & ((1 << 52) - 1)).to(torch.float64) + 0.5) * 2.0 ** -52


def _depth(word):
    return -torch.log1p(-_uniform(word))


def _bessel(x):
    """e^x K_{2/3}(x) and e^x int_x^inf K_{1/3}: int_0^inf of exp(-x (cosh t - 1)) times
    cosh(2t/3) and cosh(t/3)/cosh t, by the trapezoidal rule."""
    nodes = 96
    h = torch.acosh(1.0 + 40.0 / x) / nodes
    g = torch.exp(h / 3.0)
    a = torch.ones_like(x)
    k, ki = torch.full_like(x, 0.5), torch.full_like(x, 0.5)
    for _ in range(nodes):
        a = a * g
        c = 0.5 * (a + 1.0 / a)                      # cosh(t/3)
        ct = c * (4.0 * c * c - 3.0)
        e = torch.exp(-x * (ct - 1.0))
        k = k + e * (2.0 * c * c - 1.0)
        ki = ki + e * c / ct
    return k * h, ki * h


def _panels(edges, n=16):
    x, w = np.polynomial.legendre.leggauss(n)
    e = np.asarray(edges)
    mid, half = 0.5 * (e[1:] + e[:-1])[:, None], 0.5 * (e[1:] - e[:-1])[:, None]
    return torch.tensor(mid + half * x, **F8), torch.tensor(half * w, **F8)


_EDGES = np.concatenate([[0.0], np.geomspace(0.02, 1.5, 18), np.arange(1.75, 6.6, 0.25)])


def _photon_pdf(w, chi, kk=None):
    """dI/dw of the emitted photon, s = 3 chi w^3 / 2."""
    x = w ** 3
    k, ki = kk if kk is not None else _bessel(x)
    s1 = 1.0 + 1.5 * chi * x
    return w * w / s1 ** 3 * ((1.0 + s1 * s1) * k - s1 * ki) * torch.exp(-x)


def _pair_pdf(u, chi, kk=None):
    """dI/du of the created pair, u^2 = eta0 v^2 / (1 - v^2), eta0 = 8/(3 chi), times e^eta0."""
    y, eta0 = u * u, 8.0 / (3.0 * chi)
    k, ki = _bessel(eta0 + y)
    return torch.exp(-y) * (2.0 * (2.0 * y + eta0) * k + eta0 * ki) * (y + eta0) ** -1.5


def _invert(pdf, chi, q, shared):
    """The upper limit at which the integral of pdf reaches the fraction q, for every (chi, q)."""
    nodes, weights = _panels(_EDGES)
    kk = _bessel(nodes.reshape(1, -1) ** 3) if shared else None
    xg = torch.tensor(np.polynomial.legendre.leggauss(16)[0], **F8)
    wg = torch.tensor(np.polynomial.legendre.leggauss(16)[1], **F8)
    edges = torch.tensor(_EDGES, **F8)
    out = []
    for c, r in zip(chi.split(1 << 16), q.split(1 << 16)):
        f = pdf(nodes.reshape(1, -1), c[:, None], kk).reshape(len(c), *nodes.shape)
        cdf = torch.cumsum((f * weights).sum(2), 1)
        level = r * cdf[:, -1]
        j = torch.searchsorted(cdf, level[:, None]).clamp_(max=cdf.shape[1] - 1)
        below = torch.where(j > 0, torch.gather(cdf, 1, (j - 1).clamp(min=0)), 0.0)
        a, b = edges[j[:, 0]], edges[j[:, 0] + 1]
        need = level - below[:, 0]
        x = a + (b - a) * (need / (torch.gather(cdf, 1, j) - below)[:, 0])
        for _ in range(7):
            half = 0.5 * (x - a)
            pts = torch.cat([(a + half)[:, None] + half[:, None] * xg, x[:, None]], 1)
            v = pdf(pts, c[:, None])
            g = half * (v[:, :16] * wg).sum(1) - need
            x = torch.minimum(torch.maximum(x - g / v[:, 16], a), b)
        out.append(x)
    return torch.cat(out) if out else torch.empty_like(chi)


def _photon_energies(gamma, chi, r):
    s = 1.5 * chi * _invert(_photon_pdf, chi, r, True) ** 3
    return gamma * (s / (1.0 + s)), gamma / (1.0 + s)


def _pair_energies(gamma, chi, r):
    y = _invert(_pair_pdf, chi, (2.0 * r - 1.0).abs(), False) ** 2
    eta0 = 8.0 / (3.0 * chi)
    v = torch.sqrt(y / (y + eta0))
    hi, lo = 0.5 * gamma * (1.0 + v), 0.5 * gamma * (eta0 / (y + eta0)) / (1.0 + v)
    return torch.where(r < 0.5, lo, hi), torch.where(r < 0.5, hi, lo)


def _in_log_chi(f, chi, lo, hi, degree=200):
    """f(chi) from its Chebyshev interpolant in log chi on [lo, hi]."""
    k = np.arange(degree)
    nodes = np.cos(np.pi * (k + 0.5) / degree)
    a, b = math.log(lo), math.log(hi)
    v = f(torch.tensor(np.exp(0.5 * (a + b) + 0.5 * (b - a) * nodes), **F8)).cpu().numpy()
    c = 2.0 / degree * np.cos(np.outer(k, np.pi * (k + 0.5) / degree)) @ v
    c[0] *= 0.5
    x = (2.0 * torch.log(chi) - (a + b)) / (b - a)
    b1, b2 = torch.zeros_like(x), torch.zeros_like(x)
    for ck in c[:0:-1]:
        b1, b2 = 2.0 * x * b1 - b2 + float(ck), b1
    return x * b1 - b2 + float(c[0])


def _rate_compton(gamma, chi):
    """alpha/(sqrt3 pi) chi/gamma int R(v chi) K_{2/3}(v) dv, v = w^3, R(x) = (45 x^2 + 42 x +
    20)/(2 + 3 x)^3."""
    def wt(c):
        w, wg = _panels(_EDGES)
        w, wg = w.reshape(1, -1), wg.reshape(1, -1)
        vc = w ** 3 * c[:, None]
        k = _bessel(w ** 3)[0] * torch.exp(-w ** 3) * 3.0 * w * w
        return ((45.0 * vc * vc + 42.0 * vc + 20.0) / (2.0 + 3.0 * vc) ** 3 * k * wg).sum(1)
    return K_RATE * chi / gamma * _in_log_chi(wt, chi, 1e-9, 1e5)


def _rate_pair(gamma, chi):
    """alpha/(sqrt3 pi) / gamma int (9 - v^2)/(3 (1 - v^2)) K_{2/3}(eta) dv, zero below 0.01."""
    def wt(c):
        u, wg = _panels(_EDGES)
        u, wg = u.reshape(1, -1), wg.reshape(1, -1)
        y, eta0 = u * u, 8.0 / (3.0 * c[:, None])
        k = _bessel(eta0 + y)[0] * torch.exp(-y)
        return ((9.0 - y / (y + eta0)) / 3.0 * k / torch.sqrt(eta0 + y) * wg).sum(1) / c
    on = chi >= 0.01
    x = torch.where(on, chi, 1.0)
    w = x * torch.exp(-8.0 / (3.0 * x)) * _in_log_chi(wt, x, 0.005, 1e5)
    return torch.where(on, K_RATE / gamma * w, 0.0)


def _cross(a, b):
    return [a[1] * b[2] - a[2] * b[1], a[2] * b[0] - a[0] * b[2], a[0] * b[1] - a[1] * b[0]]


def _dot(a, b):
    return a[0] * b[0] + a[1] * b[1] + a[2] * b[2]


def _gamma_chi(p, E, B, photon):
    gamma = torch.sqrt(_dot(p, p) + torch.where(photon, 0.0, 1.0))
    f = [gamma * e + c for e, c in zip(E, _cross(p, B))]
    return gamma, LC * torch.sqrt((_dot(f, f) - _dot(p, E) ** 2).clamp(min=0.0))


def _boris(p, E, B, hq):
    m = [a + hq * e for a, e in zip(p, E)]
    t = [hq / torch.sqrt(1.0 + _dot(m, m)) * b for b in B]
    u = [a + b for a, b in zip(m, _cross(m, t))]
    f = 2.0 / (1.0 + _dot(t, t))
    return [a + f * b + hq * e for a, b, e in zip(m, _cross(u, t), E)]


def _exact_step(case, seed):
    s = _particles(case, seed)
    uid, photon, local = s["uid"], s["photon"], case.get("decision") == "local"
    species = torch.cat([torch.full((m,), sp, device=DEV) for sp, m in s["tiles"]])
    p, E, B = s["p"], [f.expand(s["n"]) for f in s["E"]], [f.expand(s["n"]) for f in s["B"]]
    if case.get("push"):
        hq = torch.where(species == POSITRON, 0.5, -0.5).to(torch.float64) * DT
        p = [torch.where(photon, a, b) for a, b in zip(p, _boris(p, E, B, hq))]
    gamma, chi = _gamma_chi(p, E, B, photon)
    del E, B
    W = torch.where(photon, _rate_pair(gamma, chi), _rate_compton(gamma, chi))
    if local:
        tau = None
        emit = W * DT > _uniform(_philox(seed, uid, 1, 4)[0])
    else:
        tau = _depth(_philox(seed, uid, 0, 0)[0]) - W * DT
        emit = tau < 0.0
    leptons, converts = (emit & ~photon).nonzero()[:, 0], (emit & photon).nonzero()[:, 0]

    def at(i):
        return uid[i], gamma[i], chi[i], [a[i] for a in p], torch.sqrt(_dot(*[[a[i] for a in p]] * 2))

    u, g, c, q, pn = at(leptons)
    ea, eb = _philox(seed, u, 1, 1)
    ca, cb = _philox(seed, u, 1, 2)
    photon_e, left = _photon_energies(g, c, _uniform(ea))
    photons = dict(zip(("px", "py", "pz"), [a * (photon_e / pn) for a in q]),
                   tau=_depth(ca), uid=cb, parent=u)
    p = [a.clone() for a in p]
    f = torch.sqrt(((left - 1.0) * (left + 1.0)).clamp(min=0.0)) / pn
    for a, b in zip(p, q):
        a[leptons] = b * f
    if not local:
        tau[leptons] = _depth(eb)
    u, g, c, q, pn = at(converts)
    ea, eb = _philox(seed, u, 1, 1)
    ca, cb = _philox(seed, u, 1, 2)
    made = {}
    for name, e, t, i in zip(("electrons", "positrons"), _pair_energies(g, c, _uniform(ea)),
                             (eb, ca), (cb, _philox(seed, u, 1, 3)[0])):
        f = torch.sqrt(((e - 1.0) * (e + 1.0)).clamp(min=0.0)) / pn
        made[name] = dict(zip(("px", "py", "pz"), [a * f for a in q]), tau=_depth(t), uid=i,
                          parent=u)
    out = dict(px=p[0], py=p[1], pz=p[2], alive=None, counts=None, counters=None)
    if not local:
        out["tau"] = tau
    if case.get("products"):
        n = _capacities(s)
        out["products"] = {}
        for name, b in dict(photons=photons, **made).items():
            out["products"][name] = {f: torch.cat([v, v.new_zeros(n[name] - len(v))])
                                     for f, v in b.items()}
    return out


def exact(case, seed):
    if case["kind"] in ("step", "tiles"):
        return _exact_step(case, seed)
    if case["kind"] == "served":
        return None
    s = _call_inputs(case, seed)
    if case["kind"] == "load":
        photon = torch.full((case["n"],), case["species"] == PHOTON, device=DEV)
        gamma, chi = _gamma_chi(s["p"], s["E"], s["B"], photon)
        rate = _rate_pair if case["species"] == PHOTON else _rate_compton
        return dict(tau=_depth(_philox(seed, s["uid"], 0, 0)[0]), gamma=gamma, chi=chi,
                    rate=rate(gamma, chi))
    f = _photon_energies if case["kind"] == "photons" else _pair_energies
    first, second = f(s["gamma"], s["chi"], s["r"])
    return dict(first=first, second=second)
