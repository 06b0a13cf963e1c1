"""The work users have this library do, as cases to time: whole collision
intervals of the stated workloads, a run's first neighbour search, a fleet of
runs stepped as one, the product-kernel refresh, the diffusion operator and
the paper's step cadence, each through the entry points a program calls.

Intervals are sampled without flipping the mass buffers (the new masses are
returned, the next pass samples the same masses with new draws), so that a
pass costs the same however many came before it; positions do move.

Exact values: neighbour distances and rate sums of the smaller cases by brute
force, and the diffusion step, in plain torch in 64 bits.
"""
from __future__ import annotations

import math

import torch

import workloads
from paper_2609_35967_amd import Engine
from paper_2609_35967_amd.binding import ManyRuns

DEV = "cuda"
EXACT_MAX = 140_000  # brute-force neighbours up to this many particles


def listed():
    return [
        # the smallest interval: the constant-kernel box of the coagulation test, lists built once
        # (a convergence run makes a thousand of these; launches and latency count)
        dict(name="box_4k", kind="static", setup="const_box", n=4096, k=32),
        # a settling column, additive kernel, lists rebuilt every interval
        dict(name="column_64k", kind="interval", setup="additive_col", n=65536, k=32),
        # a small served disk run, ragged size
        dict(name="disk_10k", kind="interval", setup="disk3d", n=10007, k=32),
        # the benchmark disk: a million micron grains, full physics
        dict(name="disk_1m", kind="interval", setup="disk3d", n=1 << 20, k=32),
        # larger neighbourhoods in single-precision rates, ragged size
        dict(name="disk_200k_k48_f32", kind="interval", setup="disk3d", n=200_003, k=48, fp32=True),
        # the neighbourhood size the paper recommends (256)
        dict(name="disk_128k_k256", kind="interval", setup="disk3d", n=1 << 17, k=256),
        # polydisperse grains: erosion, fragmentation, grouping, long event chains
        dict(name="warm_1m", kind="interval", setup="disk3d_warm", n=1 << 20, k=32),
        # the first search of a run: no previous distances to start from
        dict(name="first_search_300k", kind="first", setup="disk3d", n=300_007, k=32),
        # ten served disk runs of 2^10..2^15 particles stepped as one
        dict(name="fleet_10", kind="fleet", setup="disk3d", n=1 << 15, k=32, runs=10),
        # the ring-spreading test: one diffusion step
        dict(name="ring_1m", kind="diffuse", setup="diffusion_ring", n=1 << 20, form="concentration", St=1.0),
        # the product-kernel test: relabelling before every interval
        dict(name="product_500k", kind="product", setup="const_box", n=500_009, k=32),
        # the paper's symmetric step C D T D C with diffusion
        dict(name="cadence_128k", kind="cadence", setup="disk3d", n=1 << 17, k=32, groups=0),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["static", "interval", "interval", "interval", "interval", "first", "fleet", "diffuse", "product",
                       "cadence"])
    if kind == "static":
        return dict(kind=kind, setup="const_box", n=_logint(rng, 2048, 262144), k=rng.choice([16, 32, 32, 64]))
    if kind == "interval":
        setup = rng.choice(["additive_col", "disk3d", "disk3d", "disk3d_warm"])
        k = rng.choice([20, 32, 32, 32, 33, 48, 64, 100, 128, 200, 256])
        top = {"additive_col": 1 << 19, "disk3d": 1 << 20, "disk3d_warm": 1 << 19}[setup]
        if k > 33:
            top = min(top, (1 << 25) // k)
        return dict(kind=kind, setup=setup, n=_logint(rng, 4000, top), k=k, fp32=rng.random() < 0.25)
    if kind == "first":
        return dict(kind=kind, setup="disk3d", n=_logint(rng, 4000, 1 << 20), k=rng.choice([24, 32, 32, 48]))
    if kind == "fleet":
        return dict(kind=kind, setup="disk3d", n=_logint(rng, 1 << 13, 1 << 16), k=32, runs=rng.randint(2, 10))
    if kind == "diffuse":
        return dict(kind=kind, setup="diffusion_ring", n=_logint(rng, 1 << 16, 1 << 20),
                    form=rng.choice(["concentration", "density"]), St=rng.choice([0.1, 1.0, 10.0]))
    if kind == "product":
        return dict(kind=kind, setup="const_box", n=_logint(rng, 1 << 14, 1 << 20), k=rng.choice([20, 32, 32, 64]))
    return dict(kind=kind, setup="disk3d", n=_logint(rng, 1 << 13, 1 << 18), k=32, groups=rng.choice([0, 0, 8]))


# --------------------------------------------------------------------------- #
def _inputs(case, seed):
    """(params, state) of a case's workload."""
    setup, n = case["setup"], int(case["n"])
    if setup == "diffusion_ring":
        P = workloads.diffusion_ring_params(case["form"], St=case["St"], n=n, axisym=0)
        return P, workloads.diffusion_ring(seed, n)
    P, st = workloads.by_name(setup, seed, n)
    P = dict(P, k=int(case["k"]), rates_fp32=int(bool(case.get("fp32", False))))
    if case["kind"] == "product":
        P["kernel"] = "product"
    if case["kind"] == "cadence":
        P.update(diffusion="concentration", vint=0, axisym=1, Sc=(1.0, 1.0, 1.0))
    return P, st


def _fleet_sizes(case):
    """Sizes of a fleet's runs, log-uniform from 2^10 to the case's n."""
    r, top = int(case["runs"]), int(case["n"])
    return [int(round(math.exp(math.log(1024.0) + (math.log(top) - math.log(1024.0)) * i / max(1, r - 1))))
            for i in range(r)]


class _Fleet:
    def __init__(self, case, seed):
        self.engines = []
        for i, n in enumerate(_fleet_sizes(case)):
            P, st = _inputs(dict(case, n=n), seed * 64 + i)
            e = Engine(P, st, seed=seed * 64 + i, device=DEV, device_interval=True)
            e.build_neighbors()
            self.engines.append(e)
        self.many = ManyRuns(self.engines)


def prepare(case, seed):
    if case["kind"] == "fleet":
        return dict(case=case, fleet=_Fleet(case, seed))
    P, st = _inputs(case, seed)
    eng = Engine(P, st, seed=seed, device=DEV)
    if case["kind"] in ("static", "interval", "product"):
        eng.build_neighbors()  # a run in progress: its lists, or the distances its next search starts from
    if case["kind"] == "cadence" and case["groups"]:
        eng.set_groups(int(case["groups"]), device=True)
    return dict(case=case, eng=eng, refresh=0)


def _interval_state(e):
    d, i = e.iv.view(torch.float64), e.iv.view(torch.int64)
    return dict(dt=d[0:5], worst=d[9:10], counts=i[5:9])


def _lists(e):
    return dict(nbr=e.nbr, cnt=e.cnt, dmax=e.dmax)


def _particles(e):
    out = {k: v for k, v in e.A.t.items() if k not in ("m0", "m1")}
    out["m"] = e.A.m()
    return out


def _sampled(e):
    """What sampling left: events and the masses they gave (the buffers were not flipped)."""
    return dict(lam=e.lam, events=e.events, m_new=e.A.t["m1" if e.A.cur == 0 else "m0"])


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "fleet":
        f = state["fleet"]
        f.many.interval()
        return [dict(nbr=e.nbr, lam=e.lam, m=e.A.m(), x=e.A.t["x"], dt=e.iv.view(torch.float64)[0:5],
                     counts=e.iv.view(torch.int64)[5:9]) for e in f.engines]
    eng = state["eng"]
    if kind == "static":
        eng.collision_rates()
        eng.sample_collisions(flip=False)
        return dict(_sampled(eng), iv=_interval_state(eng))
    if kind == "interval":
        eng.build_neighbors()
        eng.collision_rates()
        eng.sample_collisions(flip=False)
        if case["setup"] == "additive_col":
            eng.push(dt=1e-3)  # a short step: the column keeps its height over many passes
        else:
            eng.push()
        return dict(_lists(eng), **_sampled(eng), state=_particles(eng), iv=_interval_state(eng))
    if kind == "first":
        eng.dmax.zero_()  # a new state: no previous distances
        eng.build_neighbors()
        return dict(_lists(eng), state=_particles(eng))
    if kind == "diffuse":
        eng.diffuse(1e-3, state["refresh"])
        state["refresh"] += 1
        return _particles(eng)
    if kind == "product":
        eng.reshuffle_neighbors(state["refresh"])
        state["refresh"] += 1
        eng.collision_rates()
        eng.sample_collisions(flip=False)
        return dict(_sampled(eng), nbr=eng.nbr, iv=_interval_state(eng))
    eng.strang_step()
    return dict(_lists(eng), lam=eng.lam, events=eng.events, state=_particles(eng))


def work(case):
    """Each input read once, each output written once; the operations of the distances kept, the pairs and the
    per-particle steps (divisions and functions counted as 10)."""
    kind = case["kind"]
    if kind == "fleet":
        ws = [work(dict(case, kind="interval", n=n)) for n in _fleet_sizes(case)]
        return dict(bytes=sum(w["bytes"] for w in ws), flops=sum(w["flops"] for w in ws))
    n = float(case["n"])
    if kind == "diffuse":
        return dict(bytes=132.0 * n, flops=250.0 * n)
    k = float(case["k"])
    arrays = {"const_box": 5, "additive_col": 7}.get(case["setup"], 11)
    pair = 160.0 if case["setup"].startswith("disk") else 15.0
    search_b = 2 * (8 * arrays + 4) + 4 * k + 12
    search_f = 8 * k + 60
    coll_b = 4 * k + 40 + 8 + 8 + 12 + 12
    coll_f = pair * k + 100
    push_b, push_f = (128, 300) if case["setup"].startswith("disk") else (40, 40)
    if kind == "first":
        return dict(bytes=search_b * n, flops=search_f * n)
    if kind == "static":
        return dict(bytes=coll_b * n, flops=coll_f * n)
    if kind == "product":
        return dict(bytes=(coll_b + 4 * k) * n, flops=coll_f * n)
    if kind == "cadence":
        return dict(bytes=(search_b + 2 * coll_b + push_b + 2 * 132) * n,
                    flops=(search_f + 2 * coll_f + push_f + 2 * 250) * n)
    return dict(bytes=(search_b + coll_b + push_b) * n, flops=(search_f + coll_f + push_f) * n)


# --------------------------------------------------------------------------- #
# Exact values in 64 bits, in plain torch.
def _f64(a):
    return torch.as_tensor(a, dtype=torch.float64, device=DEV)


def _morton_order(x, y, z):
    """Stable order of the 30-bit Morton keys over the bounding box's largest side."""
    lo = [c.min() for c in (x, y, z)]
    ext = torch.stack([c.max() - l for c, l in zip((x, y, z), lo)]).max()
    inv = 1024.0 / ext
    key = torch.zeros(x.numel(), dtype=torch.int64, device=DEV)
    for a, c in enumerate((x, y, z)):
        q = ((c - lo[a]) * inv).to(torch.int64).clamp_(0, 1023)
        for b in range(10):
            key |= ((q >> b) & 1) << (3 * b + a)
    return torch.sort(key, stable=True)[1]


def _neighbours(P, x, y, z, k):
    """(indices, distance of the farthest) of the k nearest, self included."""
    n = x.numel()
    step = max(64, (1 << 27) // n)
    idx = torch.empty((n, k), dtype=torch.int64, device=DEV)
    d = torch.empty(n, dtype=torch.float64, device=DEV)
    for s in range(0, n, step):
        e = min(n, s + step)
        d2 = None
        for a, c in enumerate((x, y, z)):
            dc = c[None, :] - c[s:e, None]
            if P["periodic"][a]:
                L = P["L"][a]
                dc = torch.where(dc > 0.5 * L, dc - L, torch.where(dc < -0.5 * L, dc + L, dc))
            d2 = dc * dc if d2 is None else d2 + dc * dc
        v, i = torch.topk(d2, k, dim=1, largest=False, sorted=True)
        idx[s:e] = i
        d[s:e] = v[:, -1].sqrt()
    return idx, d


def _oc07(St1, St2, Vg2, t):
    """Turbulent relative speed squared (Ormel & Cuzzi 2007), St1 >= St2."""
    tight = (St1 - St2) ** 2 * (St1 * St2 + t * (St1 + St2)) / ((St1 + St2) * (St1 + t) * (St2 + t))
    e = St2 / St1
    mid = St1 * (3.2 - (1.0 + e) + 2.0 / (1.0 + e) * (1.0 / 2.6 + e ** 3 / (1.6 + e)))
    heavy = 1.0 / (1.0 + St1) + 1.0 / (1.0 + St2)
    return Vg2 * torch.where(St1 < t, tight, torch.where(St1 < 1.0, mid, heavy))


def _rate_sums(P, x, y, z, d, idx, m, M, rows):
    """lambda*_i of a slice of the particles over their neighbour sets (the particle itself included)."""
    x, y, z, d, idx = x[rows], y[rows], z[rows], d[rows], idx[rows]
    mi, mj = m[rows][:, None], m[idx]
    if P["kernel"] != "physical":
        K = torch.ones_like(mj)
        if P["kernel"] == "additive":
            K = (mi + mj) / P["m0"]
        elif P["kernel"] == "product":
            K = mi * mj / P["m0"] ** 2
        rate = P["m0"] / mj * K / (P["t0"] * P["k"])
        fast = torch.zeros_like(mj, dtype=torch.bool)
    else:
        R = torch.sqrt(x * x + y * y)
        r = torch.sqrt(R * R + z * z)
        xr, w = R / P["R0"], 1.0 - R / r
        Om = torch.sqrt(P["GM"] / R ** 3)
        hg = P["h_g0"] * xr ** ((P["q"] + 1.0) / 2.0)
        H = hg * R
        cs = H * Om
        rho = P["Sigma_g0"] * xr ** P["p"] / (math.sqrt(2.0 * math.pi) * H) * torch.exp(-w / hg ** 2)
        eta = -0.5 * ((P["p"] + 0.5 * P["q"] - 1.5) * hg ** 2 + P["q"] * w)
        stf = P["St0"] / P["s0"] * xr ** -P["p"] * torch.exp(w / hg ** 2)
        V = 4.0 * math.pi * d ** 3 / 3.0
        for de in (r - P["r_in"], P["r_out"] - r):
            h = d - de
            V = V - torch.where(de < d, math.pi * h * h * (3.0 * d - h) / 3.0, torch.zeros_like(h))
        Vg2 = 1.5 * P["alpha"] * cs * cs
        nu = 0.5 * math.sqrt(8.0 / math.pi) * cs * P["mu_mH"] / (rho * P["sigma_H2"])
        t = 1.0 / torch.sqrt(P["alpha"] * cs * H / nu)
        s = (6.0 * m / (math.pi * P["rho_s"])) ** (1.0 / 3.0)
        c = lambda v: v[:, None]  # noqa: E731
        si, sj = c(s[rows]), s[idx]
        Si, Sj = c(stf) * si, c(stf) * sj
        dv2 = (2.0 * c(eta * R * Om) * (Si / (1.0 + Si ** 2) - Sj / (1.0 + Sj ** 2))) ** 2
        dv2 += (c(z * Om) * (torch.clamp(Si, max=0.5) - torch.clamp(Sj, max=0.5))) ** 2
        dv2 += (c(eta * R * Om) * (1.0 / (1.0 + Si ** 2) - 1.0 / (1.0 + Sj ** 2))) ** 2
        kT = P["mu_mH"] * c(cs) ** 2
        dv2 += torch.minimum(8.0 * kT * (1.0 / mi + 1.0 / mj) / math.pi, c(cs) ** 2)
        dv2 += _oc07(torch.maximum(Si, Sj), torch.minimum(Si, Sj), c(Vg2), c(t))
        dv = torch.sqrt(dv2)
        rate = M[idx] / mj * math.pi * (si + sj) ** 2 * dv * 0.25 / c(V)
        fast = dv >= P["v_frag"]
    psi = mj / mi
    Ng = torch.where(psi <= 1e-6, torch.floor(1e-4 / psi), torch.ones_like(psi)) if P["grouping"] else 1.0
    erode = fast & (psi <= 0.1) if P["erosion"] else torch.zeros_like(fast)
    star = torch.where(erode, (1.0 - psi) * rate / Ng + psi * rate, torch.where(fast, rate, rate / Ng))
    return star.sum(1)


def _philox(c, k0, k1):
    """Philox4x32-10 on int64 tensors holding 32-bit words."""
    m32 = 0xFFFFFFFF
    for _ in range(10):
        p0, p1 = c[0] * 0xD2511F53, c[2] * 0xCD9E8D57
        c = [((p1 >> 32) & m32) ^ c[1] ^ k0, p1 & m32, ((p0 >> 32) & m32) ^ c[3] ^ k1, p0 & m32]
        k0, k1 = (k0 + 0x9E3779B9) & m32, (k1 + 0xBB67AE85) & m32
    return c


def _normals(ids, step, w, seed):
    z = torch.zeros_like(ids)
    c = _philox([ids, z + step, z + 0x44494646, z + w], seed & 0xFFFFFFFF, seed >> 32)
    u = [((((c[2 * i + 1] << 32) | c[2 * i]) >> 11) & ((1 << 53) - 1)).double() for i in (0, 1)]
    rad = torch.sqrt(-2.0 * torch.log((u[0] + 1.0) * 2.0 ** -53))
    ang = 2.0 * math.pi * u[1] * 2.0 ** -53
    return rad * torch.cos(ang), rad * torch.sin(ang)


def _diffused(P, st, seed, dt):
    """The ring after one step: vertically integrated disk, radial and azimuthal diffusion."""
    R, ph = _f64(st["r"]), _f64(st["ph"])
    ids = torch.arange(R.numel(), dtype=torch.int64, device=DEV)
    x = R / P["R0"]
    h2 = P["h_g0"] ** 2 * x ** (P["q"] + 1.0)
    nu = P["alpha"] * h2 * R ** 2 * torch.sqrt(P["GM"] / R ** 3)
    D = nu / (1.0 + P["St_diff"] ** 2)
    drift = (1.0 + P["q"] + 1.5 + (P["p"] if P["diffusion"] == "concentration" else 0.0)) / R
    zR, _ = _normals(ids, 0, 0, seed)
    zP, _ = _normals(ids, 0, 1, seed)
    amp = torch.sqrt(2.0 * D * dt)
    R1, ph1 = R + amp * zR + D * drift * dt, ph + amp * zP / R
    ph1 = torch.where(R1 < 0.0, ph1 + math.pi, ph1)
    R1 = R1.abs()
    return dict(r=R1, ph=ph1, x=R1 * torch.cos(ph1), y=R1 * torch.sin(ph1))


def exact(case, seed):
    kind, n = case["kind"], int(case["n"])
    if kind == "diffuse":
        P, st = _inputs(case, seed)
        return _diffused(P, st, seed, 1e-3)
    if kind not in ("static", "interval", "first") or n > EXACT_MAX:
        return None
    P, st = _inputs(case, seed)
    x, y, z, m, M = (_f64(st[a]) for a in ("x", "y", "z", "m", "M"))
    o = _morton_order(x, y, z)
    x, y, z, m, M = x[o], y[o], z[o], m[o], M[o]
    idx, d = _neighbours(P, x, y, z, P["k"])
    if kind == "first":
        return dict(dmax=d)
    lam = torch.empty_like(d)
    for s in range(0, n, 1 << 15):
        rows = slice(s, min(n, s + (1 << 15)))
        lam[rows] = _rate_sums(P, x, y, z, d, idx, m, M, rows)
    return dict(dmax=d, lam=lam) if kind == "interval" else dict(lam=lam)
