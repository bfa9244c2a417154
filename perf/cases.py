"""Performance cases of the near-field library: what its users call, at the
sizes they call it with, and the same results in 64 bits.

    listed()             the named cases
    draw(rng)            one more case of the same ranges
    prepare(case, seed)  what a program holds before the call, on the GPU
    run(state)           one pass through the public entry points
    work(case)           bytes and flops a pass cannot do without
    exact(case, seed)    the same outputs in float64, by plain torch

Kinds of pass:
    force   bin a box, then its accelerations (a user with new positions)
    accel   accelerations of a box already binned
    vjp     their vector-Jacobian product, box already binned
    grad    forward and backward through the autograd function
    batch   many uneven boxes binned and summed in one call
    replay  the same as one captured graph (binning and forces)
    bin     binning alone, into the buffers of an earlier call
    multi   multipole moments of every cell
    step    step statistics, step choice, kick and drift (forces in hand)
    cycle   one whole time step: bin, forces, statistics, choice, kick, drift

Boxes are drawn on the GPU: iid uniform, or clustered by a lognormal
re-weighting of the cells with a Gaussian field of power P(k) ~ k^-2, which
gives the heavy-tailed cell counts of late-time simulation boxes.
"""
from __future__ import annotations

import math

import torch

from paper_1810_02916_amd import nearfield as nf

DEV = torch.device("cuda:0" if torch.cuda.is_available() else "cpu")

SPLINE = 2.16      # spline radius over the Plummer-equivalent length
FLOP_ACCEL = 23    # per pair interaction (22 add/mul and a reciprocal root)
FLOP_VJP = 36


def _box(n, K, sigma, L=1.0, eps=0.041, **kw):
    """n particles in K^3 cells, side L, Plummer-equivalent softening of eps
    mean spacings, sigma: the spread of ln(cell density), 0 for uniform."""
    return dict(n=n, K=K, sigma=sigma, L=L, eps=eps, **kw)


def listed():
    return [
        # a call on a toy box: nothing but launches
        dict(name="force 1k plummer", kind="force", comp=False, plummer=True, **_box(1000, 5, 0.0)),
        # a small differentiable box inside a larger fit
        dict(name="grad 4k", kind="grad", comp=True, plummer=False, **_box(4096, 8, 1.5)),
        # the uniform 32^3 box
        dict(name="force uniform 32k", kind="force", comp=False, plummer=False,
             **_box(32768, 16, 0.0, eps=0.04)),
        # a whole time step of a ragged mid-size box
        dict(name="cycle 50k", kind="cycle", comp=False, plummer=False, **_box(50021, 18, 1.0)),
        # differentiation of the 64^3 clustered box
        dict(name="grad 262k", kind="grad", comp=True, plummer=False, **_box(64 ** 3, 32, 1.5)),
        # uneven boxes in one call, compensated
        dict(name="batch 16", kind="batch", comp=True, plummer=False, boxes=16,
             **_box(65000, 20, 1.5)),
        # the 128^3 clustered box, pass by pass
        dict(name="accel 2m", kind="accel", comp=False, plummer=False, **_box(128 ** 3, 64, 1.5)),
        dict(name="vjp 2m", kind="vjp", comp=True, plummer=False, **_box(128 ** 3, 64, 1.5)),
        dict(name="bin 2m", kind="bin", **_box(128 ** 3, 64, 1.5)),
        dict(name="multipoles 2m", kind="multi", order=8, **_box(128 ** 3, 64, 1.5)),
        dict(name="step 2m", kind="step", **_box(128 ** 3, 64, 1.5)),
        # the largest: 256^3, as strongly clustered as late-time boxes are
        dict(name="accel 16m", kind="accel", comp=True, plummer=False,
             **_box(256 ** 3, 128, 2.0, L=62.5)),
    ]


# kind: (smallest n, largest n) of the drawn cases
_RANGE = {"force": (300, 2_000_000), "accel": (20_000, 4_000_000), "vjp": (20_000, 2_000_000),
          "grad": (500, 1_000_000), "batch": (2_000, 100_000), "replay": (500, 50_000),
          "bin": (10_000, 8_000_000), "multi": (10_000, 4_000_000), "step": (5_000, 4_000_000),
          "cycle": (2_000, 1_000_000)}


def draw(rng):
    kind = rng.choice(sorted(_RANGE))
    lo, hi = _RANGE[kind]
    n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    per_cell = rng.uniform(4.0, 14.0)
    K = max(5, int(round((n / per_cell) ** (1.0 / 3.0))))
    sigma = 0.0 if rng.random() < 0.25 else round(rng.uniform(0.8, 1.8), 2)
    case = dict(kind=kind, **_box(n, K, sigma, L=rng.choice([1.0, 3.0, 125.0]),
                                  eps=round(rng.uniform(0.02, 0.08), 4)))
    if kind not in ("bin", "multi", "step"):
        case["comp"] = rng.random() < 0.5
        case["plummer"] = rng.random() < 0.2
    if kind in ("batch", "replay"):
        case["boxes"] = rng.randint(2, 24)
    if kind == "multi":
        case["order"] = rng.choice([2, 4, 5, 8, 8])
    return case


# ------------------------------------------------------------------ inputs

def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _positions(n, K, sigma, L, seed):
    """(n, 3) float64 positions in [0, L)^3, in random order; the same bits for
    the same arguments (the cell weights are summed as integers)."""
    g = _gen(seed)
    if sigma == 0.0:
        return torch.rand((n, 3), generator=g, device=DEV, dtype=torch.float64) * L
    w = torch.randn((K, K, K), generator=g, device=DEV, dtype=torch.float64)
    f = torch.fft.fftfreq(K, d=1.0 / K, device=DEV, dtype=torch.float64)
    fz = torch.fft.rfftfreq(K, d=1.0 / K, device=DEV, dtype=torch.float64)
    k2 = f[:, None, None] ** 2 + f[None, :, None] ** 2 + fz[None, None, :] ** 2
    amp = torch.where(k2 > 0, 1.0 / torch.sqrt(k2.clamp_min(1e-300)), torch.zeros_like(k2))
    field = torch.fft.irfftn(torch.fft.rfftn(w) * amp, s=(K, K, K)).reshape(-1)
    field = (field - field.mean()) / field.std()
    wt = torch.exp(sigma * (field - field.max()))
    cdf = torch.cumsum((wt * 2.0 ** 36).to(torch.int64) + 1, 0)
    u = torch.randint(0, int(cdf[-1]), (n,), generator=g, device=DEV)
    cell = torch.searchsorted(cdf, u, right=True).clamp_max(K ** 3 - 1)
    pos = torch.rand((n, 3), generator=g, device=DEV, dtype=torch.float64)
    pos += torch.stack((cell // (K * K), (cell // K) % K, cell % K), 1)
    pos *= L / K
    return pos


def _eps(c, n):
    """The softening length the library takes: eps_s of the spline, or the
    Plummer length itself."""
    eps_p = c["eps"] * c["L"] / n ** (1.0 / 3.0)
    return eps_p if c.get("plummer") else SPLINE * eps_p


def _normal(n, seed, scale=1.0):
    return torch.randn((n, 3), generator=_gen(seed), device=DEV, dtype=torch.float32) * scale


def _batch_sizes(c):
    """Uneven boxes: sizes spread around n over a factor of nine, about the
    same particles per cell."""
    m = c["boxes"]
    ns = [max(200, int(c["n"] * 3.0 ** (2.0 * (((7 * b + 3) % m) / max(1, m - 1)) - 1.0)) + b)
          for b in range(m)]
    per = c["n"] / c["K"] ** 3
    return [(n, max(5, int(round((n / per) ** (1.0 / 3.0))))) for n in ns]


# step factors: a typical particle moves by about a hundredth of a cell; the
# kick changes a typical velocity by a thousandth (accelerations are about
# particles per cell / cell width^2)
def _step_scales(c):
    cell = c["L"] / c["K"]
    acc = c["n"] / c["K"] ** 3 / cell ** 2
    return dict(vel=cell, acc=acc, kick=1e-3 * cell / acc, drift=0.01)


def _accelerations(n, seed, scale):
    """Accelerations with the spread of a clustered box: normal directions,
    lognormal sizes."""
    g = _gen(seed)
    a = torch.randn((n, 3), generator=g, device=DEV, dtype=torch.float32)
    return a * (scale * torch.exp(torch.randn((n, 1), generator=g, device=DEV,
                                              dtype=torch.float32)))


_CHOOSE = dict(dlna_max=0.03, hubble=1.0, eta=0.15)


def prepare(case, seed):
    c = case
    kind = c["kind"]
    st = {"c": c, "kind": kind}
    if kind in ("batch", "replay"):
        sizes = _batch_sizes(c)
        st["pos"] = [_positions(n, K, c["sigma"], c["L"], seed * 1000 + b)
                     for b, (n, K) in enumerate(sizes)]
        st["K"] = [K for _, K in sizes]
        st["L"] = [c["L"]] * len(sizes)
        st["eps"] = [_eps(c, n) for n, _ in sizes]
        if kind == "replay":
            st["graph"] = nf.CapturedForce(st["pos"], st["K"], st["L"], st["eps"], 1.0,
                                           compensated=c["comp"], plummer=c["plummer"])
        return st
    n, K, L = c["n"], c["K"], c["L"]
    st["pos"] = _positions(n, K, c["sigma"], L, seed)
    st["eps"] = _eps(c, n)
    if kind in ("accel", "vjp", "bin", "multi", "step", "cycle"):
        st["b"] = nf.bin_particles(st["pos"], K, L, st["eps"])
    if kind in ("vjp", "grad"):
        st["cot"] = _normal(n, seed + 1)
    if kind == "grad":
        st["pos"].requires_grad_(True)
    if kind in ("step", "cycle"):
        st["s"] = _step_scales(c)
        st["vel"] = _normal(n, seed + 2, st["s"]["vel"])
    if kind == "step":
        st["acc"] = _accelerations(n, seed + 3, st["s"]["acc"])
        st["moved"] = st["pos"].clone()
    return st


def _advance(st, acc, pos):
    """Statistics, step choice, kick and drift of one box."""
    b, vel, s = st["b"], st["vel"], st["s"]
    amax, vrms, glob = nf.step_stats(b, acc, vel)
    bounds = nf.step_bounds(b, amax, vrms, glob, **_CHOOSE)
    nf.kick_drift(b, acc, vel, pos, s["kick"], s["drift"])
    return {"amax": amax, "vrms": vrms, "glob": glob, "bounds": bounds, "vel": vel, "pos": pos}


def run(state):
    st = state
    c, kind = st["c"], st["kind"]
    if kind == "force":
        b = nf.bin_particles(st["pos"], c["K"], c["L"], st["eps"])
        return nf.accel(b, 1.0, compensated=c["comp"], plummer=c["plummer"])
    if kind == "accel":
        return nf.accel(st["b"], 1.0, compensated=c["comp"], plummer=c["plummer"])
    if kind == "vjp":
        return nf.accel_vjp(st["b"], st["cot"], 1.0, compensated=c["comp"], plummer=c["plummer"])
    if kind == "grad":
        p = st["pos"]
        p.grad = None
        a = nf.nearfield_accel(p, c["K"], c["L"], st["eps"], 1.0, c["comp"], c["plummer"])
        a.backward(st["cot"])
        return {"acc": a.detach(), "grad": p.grad}
    if kind == "batch":
        b = nf.bin_particles_batched(st["pos"], st["K"], st["L"], st["eps"], check=False)
        return nf.accel(b, 1.0, compensated=c["comp"], plummer=c["plummer"])
    if kind == "replay":
        return st["graph"].replay()
    if kind == "bin":
        x = nf.rebin(st["b"], check=False).boxes[0]
        return {"off": x.off, "cell_start": x.cell_start, "order": x.order, "nbad": x.nbad}
    if kind == "multi":
        return nf.multipoles(st["b"], c["order"])
    if kind == "step":
        return _advance(st, st["acc"], st["moved"])
    if kind == "cycle":
        nf.rebin(st["b"])
        acc = nf.accel(st["b"], 1.0, compensated=c["comp"], plummer=c["plummer"])
        return {"acc": acc, **_advance(st, acc, st["b"].boxes[0].pos)}
    raise ValueError(kind)


# ------------------------------------------------------------------ work

def _interactions(n, K, sigma, L):
    """Pair interactions of one draw of the box (self pairs included)."""
    cell = _cells(_positions(n, K, sigma, L, 0), K, L)[0]
    cnt = torch.bincount(cell, minlength=K ** 3).reshape(K, K, K)
    s = cnt
    for ax in range(3):
        s = sum(torch.roll(s, d, dims=ax) for d in range(-2, 3))
    return float((cnt * s).sum())


def work(case):
    c = case
    kind = c["kind"]
    sizes = _batch_sizes(c) if kind in ("batch", "replay") else [(c["n"], c["K"])]
    by = fl = 0.0
    for n, K in sizes:
        cells = K ** 3
        pairs = 0.0
        if kind not in ("bin", "multi", "step"):
            pairs = _interactions(n, K, c["sigma"], c["L"])
        binning = 24.0 * n + 20.0 * n + 4.0 * cells
        sorted_in = 16.0 * n + 4.0 * n + 4.0 * cells
        stepping = 2 * 12.0 * n + 4.0 * n + 8.0 * cells + 12.0 * n + 2 * 24.0 * n
        if kind in ("force", "batch", "replay"):
            by += binning + 12.0 * n
            fl += FLOP_ACCEL * pairs
        elif kind == "accel":
            by += sorted_in + 12.0 * n
            fl += FLOP_ACCEL * pairs
        elif kind == "vjp":
            by += sorted_in + 24.0 * n
            fl += FLOP_VJP * pairs
        elif kind == "grad":
            by += binning + 12.0 * n + 12.0 * n + 24.0 * n
            fl += (FLOP_ACCEL + FLOP_VJP) * pairs
        elif kind == "bin":
            by += binning
            fl += 12.0 * n
        elif kind == "multi":
            p = c["order"]
            t = (p + 1) * (p + 2) * (p + 3) // 6
            by += 16.0 * n + 4.0 * cells + 4.0 * t * cells
            fl += 2.0 * t * n
        elif kind == "step":
            by += stepping
            fl += 25.0 * n
        elif kind == "cycle":
            by += binning + 12.0 * n + stepping
            fl += FLOP_ACCEL * pairs + 37.0 * n
    return {"bytes": by, "flops": fl}


# ------------------------------------------------------------------ float64

def _cells(pos, K, L):
    """(linear cell, (n, 3) offsets from the cell centre in cell widths)."""
    s = pos.detach() * (K / L)
    f = torch.floor(s)
    c = torch.remainder(f.to(torch.int64), K)
    return (c[:, 0] * K + c[:, 1]) * K + c[:, 2], (s - f) - 0.5


def _pair_sums(pos, K, L, eps, plummer, cot=None, elements=12_000_000):
    """Accelerations (cot None) or the vector-Jacobian product of the
    accelerations with ``cot``, gm = 1, in caller order: for each of the 125
    cell offsets, the sinks in order of how many sources they meet there, in
    blocks of (sinks, sources)."""
    n = pos.shape[0]
    cell, off = _cells(pos, K, L)
    cell, order = torch.sort(cell, stable=True)
    off = off[order].contiguous()
    cnt = torch.bincount(cell, minlength=K ** 3)
    start = torch.cumsum(cnt, 0) - cnt
    e = eps * K / L
    cx, cy, cz = cell // (K * K), (cell // K) % K, cell % K
    out = torch.zeros((n, 3), device=pos.device, dtype=torch.float64)
    v = None if cot is None else cot.to(torch.float64)[order].contiguous()
    for d in range(125):
        dx, dy, dz = d // 25 - 2, (d // 5) % 5 - 2, d % 5 - 2
        src = ((cx + dx) % K * K + (cy + dy) % K) * K + (cz + dz) % K
        m, rank = torch.sort(cnt[src], descending=True)
        first = start[src[rank]]
        sink = off[rank] - torch.tensor([dx, dy, dz], device=pos.device, dtype=torch.float64)
        mh = m.cpu()
        live = int((mh > 0).sum())
        lo = 0
        while lo < live:
            width = int(mh[lo])
            hi = min(live, lo + max(1, elements // width))
            # no wider than twice the narrowest sink of the block
            while hi - lo > 64 and 2 * int(mh[hi - 1]) < width:
                hi = lo + max(64, (hi - lo) // 2)
            k = torch.arange(width, device=pos.device)
            here = k[None, :] < m[lo:hi, None]
            j = torch.where(here, first[lo:hi, None] + k[None, :], 0)
            r = [off[:, a][j] - sink[lo:hi, a, None] for a in range(3)]
            r2 = r[0] * r[0] + r[1] * r[1] + r[2] * r[2]
            if plummer:
                q2 = 1.0 / (r2 + e * e)
                g = q2 * torch.sqrt(q2)
                h = -3.0 * g * q2
            else:
                rho = torch.sqrt(r2)
                safe = rho.clamp_min(1e-300)
                inside = rho < e
                g = torch.where(inside, (10.0 - 15.0 * (rho / e) + 6.0 * r2 / (e * e)) / e ** 3,
                                1.0 / (safe * safe.clamp_min(1e-150) ** 2).clamp_min(1e-300))
                if cot is not None:
                    h = torch.where(inside, (-15.0 / e + 12.0 * rho / (e * e)) / e ** 3 / safe,
                                    -3.0 * g / r2.clamp_min(1e-300))
                    h = torch.where(r2 > 0, h, torch.zeros_like(h))
            g = torch.where(here, g, 0.0)
            at = rank[lo:hi]
            if cot is None:
                for a in range(3):
                    out[at, a] += (g * r[a]).sum(1)
            else:
                u = [v[:, a][j] - v[at, a][:, None] for a in range(3)]
                t = torch.where(here, h, 0.0) * (r[0] * u[0] + r[1] * u[1] + r[2] * u[2])
                for a in range(3):
                    out[at, a] += (g * u[a] + t * r[a]).sum(1)
            lo = hi
    kappa = K / L
    res = torch.empty_like(out)
    res[order] = out * (kappa ** 2 if cot is None else kappa ** 3)
    return res


def _exact_stats(pos, K, L, acc, vel):
    """Per-cell a_max and v_rms, the global triple and the step bounds."""
    cell, _ = _cells(pos, K, L)
    a = acc.to(torch.float64).square().sum(1).sqrt()
    v2 = vel.to(torch.float64).square().sum(1)
    cnt = torch.bincount(cell, minlength=K ** 3)
    zero = torch.zeros(K ** 3, device=pos.device, dtype=torch.float64)
    amax = zero.scatter_reduce(0, cell, a, "amax")
    vrms = torch.sqrt(zero.index_add(0, cell, v2) / cnt.clamp_min(1))
    glob = torch.stack((a.max(), v2.mean().sqrt(), v2.max().sqrt()))
    ratio = torch.where(amax > 0, vrms / amax.clamp_min(1e-300), math.inf).min()
    b = torch.stack((torch.tensor(_CHOOSE["dlna_max"] / _CHOOSE["hubble"], device=pos.device,
                                  dtype=torch.float64),
                     _CHOOSE["eta"] * torch.maximum(ratio, glob[1] / glob[0]),
                     0.8 * (L / K) / glob[2]))
    return {"amax": amax, "vrms": vrms, "glob": glob,
            "bounds": torch.cat((b, b.min()[None]))[None, :]}


def _exact_advance(c, s, pos, acc, vel):
    out = _exact_stats(pos, c["K"], c["L"], acc, vel)
    v = vel.to(torch.float64) + s["kick"] * acc.to(torch.float64)
    # the stored velocity is a float: positions drift with that one
    return {**out, "vel": v, "pos": pos + s["drift"] * v.to(torch.float32).to(torch.float64)}


def _exact_multipoles(pos, K, L, order):
    cell, off = _cells(pos, K, L)
    x = [[torch.ones_like(off[:, a])] for a in range(3)]
    for a in range(3):
        for _ in range(order):
            x[a].append(x[a][-1] * off[:, a])
    cols = []
    for d in range(order + 1):
        for a in range(d, -1, -1):
            for b in range(d - a, -1, -1):
                z = torch.zeros(K ** 3, device=pos.device, dtype=torch.float64)
                cols.append(z.index_add(0, cell, x[0][a] * x[1][b] * x[2][d - a - b]))
    return torch.stack(cols, 1)


def exact(case, seed):
    c = case
    kind = c["kind"]
    if kind in ("batch", "replay"):
        return [_pair_sums(_positions(n, K, c["sigma"], c["L"], seed * 1000 + b), K, c["L"],
                           _eps(c, n), c["plummer"])
                for b, (n, K) in enumerate(_batch_sizes(c))]
    n, K, L = c["n"], c["K"], c["L"]
    if kind in ("force", "accel", "vjp", "grad", "cycle") and n > 6_000_000:
        return None   # minutes in float64
    pos = _positions(n, K, c["sigma"], L, seed)
    eps = _eps(c, n)
    if kind in ("force", "accel"):
        return _pair_sums(pos, K, L, eps, c["plummer"])
    if kind == "vjp":
        return _pair_sums(pos, K, L, eps, c["plummer"], _normal(n, seed + 1))
    if kind == "grad":
        return {"acc": _pair_sums(pos, K, L, eps, c["plummer"]),
                "grad": _pair_sums(pos, K, L, eps, c["plummer"], _normal(n, seed + 1))}
    if kind == "bin":
        cell, off = _cells(pos, K, L)
        cell, order = torch.sort(cell, stable=True)
        return {"off": torch.cat((off[order], (cell % K).to(torch.float64)[:, None]), 1),
                "cell_start": None, "order": None, "nbad": None}
    if kind == "multi":
        return _exact_multipoles(pos, K, L, c["order"])
    s = _step_scales(c)
    vel = _normal(n, seed + 2, s["vel"])
    if kind == "step":
        return _exact_advance(c, s, pos, _accelerations(n, seed + 3, s["acc"]), vel)
    if kind == "cycle":
        acc = _pair_sums(pos, K, L, eps, c["plummer"])
        return {"acc": acc, **_exact_advance(c, s, pos, acc, vel)}
    raise ValueError(kind)
