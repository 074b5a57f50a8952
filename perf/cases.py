"""Workloads whose speed this framework is judged by, through its public calls.

A case is one thing a user's program does again and again with a problem it
keeps: sweep a design grid, smooth the surface and take the best design; the
objective and gradient at continuous designs; a refinement; a thin-plate fit;
the paper's two-layer estimate.  Sizes are those of the workloads, the tests
and the paper, from the smallest to the largest, odd ones included; the
library's default precision is "fp64", and "fp32" (FP32 integrand, FP64 sums)
is what its large sweeps use.

``listed()`` names the standing cases, ``draw(rng)`` gives another of the same
ranges, ``prepare(case, seed)`` makes what a program holds before the call,
``run(state)`` is one pass, ``work(case)`` the bytes and operations a pass
cannot do without, and ``exact(case, seed)`` the results in 64 bits from plain
torch and numpy, where those take a reasonable time.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2005_10494_amd as bmd
from paper_2005_10494_amd import workloads as W


def listed():
    return [
        # One biomarker, 201 cutoffs, M = 1e4: the smallest study, an
        # interactive call in which launches and latency count.
        dict(name="cutoff_1d_201_f64", kind="sweep", design="cutoffs", m="201", draws=10_000, prec="fp64", var=False),
        # Three biomarkers on 64^3 designs, M = 1e5, FP32 integrand: the
        # headline sweep of the benchmark.
        dict(name="cutoff_3d_64_f32", kind="sweep", design="cutoffs", m="64x64x64", draws=100_000, prec="fp32",
             var=False),
        # Three biomarkers on axes of odd lengths in the default precision,
        # with the estimate's variance (the standard errors a report prints).
        dict(name="cutoff_3d_ragged_f64", kind="sweep", design="cutoffs", m="33x40x27", draws=20_000, prec="fp64",
             var=True),
        # Five biomarkers, 14 points an axis: the high-dimensional sweep, in
        # which the responder-overlap products weigh most.
        dict(name="cutoff_5d_14_f32", kind="sweep", design="cutoffs", m="14x14x14x14x14", draws=50_000, prec="fp32",
             var=False),
        # The paper's two-population experiment (Sec. 3, condition (b)) on its
        # (r_2, alpha_1) grid, default precision.
        dict(name="alpha_181x241_f64", kind="sweep", design="alpha", m="181x241", draws=100_000, prec="fp64",
             var=False),
        # Condition (c) of Sec. 3, three populations, 97 x 97 levels.
        dict(name="alpha3_97_f32", kind="sweep", design="alpha3", m="97x97", draws=100_000, prec="fp32", var=False),
        # Three cutoffs on one biomarker (four populations), default precision.
        dict(name="nested4_24_f64", kind="sweep", design="nested4", m="24x24x24", draws=20_000, prec="fp64",
             var=False),
        # Objective and gradient at many continuous five-biomarker designs
        # (the forward and backward of the differentiation form).
        dict(name="grad_5d_2048_f32", kind="grad", d=5, points=2048, draws=500_000, prec="fp32", width=0.01),
        # Refinement of one design by gradient steps: eight trial points a call,
        # the host reads each result back.
        dict(name="refine_5d_f64", kind="refine", d=5, draws=200_000, prec="fp64", width=0.01, max_iter=4),
        # Smoothing of the five-biomarker surface of 24^5 designs, bound by
        # memory, and its best design.
        dict(name="smooth_5d_24_f64", kind="smooth", m="24x24x24x24x24", prec="fp64"),
        # Thin-plate spline of a 97 x 97 level surface (Sec. 2.3), its designs
        # without a third level left out, with Newton on the fit.
        dict(name="tps_97x97", kind="tps", m="97x97", corner=86, lam=1e-4),
        # The paper's own two-layer estimate at its sample sizes (Sec. 3:
        # N1 = 10,240, N2 = 20,480) on a three-population level grid.
        dict(name="two_layer_49_f32", kind="two_layer", design="alpha3", m="49x49", outer=10_240, inner=20_480,
             prec="fp32", groups=16),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# What a drawn sweep may cost: summands a second of the two precisions, at
# which a drawn case takes no longer than the largest listed one, and the
# share of a grid's designs that exist.
_RATE = {"cutoffs": (5e10, 4e11), "alpha": (5e10, 5e11), "alpha3": (2.5e9, 4e10), "alpha4": (3.5e8, 1.4e10),
         "nested3": (1.4e9, 1.9e10), "nested4": (2e8, 6e9)}
_SHARE = {"cutoffs": 1.0, "alpha": 1.0, "alpha3": 0.61, "alpha4": 0.35, "nested3": 0.49, "nested4": 0.14}
_SECONDS = 0.05


def _draws_for(rng, G, design, prec, lo, hi):
    cap = _SECONDS * _RATE[design][prec == "fp32"] / (_SHARE[design] * G)
    return _log(rng, lo, max(lo, min(hi, cap)))


def draw(rng):
    kind = rng.choice(["sweep", "sweep", "sweep", "sweep", "sweep", "sweep", "grad", "refine", "smooth", "tps",
                       "two_layer"])
    prec = rng.choice(["fp64", "fp32"])
    if kind == "sweep":
        design = rng.choice(["cutoffs", "cutoffs", "cutoffs", "alpha", "alpha3", "alpha4", "nested3", "nested4"])
        if design == "cutoffs":
            d = rng.randint(1, 6)
            hi = (401, 160, 48, 20, 11, 8)[d - 1]
            m = [_log(rng, max(3, hi // 4), hi) for _ in range(d)]
        elif design == "alpha":
            m = [rng.randint(17, 181), rng.randint(17, 241)] if rng.random() < 0.7 else [rng.randint(49, 401)]
        elif design in ("alpha3", "nested3"):
            m = [rng.randint(13, 97), rng.randint(13, 97)]
        else:
            m = [rng.randint(7, 24) for _ in range(3)]
        G = math.prod(m)
        # the FP32 integrand is for large samples: its rounding averages out
        n = _draws_for(rng, G, design, prec, 2_000 if prec == "fp64" else 100_000, 1_000_000)
        return dict(kind=kind, design=design, m="x".join(map(str, m)), draws=n, prec=prec,
                    var=bool(rng.random() < 0.3))
    if kind == "grad":
        d = rng.randint(1, 6)
        b = _log(rng, 1, 4096)
        n = _log(rng, 200_000, max(200_000, min(1_000_000, (8e8 if prec == "fp32" else 1e8) / b)))
        return dict(kind=kind, d=d, points=b, draws=n, prec=prec, width=rng.choice([0.01, 0.01, 0.02, 0.0]))
    if kind == "refine":
        return dict(kind=kind, d=rng.randint(2, 6), draws=_log(rng, 20_000, 400_000), prec="fp64", width=0.01,
                    max_iter=rng.randint(2, 4))
    if kind == "smooth":
        d = rng.randint(1, 6)
        hi = (2048, 600, 150, 48, 24, 13)[d - 1]
        m = [_log(rng, max(5, hi // 5), hi) for _ in range(d)]
        return dict(kind=kind, m="x".join(map(str, m)), prec=prec)
    if kind == "tps":
        d = rng.randint(1, 3)
        m = [_log(rng, *((33, 401), (9, 81), (5, 18))[d - 1]) for _ in range(d)]
        return dict(kind=kind, m="x".join(map(str, m)), corner=rng.choice([0, sum(m) // (3 * d)]),
                    lam=rng.choice([1e-3, 1e-4, 1e-5]))
    design = rng.choice(["alpha", "alpha3", "alpha4"])
    m = {"alpha": [rng.randint(5, 15), rng.randint(9, 49)], "alpha3": [rng.randint(9, 49) for _ in range(2)],
         "alpha4": [rng.randint(5, 12) for _ in range(3)]}[design]
    groups = rng.choice([4, 8, 16])
    return dict(kind=kind, design=design, m="x".join(map(str, m)), outer=groups * rng.randint(16, 640),
                inner=1024 * groups * rng.randint(1, 20 // groups if groups < 16 else 1), prec=prec, groups=groups)


# ---------------------------------------------------------------------------
# the framework's calls
# ---------------------------------------------------------------------------
def _axes(case):
    return [int(x) for x in case["m"].split("x")]


def _spec(case, seed):
    """Problem settings of a case (the workloads' own), its draws from `seed`."""
    m = _axes(case) if "m" in case else None
    kind, design = case["kind"], case.get("design", "cutoffs")
    if kind in ("grad", "refine"):
        s = W.base_problem(case["d"], None, 0.3, 0.03, width=case["width"])
    elif kind == "tps":
        s = W.alpha3_design(m[0]) if len(m) == 2 else W.base_problem(len(m), m, 0.3, 0.03)
        s["m"] = m
    elif kind == "smooth" or design == "cutoffs":
        s = W.base_problem(len(m), m, 0.0 if len(m) == 1 else 0.3, 0.02 if len(m) == 1 else 0.03)
    elif design == "alpha":
        s = W.alpha_design(m[1], m_r=m[0], bandwidth=(0.02, 0.0005)) if len(m) == 2 else W.alpha_design(m[0])
    elif design == "alpha3":
        s = dict(W.alpha3_design(m[0]), m=m)
    elif design == "alpha4":
        s = dict(W.alpha4_design(m[0]), m=m)
    elif design == "nested3":
        s = W.nested3_design(m)
    else:
        s = W.nested4_design(m)
    s["seed"] = int(seed)
    return s


def _surface(m, corner, seed, device):
    """A bump and noise over the grid; the `corner` of designs whose axis
    indices add up highest has no value (as levels that already spend alpha0)."""
    gen = torch.Generator(device="cpu").manual_seed(int(seed))
    bump, total = torch.zeros((), device=device, dtype=torch.float64), torch.zeros((), device=device)
    for j, k in enumerate(m):
        shape = [1] * len(m)
        shape[j] = k
        i = torch.arange(k, device=device, dtype=torch.float64)
        bump = bump + ((i / max(k - 1, 1) - 0.6) ** 2).reshape(shape)
        total = total + i.reshape(shape)
    f = 0.3 + 0.4 * torch.exp(-bump / 0.1)
    f = f + 0.02 * torch.randn(math.prod(m), generator=gen, dtype=torch.float64).to(device).reshape(m)
    if corner > 0:
        f = torch.where(total >= sum(m) - corner, torch.full_like(f, math.nan), f)
    return f.reshape(-1).contiguous()


def prepare(case, seed):
    state = dict(case, problem=bmd.Problem(_spec(case, seed)))
    if case["kind"] == "grad":
        state["q"] = torch.from_numpy(W.design_points(case["points"], case["d"], seed=seed)).cuda()
    elif case["kind"] == "refine":
        state["q0"] = W.design_points(1, case["d"], seed=seed, lo=0.45, hi=0.55)[0]
    elif case["kind"] in ("smooth", "tps"):
        state["surface"] = _surface(_axes(case), case.get("corner", 0), seed, "cuda")
    return state


def run(s):
    p, kind = s["problem"], s["kind"]
    if kind == "sweep":
        got = p.eval_grid(s["draws"], s["prec"], want_var=s["var"])
        mean, var = got if s["var"] else (got, None)
        smoothed = p.smooth(mean)
        index, value, _ = p.argmax(smoothed)
        return {"mean": mean, "var": var, "smoothed": smoothed, "index": index, "value": value}
    if kind == "grad":
        obj, gq, gmu = p.grad_design(s["q"], s["draws"], s["prec"])
        return {"obj": obj, "gq": gq, "gmu": gmu}
    if kind == "refine":
        q, obj, steps = p.refine_design(s["q0"], s["draws"], s["prec"], max_iter=s["max_iter"])
        return {"q": q, "obj": obj, "steps": steps}
    if kind == "smooth":
        smoothed = p.smooth(s["surface"], s["prec"])
        index, value, _ = p.argmax(smoothed)
        return {"smoothed": smoothed, "index": index, "value": value}
    if kind == "tps":
        fit, n = p.smooth_tps(s["surface"], s["lam"])
        index, value, cell = p.argmax(fit)
        out = {"fit": fit, "n": n, "index": index, "value": value}
        if p.d < 3:   # in three dimensions the spline has a kink at every centre
            lo, hi = p.spec["q_lo"], p.spec["q_hi"]
            q0 = [lo + (hi - lo) * i / (k - 1) for i, k in zip(cell, p.spec["m"])]
            out["q"], out["best"], _ = p.refine_tps(q0)
        return out
    mean, var = p.eval_grid_two_layer(s["outer"], s["inner"], s["prec"], blocks=(s["groups"], s["groups"]))
    return {"mean": mean, "var": var}


def work(case):
    kind = case["kind"]
    if kind in ("grad", "refine"):
        d, B, M = case["d"], case.get("points", 1 + 8 * case.get("max_iter", 0)), case["draws"]
        per = 60 + (0 if d == 1 else (6 * d - 2) * 24)   # normal CDFs and partials; overlap products and partials
        return {"bytes": 8.0 * B * (2 * d + 3), "flops": float(B) * M * per}
    m = _axes(case)
    G, d = math.prod(m), len(m)
    if kind == "smooth":
        return {"bytes": 16.0 * G, "flops": 2.0 * G * sum(m)}
    if kind == "tps":
        n = G - int(np.isnan(_surface(m, case["corner"], 0, "cpu").numpy()).sum())
        return {"bytes": 16.0 * G, "flops": n ** 3 / 3 + 4.0 * (d + 1) * n * n + 10.0 * n * n}
    if kind == "two_layer":
        n = {"alpha": 2, "alpha3": 3, "alpha4": 4}[case["design"]]
        # ranking every threshold among the inner draws, population by population
        return {"bytes": 16.0 * G, "flops": float(G) * n * case["outer"] * math.log2(case["inner"])}
    f64 = case["prec"] == "fp64"
    design = case["design"]
    if design in ("cutoffs", "alpha"):   # drift, two CDFs and the node sum; overlap products
        per = 23 + 6 * (8 if f64 else 4) + (0 if design == "alpha" or d == 1 else 12 * d)
    elif design in ("alpha3", "nested3"):
        per = 22 + 176 * (8 if f64 else 3)
    else:
        per = 28 + 8 * (12 if f64 else 4) * (35 + 6 * (10 if f64 else 4))
    return {"bytes": 16.0 * G, "flops": per * _SHARE[design] * G * float(case["draws"])}


# ---------------------------------------------------------------------------
# the same in 64 bits, from plain torch and numpy
# ---------------------------------------------------------------------------
def _dev():
    return "cuda" if torch.cuda.is_available() else "cpu"


def _Phi(x):
    return 0.5 * torch.special.erfc(x * -math.sqrt(0.5))


def _phi(x):
    return torch.exp(-0.5 * x * x) / math.sqrt(2 * math.pi)


def _quantile(p):
    x = torch.special.ndtri(p)
    for _ in range(2):   # Newton in the tail that keeps relative accuracy
        x = x - torch.where(p < 0.5, _Phi(x) - p, (1 - p) - _Phi(-x)) / _phi(x)
    return x


def _legendre(n, a=-1.0, b=1.0):
    x, w = np.polynomial.legendre.leggauss(n)
    return 0.5 * (b - a) * x + 0.5 * (a + b), 0.5 * (b - a) * w


def _hermite(n):
    x, w = np.polynomial.hermite_e.hermegauss(n)
    return x, w / w.sum()


def _uniforms(seed, k, n, top=0):
    """u_0 .. u_{n-1} of draws k: Philox4x32-10, 52-bit uniforms."""
    key = [np.uint64(seed & 0xFFFFFFFF), np.uint64(seed >> 32)]
    mask, out = np.uint64(0xFFFFFFFF), []
    for block in range((n + 1) // 2):
        c = [k & mask, k >> np.uint64(32), np.zeros_like(k), np.full_like(k, top | block)]
        k0, k1 = key
        for _ in range(10):
            a, b = np.uint64(0xD2511F53) * c[0], np.uint64(0xCD9E8D57) * c[2]
            c = [(b >> np.uint64(32)) ^ c[1] ^ k0, b & mask, (a >> np.uint64(32)) ^ c[3] ^ k1, a & mask]
            k0, k1 = (k0 + np.uint64(0x9E3779B9)) & mask, (k1 + np.uint64(0xBB67AE85)) & mask
        for hi, lo in ((c[0], c[1]), (c[2], c[3])):
            n52 = ((hi >> np.uint64(6)) << np.uint64(26)) | (lo >> np.uint64(6))
            out.append((n52.astype(np.float64) + 0.5) * 2.0 ** -52)
    return torch.from_numpy(np.stack(out[:n])).to(_dev())


def _bvn(h, k, rho, n=32):
    """Phi_2 by Plackett's identity in the angle."""
    x, w = _legendre(n, 0.0, 1.0)
    th = torch.asin(rho)
    hk, hs = h * k, 0.5 * (h * h + k * k)
    acc = torch.zeros_like(hk)
    for xi, wi in zip(x, w):
        s = torch.sin(th * xi)
        a = 1.0 / ((1 - s) * (1 + s))
        acc += wi * torch.exp(a * (s * hk - hs))
    return _Phi(h) * _Phi(k) + th / (2 * math.pi) * acc


def _root(F, lo, hi):
    """Root of a falling function by bisection, element by element."""
    for _ in range(70):
        mid = 0.5 * (lo + hi)
        up = F(mid) > 0
        lo, hi = torch.where(up, mid, lo), torch.where(up, hi, mid)
    return 0.5 * (lo + hi)


def _grid(lo, hi, m):
    return lo + ((hi - lo) * torch.arange(m, dtype=torch.float64, device=_dev())) / (m - 1)


def _step_draws(spec, M, nbio):
    u = _uniforms(spec["seed"], np.arange(M, dtype=np.uint64), 2 + nbio)
    b0 = spec["mu_b0"] + spec["sd_b0"] * _quantile(u[0])
    b1 = spec["mu_b1"] + spec["sd_b1"] * _quantile(u[1])
    return b0, b1, spec["tau_lo"] + (spec["tau_hi"] - spec["tau_lo"]) * u[2:]


def _factors(spec, c, x):
    """Phi((sqrt(rho_b) x_m - c) / sqrt(1 - rho_b)) with a last axis m."""
    return _Phi((math.sqrt(spec["rho_b"]) * x - c[..., None]) / math.sqrt(1 - spec["rho_b"]))


def _exact_cutoffs(spec, M, moment):
    m, d, info = spec["m"], spec["d"], spec["info"]
    G = math.prod(m)
    q = _grid(spec["q_lo"], spec["q_hi"], max(m)) if d == 1 else [_grid(spec["q_lo"], spec["q_hi"], k) for k in m]
    b0, b1, tau = _step_draws(spec, M, d)
    xs, ws = (torch.from_numpy(a).to(_dev()) for a in _hermite(64))
    if d == 1:
        r = 1 - q
    else:
        A = [_factors(spec, _quantile(a), xs) for a in q]          # [m_j, 64]
        B = [_factors(spec, _quantile(t), xs) for t in tau]        # [M, 64]
        r = ws
        for a in A:
            r = r[..., None, :] * a
        r = r.sum(-1).reshape(-1)
    rho = r.sqrt()
    one = torch.ones_like(r)
    z = _root(lambda t: 2 * _Phi(-t) - _bvn(-t, -t, rho) - spec["alpha0"],
              one * float(-_quantile(torch.tensor(spec["alpha0"], dtype=torch.float64))),
              one * float(-_quantile(torch.tensor(0.5 * spec["alpha0"], dtype=torch.float64))))
    split = max(1, d // 2)
    chunk = max(1, int(2e7 // G))
    for k0 in range(0, M, chunk):
        k = slice(k0, min(M, k0 + chunk))
        if d == 1:
            O = torch.where(q[:, None] > tau[0][None, k], 1 - q[:, None], 1 - tau[0][None, k])
            PR = 1 - tau[0][k]
        else:
            PR = ws * torch.ones_like(B[0][k])
            for b in B:
                PR = PR * b[k]
            PR = PR.sum(-1)
            half = [ws.expand(PR.numel(), 1, -1), torch.ones_like(ws).expand(PR.numel(), 1, -1)]
            for j in range(d):
                v = torch.where((q[j][None, :] > tau[j][k][:, None])[..., None], A[j][None], B[j][k][:, None, :])
                s = int(j >= split)
                half[s] = (half[s][:, :, None, :] * v[:, None]).reshape(PR.numel(), -1, ws.numel())
            O = torch.bmm(half[0], half[1].transpose(1, 2).contiguous()).reshape(PR.numel(), -1).T
        mu1 = math.sqrt(info) * (b0[k] + b1[k] * PR)
        mu2 = (r * info).sqrt()[:, None] * (b0[k] + b1[k] * O / r[:, None])
        moment(1 - _bvn(z[:, None] - mu1, z[:, None] - mu2, rho[:, None], 24))


def _paper(spec, r):
    th = -torch.log1p(-(spec["paper_a"] - spec["paper_b"] * r))
    return (r * spec["info"]).sqrt() * th, (4 * spec["info"] / spec["paper_events"]) ** 0.5


def _exact_alpha(spec, M, moment):
    a1 = _grid(spec["q_lo"], spec["q_hi"], spec["m"][-1])
    r = _grid(spec["r_lo"], spec["r_hi"], spec["m"][0]) if spec["d"] == 2 else torch.tensor([spec["r_lo"]], device=_dev(), dtype=torch.float64)
    r, a1 = (t.reshape(-1) for t in torch.meshgrid(r, a1, indexing="ij"))
    rho, z1 = r.sqrt(), -_quantile(a1)
    z2 = _root(lambda t: a1 + _Phi(-t) - _bvn(-z1, -t, rho) - spec["alpha0"],
               -_quantile(torch.full_like(a1, spec["alpha0"])), -_quantile(spec["alpha0"] - a1))
    e = _quantile(_uniforms(spec["seed"], np.arange(M, dtype=np.uint64), 2))
    (m1, sc), (m2, _) = _paper(spec, torch.ones_like(r)), _paper(spec, r)
    chunk = max(1, int(2e7 // r.numel()))
    for k0 in range(0, M, chunk):
        k = slice(k0, min(M, k0 + chunk))
        h1 = (z1 - m1)[:, None] - sc * e[0, k]
        h2 = (z2 - m2)[:, None] - sc * (rho[:, None] * e[0, k] + (1 - r).sqrt()[:, None] * e[1, k])
        moment(1 - _bvn(h1, h2, rho[:, None], 24))


def _tvn(h1, h2, h3, r2, r3, panels):
    """Phi_3 of three nested populations, given the second statistic."""
    x, w = _legendre(8, 0.0, 1.0)
    a, b = math.sqrt(r2), math.sqrt(r3 / r2)
    sa, sb = math.sqrt(1 - r2), math.sqrt(1 - r3 / r2)
    hi = torch.minimum(torch.minimum(h2, torch.full_like(h2, 8.5)),
                       torch.minimum((h1 + 8.5 * sa) / a, (h3 + 8.5 * sb) / b))
    width = torch.clamp(hi + 8.5, min=0.0) / panels
    acc = torch.zeros_like(width + h3)
    for p in range(panels):
        for xi, wi in zip(x, w):
            y = -8.5 + width * (p + xi)
            acc += wi * _phi(y) * _Phi((h1 - a * y) / sa) * _Phi((h3 - b * y) / sb)
    return acc * width


def _third_level(spec):
    """Critical values of the three-population level grid; NaN without a third."""
    r2, r3 = spec["r_lo"], spec["r_hi"]
    a = torch.meshgrid(*[_grid(spec["q_lo"], spec["q_hi"], k) for k in spec["m"]], indexing="ij")
    z1, z2 = (-_quantile(t.reshape(-1)) for t in a)
    a12 = 1 - _bvn(z1, z2, torch.full_like(z1, math.sqrt(r2)))
    ok = a12 < spec["alpha0"]
    lo = -_quantile(torch.full_like(z1, spec["alpha0"]))
    hi = -_quantile(torch.where(ok, spec["alpha0"] - a12, torch.full_like(z1, spec["alpha0"])))
    z3 = _root(lambda t: 1 - _tvn(z1, z2, t, r2, r3, 16) - spec["alpha0"], lo, hi)
    return z1, z2, torch.where(ok, z3, torch.full_like(z3, math.nan)), ok


def _chain(spec, e, n):
    """Nested statistics' normals from independent ones, and their means."""
    r = torch.tensor([1.0, spec["r_lo"], spec["r_hi"], spec.get("r_4", 0.0)], dtype=torch.float64, device=_dev())[:n]
    y = [e[0]]
    for i in range(1, n):
        f = (r[i] / r[i - 1]).item()
        y.append(math.sqrt(f) * y[-1] + math.sqrt(1 - f) * e[i])
    mean, sc = _paper(spec, r)
    return torch.stack(y), mean, sc


def _exact_alpha3(spec, M, moment):
    z1, z2, z3, ok = _third_level(spec)
    e = _quantile(_uniforms(spec["seed"], np.arange(M, dtype=np.uint64), 3))
    y, mean, sc = _chain(spec, e, 3)
    z = torch.stack([z1[ok], z2[ok], z3[ok]])
    chunk = max(1, int(2e7 // z.shape[1]))
    for k0 in range(0, M, chunk):
        k = slice(k0, min(M, k0 + chunk))
        h = [z[i][:, None] - mean[i] - sc * y[i, k] for i in range(3)]
        f = torch.full((ok.numel(), h[0].shape[1]), math.nan, dtype=torch.float64, device=_dev())
        f[ok] = 1 - _tvn(*h, spec["r_lo"], spec["r_hi"], 10)
        moment(f)


def _smooth(spec, f):
    """Nadaraya-Watson over the grid, axis by axis; over the designs with a
    value only where the design space has designs without."""
    m = spec["m"]

    def separable(v):
        v = v.reshape(m)
        for j, k in enumerate(m):
            lo, hi = (spec["r_lo"], spec["r_hi"]) if spec.get("design") == "alpha" and spec["d"] == 2 and j == 0 else \
                (spec["q_lo"], spec["q_hi"])
            q = _grid(lo, hi, k)
            w = torch.exp(-0.5 * ((q[:, None] - q[None]) / spec["bandwidth"][j]) ** 2)
            w = w / w.sum(1, keepdim=True)
            v = torch.tensordot(w, v, dims=([1], [j])).movedim(0, j)
        return v.reshape(-1)

    if spec.get("design") not in ("alpha3", "alpha4", "nested3", "nested4"):
        return separable(f)
    ok = ~torch.isnan(f)
    return torch.where(ok, separable(torch.where(ok, f, torch.zeros_like(f))) / separable(ok.double()), f)


def _best(f):
    v = f[~torch.isnan(f)]
    return float(v.max())


def _exact_sweep(case, spec):
    M, design, G = case["draws"], case["design"], math.prod(spec["m"])
    cost = {"cutoffs": G * M * (1 + spec["d"]), "alpha": G * M, "alpha3": 20 * G * M}.get(design, math.inf)
    if cost > 4e10:   # over about 20 seconds; the four-population integrals always
        return None
    sums = [torch.zeros(G, dtype=torch.float64, device=_dev()) for _ in range(2)]

    def moment(f):
        sums[0] += f.sum(1)
        sums[1] += (f * f).sum(1)

    {"cutoffs": _exact_cutoffs, "alpha": _exact_alpha, "alpha3": _exact_alpha3}[design](spec, M, moment)
    mean = sums[0] / M
    var = (sums[1] - sums[0] * mean) / (M - 1) if case["var"] else None
    smoothed = _smooth(spec, mean)
    return {"mean": mean, "var": var, "smoothed": smoothed, "index": None, "value": _best(smoothed)}


def _exact_grad(case, spec, seed):
    d, B, M, info, width = case["d"], case["points"], case["draws"], spec["info"], case["width"]
    if B * M * (1 if d == 1 else 24 * d) > 6e9:   # over about 20 seconds
        return None
    q = torch.from_numpy(W.design_points(B, d, seed=seed)).to(_dev()).requires_grad_()
    mu = torch.tensor([[spec["mu_b0"], spec["mu_b1"]]], dtype=torch.float64, device=_dev()).repeat(B, 1).requires_grad_()
    b0, b1, tau = _step_draws(spec, M, d)
    b0, b1 = b0 - spec["mu_b0"], b1 - spec["mu_b1"]
    xs, ws = (torch.from_numpy(a).to(_dev()) for a in _hermite(64))
    xk, wk = (torch.from_numpy(a).to(_dev()) for a in _hermite(32))

    def design(q):
        """r, z* of the points and their node factors, differentiable in q."""
        c = torch.special.ndtri(q.detach())
        c = c + (q - _Phi(c)) / _phi(c)   # value and derivative of the quantile
        r = 1 - q[:, 0] if d == 1 else (ws * _factors(spec, c, xs).prod(1)).sum(-1)
        rho = r.sqrt()
        F = lambda t, s: 2 * _Phi(-t) - _bvn(-t, -t, s) - spec["alpha0"]  # noqa: E731
        with torch.no_grad():
            one = torch.ones_like(r)
            z = _root(lambda t: F(t, rho), one * 1.5, one * 4.5)
            slope = -2 * _phi(z) * _Phi(z * ((1 - rho) / (1 + rho)).sqrt())
        return r, rho, z - F(z, rho) / slope, None if d == 1 else _factors(spec, c, xk)

    total = torch.zeros(B, dtype=torch.float64, device=_dev())
    chunk = max(1, int(4e6 // (B * (1 if d == 1 else 8 * d))))
    grads = [torch.zeros_like(q), torch.zeros_like(mu)]
    for k0 in range(0, M, chunk):
        k = slice(k0, min(M, k0 + chunk))
        r, rho, z, A = design(q)
        t = tau[:, k]
        s = (torch.sigmoid((q[:, :, None] - t[None]) / width) if width > 0 else (q[:, :, None] > t[None]).double())
        if d == 1:
            O = 1 - (s[:, 0] * q + (1 - s[:, 0]) * t)
            PR = 1 - t[0]
        else:
            Bt = _factors(spec, _quantile(t), xk)               # [d, k, 32]
            PR = (wk * Bt.prod(0)).sum(-1)
            O = wk
            for j in range(d):
                O = O * (s[:, j, :, None] * A[:, j, None, :] + (1 - s[:, j, :, None]) * Bt[j][None])
            O = O.sum(-1)
        e0, e1 = mu[:, :1] + b0[k], mu[:, 1:] + b1[k]
        mu1 = math.sqrt(info) * (e0 + e1 * PR)
        mu2 = (r * info).sqrt()[:, None] * (e0 + e1 * O / r[:, None])
        f = (1 - _bvn(z[:, None] - mu1, z[:, None] - mu2, rho[:, None], 24)).sum(1) / M
        for g, x in zip(grads, torch.autograd.grad(f.sum(), [q, mu])):
            g += x
        total += f.detach()
    return {"obj": total, "gq": grads[0], "gmu": grads[1]}


def _exact_tps(case, spec, seed):
    m = spec["m"]
    d = len(m)
    f = _surface(m, case["corner"], seed, "cpu")
    ok = ~torch.isnan(f)
    u = torch.stack([t.reshape(-1) for t in torch.meshgrid(
        *[torch.arange(k, dtype=torch.float64) / (k - 1) for k in m], indexing="ij")], 1)[ok]
    y, n = f[ok], int(ok.sum())
    r = (u[:, None] - u[None]).square().sum(-1).sqrt()
    phi = r ** 3 if d == 1 else torch.where(r > 0, r * r * torch.log(torch.clamp(r, min=1e-300)), r) if d == 2 else -r
    P = torch.cat([torch.ones(n, 1, dtype=torch.float64), u], 1)
    S = torch.zeros(n + d + 1, n + d + 1, dtype=torch.float64)
    S[:n, :n] = phi + case["lam"] * torch.eye(n, dtype=torch.float64)
    S[:n, n:] = P
    S[n:, :n] = P.T
    c = torch.linalg.solve(S, torch.cat([y, torch.zeros(d + 1, dtype=torch.float64)]))
    fit = f.clone()
    fit[ok] = y - case["lam"] * c[:n]   # the smoothing system at the centres
    return {"fit": fit, "n": None, "index": None, "value": _best(fit), "q": None, "best": None}


def _exact_two_layer(case, spec):
    design, N1, N2, A = case["design"], case["outer"], case["inner"], case["groups"]
    G = math.prod(spec["m"])
    if design != "alpha3" or float(G) * N1 * N2 > 6e11:   # over about 20 seconds
        return None
    z1, z2, z3, ok = _third_level(spec)
    y, mean, sc = _chain(spec, _quantile(_uniforms(spec["seed"], np.arange(N1, dtype=np.uint64), 3)), 3)
    x, _, _ = _chain(spec, _quantile(_uniforms(spec["seed"], np.arange(N2, dtype=np.uint64), 3, 1 << 31)), 3)
    est, var = (torch.full((G,), math.nan, dtype=torch.float64, device=_dev()) for _ in range(2))
    for g in torch.nonzero(ok).reshape(-1).tolist():
        t = [float(z[g]) - (mean[i] + sc * y[i]) for i, z in enumerate((z1, z2, z3))]
        inside = x[0][None] <= t[0][:, None]
        for i in (1, 2):
            inside &= x[i][None] <= t[i][:, None]
        n = inside.reshape(A, N1 // A, A, N2 // A).sum((1, 3)).double() / ((N1 // A) * (N2 // A))
        R, C, all_ = n.mean(1, keepdim=True), n.mean(0, keepdim=True), n.mean()
        msa, msb = A * (R - all_).square().sum() / (A - 1), A * (C - all_).square().sum() / (A - 1)
        mse = (n - R - C + all_).square().sum() / (A - 1) ** 2
        est[g], var[g] = 1 - all_, (msa + msb - mse) / (A * A)
    return {"mean": est, "var": var}


def exact(case, seed):
    spec = _spec(case, seed)
    with torch.no_grad():
        if case["kind"] == "sweep":
            return _exact_sweep(case, spec)
        if case["kind"] == "smooth":
            s = _smooth(spec, _surface(spec["m"], 0, seed, _dev()))
            return {"smoothed": s, "index": None, "value": _best(s)}
        if case["kind"] == "tps":
            return _exact_tps(case, spec, seed)
        if case["kind"] == "two_layer":
            return _exact_two_layer(case, spec)
    if case["kind"] == "grad":
        return _exact_grad(case, spec, seed)
    return None   # a refinement's end point depends on the path that it takes
