"""The work that users of this package have it do, as cases to be timed.

Kinds of case, each through the package's public entry points:

  sim        a batch of reaction-diffusion solves advanced a number of steps
             (``cil_simulate_patterns``, IMEX Euler or the second-order scheme)
  relax      a batch run to its stationary patterns (residual < 1e-8)
  plan       an uneven batch bound to a simulate plan, one graph launch
  statistic  range, radii, bins, bootstrap and likelihood of two pattern sets
             (``cil_statistic_adaptive``)
  proposals  the cost of a batch of parameter proposals from their synthetic
             patterns (``SyntheticCIL.costs_from_patterns``)
  norms      the six-norm statistic of two pattern sets

Sizes are those of ``cil_synth.WORKLOADS`` and the tests, or scaled from them.
The trajectories of these models amplify rounding while a pattern is selected
(a unit in the last place of FP32 becomes 1e-2 of a solve's pattern on the way
from noise to stationarity), so FP32 cases stop before that phase or start
after it, and the residual a solve stops at (rounding noise at that point) is
not among the outputs.
"""
import math

import numpy as np
import torch

import paper_2203_14742_amd as cil
from paper_2203_14742_amd.inference import SyntheticCIL

DEV = "cuda"

# model: id, parameters, diffusion coefficients, domain length at 64 nodes (0: the same at every side), dt, noise law
MODELS = {
    "fhn": (cil.CIL_FHN, (1.0, 10.0, 1.0), (0.05, 0.00028), 1.0, False, 0.05),
    "gm_source": (cil.CIL_GM_SOURCE, (0.5, 1.0), (1.0, 100.0), 120.0, True, 0.2),
    "brusselator": (cil.CIL_BRUSSELATOR, (4.5, 6.96), (0.0016, 0.0132), 1.0, False, 0.05),
}
DTYPES = {"f32": torch.float32, "f64": torch.float64}
# most steps from noise over which FP32 trajectories stay comparable
FP32_STEPS = {"fhn": 90, "gm_source": 120, "brusselator": 200}
FP64_STEPS = {"fhn": 1000, "gm_source": 300, "brusselator": 600}


def listed():
    return [
        # one solve alone, the smallest call: a user looking at one parameter point
        {"name": "sim_lone_gm64_f32", "kind": "sim", "model": "gm_source", "sides": "64", "dtype": "f32", "solves": 1,
         "steps": 100, "dt": 0.2, "scheme": "euler"},
        # two 64-pattern sets on 32x32 in double precision, the plain method's configuration
        {"name": "sim_fhn32_f64", "kind": "sim", "model": "fhn", "sides": "32", "dtype": "f64", "solves": 128,
         "steps": 1000, "dt": 0.01, "scheme": "euler"},
        # synthetic patterns of ten proposals on 128x128
        {"name": "sim_fhn128_f32", "kind": "sim", "model": "fhn", "sides": "128", "dtype": "f32", "solves": 640,
         "steps": 80, "dt": 0.05, "scheme": "euler"},
        # a grid study over sides that are no powers of two, double precision
        {"name": "sim_ragged_f64", "kind": "sim", "model": "brusselator", "sides": "20,33,48,50,63,96",
         "dtype": "f64", "solves": 192, "steps": 300, "dt": 0.05, "scheme": "euler"},
        # the second-order scheme on the 32x32 sets
        {"name": "sim_sbdf2_fhn32_f64", "kind": "sim", "model": "fhn", "sides": "32", "dtype": "f64", "solves": 128,
         "steps": 500, "dt": 0.01, "scheme": "sbdf2"},
        # 500 initial states to stationarity, double precision throughout
        {"name": "relax_gm64_f64", "kind": "relax", "n": 64, "dtype": "f64", "solves": 500, "shift": 0.0},
        # the same batch's patterns carried on to a neighbouring parameter point: FP32 steps, refined to the tolerance
        {"name": "relax_gm64_f32", "kind": "relax", "n": 64, "dtype": "f32", "solves": 500, "shift": 0.02},
        # mixed sides with a parameter point each, as one plan
        {"name": "plan_bz_uneven_f32", "kind": "plan", "solves": 384, "steps": 120},
        # the statistic of 500 stationary patterns of 64x64, halves
        {"name": "statistic_250", "kind": "statistic", "nA": 250, "nB": 250, "n": 64, "M": 13, "n_boot": 200,
         "dtype": "f32"},
        # the statistic of 4096 patterns of 128x128, halves
        {"name": "statistic_2048", "kind": "statistic", "nA": 2048, "nB": 2048, "n": 128, "M": 32, "n_boot": 200,
         "dtype": "f32"},
        # one sampler step: 20 proposals with 64 synthetic patterns of 128x128 each
        {"name": "proposals_20x64", "kind": "proposals", "proposals": 20, "n_syn": 64, "n_set": 8, "n": 128, "M": 13,
         "n_boot": 200, "dtype": "f32"},
        # six norms of 500 patterns of 64x64, halves
        {"name": "norms_250", "kind": "norms", "nA": 250, "nB": 250, "n": 64, "M": 10, "n_boot": 200, "dtype": "f32"},
    ]


MOST_POINTS = 1.5e9        # grid values times steps of a drawn batch of solves


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["sim", "sim", "sim", "sim", "sim", "relax", "relax", "plan", "statistic", "statistic",
                       "proposals", "norms"])
    dtype = rng.choice(["f32", "f64"])
    if kind == "sim":
        model = rng.choice(sorted(MODELS))
        # grid sides: powers of two as often as any other
        sides = [rng.choice([32, 64, 128, rng.randint(16, 128), rng.randint(16, 128)])
                 for _ in range(rng.choice([1, 1, 1, 2, 4]))]
        scheme = rng.choice(["euler", "euler", "euler", "sbdf2"])
        steps = rng.randint(40, (FP32_STEPS if dtype == "f32" else FP64_STEPS)[model])
        mean = sum(2 * n * n for n in sides) / len(sides)
        # values cost most where a side, type or scheme has no stepper of its own: smaller batches there
        own = scheme == "euler" and all(n in (32, 64) or (n == 128 and dtype == "f32") for n in sides)
        cap = MOST_POINTS / (1 if own else 6)
        solves = _log_int(rng, 1, max(2, min(1000, cap / (mean * steps))))
        return {"kind": "sim", "model": model, "sides": ",".join(map(str, sides)), "dtype": dtype, "solves": solves,
                "steps": steps, "dt": MODELS[model][5], "scheme": scheme}
    if kind == "relax":
        n = rng.choice([32, 64, rng.randint(24, 64)])
        return {"kind": "relax", "n": n, "dtype": dtype, "solves": _log_int(rng, 16, 500 if n in (32, 64) else 64),
                "shift": round(rng.uniform(0.01, 0.03), 4) if dtype == "f32" else 0.0}
    if kind == "plan":
        return {"kind": "plan", "solves": rng.randint(9, 384), "steps": rng.randint(40, 120)}
    if kind == "statistic":
        return {"kind": "statistic", "nA": _log_int(rng, 20, 1500), "nB": _log_int(rng, 20, 1500),
                "n": rng.choice([32, 50, 64, 128, rng.randint(16, 128)]), "M": rng.randint(5, 40),
                "n_boot": rng.randint(50, 400), "dtype": dtype}
    if kind == "proposals":
        n_set = rng.randint(2, 16)
        return {"kind": "proposals", "proposals": rng.randint(1, 20), "n_syn": n_set + rng.randint(20, 60),
                "n_set": n_set, "n": rng.choice([32, 64, rng.randint(20, 128)]), "M": rng.randint(5, 16),
                "n_boot": rng.randint(50, 300), "dtype": dtype}
    return {"kind": "norms", "nA": rng.randint(20, 250), "nB": rng.randint(20, 250), "n": rng.randint(16, 64),
            "M": rng.randint(4, 10), "n_boot": rng.randint(50, 200), "dtype": dtype}


# ------------------------------------------------------------------ inputs

def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _length(model, n):
    _, _, _, L, scales, _ = MODELS[model]
    return L * (n - 1) / 63.0 if scales else L       # the same node spacing where the domain grows with the side


def _noise(model, base, n, count, g):
    """Initial states [count, 2, n, n]: the steady state with 1 % of noise (relative for gm_source)."""
    u = torch.rand((count, 2, n, n), dtype=torch.float64, device=DEV, generator=g)
    b = torch.tensor(base, dtype=torch.float64, device=DEV).reshape(-1, 2)[:, :, None, None]
    return b * (1.0 + 0.01 * (2.0 * u - 1.0)) if model == "gm_source" else b + 0.01 * u


def _patterns(count, n, g, dtype, modes=12):
    """Stand-in stationary patterns [count, 2 n^2]: tanh of cosine modes on a ring of wave numbers, of differing contrast."""
    i = (torch.arange(n, dtype=torch.float64, device=DEV) + 0.5) / n
    ring = 8.0 * min(1.0, n / 32.0)
    ang = torch.rand((count, 2, modes), dtype=torch.float64, device=DEV, generator=g) * (math.pi / 2)
    sign = torch.where(torch.rand((count, 2, modes), device=DEV, generator=g) < 0.5, 1.0, -1.0).double()
    kx, ky = (ring * torch.cos(ang)).round(), (ring * torch.sin(ang)).round()
    contrast = 0.4 + 1.2 * torch.rand((count, 1, 1, 1), dtype=torch.float64, device=DEV, generator=g)
    out = torch.empty((count, 2, n, n), dtype=dtype, device=DEV)
    for a in range(0, count, 256):
        b = min(count, a + 256)
        cx = torch.cos(math.pi * kx[a:b, :, :, None] * i) * sign[a:b, :, :, None]
        cy = torch.cos(math.pi * ky[a:b, :, :, None] * i)
        f = torch.matmul(cx.transpose(2, 3).contiguous(), cy.contiguous())
        t = torch.tanh(1.5 * f / math.sqrt(modes))
        t[:, 1] *= 0.5
        out[a:b] = (t * contrast[a:b]).to(dtype)
    return out.reshape(count, 2 * n * n)


def _indices(high, rows, cols, g):
    return torch.randint(0, high, (rows, cols), device=DEV, generator=g, dtype=torch.int32)


def _sides(case):
    each = [int(s) for s in case["sides"].split(",")]
    return [each[b % len(each)] for b in range(case["solves"])]


def _sim_inputs(case, seed):
    """Per solve the problem (side, length) and all initial states back to back, FP64."""
    name = case["model"]
    model, p, nu, _, _, _ = MODELS[name]
    g = _gen(seed)
    ns = _sides(case)
    base = cil.cil_homogeneous_state(model, p)
    parts = [None] * len(ns)
    for n in sorted(set(ns)):
        rows = [b for b, m in enumerate(ns) if m == n]
        x = _noise(name, base, n, len(rows), g).reshape(len(rows), -1)
        for k, b in enumerate(rows):
            parts[b] = x[k]
    return model, p, nu, ns, [_length(name, n) for n in ns], torch.cat(parts)


def _plan_inputs(case, seed):
    """Mixed sides, a Brusselator parameter point each within 5 % of the centre."""
    r = np.random.default_rng(seed)
    ns = [(32, 64, 128)[b % 3] for b in range(case["solves"])]
    theta = np.array([4.5, 6.96, 0.0016, 0.0132]) * (1.0 + r.uniform(-0.05, 0.05, (len(ns), 4)))
    g = _gen(seed)
    parts = [None] * len(ns)
    for n in (32, 64, 128):
        rows = [b for b, m in enumerate(ns) if m == n]
        if rows:
            base = np.stack([theta[rows, 0], theta[rows, 1] / theta[rows, 0]], axis=1)
            x = _noise("brusselator", base, n, len(rows), g).reshape(len(rows), -1)
            for k, b in enumerate(rows):
                parts[b] = x[k]
    return ns, theta, torch.cat(parts).float()


def _relax_start(case, seed):
    """Initial states of the relaxation and its parameters: noise, or the patterns of the neighbouring point."""
    n, B = case["n"], case["solves"]
    model, p, nu, _, _, dt = MODELS["gm_source"]
    x = _noise("gm_source", cil.cil_homogeneous_state(model, p), n, B, _gen(seed))
    L = _length("gm_source", n)
    if not case["shift"]:
        return x, p, L, dt
    cil.cil_simulate_patterns(model, x, cil.make_problems(n, L, nu, p, B), dt, 6000, tol=1e-8, check_every=25)
    return x, (p[0] * (1.0 + case["shift"]), p[1]), L, dt


def prepare(case, seed):
    kind = case["kind"]
    if kind == "sim":
        model, p, nu, ns, Ls, ics = _sim_inputs(case, seed)
        ics = ics.to(DTYPES[case["dtype"]])
        return {"kind": kind, "model": model, "ics": ics, "st": torch.empty_like(ics),
                "probs": cil.make_problems(ns, Ls, nu, p, len(ns)), "dt": case["dt"], "steps": case["steps"],
                "scheme": case["scheme"]}
    if kind == "relax":
        x, p, L, dt = _relax_start(case, seed)
        ics = x.to(DTYPES[case["dtype"]])
        return {"kind": kind, "model": cil.CIL_GM_SOURCE, "ics": ics, "st": torch.empty_like(ics), "dt": dt,
                "probs": cil.make_problems(case["n"], L, MODELS["gm_source"][2], p, case["solves"])}
    if kind == "plan":
        ns, theta, ics = _plan_inputs(case, seed)
        st = ics.clone()
        probs = cil.make_problems(ns, 1.0, theta[:, 2:].copy(), theta[:, :2].copy())
        return {"kind": kind, "ics": ics, "st": st,
                "plan": cil.SimPlan(cil.CIL_BRUSSELATOR, st, probs, 0.05, case["steps"], check_every=case["steps"])}
    g = _gen(seed)
    n, M, dtype = case["n"], case["M"], DTYPES[case["dtype"]]
    if kind == "proposals":
        P, n_syn, n_set, n_boot = case["proposals"], case["n_syn"], case["n_set"], case["n_boot"]
        S = _patterns(P * n_syn, n, g, dtype)
        data = _patterns(n_set, n, g, dtype)
        # resamples of the synthetic patterns: n_set of them, and n_syn - n_set of those that were not drawn
        r = np.random.default_rng(seed)
        k2 = n_syn - n_set
        s1 = r.integers(0, n_syn, (n_boot, n_set)).astype(np.int32)
        s2 = np.empty((n_boot, k2), dtype=np.int32)
        for b in range(n_boot):
            rest = np.setdiff1d(np.arange(n_syn), s1[b])
            s2[b] = rest[r.integers(0, rest.size, k2)]
        subset = r.permutation(n_syn)[:k2].astype(np.int32)
        scil = SyntheticCIL(cil.CIL_FHN, n, 1.0, (0.05, 0.00028), lambda t: (t[0], t[1], 1.0), data, n_syn, n_boot, M,
                            0.05, 2000, np.zeros((1, 2, n, n)), (s1, s2, subset))
        return {"kind": kind, "scil": scil, "S": S, "data": data, "lists": (s1, s2, subset)}
    nA, nB = case["nA"], case["nB"]
    X = _patterns(nA + nB, n, g, dtype)
    st = {"kind": kind, "X": X, "A": X[:nA], "B": X[nA:], "M": M, "n": n,
          "ia": _indices(nA, case["n_boot"], nA, g), "ib": _indices(nB, case["n_boot"], nB, g)}
    if kind == "norms":
        st["ii"] = torch.arange(nA, device=DEV).repeat_interleave(nB)
        st["jj"] = torch.arange(nB, device=DEV).repeat(nA)
    return st


def _ends(n):
    e = 2 * n * (n - 1)
    return [2 * n * n, 2 * n * n + e, 2 * n * n + 2 * e]


def _run_norms(s):
    M, ia, ib = s["M"], s["ia"], s["ib"]
    X, n = s["X"], s["n"]
    nA = s["A"].shape[0]
    aug = cil.cil_augment_patterns(X, n, 1.0)
    Ys = []
    for V in (X, aug):
        _, _, _, bins, _ = cil.cil_pair_bins_adaptive(V[:nA], V[nA:], M)
        Ys.append(cil.cil_bootstrap_features(bins, ia, ib, M, want_counts=False)[1])
    ends = _ends(n)
    D = cil.cil_pair_maxabs(aug[:nA], aug[nA:], ends)
    parts = []
    for a, b in zip([0] + ends[:-1], ends):
        part = aug[:, a:b].contiguous()
        parts.append(cil.cil_canonical_d2(part[:nA], part[nA:], s["ii"], s["jj"]).reshape(nA, -1))
    total = cil.cil_combine_segments(torch.stack(parts, dim=-1).contiguous(), 2)
    for V in (D[..., 0].contiguous(), cil.cil_combine_segments(D, 0), cil.cil_combine_segments(D, 1), total):
        lo, hi = cil.cil_value_range(V)
        bins, _ = cil.cil_bin_values(V, cil.cil_radii(lo * lo, hi * hi, M))
        Ys.append(cil.cil_bootstrap_features(bins, ia, ib, M, want_counts=False)[1])
    Y = torch.cat(Ys, dim=1).contiguous()
    _, _, m_eff, status = cil.cil_gaussian_loglik(Y, Y[0].contiguous())
    return {"Y": Y, "D": D, "total": total, "m_eff": m_eff, "status": status}


def run(state):
    s, kind = state, state["kind"]
    if kind == "sim":
        s["st"].copy_(s["ics"])
        rep = cil.cil_simulate_patterns(s["model"], s["st"], s["probs"], s["dt"], s["steps"], check_every=s["steps"],
                                        polish=0, scheme=s["scheme"])
        return {"patterns": s["st"], "steps": rep["steps_taken"], "status": rep["status"]}
    if kind == "relax":
        s["st"].copy_(s["ics"])
        rep = cil.cil_simulate_patterns(s["model"], s["st"], s["probs"], s["dt"], 6000, tol=1e-8, check_every=25,
                                        polish=cil.CIL_POLISH_REFINE)
        out = {"patterns": s["st"], "status": rep["status"]}
        if s["st"].dtype == torch.float64:           # (in FP32 the last bit can move a stop by one evaluation)
            out["steps"] = rep["steps_taken"]
        return out
    if kind == "plan":
        s["st"].copy_(s["ics"])
        s["plan"].launch()
        return {"patterns": s["st"]}
    if kind == "statistic":
        lo, hi, radii, counts, bins, Y, y_obs, (f, ll, m_eff, status) = cil.cil_statistic_adaptive(
            s["A"], s["B"], s["M"], s["ia"], s["ib"])
        return {"d2min": lo, "d2max": hi, "radii": radii, "counts": counts, "bins": bins, "Y": Y, "y_obs": y_obs,
                "f": f, "loglik": ll, "m_eff": m_eff, "status": status}
    if kind == "proposals":
        f, ll = s["scil"].costs_from_patterns(s["S"])
        return {"f": f, "loglik": ll}
    return _run_norms(s)


# ------------------------------------------------------ what a pass needs

def _step_flops(n):
    # two species, two 2D transforms each (2.5 N log2 N), divide and reaction
    return 2 * 2 * 2.5 * n * n * math.log2(n * n) + 12 * n * n


RELAX_STEPS = 730          # mean steps per solve from noise to residual < 1e-8


def work(case):
    kind = case["kind"]
    if kind in ("sim", "plan"):
        ns = _sides(case) if kind == "sim" else [(32, 64, 128)[b % 3] for b in range(case["solves"])]
        size = 8 if case.get("dtype") == "f64" else 4
        return {"bytes": sum(2 * 2 * n * n * size for n in ns), "flops": case["steps"] * sum(map(_step_flops, ns))}
    if kind == "relax":
        n, B = case["n"], case["solves"]
        return {"bytes": 2 * B * 2 * n * n * (8 if case["dtype"] == "f64" else 4),
                "flops": B * RELAX_STEPS * _step_flops(n)}
    size = 8 if case["dtype"] == "f64" else 4
    d = 2 * case["n"] ** 2
    M, n_boot = case["M"], case["n_boot"]
    if kind == "proposals":
        P, n_syn, n_set = case["proposals"], case["n_syn"], case["n_set"]
        pairs = P * (n_syn * n_syn / 2 + n_set * n_syn)
        return {"bytes": (P * n_syn + n_set) * d * size, "flops": 2 * d * pairs + P * n_boot * n_set * n_syn}
    nA, nB = case["nA"], case["nB"]
    boot = 2 * n_boot * (nA + nB) * 4 + n_boot * M * 8 + nA * nB
    if kind == "statistic":
        return {"bytes": (nA + nB) * d * size + boot, "flops": 2.0 * d * nA * nB + n_boot * nA * nB}
    da = _ends(case["n"])[-1]
    # L2, W12 and its three parts as products, three max norms as a subtraction and a comparison
    return {"bytes": (nA + nB) * d * size + 6 * boot + nA * nB * 4 * 8, "flops": nA * nB * (2 * d + 6 * da + 6 * n_boot)}


# ------------------------------------------------------- 64-bit references

def _modes(n):
    k = torch.arange(n, dtype=torch.float64, device=DEV)
    Q = torch.cos(math.pi * k[:, None] * (2 * k[None, :] + 1) / (2 * n)) * math.sqrt(2.0 / n)
    Q[0] *= math.sqrt(0.5)
    return Q, 4.0 * torch.sin(math.pi * k / (2 * n)) ** 2


def _reaction(name, p, v, w):
    if name == "fhn":
        return torch.stack([p[1] * (w - p[2] * v), -v + p[0] * w - w * w * w], 1)
    if name == "gm_source":
        return torch.stack([p[0] - p[1] * v + v * v / w, v * v - w], 1)
    vvw = v * v * w
    return torch.stack([p[0] - (p[1] + 1.0) * v + vvw, p[1] * v - vvw], 1)


class _Solver:
    """IMEX steps of solves of one side in 64 bits, diffusion solved in the cosine basis."""

    def __init__(self, name, p, nu, n, L):
        self.name, self.p = name, p
        self.Q, lam = _modes(n)
        h2 = ((n - 1) / L) ** 2
        self.Lam = (lam[:, None] + lam[None, :]) * h2
        self.nu = nu                                  # two numbers, or two tensors [B, 1, 1]

    def _diffuse(self, r, dt):
        div = torch.stack([(1.0 + dt * self.nu[0] * self.Lam).expand(r.shape[0], *self.Lam.shape),
                           (1.0 + dt * self.nu[1] * self.Lam).expand(r.shape[0], *self.Lam.shape)], 1)
        Q, Qt = self.Q, self.Q.t().contiguous()
        return torch.matmul(Qt, torch.matmul(torch.matmul(Q, torch.matmul(r, Qt)) / div, Q))

    def euler(self, u, dt):
        return self._diffuse(u + dt * _reaction(self.name, self.p, u[:, 0], u[:, 1]), dt)

    def run(self, u, dt, steps, scheme):
        if scheme == "euler":
            for _ in range(steps):
                u = self.euler(u, dt)
            return u
        up, fp = u, _reaction(self.name, self.p, u[:, 0], u[:, 1])
        u = self.euler(u, dt)
        for _ in range(steps - 1):
            f = _reaction(self.name, self.p, u[:, 0], u[:, 1])
            r = (4.0 * u - up) / 3.0 + (2.0 * dt / 3.0) * (2.0 * f - fp)
            up, fp = u, f
            u = self._diffuse(r, 2.0 * dt / 3.0)
        return u

    def relax(self, u, dt, max_steps, tol, every):
        u, steps = u.clone(), torch.zeros(u.shape[0], dtype=torch.int64, device=DEV)
        live = torch.arange(u.shape[0], device=DEV)
        x = u
        for s in range(1, max_steps + 1):
            old = x
            x = self.euler(x, dt)
            if s % every == 0 or s == max_steps:
                far = (x - old).abs().amax(dim=(1, 2, 3)) / dt >= tol
                u[live], steps[live] = x, s
                live, x = live[far], x[far]
                if not live.numel():
                    break
        return u, steps


def _exact_sim(case, seed):
    model, p, nu, ns, Ls, ics = _sim_inputs(case, seed)
    flat = ics.to(DTYPES[case["dtype"]]).double()
    out, off = [None] * len(ns), np.concatenate([[0], np.cumsum([2 * n * n for n in ns])])
    for n in sorted(set(ns)):
        rows = [b for b, m in enumerate(ns) if m == n]
        u = torch.stack([flat[off[b]:off[b + 1]].reshape(2, n, n) for b in rows])
        x = _Solver(case["model"], p, nu, n, Ls[rows[0]]).run(u, case["dt"], case["steps"], case["scheme"])
        for k, b in enumerate(rows):
            out[b] = x[k].reshape(-1)
    return {"patterns": torch.cat(out), "steps": None, "status": None}


def _exact_plan(case, seed):
    ns, theta, ics = _plan_inputs(case, seed)
    flat = ics.double()
    out, off = [None] * len(ns), np.concatenate([[0], np.cumsum([2 * n * n for n in ns])])
    for n in sorted(set(ns)):
        rows = [b for b, m in enumerate(ns) if m == n]
        t = torch.tensor(theta[rows], dtype=torch.float64, device=DEV)[:, :, None, None]
        u = torch.stack([flat[off[b]:off[b + 1]].reshape(2, n, n) for b in rows])
        sv = _Solver("brusselator", (t[:, 0], t[:, 1]), (t[:, 2], t[:, 3]), n, 1.0)
        x = sv.run(u, 0.05, case["steps"], "euler")
        for k, b in enumerate(rows):
            out[b] = x[k].reshape(-1)
    return {"patterns": torch.cat(out)}


def _square_distances(A, B):
    """All squared distances of two sets in 64 bits, from centred vectors."""
    A, B = A.double(), B.double()
    c = A.mean(dim=0, keepdim=True)
    A, B = A - c, B - c
    return ((A * A).sum(1)[:, None] + (B * B).sum(1)[None, :] - 2.0 * (A @ B.t().contiguous())).clamp_min(0.0)


def _ladder(lo, hi, M):
    """Radii between two distances' squares: R_0 b^-m, m = 1..M."""
    r0, rM = math.sqrt(float(hi)), math.sqrt(float(lo))
    b = (r0 / rM) ** (1.0 / M)
    return np.array([r0 * b ** -m for m in range(1, M + 1)])


def _bins(V, thresholds):
    t = torch.tensor(thresholds, dtype=torch.float64, device=DEV)
    out = torch.zeros(V.shape, dtype=torch.int64, device=DEV)
    for m in range(t.numel()):
        out += V < t[m]
    return out


def _resampled(bins, ia, ib, M):
    """Correlation integral vectors of the resamples [n_boot, M]."""
    nA, nB = bins.shape

    def mult(idx, n):
        w = torch.zeros((idx.shape[0], n), dtype=torch.float64, device=DEV)
        return w.scatter_add_(1, idx.long(), torch.ones(idx.shape, dtype=torch.float64, device=DEV))

    wa, wb = mult(ia, nA), mult(ib, nB)
    cols = [((wa @ (bins > m).double()) * wb).sum(1) for m in range(M)]
    return torch.stack(cols, 1) / float(ia.shape[1] * ib.shape[1])


def _exact_statistic(case, seed):
    s = prepare(case, seed)
    d2 = _square_distances(s["A"], s["B"])
    lo, hi = float(d2.min()), float(d2.max())
    radii = _ladder(lo, hi, s["M"])
    thr = radii * radii
    bins = _bins(d2, thr)
    Y = _resampled(bins, s["ia"], s["ib"], s["M"])
    y = torch.stack([(bins > m).double().mean() for m in range(s["M"])])
    # (the smallest radius is the smallest distance: whether that one pair lies under it hangs on the last bit, and the
    # likelihood of a nearly empty bin on that pair)
    return {"d2min": lo, "d2max": hi, "radii": radii, "counts": None, "bins": None, "Y": Y, "y_obs": y, "f": None,
            "loglik": None, "m_eff": None, "status": None}


def _exact_norms(case, seed):
    s = prepare(case, seed)
    X, n, M, nA = s["X"], s["n"], s["M"], case["nA"]
    x = X.double().reshape(-1, 2, n, n)
    h = 1.0 / (n - 1)
    dx, dy = (x[..., 1:] - x[..., :-1]) / h, (x[..., 1:, :] - x[..., :-1, :]) / h
    segs = [t.to(X.dtype).double().reshape(X.shape[0], -1) for t in (x, dx, dy)]
    D = torch.empty((nA, X.shape[0] - nA, 3), dtype=torch.float64, device=DEV)
    for k, t in enumerate(segs):
        for i in range(nA):
            D[i, :, k] = (t[i] - t[nA:]).abs().amax(1)
    d2 = [_square_distances(t[:nA], t[nA:]) for t in segs]
    total = d2[0].sqrt() + d2[1].sqrt() + d2[2].sqrt()
    return {"Y": None, "D": D, "total": total, "m_eff": None, "status": None}


def exact(case, seed):
    kind = case["kind"]
    if kind == "sim":
        return _exact_sim(case, seed)
    if kind == "plan":
        return _exact_plan(case, seed)
    if kind == "relax":
        x, p, L, dt = _relax_start(case, seed)
        x = x.to(DTYPES[case["dtype"]]).double()
        u, _ = _Solver("gm_source", p, MODELS["gm_source"][2], case["n"], L).relax(x, dt, 6000, 1e-8, 25)
        return {"patterns": u, "status": None, "steps": None}
    if kind == "proposals":                          # likelihoods alone: see _exact_statistic
        return None
    return {"statistic": _exact_statistic, "norms": _exact_norms}[kind](case, seed)
