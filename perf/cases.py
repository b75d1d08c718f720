"""The work that programs give this library, as measurable cases.

A case names one call path of the public binding with its sizes and options:

  fine      pr_fine_propagate over all slices of an ensemble
  restrict  pr_restrict_quantiles of k ensembles, with ranks and moments
  match     pr_match_quantiles and pr_match_knots of k ensembles
  hist      histogram-state update: pr_hist_restrict, pr_hist_jump, pr_hist_match
  coarse    set-up of a coarse model and one coarse step of all its slices
  solve     a whole small parareal solve: create, iterate, read the states
  chem      one histogram-state parareal iteration of the chemical system
  grad      observables and their parameter gradient through autograd
  batch     one batched iteration of many uneven instances

listed() holds the sizes of the library's own workloads, draw() others of the
same ranges.  Inputs are made from a seed with torch; exact() repeats a path
in plain 64-bit torch or numpy, with the noise definition of include/pr.h.
"""
import math

import numpy as np
import torch

import paper_1912_09240_amd as pr
from paper_1912_09240_amd.autograd import ParamGrad

BETA, LAM, C3, C1 = 2.0, 1.0, 1.0, -1.0
JUMPS = {"add": pr.PR_J_ADD, "mult": pr.PR_J_MULT, "rot": pr.PR_J_ROT, "quantile": pr.PR_J_QUANTILE}
MATCHES = {"marginal": pr.PR_M_MARGINAL, "reweight": pr.PR_M_REWEIGHT, "resample": pr.PR_M_RESAMPLE,
           "resample_det": pr.PR_M_RESAMPLE_DET}
# vector operations of one Philox block with its Box-Muller pair, and of the
# Euler-Maruyama update of one component, as bench.py counts them
OPS_PAIR, OPS_UPDATE = 69, 5


def listed():
    return [
        # the tiny plain-method ensemble: all 10 slices of 100 steps in one short launch
        dict(name="fine_tiny", kind="fine", d=1, dtype="f64", n=10_000, k=10, steps=1_000, dt=1e-3, eps=0.1),
        # the large plain-method ensemble: one sweep of the headline workload
        dict(name="fine_large", kind="fine", d=1, dtype="f64", n=2 ** 20, k=64, steps=100_000, dt=1e-4, eps=0.01),
        # fast part in R^32 stepped in FP32, on a shorter horizon than the library's own run
        dict(name="fine_r32_f32", kind="fine", d=32, dtype="f32", n=2 ** 16, k=32, steps=5_000, dt=1e-4, eps=0.01),
        # sort of the fine results of the large workload: knots and ranks of 64 ensembles
        dict(name="restrict_large", kind="restrict", dtype="f64", n=2 ** 20, k=64, nq=100, moments=False),
        # an FP32 run of the size of the chemical study, with an odd particle count
        dict(name="restrict_ragged_f32", kind="restrict", dtype="f32", n=99_991, k=33, nq=100, moments=True),
        # lifting of the large workload: matched states of 64 ensembles and their knots
        dict(name="match_large", kind="match", dtype="f64", n=2 ** 20, k=64, nq=100),
        # histogram-state update of a mid-sized run, quantile iterator and resampling
        dict(name="hist_resample", kind="hist", n=2 ** 18, k=64, cells=1024, jump="quantile", match="resample"),
        # coarse model of the large workload: exponentials of both slice lengths, one coarse pass
        dict(name="coarse_1024", kind="coarse", cells=1024, k=64, nq=100, steps=100_000, dt=1e-4),
        # the tiny plain-method problem from nothing to its final states: 10 slices, two iterations
        dict(name="solve_tiny", kind="solve", n=10_000, k=10, steps=1_000, dt=1e-3, eps=0.1, cells=200, nq=100,
             iters=2),
        # one iteration of the chemical study (Table 1 sizes)
        dict(name="chem_sweep", kind="chem", n=100_000, k=20, steps=40_000, dt=1e-3, cells=600, jump="quantile",
             match="marginal"),
        # the differentiated form: four observables, their gradient in four parameters
        dict(name="grad_1m", kind="grad", n=2 ** 20, steps=10_000, dt=1e-4, eps=0.1, every=256),
        # batched form: 32 uneven instances of 2^12 to 2^15 particles
        dict(name="batch_32", kind="batch", count=32, log_lo=12, log_hi=15, t_end=0.5, cells=200, nq=100),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["fine", "fine", "restrict", "restrict", "match", "hist", "coarse", "solve", "chem", "grad",
                       "batch"])
    if kind == "fine":
        d = rng.choice([1, 1, 1, 2, 3, 4, 8, 16, 32])
        n, k = _log(rng, 1_000, 2 ** 20), rng.randint(1, 64)
        per_slice = _log(rng, 20, 1_500)
        while n * k * per_slice * (1 + d // 2) > 6e9 or n * k * d > 2e8:
            n, per_slice = max(1_000, n * 2 // 3), max(20, per_slice * 3 // 4)
        eps = rng.choice([0.1, 0.05, 0.01])
        return dict(kind=kind, d=d, dtype=rng.choice(["f64", "f64", "f32"]), n=n, k=k,
                    steps=k * per_slice + rng.randint(0, k - 1), dt=eps / rng.choice([20, 50, 100]), eps=eps)
    if kind == "restrict":
        n, k = _log(rng, 1_000, 2 ** 20), rng.randint(1, 64)
        return dict(kind=kind, dtype=rng.choice(["f64", "f64", "f32"]), n=n, k=k, nq=rng.choice([50, 100, 200]),
                    moments=rng.random() < 0.5)
    if kind == "match":
        return dict(kind=kind, dtype=rng.choice(["f64", "f64", "f32"]), n=_log(rng, 4_000, 2 ** 20),
                    k=rng.randint(1, 64), nq=rng.choice([50, 100, 200]))
    if kind == "hist":
        return dict(kind=kind, n=_log(rng, 4_000, 2 ** 18), k=rng.randint(1, 64), cells=rng.randint(100, 1024),
                    jump=rng.choice(sorted(JUMPS)), match=rng.choice(sorted(MATCHES)))
    if kind == "coarse":
        k = rng.randint(4, 64)
        return dict(kind=kind, cells=_log(rng, 100, 1024), k=k, nq=rng.choice([50, 100, 200]),
                    steps=k * _log(rng, 100, 1_500) + rng.randint(0, k - 1), dt=1e-4)
    if kind == "solve":
        k = rng.randint(4, 32)
        eps = rng.choice([0.1, 0.05, 0.01])
        return dict(kind=kind, n=_log(rng, 4_000, 2 ** 17), k=k, steps=k * _log(rng, 50, 400) + rng.randint(0, k - 1),
                    dt=eps / 50, eps=eps, cells=_log(rng, 100, 512), nq=rng.choice([50, 100]), iters=rng.randint(1, 4))
    if kind == "chem":
        k = rng.randint(8, 32)
        return dict(kind=kind, n=_log(rng, 10_000, 100_000), k=k, steps=k * _log(rng, 200, 2_000), dt=1e-3,
                    cells=rng.choice([300, 600]), jump=rng.choice(sorted(JUMPS)), match=rng.choice(sorted(MATCHES)))
    if kind == "grad":
        return dict(kind=kind, n=_log(rng, 10_000, 2 ** 20), steps=_log(rng, 500, 10_000), dt=1e-4,
                    eps=rng.choice([0.1, 0.05]), every=rng.choice([8, 64, 256]))
    return dict(kind=kind, count=rng.randint(4, 32), log_lo=12, log_hi=rng.randint(12, 15), t_end=0.5, cells=200,
                nq=rng.choice([50, 100]))


# ---------------------------------------------------------------------------
# Inputs.
# ---------------------------------------------------------------------------
def _rng(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) & 0x7FFFFFFFFFFFFFFF)
    return g


def _dtype(case):
    return torch.float64 if case["dtype"] == "f64" else torch.float32


def _prec(case):
    return pr.PR_F64 if case["dtype"] == "f64" else pr.PR_F32


def _double_well(k, n, g, dtype=torch.float64):
    """k ensembles of the bistable slow variable, each with its own balance and spread."""
    x = torch.randn((k, n), generator=g, device="cuda", dtype=torch.float64)
    side = torch.rand((k, n), generator=g, device="cuda", dtype=torch.float32)
    par = torch.rand((k, 2), generator=g, device="cuda", dtype=torch.float64)
    x *= 0.25 + 0.2 * par[:, :1]
    x += torch.where(side < (0.3 + 0.4 * par[:, 1:]).float(), -0.9, 0.9)
    return x.to(dtype)


def _fine_inputs(case, seed):
    g, k, n, d = _rng(seed), case["k"], case["n"], case["d"]
    x = _double_well(k, n, g)
    a = 0.5 + torch.rand(d, generator=g, device="cuda", dtype=torch.float64) if d > 1 else None
    y = torch.empty((k, d, n), device="cuda", dtype=_dtype(case))
    for i in range(d):
        z = torch.randn((k, n), generator=g, device="cuda", dtype=torch.float64)
        y[:, i] = x * (a[i] if a is not None else 1.0) + z / math.sqrt(BETA)
    return x.to(_dtype(case)), y, a


def _levels(nq):
    return torch.arange(nq + 1, device="cuda", dtype=torch.float64) / nq


def _match_targets(case, seed, q):
    """Targets as a chain gives them: the prior's knots moved by a smooth correction of a few hundredths."""
    g = _rng(seed + 1)
    c = torch.rand((case["k"], 3), generator=g, device="cuda", dtype=torch.float64)
    p = _levels(case["nq"])
    return q + 0.03 * (c[:, :1] - 0.5) + 0.02 * c[:, 1:2] * torch.sin(math.pi * (p + c[:, 2:]))


def _hist_masses(case, seed):
    """Two neighbouring coarse histograms per slice."""
    g, k = _rng(seed + 1), case["k"]
    edges = torch.linspace(-3.0, 3.0, case["cells"] + 1, device="cuda", dtype=torch.float64)
    out = []
    c = torch.rand((k, 2), generator=g, device="cuda", dtype=torch.float64)
    for move in (0.0, 0.02):
        w = (0.35 + 0.3 * c[:, :1] + move).clamp(0.0, 1.0)
        sd = 0.3 + 0.15 * c[:, 1:] + move

        def cdf(e):
            return w * torch.special.ndtr((e + 0.9 - move) / sd) + (1 - w) * torch.special.ndtr((e - 0.9 - move) / sd)

        f = cdf(edges[None, :])
        f[:, 0], f[:, -1] = 0.0, 1.0
        out.append((f[:, 1:] - f[:, :-1]).contiguous())
    return out


def _coarse_knots(case, seed):
    x = _double_well(case["k"], 20_000, _rng(seed))
    return _hazen(x.sort(dim=1).values, case["nq"])


def _batch_problem(case, seed):
    r = np.random.default_rng(seed)
    sdes, scheds, ns = [], [], []
    count, span = case["count"], case["log_hi"] - case["log_lo"] + 1
    for i in range(count):  # the parameters from the seed, the sizes spread evenly over the case's ranges
        eps, lam = 10.0 ** (-2.5 + 1.5 * ((7 * i) % count + r.random()) / count), r.uniform(0.5, 2.0)
        s = int(round(case["t_end"] * 20 / eps))
        sdes.append(pr.Sde(lam=lam, eps=eps, beta=BETA))
        scheds.append(pr.Schedule(s, 8 + (11 * i) % 25, case["t_end"] / s))
        ns.append(2 ** (case["log_lo"] + i % span))
    return sdes, scheds, ns


class _Handle:
    """A library handle that is released with the state that holds it."""

    def __init__(self, h, destroy):
        self.h, self._destroy = h, destroy

    def __del__(self):
        if self.h is not None:
            self._destroy(self.h)
            self.h = None


def _bytes(n):
    return torch.empty(max(1, n), dtype=torch.uint8, device="cuda")


def _f64(*shape):
    return torch.empty(shape, dtype=torch.float64, device="cuda")


def prepare(case, seed):
    k = case.get("k")
    n = case.get("n")
    s = dict(case=case, kind=case["kind"], seed=int(seed) & 0xFFFFFFFF)
    if case["kind"] == "fine":
        s["x"], s["y"], s["a"] = _fine_inputs(case, seed)
        s["sde"] = pr.Sde(lam=LAM, eps=case["eps"], beta=BETA, c3=C3, c1=C1, d=case["d"], precision=_prec(case),
                          a=s["a"])
        s["sched"] = pr.Schedule(case["steps"], k, case["dt"])
    elif case["kind"] == "restrict":
        s["x"] = _double_well(k, n, _rng(seed), _dtype(case))
        s["ws"] = _bytes(pr.pr_restrict_workspace_size(n, k, _prec(case)))
        s["q"], s["rank"] = _f64(k, case["nq"] + 1), torch.empty((k, n), dtype=torch.int32, device="cuda")
        s["moments"] = _f64(k, 4) if case["moments"] else None
    elif case["kind"] == "match":
        s["x"] = _double_well(k, n, _rng(seed), _dtype(case))
        s["ws"] = _bytes(pr.pr_restrict_workspace_size(n, k, _prec(case)))
        s["q"], s["rank"] = _f64(k, case["nq"] + 1), torch.empty((k, n), dtype=torch.int32, device="cuda")
        pr.pr_restrict_quantiles(s["x"], _prec(case), n, k, case["nq"], s["q"], s["ws"], rank=s["rank"])
        s["qt"] = _match_targets(case, seed, s["q"])
        s["out"], s["qn"] = torch.empty_like(s["x"]), torch.empty_like(s["q"])
        s["flag"] = torch.zeros(1, dtype=torch.int32, device="cuda")
    elif case["kind"] == "hist":
        g, I = _rng(seed), case["cells"]
        s["x"] = _double_well(k, n, g)
        s["y"] = s["x"] + torch.randn((k, n), generator=g, device="cuda", dtype=torch.float64) / math.sqrt(BETA)
        s["rc"], s["rcs"] = _hist_masses(case, seed)
        s["grid"] = pr.Grid(n_cells=I)
        s["rf"], s["rn"] = _f64(k, I), _f64(k, I)
        s["ws"] = _bytes(pr.pr_hist_workspace_size(k, I))
        s["jws"] = _bytes(pr.pr_hist_jump_workspace_size(k, I))
        s["mws"] = _bytes(pr.pr_hist_match_workspace_size(n, k, I))
        s["xo"], s["yo"], s["wo"] = _f64(k, n), _f64(k, n), _f64(k, n)
    elif case["kind"] == "coarse":
        s["sde"] = pr.Sde(lam=LAM, eps=0.01, beta=BETA, c3=C3, c1=C1)
        s["sched"] = pr.Schedule(case["steps"], k, case["dt"])
        s["grid"] = pr.Grid(n_cells=case["cells"], n_q=case["nq"])
        s["q"] = _coarse_knots(case, seed)
        s["qo"], s["rho"] = torch.empty_like(s["q"]), _f64(k, case["cells"])
    elif case["kind"] == "solve":
        s["sde"] = pr.Sde(lam=LAM, eps=case["eps"], beta=BETA, c3=C3, c1=C1)
        s["sched"] = pr.Schedule(case["steps"], k, case["dt"])
        s["grid"] = pr.Grid(n_cells=case["cells"], n_q=case["nq"])
        s["x"], s["y"], s["q"] = _f64(n), _f64(n), _f64(k + 1, case["nq"] + 1)
    elif case["kind"] == "chem":
        grid = pr.Grid(n_cells=case["cells"], x_lo=0.0, x_hi=600.0)
        h = pr.pr_parareal_hist_create_chem(pr.Chem(), pr.Schedule(case["steps"], k, case["dt"]), grid, s["seed"], 0,
                                            n, JUMPS[case["jump"]], MATCHES[case["match"]])
        s["h"] = _Handle(h, pr.pr_parareal_hist_destroy)
        s["x"], s["y"], s["w"], s["rho"] = _f64(n), _f64(n), _f64(n), _f64(k + 1, case["cells"])
    elif case["kind"] == "grad":
        g = np.random.default_rng(seed)
        s["theta"] = torch.tensor([LAM + 0.1 * g.random(), case["eps"], BETA, C3 + 0.1 * g.random()],
                                  dtype=torch.float64, device="cuda")
        s["weights"] = torch.tensor([1.0, 0.3, -0.2, 0.5], dtype=torch.float64, device="cuda")
        s["cfg"] = dict(n=n, S=case["steps"], dt=case["dt"], every=case["every"], seed=s["seed"])
    else:
        sdes, scheds, ns = _batch_problem(case, seed)
        h = pr.pr_parareal_batch_create(sdes, scheds, ns, pr.Grid(n_cells=case["cells"], n_q=case["nq"]), s["seed"])
        s["h"] = _Handle(h, pr.pr_parareal_batch_destroy)
        s["ends"] = [c.n_slices for c in scheds]
        s["q"] = _f64(case["count"], case["nq"] + 1)
        s["x"] = [_f64(v) for v in ns]
    return s


def run(s):
    case, kind = s["case"], s["kind"]
    k, n = case.get("k"), case.get("n")
    if kind == "fine":
        pr.pr_fine_propagate(s["sde"], s["sched"], s["seed"], 0, n, 0, k, s["x"], s["y"])
        return s["x"], s["y"]
    if kind == "restrict":
        pr.pr_restrict_quantiles(s["x"], _prec(case), n, k, case["nq"], s["q"], s["ws"], rank=s["rank"],
                                 moments=s["moments"])
        return s["q"], s["rank"], s["moments"]
    if kind == "match":
        pr.pr_match_quantiles(s["qt"], s["q"], s["rank"], n, k, case["nq"], s["x"], s["out"], precision=_prec(case))
        pr.pr_match_knots(s["qt"], s["q"], n, k, case["nq"], s["ws"], s["qn"], s["flag"], precision=_prec(case))
        return s["out"], s["qn"], s["flag"]
    if kind == "hist":
        pr.pr_hist_restrict(s["x"], None, n, k, s["grid"], s["rf"], s["ws"])
        pr.pr_hist_jump(JUMPS[case["jump"]], s["rc"], s["rf"], s["rcs"], k, s["grid"], s["rn"], s["jws"])
        pr.pr_hist_match(MATCHES[case["match"]], s["rn"], s["rf"], n, k, 1, s["grid"], s["x"], s["y"], None, n,
                         s["xo"], s["yo"], s["wo"], s["mws"], seed=s["seed"], t_first=1)
        out = [s["rf"], s["rn"]]
        if case["match"] != "reweight":
            out.append(s["xo"])
        if case["match"] != "marginal":
            out.append(s["wo"])
        if case["match"].startswith("resample"):
            out.append(s["yo"])
        return out
    if kind == "coarse":
        h = pr.pr_coarse_create(s["sde"], s["sched"], s["grid"])
        pr.pr_coarse_fp_step(h, 0, k, s["q"], s["qo"], rho_out=s["rho"])
        pr.pr_coarse_destroy(h)
        return s["qo"], s["rho"]
    if kind == "solve":
        h = pr.pr_parareal_create(s["sde"], s["sched"], s["grid"], s["seed"], 0, n)
        pr.pr_parareal_iterate(h, case["iters"])
        for t in range(k):
            pr.pr_parareal_state(h, t, q=s["q"][t])
        pr.pr_parareal_state(h, k, x=s["x"], y=s["y"], q=s["q"][k])
        pr.pr_parareal_destroy(h)
        return s["x"], s["y"], s["q"]
    if kind == "chem":
        pr.pr_parareal_hist_iterate(s["h"].h, 1)
        for t in range(k):
            pr.pr_parareal_hist_state(s["h"].h, t, rho=s["rho"][t])
        pr.pr_parareal_hist_state(s["h"].h, k, x=s["x"], y=s["y"], w=s["w"], rho=s["rho"][k])
        return s["x"], s["y"], s["w"], s["rho"]
    if kind == "grad":
        theta = s["theta"].detach().requires_grad_()
        obs = ParamGrad.apply(theta, s["cfg"])
        (obs * s["weights"]).sum().backward()
        return obs.detach(), theta.grad
    pr.pr_parareal_batch_iterate(s["h"].h, 1, pr.PR_LAUNCH_BATCHED)
    for i, t in enumerate(s["ends"]):
        pr.pr_parareal_batch_state(s["h"].h, i, t, x=s["x"][i], q=s["q"][i])
    return s["q"], s["x"]


# ---------------------------------------------------------------------------
# The least work of one pass: every input read once, every output written
# once; operations of the stepping and of the dense products.
# ---------------------------------------------------------------------------
def _step_ops(d):
    return OPS_PAIR * ((d + 2) // 2) + OPS_UPDATE * (1 + d)


def work(case):
    kind, k, n = case["kind"], case.get("k"), case.get("n")
    if kind == "fine":
        return dict(bytes=2 * n * k * (1 + case["d"]) * (8 if case["dtype"] == "f64" else 4),
                    flops=n * case["steps"] * _step_ops(case["d"]))
    if kind == "restrict":
        return dict(bytes=n * k * (12 if case["dtype"] == "f64" else 8), flops=0)
    if kind == "match":  # values and ranks in, values out; the sorted keys behind the knots
        return dict(bytes=n * k * (28 if case["dtype"] == "f64" else 16), flops=0)
    if kind == "hist":  # x for the histogram; x (and y) in and out and the weights for the matching
        per = {"marginal": 8 + 16, "reweight": 8 + 16}.get(case["match"], 8 + 16 + 24)
        return dict(bytes=n * k * per, flops=0)
    if kind == "coarse":  # the exponentials written once; squarings of full matrices
        return dict(bytes=2 * 8 * case["cells"] ** 2, flops=2 * k * case["cells"] ** 2)
    if kind == "solve":
        return dict(bytes=n * k * 40 * case["iters"], flops=n * case["steps"] * _step_ops(1) * case["iters"])
    if kind == "chem":
        return dict(bytes=n * k * 48, flops=n * case["steps"] * 98)
    if kind == "grad":  # forward, one replay and the reverse recursion with four seeds
        return dict(bytes=n * 32 * (1 + case["steps"] // case["every"]),
                    flops=n * case["steps"] * (2 * _step_ops(1) + 69))
    # mean particle count and 1/eps of the draw
    lo, hi = case["log_lo"], case["log_hi"]
    mean_n = sum(2 ** e for e in range(lo, hi + 1)) / (hi - lo + 1)
    inv_eps = (10 ** 2.5 - 10) / (1.5 * math.log(10))
    return dict(bytes=case["count"] * mean_n * 20 * 40,
                flops=case["count"] * mean_n * case["t_end"] * 20 * inv_eps * _step_ops(1))


# ---------------------------------------------------------------------------
# The same results in plain 64-bit arithmetic.
# ---------------------------------------------------------------------------
M32 = 0xFFFFFFFF


def _philox(key, c0, c1, c2, c3):
    """Philox4x32-10 on int64 tensors (or ints) holding 32-bit words."""
    k0, k1 = key & M32, (key >> 32) & M32
    for _ in range(10):
        p0, p1 = 0xD2511F53 * c0, 0xCD9E8D57 * c2
        c0, c1, c2, c3 = ((p1 >> 32) & M32) ^ c1 ^ k0, p1 & M32, ((p0 >> 32) & M32) ^ c3 ^ k1, p0 & M32
        k0, k1 = (k0 + 0x9E3779B9) & M32, (k1 + 0xBB67AE85) & M32
    return c0, c1, c2, c3


def _normals(seed, tag, m, p, j, single):
    """The normal pair of particles p (int64 tensor): the FP64 bit layout, or the one of FP32 stepping."""
    w0, w1, w2, w3 = _philox(seed, m, p, (tag << 16) | j, 0)
    if single:
        u = ((w0 >> 8).double() + 0.5) * 2.0 ** -24
        t = (((w2 >> 4) & 255).double() + (w2 >> 12).double() * 2.0 ** -20) / 128
        s, c = torch.sin(math.pi * t), torch.cos(math.pi * t)
    else:
        u = (((w0 >> 12) << 32) + w1).double() * 2.0 ** -52 + 2.0 ** -53
        a = math.pi * (((w2 >> 4) & 255).double() + 0.5) / 128
        b = math.pi / 128 * ((((w2 >> 12) << 32) + w3).double() * 2.0 ** -52 - 0.5)
        sa, ca, sb, cb = torch.sin(a), torch.cos(a), torch.sin(b), torch.cos(b)
        s, c = sa * cb + ca * sb, ca * cb - sa * sb
    r = torch.sqrt(-2.0 * torch.log(u))
    return r * c, r * s


def _exact_fine(case, seed):
    n, k, d, S = case["n"], case["k"], case["d"], case["steps"]
    if n * S * ((d + 2) // 2) > 6e9 or S // k * ((d + 2) // 2) > 20_000:
        return None
    x, y, a = _fine_inputs(case, seed)
    x, y = x.double(), y.double()
    dt, eps = case["dt"], case["eps"]
    sx, sy = math.sqrt(2 * dt / BETA), math.sqrt(2 * dt / (BETA * eps))
    p = torch.arange(n, device="cuda")
    seed &= M32
    aa = a if a is not None else torch.ones(1, device="cuda", dtype=torch.float64)
    first = torch.tensor([i * S // k for i in range(k)], device="cuda")
    last = torch.tensor([(i + 1) * S // k for i in range(k)], device="cuda")
    for i in range(int((last - first).max())):
        m = (first + i)[:, None]
        z = []
        for j in range((d + 2) // 2):
            z += _normals(seed, 0, m, p[None, :], j, case["dtype"] == "f32")
        xn = x - dt * (C3 * x ** 3 + C1 * x + LAM * (x - y.mean(dim=1))) + sx * z[0]
        yn = torch.empty_like(y)
        for c in range(d):
            yn[:, c] = y[:, c] - dt / eps * (y[:, c] - aa[c] * x) + sy * z[1 + c]
        if bool((m >= last[:, None]).any()):
            go = m < last[:, None]
            xn, yn = torch.where(go, xn, x), torch.where(go[:, None], yn, y)
        x, y = xn, yn
    return x, y


def _hazen(xs, nq):
    """Midpoint-convention knots of rows in ascending order."""
    n = xs.shape[1]
    t = torch.arange(nq + 1, device=xs.device, dtype=torch.float64) / nq * n - 0.5
    r = t.floor().clamp(0, n - 1)
    hi = (r + 1).clamp(max=n - 1)
    f = (t - r).clamp(0.0, 1.0)
    lo_v, hi_v = xs[:, r.long()], xs[:, hi.long()]
    return lo_v + f * (hi_v - lo_v)


def _exact_restrict(case, seed):
    x = _double_well(case["k"], case["n"], _rng(seed), _dtype(case)).double()
    q = torch.cat([_hazen(r.sort().values[None], case["nq"]) for r in x])
    m = torch.stack([(x ** e).mean(dim=1) for e in (1, 2, 3, 4)], dim=1) if case["moments"] else None
    return q, None, m


def _exact_match(case, seed):
    n, nq = case["n"], case["nq"]
    x = _double_well(case["k"], n, _rng(seed), _dtype(case)).double()
    xs = x.sort(dim=1, stable=True)
    q = _hazen(xs.values, nq)
    qt = _match_targets(case, seed, q)
    d = qt - q
    u = (torch.arange(n, device="cuda", dtype=torch.float64) + 0.5) / n * nq
    j = u.floor().clamp(max=nq - 1)
    w = u - j
    j = j.long()
    moved = xs.values + (1 - w) * d[:, j] + w * d[:, j + 1]  # in rank order
    out = torch.empty_like(x).scatter_(1, xs.indices, moved)
    qn = _hazen(out.to(_dtype(case)).double().sort(dim=1).values, nq)
    return out, qn, None


def _exact_hist(case, seed):
    x = _double_well(case["k"], case["n"], _rng(seed))
    I, k = case["cells"], case["k"]
    cell = torch.floor((x + 3.0) * I / 6.0).clamp(0, I - 1).long() + I * torch.arange(k, device="cuda")[:, None]
    rf = torch.bincount(cell.reshape(-1), minlength=k * I).reshape(k, I).double() / case["n"]
    return [rf] + [None] * 3


def _exact_coarse(case, seed):
    """exp(A tau) rho by uniformisation (non-negative terms only) in extended precision."""
    I, k, nq, S = case["cells"], case["k"], case["nq"], case["steps"]
    L = np.longdouble
    h = 6.0 / I
    mid, edge = L(-3) + (np.arange(I, dtype=L) + L(0.5)) * L(h), L(-3) + np.arange(I + 1, dtype=L) * L(h)
    g = L(h) * np.exp(-L(BETA) * (L(C3) * mid ** 4 / 4 + L(C1) * mid ** 2 / 2))
    a = np.exp(-L(BETA) * (L(C3) * edge ** 4 / 4 + L(C1) * edge ** 2 / 2)) / (L(BETA) * L(h))
    a[0] = a[-1] = 0
    out_rate = (a[:-1] + a[1:]) / g
    rate = out_rate.max()
    taus = np.array([((i + 1) * S // k - i * S // k) * case["dt"] for i in range(k)], dtype=L)
    mean = rate * taus
    if mean.max() * I * k > 6e8 or mean.max() > 10_000:
        return None
    q = _coarse_knots(case, seed).cpu().numpy().astype(L)
    rho = np.empty((k, I), dtype=L)
    for s in range(k):
        c = np.interp(np.asarray(edge, dtype=np.float64), np.asarray(q[s], dtype=np.float64), np.arange(nq + 1) / nq)
        j = np.clip(np.searchsorted(q[s], edge, side="left") - 1, 0, nq - 1)
        c = (j + (edge - q[s][j]) / (q[s][j + 1] - q[s][j])) / L(nq)
        c = np.where(edge <= q[s][0], L(0), np.where(edge > q[s][-1], L(1), c))
        c[0], c[-1] = 0, 1
        rho[s] = np.diff(c)
    stay, right, left = 1 - out_rate / rate, a[1:-1] / (g[:-1] * rate), a[1:-1] / (g[1:] * rate)
    acc, v, logp = np.zeros_like(rho), rho.copy(), -mean
    top = float(mean.max())
    for i in range(int(top + 12 * math.sqrt(top) + 40)):
        if i:
            nv = v * stay
            nv[:, 1:] += v[:, :-1] * right
            nv[:, :-1] += v[:, 1:] * left
            v = nv
            logp = logp + np.log(mean) - np.log(L(i))
        if float(logp.max()) > -60.0:
            acc += np.exp(logp)[:, None] * v
    qo = np.empty((k, nq + 1))
    for s in range(k):
        cum = np.concatenate([[L(0)], np.cumsum(acc[s])])
        lev = np.arange(1, nq, dtype=L) / L(nq) * cum[-1]
        i = np.clip(np.searchsorted(cum, lev, side="left"), 1, I) - 1
        qo[s, 1:nq] = edge[i] + (lev - cum[i]) / acc[s][i] * L(h)
        qo[s, 0], qo[s, nq] = edge[0], edge[I]
    return torch.from_numpy(qo).cuda(), torch.from_numpy(acc.astype(np.float64)).cuda()


def _exact_grad(case, seed):
    """The ensemble with its tangents in (lambda, eps, beta, c3); quantiles with the order frozen."""
    n, S, dt = case["n"], case["steps"], case["dt"]
    if n * S > 1.2e10:
        return None
    g = np.random.default_rng(seed)
    lam, eps, beta, c3 = LAM + 0.1 * g.random(), case["eps"], BETA, C3 + 0.1 * g.random()
    seed &= M32
    p = torch.arange(n, device="cuda")
    z0, z1 = _normals(seed, 1, 0, p, 0, False)
    x = 0.5 * z0
    y = x + z1 / math.sqrt(beta)
    tx, ty = torch.zeros((4, n), device="cuda", dtype=torch.float64), torch.zeros((4, n), device="cuda",
                                                                                dtype=torch.float64)
    ty[2] = -0.5 * z1 * beta ** -1.5
    sx, sy = math.sqrt(2 * dt / beta), math.sqrt(2 * dt / (beta * eps))
    for m in range(S):
        z0, z1 = _normals(seed, 0, m, p, 0, False)
        dx = x - y
        jxx = (1.0 - dt * (C1 + lam)) - (3.0 * dt * c3) * (x * x)
        nx, ny = tx * jxx + (dt * lam) * ty, torch.lerp(ty, tx, dt / eps)
        nx[0] -= dt * dx
        nx[2] -= (0.5 * sx / beta) * z0
        nx[3] -= dt * x ** 3
        ny[1] -= (dt / eps ** 2) * dx + (0.5 * sy / eps) * z1
        ny[2] -= (0.5 * sy / beta) * z1
        x, y = x - dt * (c3 * x ** 3 + C1 * x + lam * dx) + sx * z0, y + (dt / eps) * dx + sy * z1
        tx, ty = nx, ny
    obs, jac = [(x * x).mean()], [(2.0 * x * tx).mean(dim=1)]
    order = x.sort()
    for al in (0.1, 0.5, 0.9):
        t = al * n - 0.5
        r = int(math.floor(t))
        f = t - r
        i, j = order.indices[r], order.indices[r + 1]
        obs.append((1 - f) * x[i] + f * x[j])
        jac.append((1 - f) * tx[:, i] + f * tx[:, j])
    w = torch.tensor([1.0, 0.3, -0.2, 0.5], dtype=torch.float64, device="cuda")
    return torch.stack(obs), (w[:, None] * torch.stack(jac)).sum(dim=0)


def exact(case, seed):
    f = {"fine": _exact_fine, "restrict": _exact_restrict, "match": _exact_match, "hist": _exact_hist,
         "coarse": _exact_coarse, "grad": _exact_grad}.get(case["kind"])
    return f(case, seed) if f else None
