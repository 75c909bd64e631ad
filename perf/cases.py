"""The workloads this library's speed is measured on, through its public entry points.

A case is a dict of plain values whose "kind" names the path:

  jj           sde_jj_integrate: points of the Josephson junction (or of the
               paper's washboard) over many paths, FP32
  jj_f64       sde_jj_integrate_f64: the same in double precision
  mean_field   sde_kuramoto_integrate, Eq. 3 sums (held in registers, or
               streamed through HBM when a realization is too large)
  all_pairs    sde_kuramoto_integrate, the O(N^2) sum of Alg. 3
  dense        sde_kuramoto_integrate with an explicit coupling matrix
  observables  sde_observables: ensemble means, standard errors, order
               parameters of device arrays
  density      sde_position_histograms and sde_phase_histograms: P(x; t) from
               recorded windings and the density of the phases
  predict      sde_surrogate_predict: the ensemble of MLPs over query points
  train        sde_surrogate_train: epochs of minibatch Adam

listed() holds one or two cases of each at the sizes of the library's own
configurations (shorter in steps, where a full run takes seconds: the time
per step does not depend on their number), draw() others of the same ranges.
"""
import math

import numpy as np
import torch

import paper_0903_3852_amd as sde

DEV = "cuda"
WIDTHS = [5, 256, 256, 256, 1]
MEMBERS = 5
CENTER = [4.0, 5.0, 0.25, -2.5, 1.0]
SCALE = [2.0, 2.0, 0.25, 1.5, 0.5]


def listed():
    return [
        # One junction point at the parameters of the paper's Fig. 2 run, 4096 paths x 10^4 steps:
        # the interactive call, which leaves most of the chip idle.
        dict(name="jj_single", kind="jj", points="single", n_points=1, paths=4096, steps=10000, period=400,
             transient=0, scheme=0, resume=False, state=True),
        # Part of the 128 x 128 (f, D) parameter scan with 1024 paths a point: the headline workload.
        dict(name="jj_scan", kind="jj", points="scan", n_points=4096, paths=1024, steps=5000, period=200,
             transient=2500, scheme=0, resume=False, state=False),
        # A ragged batch of random points (paths and steps of each differ), every path's state kept.
        dict(name="jj_batch", kind="jj", points="batch", n_points=192, paths=8192, steps=8000, period=200,
             transient=4000, scheme=0, resume=False, state=True),
        # The precision study of Fig. 2 in FP64: V(x) = sin(2 pi x), dt = 0.01 of the drive period.  Four
        # periods: this potential's paths separate by e every ~130 steps, so later ones cannot be compared.
        dict(name="jj_fig2_f64", kind="jj_f64", points="fig2", n_points=1, paths=1 << 18, steps=400, period=100,
             transient=0, scheme=0, resume=False, state=True),
        # 16 realizations of 65536 oscillators in the mean field, the configuration's own size.
        dict(name="mf_uniform", kind="mean_field", N=65536, R=16, steps=1000, K=3.0, D=0.1, dt=0.01, sigma=1.0,
             every=100, scheme=0, resume=False),
        # Fig. 4: 2^24 identical oscillators, one realization, streamed through HBM.
        dict(name="mf_fig4", kind="mean_field", N=1 << 24, R=1, steps=20, K=4.0, D=1.0, dt=0.01, sigma=0.0,
             every=10, scheme=0, resume=True),
        # Dense heterogeneous coupling, 256 realizations, the split BF16 product.
        dict(name="dense_bf16x3", kind="dense", coupling=sde.SDE_DENSE_BF16X3, N=4096, R=256, steps=20, K=4.0, D=0.05,
             dt=0.005, sigma=0.5, every=10, scheme=0, resume=True),
        # All pairs at a size the paper plots (its small-N end), a few realizations.
        dict(name="all_pairs", kind="all_pairs", N=16384, R=4, steps=10, K=3.0, D=0.1, dt=0.01, sigma=1.0, every=10,
             scheme=0, resume=True),
        # <v> +- its error over the Fig. 2 ensemble (one group of 2^19 paths), from v and from the FP64 window sums.
        dict(name="observables", kind="observables", what="velocity", groups=1, n=1 << 19),
        # P(x; t) of Fig. 2 from the recorded periods of 2^19 paths, and the density of their phases.
        dict(name="density", kind="density", rows=200, n=1 << 19, bins=200, phase_bins=100),
        # The surrogate over 2*10^5 query points.
        dict(name="surrogate_predict", kind="predict", n=200000, hidden=256, layers=3, members=5),
        # Two epochs of 16384 labels in minibatches of 1024.
        dict(name="surrogate_train", kind="train", n=16384, batch=1024, epochs=2, hidden=256, layers=3, members=5),
    ]


def _log(rng, lo, hi):
    """A whole number of [lo, hi], spread over its logarithm."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["jj", "jj", "jj", "jj_f64", "mean_field", "mean_field", "all_pairs", "dense", "dense",
                       "observables", "observables", "density", "predict", "predict", "train"])
    scheme = 1 if rng.random() < 0.25 else 0
    resume = rng.random() < 0.5
    if kind == "jj":
        points = rng.choice(["single", "scan", "batch"])
        if points == "single":  # one point: from a wavefront to a full chip
            paths = _log(rng, 60, 300000)
            steps = min(_log(rng, 200, 20000), max(200, 400000000 // paths))
            n_points = 1
        elif points == "scan":
            n_points, paths = _log(rng, 16, 2000), _log(rng, 100, 3000)
            steps = max(100, min(_log(rng, 500, 8000), 15000000000 // (n_points * paths)))
        else:
            n_points, paths = _log(rng, 5, 150), _log(rng, 500, 9000)
            steps = _log(rng, 1000, 9000)
        return dict(kind="jj", points=points, n_points=n_points, paths=paths, steps=steps,
                    period=rng.choice([100, 200, 365, 400]), transient=rng.choice([0, steps // 2, steps // 3]),
                    scheme=scheme, resume=resume, state=resume or rng.random() < 0.5)
    if kind == "jj_f64":
        if rng.random() < 0.5:
            return dict(kind="jj_f64", points="fig2", n_points=1, paths=_log(rng, 1000, 300000),
                        steps=rng.randint(150, 420), period=100, transient=0, scheme=scheme, resume=resume, state=True)
        paths = _log(rng, 1000, 200000)
        return dict(kind="jj_f64", points="single", n_points=1, paths=paths,
                    steps=max(200, min(_log(rng, 300, 6000), 150000000 // paths)), period=400, transient=100,
                    scheme=scheme, resume=resume, state=True)
    if kind == "mean_field":
        if rng.random() < 0.35:  # streamed
            N = _log(rng, 600000, 16000000)
            return dict(kind="mean_field", N=N, R=1, steps=rng.randint(6, 20), K=4.0, D=1.0, dt=0.01, sigma=0.0,
                        every=rng.choice([5, 10]), scheme=scheme, resume=resume)
        N = _log(rng, 200, 100000)
        R = max(1, min(_log(rng, 1, 64), (1 << 20) // N))
        return dict(kind="mean_field", N=N, R=R, steps=rng.randint(100, 600), K=3.0, D=0.1, dt=0.01, sigma=1.0,
                    every=rng.choice([10, 50, 100]), scheme=scheme, resume=resume)
    if kind == "all_pairs":
        N = _log(rng, 300, 16000)
        R = max(1, min(_log(rng, 1, 16), int(4 * (16384 / N) ** 2)))
        return dict(kind="all_pairs", N=N, R=R, steps=rng.randint(4, 10), K=3.0, D=0.1, dt=0.01, sigma=1.0,
                    every=rng.choice([2, 5]), scheme=scheme, resume=resume)
    if kind == "dense":
        N = _log(rng, 300, 4090)
        R = _log(rng, 8, 256)
        return dict(kind="dense", coupling=rng.choice([sde.SDE_DENSE_FP32, sde.SDE_DENSE_BF16X3, sde.SDE_DENSE_FP16X3]),
                    N=N, R=R, steps=rng.randint(4, 12), K=4.0, D=0.05, dt=0.005, sigma=0.5, every=rng.choice([2, 4]),
                    scheme=scheme, resume=resume)
    if kind == "observables":
        what = rng.choice(["velocity", "phase"])
        groups = _log(rng, 1, 2000)
        return dict(kind="observables", what=what, groups=groups, n=max(2 * groups, _log(rng, 1000, 4000000)))
    if kind == "density":
        n = _log(rng, 3000, 2000000)
        rows = max(1, min(_log(rng, 1, 2000), 100000000 // n))
        return dict(kind="density", rows=rows, n=n, bins=_log(rng, 20, 2000), phase_bins=_log(rng, 20, 2000))
    hidden = rng.choice([256, 256, 256, 128, 100, 200])
    layers = rng.choice([3, 3, 2])
    if kind == "predict":
        return dict(kind="predict", n=_log(rng, 1, 190000), hidden=hidden, layers=layers, members=rng.randint(2, 5))
    batch = rng.choice([256, 512, 1000, 1024])
    return dict(kind="train", n=rng.randint(3 * batch, 16000), batch=batch, epochs=rng.randint(1, 2), hidden=hidden,
                layers=layers, members=rng.randint(2, 5))


# ---------------------------------------------------------------- contexts --
_ctx = {}


def _context(kind):
    """One context per program.  Kuramoto programs that have to reproduce their phases bit for bit pin the launch
    choices (autotuner off: the documented defaults), since the split of the sums rounds differently; the path
    integrators' results do not depend on the launch, and they keep the tuner."""
    pinned = kind in ("mean_field", "all_pairs", "dense")
    if pinned not in _ctx:
        c = sde.sde_create(torch.cuda.current_device())
        if pinned:
            sde.sde_set_option(c, sde.SDE_OPT_AUTOTUNE, 0)
        _ctx[pinned] = c
    return _ctx[pinned]


class _Surrogate:
    """A surrogate handle that is given back with the state that holds it."""

    def __init__(self, ctx, widths, members, seed):
        self.h = sde.sde_surrogate_create(ctx, widths, members, seed)

    def __del__(self):
        sde.sde_surrogate_destroy(self.h)


def _gen(seed, salt=0):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed * 1000003 + salt)
    return g


def _rng(seed, salt=0):
    return np.random.default_rng([seed, salt])


# ------------------------------------------------------------------ inputs --
def _jj_points(case, seed):
    """Columns of the case's points (numpy, one entry a point)."""
    n, kind = case["n_points"], case["points"]
    r = _rng(seed, 1)
    one = np.ones(n)
    c = dict(m=one, gamma=0.9 * one, a=4.2 * one, omega=4.9 * one, f=0.1 * one, D=1e-3 * one,
             n_paths=np.full(n, case["paths"]), steps_per_period=np.full(n, case["period"]),
             n_steps=np.full(n, case["steps"]), n_transient=np.full(n, case["transient"]),
             potential=np.full(n, sde.SDE_POTENTIAL_SIN2PI if kind == "fig2" else sde.SDE_POTENTIAL_SIN))
    if kind == "scan":  # n points of the (f, D) plane
        c["f"] = 0.5 * r.random(n)
        c["D"] = 10.0 ** (-4.0 + 3.0 * np.arange(n) / max(1, n - 1))
    elif kind == "batch":
        c["a"], c["omega"] = r.uniform(2.0, 6.0, n), r.uniform(3.0, 7.0, n)
        c["f"], c["D"] = r.uniform(0.0, 0.5, n), 10.0 ** r.uniform(-4.0, -1.0, n)
        c["gamma"] = r.uniform(0.5, 1.5, n)
        sizes = _rng(n, 11)  # of the case, whatever the seed
        c["n_paths"] = sizes.integers(max(1, case["paths"] // 32), case["paths"] + 1, n)
        c["n_steps"] = sizes.integers(max(1, case["steps"] // 8), case["steps"] + 1, n)
        c["n_transient"] = c["n_steps"] // 2 if case["transient"] else 0 * c["n_steps"]
    return c


def _jj_start(case, seed, total):
    """A state to resume from at step 1000 (an earlier call's end)."""
    g = _gen(seed, 2)
    t = torch.float64 if case["kind"] == "jj_f64" else torch.float32
    theta = torch.rand(total, generator=g, device=DEV, dtype=torch.float32).to(t)
    v = (torch.randn(total, generator=g, device=DEV, dtype=torch.float32) * 0.5).to(t)
    winding = torch.randint(-3, 4, (total,), generator=g, device=DEV, dtype=torch.int32)
    acc = torch.zeros(total, dtype=torch.float64, device=DEV)
    return theta, winding, v, acc


def _omega(case, seed):
    w = (case["sigma"] * _rng(seed, 3).standard_normal(case["N"])).astype(np.float32)
    return torch.from_numpy(w).to(DEV)


def _phases(case, seed):
    """The phases an earlier call left: spread around the circle with a cluster."""
    g = _gen(seed, 4)
    shape = (case["R"], case["N"])
    p = 0.35 + 0.2 * torch.randn(shape, generator=g, device=DEV)
    return (p - torch.floor(p)).clamp_(0.0, 1.0 - 2.0 ** -24).contiguous()


def _coupling(case, seed):
    """Symmetric K_ij = (K/N)(1 + 0.5 u_ij), u_ij ~ U[-1, 1], zero diagonal."""
    N = case["N"]
    u = torch.rand((N, N), generator=_gen(seed, 5), device=DEV) * 2.0 - 1.0
    u = torch.triu(u, 1)
    k = (case["K"] / N) * (1.0 + 0.5 * (u + u.T))
    k.fill_diagonal_(0.0)
    return k.contiguous()


def _query_rows(n, seed, salt):
    """Rows (a, omega, f, log10 D, gamma) of the batch distribution."""
    u = torch.rand((n, 5), generator=_gen(seed, salt), device=DEV)
    lo = torch.tensor([2.0, 3.0, 0.0, -4.0, 0.5], device=DEV)
    hi = torch.tensor([6.0, 7.0, 0.5, -1.0, 1.5], device=DEV)
    return (lo + (hi - lo) * u).contiguous()


def _weights(case, seed, member):
    """A member's weights, of the size training leaves them at."""
    r = _rng(seed, 100 + member)
    w = [5] + [case["hidden"]] * case["layers"] + [1]
    out = []
    for i, o in zip(w, w[1:]):
        b = 1.5 / math.sqrt(i)
        out.append((r.uniform(-b, b, (o, i)).astype(np.float32), r.uniform(-b, b, o).astype(np.float32)))
    return out


def prepare(case, seed):
    kind = case["kind"]
    ctx = _context(kind)
    if kind in ("jj", "jj_f64"):
        cols = _jj_points(case, seed)
        pts = sde.make_points_np(**cols)
        total = int(cols["n_paths"].sum())
        s = dict(ctx=ctx, kind=kind, pts=pts)
        s["run"] = sde.make_run(seed=seed, step0=1000 if case["resume"] else 0, scheme=case["scheme"],
                                init=sde.SDE_INIT_FROM_STATE if case["resume"] else sde.SDE_INIT_PHILOX)
        s["state"] = _jj_start(case, seed, total) if case["state"] else (None, None, None, None)
        s["sums"] = torch.zeros((len(pts), 2), dtype=torch.float64, device=DEV)
        return s
    if kind in ("mean_field", "all_pairs", "dense"):
        coupling = {"mean_field": sde.SDE_MEANFIELD, "all_pairs": sde.SDE_TILED}.get(kind, case.get("coupling"))
        d = sde.sde_kuramoto_desc(case["N"], case["R"], case["K"] if kind != "dense" else 0.0, case["D"], case["dt"],
                                  case["steps"], coupling, 0)
        run_ = sde.make_run(seed=seed, step0=1001 if case["resume"] else 0, scheme=case["scheme"],
                            init=sde.SDE_INIT_FROM_STATE if case["resume"] else sde.SDE_INIT_PHILOX,
                            sample_every=case["every"])
        samples = torch.zeros((case["R"], case["steps"] // case["every"] + 1), dtype=torch.float64, device=DEV)
        return dict(ctx=ctx, kind=kind, desc=d, run=run_, phi=_phases(case, seed), omega=_omega(case, seed),
                    K=_coupling(case, seed) if kind == "dense" else None, samples=samples)
    if kind == "observables":
        n, g = case["n"], case["groups"]
        cuts = np.sort(_rng(seed, 6).integers(0, n + 1, g - 1)) if g > 1 else np.zeros(0, dtype=np.int64)
        counts = np.diff(np.concatenate([[0], cuts, [n]])).astype(np.uint32)
        if case["what"] == "phase":
            x = dict(theta=_phases(dict(R=1, N=n), seed).view(-1))
        else:
            v = -0.015 + 0.9 * torch.randn(n, generator=_gen(seed, 7), device=DEV)
            a = -3000.0 + 800.0 * torch.randn(n, generator=_gen(seed, 8), device=DEV, dtype=torch.float64)
            x = dict(v=v, acc=a)
        return dict(ctx=ctx, kind=kind, counts=counts, **x)
    if kind == "density":
        rows, n = case["rows"], case["n"]
        g = _gen(seed, 9)
        w = torch.empty((rows, n), dtype=torch.int32, device=DEV)
        for r in range(rows):  # the ensemble drifts and spreads from row to row
            w[r] = torch.floor(0.7 * math.sqrt(r + 1.0) * torch.randn(n, generator=g, device=DEV) - 0.02 * r).to(torch.int32)
        theta = _phases(dict(R=1, N=n), seed)
        return dict(ctx=ctx, kind=kind, winding=w, theta=theta, x0=-(case["bins"] // 2), bins=case["bins"],
                    phase_bins=case["phase_bins"],
                    pos=torch.zeros((rows, case["bins"] + 2), dtype=torch.int64, device=DEV),
                    dens=torch.zeros((1, case["phase_bins"] + 1), dtype=torch.int64, device=DEV))
    widths = [5] + [case["hidden"]] * case["layers"] + [1]
    sur = _Surrogate(ctx, widths, case["members"], seed)
    sde.sde_surrogate_set_scaling(sur.h, sde.make_scaling(CENTER, SCALE, 0.01, 0.14, 1))
    X = _query_rows(case["n"], seed, 10)
    if kind == "predict":
        for m in range(case["members"]):
            p = np.concatenate([x.ravel() for W, b in _weights(case, seed, m) for x in (W, b)])
            sde.sde_surrogate_set_params(sur.h, m, p)
        return dict(kind=kind, sur=sur, X=X, mean=torch.zeros(case["n"], device=DEV),
                    spread=torch.zeros(case["n"], device=DEV))
    y = 0.14 * torch.sin(2.0 * X[:, 0] - X[:, 1]) * torch.exp(X[:, 2]) + 0.01 * X[:, 3] * X[:, 4]
    return dict(kind=kind, sur=sur, X=X, y=y.contiguous(), members=case["members"],
                opts=sde.make_train_opts(case["epochs"], case["batch"], lr=1e-3, shuffle_seed=seed))


# --------------------------------------------------------------------- run --
def run(s):
    kind = s["kind"]
    if kind in ("jj", "jj_f64"):
        f = sde.sde_jj_integrate if kind == "jj" else sde.sde_jj_integrate_f64
        theta, winding, v, acc = s["state"]
        f(s["ctx"], s["pts"], s["run"], theta, winding, v, acc, s["sums"])
        return dict(sums=s["sums"]) if theta is None else dict(theta=theta, winding=winding, v=v, acc=acc,
                                                               sums=s["sums"])
    if kind in ("mean_field", "all_pairs", "dense"):
        sde.sde_kuramoto_integrate(s["ctx"], s["desc"], s["run"], s["phi"], s["omega"], s["K"], s["samples"])
        return dict(phi=s["phi"], r=s["samples"])
    if kind == "observables":
        if "theta" in s:
            return dict(order=sde.sde_observables(s["ctx"], sde.SDE_OBS_ORDER, s["theta"], s["counts"]))
        return dict(v=sde.sde_observables(s["ctx"], sde.SDE_OBS_MEAN_F32, s["v"], s["counts"]),
                    v2=sde.sde_observables(s["ctx"], sde.SDE_OBS_MEANSQ_F32, s["v"], s["counts"]),
                    acc=sde.sde_observables(s["ctx"], sde.SDE_OBS_MEAN_F64, s["acc"], s["counts"]))
    if kind == "density":
        sde.sde_position_histograms(s["ctx"], s["winding"], s["x0"], s["bins"], s["pos"])
        sde.sde_phase_histograms(s["ctx"], s["theta"], s["phase_bins"], s["dens"])
        return dict(pos=s["pos"], dens=s["dens"])
    if kind == "predict":
        sde.sde_surrogate_predict(s["sur"].h, s["X"], s["mean"], s["spread"])
        return dict(mean=s["mean"], spread=s["spread"])
    curve = sde.sde_surrogate_train(s["sur"].h, s["X"], s["y"], s["opts"])
    return dict(loss=curve, params=[sde.sde_surrogate_get_params(s["sur"].h, m) for m in range(s["members"])])


# -------------------------------------------------------------------- work --
def work(case):
    """Inputs once, outputs once; FLOPs of the method (a Heun path-step is two drifts, the update and its share of a
    Philox block: about 50; 63 for a mean-field oscillator-step, where the sums come on top; Euler-Maruyama less)."""
    kind = case["kind"]
    if kind in ("jj", "jj_f64"):
        c = _jj_points(case, 0)
        paths = float(c["n_paths"].sum())
        steps = float((c["n_paths"] * c["n_steps"]).sum())
        w = 8 if kind == "jj_f64" else 4
        state = paths * (2 * w + 4 + 8) * ((1 + case["resume"]) if case["state"] else 0)
        return {"bytes": state + 96.0 * case["n_points"], "flops": steps * (35 if case["scheme"] else 50)}
    if kind in ("mean_field", "all_pairs", "dense"):
        N, R, steps = float(case["N"]), case["R"], case["steps"]
        stages = 1 if case["scheme"] else 2
        b = N * R * 4 * (1 + case["resume"]) + 4 * N + 8 * R * (steps // case["every"] + 1)
        if kind == "mean_field":
            return {"bytes": b, "flops": N * R * steps * (47 if case["scheme"] else 63)}
        if kind == "all_pairs":
            return {"bytes": b, "flops": 3.0 * N * N * R * stages * steps}
        return {"bytes": b + 4 * N * N, "flops": 4.0 * N * N * R * stages * steps}
    if kind == "observables":
        n = float(case["n"])
        return {"bytes": 4 * n, "flops": 4 * n} if case["what"] == "phase" else {"bytes": (4 + 4 + 8) * n, "flops": 9 * n}
    if kind == "density":
        cells = float(case["rows"]) * (case["bins"] + 2) + case["phase_bins"] + 1
        return {"bytes": 4.0 * (case["rows"] + 1) * case["n"] + 8 * cells, "flops": 2.0 * (case["rows"] + 1) * case["n"]}
    H, L, n, m = float(case["hidden"]), case["layers"], float(case["n"]), case["members"]
    params = 5 * H + H + (L - 1) * (H * H + H) + H + 1
    macs = 5 * H + (L - 1) * H * H + H
    if kind == "predict":
        return {"bytes": n * 28 + 4 * m * params, "flops": 2 * macs * n * m}
    steps = case["n"] // case["batch"] * case["epochs"]
    return {"bytes": n * 24 + 16 * m * params * steps, "flops": 6 * macs * case["batch"] * steps * m}


# ------------------------------------------------------------------- exact --
_MASK = 0xFFFFFFFF


def _philox(c0, c1, c2, c3, seed):
    """Philox4x32-10 words (int64 tensors of 32-bit values) at the counter (c0, c1, c2, c3)."""
    k0, k1 = seed & _MASK, (seed >> 32) & _MASK
    for _ in range(10):
        p0, p1 = c0 * 0xD2511F53, c2 * 0xCD9E8D57
        c0, c1, c2, c3 = ((p1 >> 32) & _MASK) ^ c1 ^ k0, p1 & _MASK, ((p0 >> 32) & _MASK) ^ c3 ^ k1, p0 & _MASK
        k0, k1 = (k0 + 0x9E3779B9) & _MASK, (k1 + 0xBB67AE85) & _MASK
    return c0, c1, c2, c3


def _whole(x):
    return torch.as_tensor(x, dtype=torch.int64, device=DEV)


def _gauss4(block, a, b, seed):
    """The four Gaussians of block `block` of the streams (a, b): Box-Muller on 24-bit uniforms."""
    x = _philox(torch.full_like(a, block), a, b, torch.zeros_like(a), seed)
    out = []
    for i in (0, 2):
        rho = torch.sqrt(-2.0 * torch.log(((x[i] >> 8) + 1).double() * 2.0 ** -24))
        ang = 2.0 * math.pi * ((x[i + 1] >> 8).double() * 2.0 ** -24)
        out += [rho * torch.cos(ang), rho * torch.sin(ang)]
    return out


def _exact_jj(case, seed):
    cols = _jj_points(case, seed)
    paths = cols["n_paths"]
    total, longest = int(paths.sum()), int(cols["n_steps"].max())
    if float(total) * longest > 2.5e10:
        return None  # too long here
    ids = np.repeat(np.arange(len(paths)), paths)
    q = _whole(ids)
    p = _whole(np.arange(total) - np.repeat(np.cumsum(paths) - paths, paths))
    dt_ = 2.0 * math.pi / (cols["omega"] * cols["steps_per_period"])

    def per(x):  # a point's constant for each of its paths (a number, where all points share it)
        x = np.asarray(x, dtype=np.float64)
        return float(x[0]) if np.all(x == x[0]) else torch.from_numpy(x).to(DEV)[q]

    sin2pi = case["points"] == "fig2"
    period = 1.0 if sin2pi else 2.0 * math.pi  # of the coordinate
    dt, gamma, a, f, sig = (per(x) for x in (dt_, cols["gamma"], cols["a"], cols["f"],
                                             np.sqrt(2.0 * cols["gamma"] * cols["D"] * dt_)))
    n_steps, n_tr = (torch.from_numpy(cols[k].astype(np.int64)).to(DEV)[q] for k in ("n_steps", "n_transient"))
    step0 = 1000 if case["resume"] else 0
    if case["resume"]:
        theta, winding, v, acc = (x.double() for x in _jj_start(case, seed, total))
        x = (theta + winding) * period
    else:
        w = _philox(torch.zeros_like(p), p, q, torch.ones_like(p), seed)
        x = (w[0] >> 8).double() * 2.0 ** -24 * period
        v = -2.0 + 4.0 * ((w[1] >> 8).double() * 2.0 ** -24)
        acc = torch.zeros(total, dtype=torch.float64, device=DEV)
    S = case["period"]
    ragged = int(cols["n_steps"].min()) < longest

    def force(y):
        return -2.0 * math.pi * torch.cos(2.0 * math.pi * y) if sin2pi else -torch.sin(y)

    g = None
    for n in range(step0, step0 + longest):
        if g is None or n % 4 == 0:
            g = _gauss4(n >> 2, p, q, seed)
        ns = sig * g[n % 4]
        e0 = a * math.cos(2.0 * math.pi * (n % S) / S) + f
        e1 = a * math.cos(2.0 * math.pi * ((n + 1) % S) / S) + f
        F1 = force(x) - gamma * v + e0
        if case["scheme"] == sde.SDE_HEUN:
            vt = v + dt * F1 + ns
            F2 = force(x + dt * v) - gamma * vt + e1
            xn, vn = x + 0.5 * dt * (v + vt), v + 0.5 * dt * (F1 + F2) + ns
        else:
            xn, vn = x + dt * v, v + dt * F1 + ns
        if ragged:
            on = n - step0 < n_steps
            x, v = torch.where(on, xn, x), torch.where(on, vn, v)
            acc = acc + torch.where(on & (n >= n_tr), v, 0.0)
        else:
            x, v = xn, vn
            if n >= int(cols["n_transient"][0]):
                acc = acc + v
    end = step0 + cols["n_steps"]
    W = np.maximum(end - cols["n_transient"], 0)
    vbar = acc * per(np.where(W > 0, 1.0 / np.maximum(W, 1), 0.0))
    sums = torch.zeros((len(paths), 2), dtype=torch.float64, device=DEV)
    sums[:, 0].index_add_(0, q, vbar)
    sums[:, 1].index_add_(0, q, vbar * vbar)
    if not case["state"]:
        return dict(sums=sums)
    t = x / period
    return dict(theta=t - torch.floor(t), winding=None, v=v, acc=acc, sums=sums)


def _exact_kuramoto(case, seed):
    N, R, steps = case["N"], case["R"], case["steps"]
    i = _whole(np.arange(N)).repeat(R)
    r = _whole(np.arange(R)).repeat_interleave(N)
    if case["resume"]:
        th = _phases(case, seed).double()
    else:
        th = ((_philox(torch.zeros_like(i), i, r, torch.ones_like(i), seed)[0] >> 8).double() * 2.0 ** -24).view(R, N)
    omega = _omega(case, seed).double()
    K = _coupling(case, seed).double().T.contiguous() if case["kind"] == "dense" else None
    dt = case["dt"]
    sig = math.sqrt(2.0 * case["D"] * dt) / (2.0 * math.pi)
    step0 = 1001 if case["resume"] else 0
    out = []

    def sums(t):
        s, c = torch.sin(2.0 * math.pi * t), torch.cos(2.0 * math.pi * t)
        return s, c, s.sum(1, keepdim=True), c.sum(1, keepdim=True)

    def drift(t):
        s, c, S, C = sums(t)
        if K is None:
            return omega + (case["K"] / N) * (c * S - s * C)
        return omega + (c * (s @ K) - s * (c @ K))

    def order(t):
        _, _, S, C = sums(t)
        out.append(torch.sqrt(S * S + C * C)[:, 0] / N)

    g = None
    for k in range(steps):
        n = step0 + k
        if k % case["every"] == 0:
            order(th)
        if g is None or n % 4 == 0:
            g = _gauss4(n >> 2, i, r, seed)
        ns = sig * g[n % 4].view(R, N)
        F1 = drift(th)
        t = th + dt / (2.0 * math.pi) * F1 + ns
        if case["scheme"] == sde.SDE_HEUN:
            t = th + dt / (4.0 * math.pi) * (F1 + drift(t)) + ns
        th = t - torch.floor(t)
    if steps % case["every"] == 0:
        order(th)
    return dict(phi=th, r=torch.stack(out, 1))


def _exact_observables(case, seed):
    s = prepare(case, seed)
    cuts = np.cumsum(s["counts"].astype(np.int64))[:-1]

    def mean(x):
        x = x.double().cpu().numpy()
        res = np.zeros((case["groups"], 2))
        for k, part in enumerate(np.split(x, cuts)):
            if part.size:
                res[k] = part.mean(), part.std(ddof=1) / math.sqrt(part.size) if part.size > 1 else 0.0
        return res

    if "theta" in s:
        t = 2.0 * math.pi * s["theta"].double()
        z = torch.complex(torch.cos(t), torch.sin(t)).cpu().numpy()
        res = np.zeros((case["groups"], 2))
        for k, part in enumerate(np.split(z, cuts)):
            if part.size:
                res[k] = abs(part.mean()), np.angle(part.mean()) / (2.0 * math.pi)
        return dict(order=res)
    return dict(v=mean(s["v"]), v2=mean(s["v"].double() ** 2), acc=mean(s["acc"]))


def _exact_predict(case, seed):
    X = _query_rows(case["n"], seed, 10).double()
    h0 = (X - torch.tensor(CENTER, device=DEV).double()) / torch.tensor(SCALE, device=DEV).double()
    outs = []
    for m in range(case["members"]):
        h = h0
        layers = _weights(case, seed, m)
        for k, (W, b) in enumerate(layers):
            h = h @ torch.from_numpy(W).to(DEV).double().T.contiguous() + torch.from_numpy(b).to(DEV).double()
            if k + 1 < len(layers):
                h = 0.5 * h * (1.0 + torch.erf(h / math.sqrt(2.0)))
        # the scaling's two numbers are single precision
        outs.append((float(np.float32(0.01)) + float(np.float32(0.14)) * h[:, 0]) * X[:, 1])
    o = torch.stack(outs, 1)
    return dict(mean=o.mean(1), spread=o.std(1, unbiased=True))


def exact(case, seed):
    kind = case["kind"]
    if kind in ("jj", "jj_f64"):
        return _exact_jj(case, seed)
    if kind in ("mean_field", "all_pairs", "dense"):
        return _exact_kuramoto(case, seed)
    if kind == "observables":
        return _exact_observables(case, seed)
    if kind == "predict":
        return _exact_predict(case, seed)
    # The densities are counts.  Training's minibatches come from the C++ library's own shuffle, which numpy and torch
    # do not have.
    return None
