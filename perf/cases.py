"""The work that a user of the library has it do, as cases that can be timed.

A case is a dict of plain values; `listed()` gives the standing ones, `draw(rng)` one more of
the same ranges.  `prepare(case, seed)` makes on the GPU what a program holds before the call,
`run(state)` makes one pass through the public entry points and returns its outputs,
`work(case)` gives the bytes and operations that the pass cannot do without, and
`exact(case, seed)` the same outputs in 64-bit arithmetic by plain torch, where that is short.

Inputs follow the package's own recipe (`paper_1601_05904_amd/workloads.py`): data uniform or a
Gaussian mixture over a uniform background, z = sin 6x cos 6y + 0.01 noise, uniform queries;
`extent` 0 keeps coordinates on the 2^-20 lattice in [0, 1), a positive one spreads them over a
square of that side with its corner at (extent, 2 extent), as projected map coordinates are.
"""
import math

import torch

import paper_1601_05904_amd as aidw
import paper_1601_05904_amd.batch as batch
import paper_1601_05904_amd.learned as learned

LEVELS = (1.0, 2.0, 3.0, 4.0, 5.0)
OTHER_LEVELS = (0.5, 1.25, 2.0, 3.5, 7.0)
FEATURE_CELLS = 25
PAIRS_EXACT = 8e10  # n * m up to which the 64-bit sums are short


def listed():
    return [
        # a web request: a few interpolated points over a small survey, all latency and launches
        dict(name="run_small", kind="run", n=1000, m=257, k=10, data="uniform", extent=0.0, levels="default"),
        # the smallest benchmark size
        dict(name="run_4k", kind="run", n=4096, m=4096, k=10, data="uniform", extent=0.0, levels="default"),
        # the middle of the size sweep (100K = 102,400)
        dict(name="run_100k", kind="run", n=102400, m=102400, k=10, data="uniform", extent=0.0, levels="default"),
        # uneven occupancy: the 2^18 mixture
        dict(name="run_clustered_256k", kind="run", n=1 << 18, m=1 << 18, k=15, data="mixture", extent=0.0,
             levels="default"),
        # the headline size
        dict(name="run_1m", kind="run", n=1 << 20, m=1 << 20, k=10, data="uniform", extent=0.0, levels="default"),
        # some thousand points, an odd count, in a large survey in map coordinates, with levels of its own
        dict(name="run_survey", kind="run", n=700001, m=5003, k=7, data="mixture", extent=20000.0, levels="other"),
        # stage 1 alone, the neighbours wanted too (the grid is kept by the program)
        dict(name="knn_1m", kind="knn", n=1 << 20, m=1 << 20, k=10, data="uniform", extent=0.0),
        # the grid of a new survey
        dict(name="grid_1m", kind="grid", n=1 << 20, m=1 << 20, k=10, data="mixture", extent=0.0),
        # stage 2 alone, without a grid: another field z over known neighbour distances
        dict(name="interp_ragged", kind="interp", n=65539, m=200003, k=10, data="uniform", extent=1000.0,
             levels="default"),
        # the learned form: the network decides where the certificate is tried
        dict(name="learned_1m", kind="learned", n=1 << 20, m=1 << 20, k=15, data="mixture", extent=0.0,
             levels="default"),
        # training the network: two epochs over 100 k pairs
        dict(name="train_100k", kind="train", pairs=100000, epochs=2, batch=1024),
        # many jobs of uneven size as one plan, replayed
        dict(name="batch_48", kind="batch", jobs=48, lo=1024, hi=65536, graph=True),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("run", "run", "run", "run", "knn", "grid", "interp", "learned", "batch", "train"))
    if kind == "train":
        return dict(kind=kind, pairs=_log(rng, 5000, 100000), epochs=rng.randint(1, 2),
                    batch=rng.choice((256, 1000, 1024)))
    if kind == "batch":
        hi = _log(rng, 4096, 65536)
        return dict(kind=kind, jobs=rng.randint(3, 48), lo=max(100, hi // 64), hi=hi, graph=rng.random() < 0.5)
    c = dict(kind=kind, n=_log(rng, 300, 1 << 20), m=_log(rng, 100, 1 << 20), k=rng.choice((7, 8, 10, 12, 15)),
             data=rng.choice(("uniform", "mixture")), extent=rng.choice((0.0, 0.0, 1000.0, 20000.0)))
    if kind in ("run", "interp", "learned"):
        c["levels"] = rng.choice(("default", "default", "other"))
    if kind == "learned":
        c["n"], c["k"], c["levels"] = max(c["n"], 4096), 15, "default"
    return c


# ---------------------------------------------------------------- inputs

def _uniform(g, count):
    return torch.floor(torch.rand(count, generator=g, device="cuda", dtype=torch.float64) * 2 ** 20) / 2 ** 20


def _points(g, n, data, ncomp):
    x, y = _uniform(g, n), _uniform(g, n)
    if data == "mixture":
        cx, cy = _uniform(g, ncomp), _uniform(g, ncomp)
        comp = torch.randint(0, ncomp, (n,), generator=g, device="cuda")
        px = cx[comp] + 0.02 * torch.randn(n, generator=g, device="cuda", dtype=torch.float64)
        py = cy[comp] + 0.02 * torch.randn(n, generator=g, device="cuda", dtype=torch.float64)
        keep = (px >= 0) & (px < 1) & (py >= 0) & (py < 1)
        keep &= torch.rand(n, generator=g, device="cuda") >= 0.1
        x = torch.where(keep, torch.floor(px * 2 ** 20) / 2 ** 20, x)
        y = torch.where(keep, torch.floor(py * 2 ** 20) / 2 ** 20, y)
    return x, y


def _dataset(g, n, m, data, extent, ncomp=16):
    x, y = _points(g, n, data, ncomp)
    z = torch.sin(6 * x) * torch.cos(6 * y) + 0.01 * torch.randn(n, generator=g, device="cuda", dtype=torch.float64)
    qx, qy = _uniform(g, m), _uniform(g, m)
    if extent > 0:
        x, qx = (extent + extent * v for v in (x, qx))
        y, qy = (2 * extent + extent * v for v in (y, qy))
    return tuple(v.float() for v in (x, y, z, qx, qy))


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _levels(case):
    return OTHER_LEVELS if case.get("levels") == "other" else LEVELS


def _jobs(case, seed):
    """The jobs of a batch: sizes by the seed, n log-uniform, m = n, k from {8, 10, 15}, half of
    them uniform and half 8-component mixtures."""
    g = _gen(seed)
    count = case["jobs"]
    u = torch.linspace(0, 1, count, dtype=torch.float64)
    jobs = []
    for j in range(count):
        n = int(round(case["lo"] * (case["hi"] / case["lo"]) ** float(u[j])))
        k = (8, 10, 15)[j % 3]
        jobs.append((_dataset(g, n, n, "mixture" if j % 2 else "uniform", 0.0, 8), k))
    return jobs


def _train_set(case, seed):
    """Feature rows with the counts' and offsets' ranges, and targets in [0, 3]."""
    g = _gen(seed)
    feat = torch.empty((case["pairs"], learned.N_IN), device="cuda")
    counts = torch.poisson(torch.full((case["pairs"], FEATURE_CELLS), 2.0, device="cuda"), generator=g)
    feat[:, :FEATURE_CELLS] = counts / 2.0
    feat[:, FEATURE_CELLS:] = torch.rand((case["pairs"], 2), generator=g, device="cuda")
    target = (1.5 / feat[:, :FEATURE_CELLS].mean(1).clamp_min(0.2).sqrt()).clamp_max(3.0)
    return feat.contiguous(), target.contiguous()


def prepare(case, seed):
    kind = case["kind"]
    s = dict(kind=kind)
    if kind == "train":
        s["feat"], s["target"] = _train_set(case, seed)
        s["epochs"], s["batch"] = case["epochs"], case["batch"]
        return s
    if kind == "batch":
        jobs = [batch.Job(*t, params=aidw.Params(k=k)) for t, k in _jobs(case, seed)]
        torch.cuda.synchronize()
        s["plan"] = batch.Plan(jobs, batch.Config(q=1, split_points=4096, workers_per_cu=8,
                                                  use_graph=1 if case["graph"] else 0))
        s["stream"] = torch.cuda.Stream()
        return s
    g = _gen(seed)
    x, y, z, qx, qy = _dataset(g, case["n"], case["m"], case["data"], case["extent"])
    p = aidw.Params(k=case["k"], levels=_levels(case))
    s.update(x=x, y=y, z=z, qx=qx, qy=qy, p=p)
    if kind == "knn":
        s["grid"] = aidw.build_grid(x, y, qx, qy, p)
    elif kind == "interp":
        grid = aidw.build_grid(x, y, qx, qy, p)
        s["r_obs"], s["d1sq"], _ = aidw.knn(grid, qx, qy, p.k)
        s["p"] = aidw.Params(k=p.k, levels=p.levels, area=grid.describe()["area"])
        grid.close()
    elif kind == "learned":
        tx, ty, _, tqx, tqy = _dataset(g, 1 << 16, 40000, case["data"], case["extent"])
        grid = aidw.build_grid(tx, ty, tqx, tqy, p)
        feat, _ = learned.features(grid, tqx, tqy, want_d1sq=False)
        target = aidw.nn_statistic(grid, tqx, tqy, p.k, 3.0)
        grid.close()
        s["mlp"] = learned.MLP(seed=1)
        s["mlp"].train(feat, target, epochs=8, batch=1024, lr=2e-3, seed=1)
    return s


def run(s):
    kind = s["kind"]
    if kind == "run":
        qz, alpha, r_obs = aidw.run(s["x"], s["y"], s["z"], s["qx"], s["qy"], s["p"], want_alpha=True, want_robs=True)
        return {"qz": qz, "alpha": alpha, "r_obs": r_obs}
    if kind == "knn":
        r_obs, d1sq, idx = aidw.knn(s["grid"], s["qx"], s["qy"], s["p"].k, want_d1sq=True, want_idx=True)
        return {"r_obs": r_obs, "d1sq": d1sq, "idx": idx}
    if kind == "grid":
        grid = aidw.build_grid(s["x"], s["y"], s["qx"], s["qy"], s["p"])
        starts, sx, sy, sidx = grid.arrays()
        grid.close()
        return {"starts": starts, "sx": sx, "sy": sy, "sidx": sidx}
    if kind == "interp":
        qz, alpha = aidw.interpolate(s["x"], s["y"], s["z"], s["qx"], s["qy"], s["r_obs"], s["d1sq"], s["p"],
                                     want_alpha=True)
        return {"qz": qz, "alpha": alpha}
    if kind == "learned":
        qz, alpha, _, count = learned.run_learned(s["x"], s["y"], s["z"], s["qx"], s["qy"], s["p"], s["mlp"],
                                                  rule=learned.NETWORK_GATED_CERTIFICATE, delta=0.3, want_alpha=True)
        return {"qz": qz, "alpha": alpha, "knn_queries": count}
    if kind == "train":
        mlp = learned.MLP(seed=3)
        losses = mlp.train(s["feat"], s["target"], epochs=s["epochs"], batch=s["batch"], lr=2e-3, seed=7)
        params = mlp.get_params()
        mlp.close()
        return {"params": params, "losses": losses}
    s["plan"].run(s["stream"])
    return s["plan"].qz


# ---------------------------------------------------------------- bounds and 64-bit results

def _search_work(n, m, k):
    """Stage 1: each point binned, each query compared with its k neighbours at least."""
    return 12.0 * n + 8.0 * k * m


def work(case):
    """Each input read once and each output written once.  The sums over all n points of a query
    are not n * m operations that nothing can avoid (a hierarchical summation forms them in far
    fewer), so only the operations per point, per query and per neighbour are counted."""
    kind = case["kind"]
    if kind == "train":
        steps = case["pairs"] * case["epochs"]
        return {"bytes": 4.0 * (case["pairs"] * (learned.N_IN + 1) + learned.N_PARAMS),
                "flops": 6.0 * (27 * 64 + 64 * 64 + 64) * steps}
    if kind == "batch":
        sizes = [(int(round(case["lo"] * (case["hi"] / case["lo"]) ** (j / max(1, case["jobs"] - 1)))), (8, 10, 15)[j % 3])
                 for j in range(case["jobs"])]
        return {"bytes": sum(24.0 * n for n, _ in sizes),
                "flops": sum(_search_work(n, n, k) + 10.0 * (k + 1) * n for n, k in sizes)}
    n, m, k = case["n"], case["m"], case["k"]
    if kind == "grid":
        cells = n / 2
        return {"bytes": 8.0 * (n + m) + 12.0 * n + 4.0 * cells, "flops": 12.0 * n + 4.0 * m}
    if kind == "knn":
        return {"bytes": 8.0 * n + 8.0 * m + (8.0 + 4.0 * k) * m, "flops": _search_work(n, m, k)}
    if kind == "interp":
        return {"bytes": 12.0 * n + 16.0 * m + 8.0 * m, "flops": 4.0 * n + 10.0 * k * m}
    outs = 8.0 if kind == "learned" else 12.0
    return {"bytes": 12.0 * n + 8.0 * m + outs * m, "flops": _search_work(n, m, k) + 4.0 * n + 10.0 * k * m}


def _alpha64(R, levels, r_min=0.0, r_max=2.0):
    mu = 0.5 - 0.5 * torch.cos(math.pi / r_max * (R - r_min))
    mu = torch.where(R <= r_min, torch.zeros_like(R), torch.where(R >= r_max, torch.ones_like(R), mu))
    knots = (0.1, 0.3, 0.5, 0.7, 0.9)
    a = torch.full_like(mu, levels[0])
    for i in range(4):
        t = 5.0 * (mu - knots[i])
        a = torch.where(mu > knots[i], levels[i] * (1.0 - t) + levels[i + 1] * t, a)
    return torch.where(mu > knots[4], torch.full_like(mu, levels[4]), a)


def _aidw64(x, y, z, qx, qy, k, levels):
    """(z, alpha, r_obs) of every query by Eq. 1-6 in float64."""
    n, m = x.numel(), qx.numel()
    area = ((torch.maximum(x.max(), qx.max()).double() - torch.minimum(x.min(), qx.min()).double())
            * (torch.maximum(y.max(), qy.max()).double() - torch.minimum(y.min(), qy.min()).double()))
    r_exp = 1.0 / (2.0 * torch.sqrt(n / area))
    xd, yd, zd = x.double(), y.double(), z.double()
    out = [[], [], []]
    step = max(1, (1 << 26) // n)
    for lo in range(0, m, step):
        d2 = (qx[lo:lo + step].double()[:, None] - xd) ** 2
        d2 += (qy[lo:lo + step].double()[:, None] - yd) ** 2
        near = torch.topk(d2, k, dim=1, largest=False, sorted=True).values
        r_obs = near.sqrt().mean(1)
        alpha = _alpha64(r_obs / r_exp, levels)
        d1 = near[:, :1]
        w = (d2 / torch.where(d1 > 0, d1, torch.ones_like(d1))).log_()
        w *= -0.5 * alpha[:, None]
        w.exp_()
        hit = d1[:, 0] == 0
        if bool(hit.any()):
            w[hit] = (d2[hit] == 0).double()
        out[0].append((w @ zd) / w.sum(1))
        out[1].append(alpha)
        out[2].append(r_obs)
    return tuple(torch.cat(v) for v in out)


def exact(case, seed):
    kind = case["kind"]
    if kind == "batch":
        if case["jobs"] * case["hi"] ** 2 > PAIRS_EXACT * 4:
            return None
        return [_aidw64(*t, k, LEVELS)[0] for t, k in _jobs(case, seed)]
    if kind not in ("run", "interp", "learned", "knn") or float(case["n"]) * case["m"] > PAIRS_EXACT:
        return None
    x, y, z, qx, qy = _dataset(_gen(seed), case["n"], case["m"], case["data"], case["extent"])
    qz, alpha, r_obs = _aidw64(x, y, z, qx, qy, case["k"], _levels(case))
    if kind == "knn":
        return {"r_obs": r_obs, "d1sq": None, "idx": None}
    if kind == "run":
        return {"qz": qz, "alpha": alpha, "r_obs": r_obs}
    if kind == "interp":
        return {"qz": qz, "alpha": alpha}
    return {"qz": qz, "alpha": alpha, "knn_queries": None}
