"""The hierarchical summation of Eq. 1 (large jobs) against Eq. 1 in float64 over all pairs, at
the shapes where its parts can go wrong: ragged sizes, strips, gaps between clusters, queries in
voids, coincident points, every kind of level, fields that vanish near the query, and inputs it
hands back to the pair kernel.

Bars: the library's stated 1e-5 in the normwise relative metric for every query, and 2e-7 in the
root mean square: a weight t^(-alpha/2) of the pair kernels carries up to about alpha/2 + 2 float32
roundings (alpha <= 7: 6 x 6e-8 = 4e-7 at most, half of it typical), which the weighted mean
averages; the truncation bound of a square is 2^-22 = 2.4e-7 of a query's sums, met only by points
in the square's corner."""
import numpy as np
import pytest

from paper_1601_05904_amd import workloads as W

pytestmark = pytest.mark.gpu

MAX_TOL, RMS_TOL = 1e-5, 2e-7


@pytest.fixture(scope="module")
def T():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1601_05904_amd as aidw
    aidw.load(build_if_missing=False)
    return torch


def aidw_mod():
    import paper_1601_05904_amd as aidw
    return aidw


def reference(T, x, y, z, qx, qy, alpha, sel):
    """(z, sum w|z| / sum w) of the selected queries by Eq. 1 in float64 with the given alpha."""
    out, norm = [], []
    xd, yd, zd = x.double(), y.double(), z.double()
    for i in range(0, len(sel), 16):
        s = sel[i:i + 16]
        d2 = (qx[s].double()[:, None] - xd) ** 2 + (qy[s].double()[:, None] - yd) ** 2
        d1 = d2.min(1, keepdim=True).values
        w = T.exp(T.log(d2 / T.where(d1 > 0, d1, T.ones_like(d1))) * (-0.5 * alpha[s].double()[:, None]))
        w = T.where(d1 == 0, (d2 == 0).double(), w)
        den = w.sum(1)
        out.append((w * zd).sum(1) / den)
        norm.append((w * zd.abs()).sum(1) / den)
    return T.cat(out), T.cat(norm)


def check(T, data, params, sample=384, rms_tol=RMS_TOL):
    aidw = aidw_mod()
    x, y, z, qx, qy = (T.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).to("cuda") for a in data)
    qz, al, ro = aidw.run(x, y, z, qx, qy, params, want_alpha=True, want_robs=True)
    again = aidw.run(x, y, z, qx, qy, params)
    assert T.equal(qz, again)  # the same inputs, the same bits
    rng = np.random.default_rng(5)
    sel = T.from_numpy(np.sort(rng.choice(len(qx), size=min(sample, len(qx)), replace=False))).to("cuda")
    ref, norm = reference(T, x, y, z, qx, qy, al, sel)
    e = (qz[sel].double() - ref).abs() / T.maximum(ref.abs(), norm).clamp_min(1e-300)
    assert bool(T.isfinite(qz).all())
    print("max %.2e rms %.2e" % (float(e.max()), float(e.square().mean().sqrt())))
    assert float(e.max()) <= MAX_TOL
    assert float(e.square().mean().sqrt()) <= rms_tol
    return x, y, z, qx, qy, qz, al, ro


def make(n, m, seed, kind="uniform"):
    ds = W.make(n, m, 10, seed, kind, 8)
    return [ds.x, ds.y, ds.z, ds.qx, ds.qy]


@pytest.mark.parametrize("occupancy", [0.5, 2.0, 8.0, 40.0])
def test_dense_places(T, occupancy):
    """Clusters of thousands of points inside one leaf, whose squares go on below it (two levels where a
    leaf is 4 x 4 cells or more, one at 2 x 2, none at one cell), in a sparse rest."""
    aidw = aidw_mod()
    rng = np.random.default_rng(61)

    def places(n):
        p = rng.random((n, 2))
        c = rng.integers(0, 4, n // 2)
        p[: n // 2] = np.array([[0.2, 0.3], [0.7, 0.2], [0.25, 0.8], [0.5, 0.5]])[c] + rng.normal(0, 1, (n // 2, 2)) * (
            np.array([0.002, 0.004, 0.008, 0.016])[c, None])
        return W.quantise(p[rng.permutation(n)].clip(0, 1))

    p, q = places(60000), places(40000)
    z = np.sin(9 * p[:, 0]) + np.cos(7 * p[:, 1]) + 0.3
    check(T, [p[:, 0], p[:, 1], z, q[:, 0], q[:, 1]], aidw.Params(k=10, occupancy=occupancy))


@pytest.mark.parametrize("case", ["ragged", "mixture", "levels", "levels_low", "strip", "tall", "few_queries", "few_data",
                                  "map_coords", "fine_cells", "wide_cells", "cell_width"])
def test_shapes(T, case):
    aidw = aidw_mod()
    p = aidw.Params(k=10)
    if case == "ragged":
        d = make(40961, 50009, 801)
    elif case == "mixture":
        d = make(65537, 40001, 802, "mixture")
    elif case == "levels":  # no integer class, alpha up to 7
        d, p = make(50001, 45000, 803, "mixture"), aidw.Params(k=8, levels=(0.5, 1.25, 2.0, 3.5, 7.0))
    elif case == "levels_low":
        d, p = make(50001, 45000, 804), aidw.Params(k=8, levels=(0.05, 0.1, 0.2, 0.4, 0.8))
    elif case in ("strip", "tall"):
        d = make(50000, 50000, 805)
        i = 1 if case == "strip" else 0
        d[i] = d[i] * np.float32(2e-4)
        d[i + 3] = d[i + 3] * np.float32(2e-4)
    elif case == "few_queries":
        d = make((1 << 20) + 13, 9001, 806, "mixture")
    elif case == "few_data":
        d = make(4099, (1 << 19) + 77, 807)
    elif case == "map_coords":
        d = make(60000, 41000, 808)
        d[0], d[3] = (np.float32(20000.0) + np.float32(20000.0) * v for v in (d[0], d[3]))
        d[1], d[4] = (np.float32(40000.0) + np.float32(20000.0) * v for v in (d[1], d[4]))
    elif case == "fine_cells":
        d, p = make(50000, 45000, 809, "mixture"), aidw.Params(k=10, occupancy=0.02)
    elif case == "wide_cells":
        d, p = make(50000, 45000, 810, "mixture"), aidw.Params(k=10, occupancy=60.0)
    else:
        d, p = make(50000, 45000, 811), aidw.Params(k=10, cell_width=0.013)
    check(T, d, p)


@pytest.mark.parametrize("case", ["gap", "void", "diagonal", "lattice", "outlier"])
def test_uneven_places(T, case):
    """Queries on both sides of a gap, queries where no data are near, data and queries along a
    line, coincident points, and one point far from all others."""
    aidw = aidw_mod()
    rng = np.random.default_rng(820)
    n, m = 50000, 45000
    d = make(n, m, 821)
    if case == "gap":  # two squares of data, queries in both and between
        left = rng.random(n) < 0.5
        d[0] = np.where(left, d[0] * 0.1, 0.9 + d[0] * 0.1)
        d[3] = np.where(rng.random(m) < 0.9, np.where(rng.random(m) < 0.5, d[3] * 0.1, 0.9 + d[3] * 0.1), d[3])
    elif case == "void":  # data in a corner, queries everywhere
        d[0], d[1] = d[0] * 0.2, d[1] * 0.2
    elif case == "diagonal":
        t = rng.random(n)
        d[0], d[1] = t, np.clip(t + 0.001 * rng.standard_normal(n), 0, 1)
        t = rng.random(m)
        d[3], d[4] = t, np.clip(t + 0.01 * rng.standard_normal(m), 0, 1)
    elif case == "lattice":
        d[0], d[1] = rng.integers(0, 256, n) / 256.0, rng.integers(0, 256, n) / 256.0
        d[3], d[4] = rng.integers(0, 512, m) / 512.0, rng.integers(0, 512, m) / 512.0
    else:
        d[0][0], d[1][0] = 40.0, 35.0
    check(T, d, aidw.Params(k=10))


@pytest.mark.parametrize("case", ["zero_half", "spikes", "offset", "constant", "tiny"])
def test_fields(T, case):
    """Fields whose values near a query say nothing about the far ones: exact zeros near by, rare
    large spikes, a large offset, a constant, values near the smallest floats."""
    aidw = aidw_mod()
    d = make(50000, 45000, 830)
    rng = np.random.default_rng(831)
    z = d[2].astype(np.float64)
    if case == "zero_half":
        z = np.where(d[0] < 0.5, 0.0, 1.0 + z)
    elif case == "spikes":
        z = np.where(rng.random(z.size) < 1e-3, 1e6 * rng.standard_normal(z.size), 1e-3 * z)
    elif case == "offset":
        z = 1e4 + z
    elif case == "constant":
        z = np.full(z.size, 0.6180339887)
    else:
        z = 1e-30 * z
    d[2] = z.astype(np.float32)
    x, y, z, qx, qy, qz, _, _ = check(T, d, aidw.Params(k=10))
    if case == "constant":
        assert float((qz - z[0]).abs().max()) <= 4e-7


def test_interpolate_alone(T):
    """aidw_interpolate: with and without a grid, data and query arrays off 16-byte alignment,
    queries far outside the data's box and a query whose coordinate is NaN."""
    aidw = aidw_mod()
    d = make(50003, 45001, 840)
    x, y, z, qx, qy = (T.cat([T.zeros(1, device="cuda"), T.from_numpy(a).to("cuda")])[1:] for a in d)
    qx[5], qy[5] = 30.0, -20.0
    p = aidw.Params(k=10)
    g = aidw.build_grid(x, y, qx, qy, p)
    r, d1, _ = aidw.knn(g, qx, qy, 10)
    p = aidw.Params(k=10, area=g.describe()["area"])
    with_grid, al = aidw.interpolate(x, y, z, qx, qy, r, d1, p, grid=g, want_alpha=True)
    g.close()
    without = aidw.interpolate(x, y, z, qx, qy, r, d1, p)
    assert T.equal(with_grid, without)
    sel = T.arange(0, 45001, 150, device="cuda")
    sel[0] = 5
    ref, norm = reference(T, x, y, z, qx, qy, al, sel)
    e = (without[sel].double() - ref).abs() / T.maximum(ref.abs(), norm)
    assert float(e.max()) <= MAX_TOL
    qx2 = qx.clone()
    qx2[7] = float("nan")
    odd = aidw.interpolate(x, y, z, qx2, qy, r, d1, p)
    assert bool(T.isnan(odd[7]))
    keep = T.ones_like(odd, dtype=T.bool)
    keep[7] = False
    assert float((odd[keep] - without[keep]).abs().max()) <= 1e-5


@pytest.mark.parametrize("case", ["nan", "inf", "huge", "dense", "no_area"])
def test_handed_back_to_the_pair_kernel(T, case):
    """Values beyond the moments' range, a leaf of very many points, data without an area: the sums
    are those of the pair kernel (NaN where it gives NaN)."""
    aidw = aidw_mod()
    d = make(50000, 40000, 850)
    if case == "nan":
        d[2][17] = np.nan
    elif case == "inf":
        d[2][17] = np.inf
    elif case == "huge":
        d[2] = d[2] * np.float32(1e33)
    elif case == "dense":
        d[0][:30000] = W.quantise(0.5 + 1e-4 * np.random.default_rng(1).random(30000))
        d[1][:30000] = W.quantise(0.5 + 1e-4 * np.random.default_rng(2).random(30000))
    x, y, z, qx, qy = (T.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).to("cuda") for a in d)
    p = aidw.Params(k=10)
    if case == "no_area":  # interpolation alone, over points on one line
        r = T.full((40000,), 0.01, device="cuda")
        d1 = T.full((40000,), 1e-6, device="cuda")
        x.fill_(0.25)
        p = aidw.Params(k=10, area=1.0)
        run = lambda: aidw.interpolate(x, y, z, qx, qy, r, d1, p)  # noqa: E731
    else:
        run = lambda: aidw.run(x, y, z, qx, qy, p)  # noqa: E731
    got = run()
    aidw.set_interp_config(1, 0, -1)
    try:
        want = run()
    finally:
        aidw.set_interp_config(0, 0, -1)
    assert T.equal(T.isnan(got), T.isnan(want))
    ok = T.isfinite(want)
    scale = float(z[T.isfinite(z)].abs().max())
    if bool(ok.any()):
        assert float((got[ok].double() - want[ok].double()).abs().max()) <= 1e-5 * scale


def test_streams_share_nothing(T):
    """Two hierarchical runs in flight on two streams, over other data, give what each gives alone."""
    aidw = aidw_mod()
    sets = [[T.from_numpy(a).to("cuda") for a in make(50000, 45000, 860 + i, "mixture")] for i in range(2)]
    p = aidw.Params(k=10)
    want = [aidw.run(*s, p) for s in sets]
    T.cuda.synchronize()
    streams = [T.cuda.Stream(), T.cuda.Stream()]
    for _ in range(3):
        got = [aidw.run(*s, p, stream=st) for s, st in zip(sets, streams)]
        T.cuda.synchronize()
        assert all(T.equal(a, b) for a, b in zip(got, want))


@pytest.mark.parametrize("size", ["small", "large"])
def test_batch_jobs(T, size):
    """Jobs on both sides of the batched form's size rule in one plan, replayed as a graph after the
    fields change, against Eq. 1 in float64: uneven kinds and levels, a job whose z holds a NaN, one
    with a leaf of very many points, one without an area."""
    aidw = aidw_mod()
    import paper_1601_05904_amd.batch as B
    specs = [(8191, 700, "uniform", {}), (8192, 256, "uniform", {}), (8192, 255, "mixture", {}), (20011, 9001, "mixture", {}),
             (30000, 12000, "mixture", dict(levels=(0.5, 1.25, 2.0, 3.5, 7.0))), (40000, 3000, "uniform", dict(levels=(1, 2, 3, 4, 9))),
             (10000, 5000, "uniform", {}), (40000, 2000, "uniform", {}), (9000, 500, "uniform", {}), (500, 30000, "uniform", {})]
    if size == "large":  # enough pairs for the hierarchical sums, on both sides of the rules for a job
        specs = [(8191, 60000, "uniform", {}), (8192, 60000, "uniform", {}), (65536, 255, "mixture", {}),
                 (20011, 9001, "mixture", {}), (60000, 40000, "mixture", dict(levels=(0.5, 1.25, 2.0, 3.5, 7.0))),
                 (40000, 40000, "uniform", dict(levels=(1, 2, 3, 4, 9))), (50000, 50000, "uniform", {}),
                 (50000, 40000, "uniform", {}), (9000, 30000, "uniform", {}), (500, 30000, "uniform", {})]
    jobs = []
    for i, (n, m, kind, kw) in enumerate(specs):
        d = make(n, m, 870 + i, kind)
        if i == 6:
            d[2][11] = np.nan
        if i == 7:
            d[0][:30000] = W.quantise(0.5 + 1e-4 * np.random.default_rng(1).random(30000))
            d[1][:30000] = W.quantise(0.5 + 1e-4 * np.random.default_rng(2).random(30000))
        if i == 8:
            d[0][:] = d[3][:] = 0.25
        jobs.append(B.Job(*(T.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).to("cuda") for a in d),
                          params=aidw.Params(k=10, **kw)))
    plan = B.Plan(jobs, B.Config(use_graph=1), want_alpha=True)
    side = T.cuda.Stream()
    T.cuda.synchronize()
    for rep in range(3):
        if rep:
            for jb in jobs:
                jb.z.mul_(1.5).add_(0.125)
            T.cuda.synchronize()
        plan.run(side)
        assert plan.status(side) == [aidw.OK] * 8 + [aidw.EDEGENERATE, aidw.OK]
        for i, jb in enumerate(jobs):
            if i == 8 or i == 6:
                assert bool(T.isnan(plan.qz[i]).all())
                continue
            sel = T.arange(0, plan.qz[i].numel(), max(1, plan.qz[i].numel() // 100), device="cuda")
            ref, norm = reference(T, jb.x, jb.y, jb.z, jb.qx, jb.qy, plan.alpha[i], sel)
            e = (plan.qz[i][sel].double() - ref).abs() / T.maximum(ref.abs(), norm)
            assert float(e.max()) <= MAX_TOL, (rep, i, float(e.max()))
    direct = B.Plan(jobs, B.Config(), want_alpha=True)
    direct.run()
    T.cuda.synchronize()
    for a, b in zip(plan.qz, direct.qz):
        assert T.equal(a.nan_to_num(7.0), b.nan_to_num(7.0))
    for p in (plan, direct):
        p.close()


@pytest.mark.parametrize("n,m", [(60000, 60000), (4300001, 9000)])
def test_points_on_a_line(T, n, m):
    """aidw_interpolate alone needs no area of the data's own: points on a line, which no grid spans, on both
    sides of the size from which the grid it builds is sized by the host."""
    aidw = aidw_mod()
    g = T.Generator(device="cuda").manual_seed(n)
    x = T.rand(n, generator=g, device="cuda")
    z = T.rand(n, generator=g, device="cuda") + 0.5
    qx, qy = T.rand(m, generator=g, device="cuda"), T.rand(m, generator=g, device="cuda")
    y = T.full_like(x, 0.25)
    d1 = (qy - 0.25) ** 2 + 1e-9
    r_obs = T.full_like(qx, 0.01)
    p = aidw.Params(k=10, area=1.0)
    got = aidw.interpolate(x, y, z, qx, qy, r_obs, d1, p)
    aidw.set_interp_config(1, 0, -1)
    try:
        want = aidw.interpolate(x, y, z, qx, qy, r_obs, d1, p)
    finally:
        aidw.set_interp_config(0, 0, -1)
    assert bool(T.isfinite(got).all())
    assert float(((got - want).abs() / want.abs()).max()) <= 2 * MAX_TOL
