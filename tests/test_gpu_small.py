"""Few queries: the data ranges that fill the chip with them, and the kernel that combines the ranges
and replaces coincident queries.

Bar: the library's stated 1e-5 in the normwise relative metric holds for each form, so two forms differ
by at most twice that."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,m", [(12, 5), (127, 1), (128, 257), (129, 64), (513, 255), (1000, 256), (4097, 3000),
                                 (16400, 20), (70001, 300)])
def test_ranges_of_few_queries(n, m):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1601_05904_amd as aidw
    aidw.load(build_if_missing=False)
    rng = np.random.default_rng(n)
    x, y = rng.random((2, n)).astype(np.float32)
    x[n // 2:n // 2 + 3], y[n // 2:n // 2 + 3] = x[0], y[0]  # coincident data points
    z = (rng.random(n) + 0.5).astype(np.float32)
    qx, qy = rng.random((2, m)).astype(np.float32)
    same = rng.random(m) < 0.2
    own = rng.integers(0, n, m)
    own[0] = 0
    same[0] = True
    qx[same], qy[same] = x[own[same]], y[own[same]]
    x, y, z, qx, qy = (torch.from_numpy(a).cuda() for a in (x, y, z, qx, qy))
    p = aidw.Params(k=10)
    got, alpha, r_obs = aidw.run(x, y, z, qx, qy, p, want_alpha=True, want_robs=True)
    grid = aidw.build_grid(x, y, qx, qy, p)
    area = grid.describe()["area"]
    _, d1, _ = aidw.knn(grid, qx, qy, 10)
    grid.close()
    d1 = d1.clone()
    d1[-1] = 0.0  # claims a data point at its place: where there is none, the sums stand
    pa = aidw.Params(k=10, area=area)
    alone = aidw.interpolate(x, y, z, qx, qy, r_obs, d1, pa)
    alone = alone[0] if isinstance(alone, tuple) else alone
    aidw.set_interp_config(1, 1, 1)
    try:
        whole = aidw.run(x, y, z, qx, qy, p)
        whole_alone = aidw.interpolate(x, y, z, qx, qy, r_obs, d1, pa)
        whole_alone = whole_alone[0] if isinstance(whole_alone, tuple) else whole_alone
    finally:
        aidw.set_interp_config(0, 0, -1)
    ref = (z[None].double() * ((qx[:, None] == x) & (qy[:, None] == y))).sum(1) / (
        (qx[:, None] == x) & (qy[:, None] == y)).sum(1)
    at = torch.isfinite(ref)
    assert bool(at[0]) and torch.allclose(got[at].double(), ref[at], rtol=1e-6, atol=0)
    for a, b in ((got, whole), (alone, whole_alone)):
        assert bool(torch.isfinite(a).all())
        assert float(((a - b).abs() / b.abs()).max()) <= 2e-5


@pytest.mark.parametrize("n,m", [(1000, 300), (4096, 4096), (300, 100000), (40961, 50009), (65536, 65536),
                                 (20000, 150000), (333333, 100000)])
def test_captured_after_one_call(n, m):
    """aidw_interpolate captured into a graph right after its first call on a stream, with no other
    memory cached, and replayed after the field has changed."""
    import ctypes
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1601_05904_amd as aidw
    lib = aidw.load(build_if_missing=False)
    rng = np.random.default_rng(n + m)
    x, y, z = (torch.from_numpy(a).cuda() for a in rng.random((3, n)).astype(np.float32))
    qx, qy = (torch.from_numpy(a).cuda() for a in rng.random((2, m)).astype(np.float32))
    grid = aidw.build_grid(x, y, qx, qy, aidw.Params(k=10))
    r_obs, d1, _ = aidw.knn(grid, qx, qy, 10)
    p = aidw.Params(k=10, area=grid.describe()["area"])._c()
    grid.close()
    aidw.release_cached_memory()
    qz = torch.empty(m, device="cuda")
    side = torch.cuda.Stream()
    torch.cuda.synchronize()

    def call():
        assert lib.aidw_interpolate(x.data_ptr(), y.data_ptr(), z.data_ptr(), n, qx.data_ptr(), qy.data_ptr(), m,
                                    r_obs.data_ptr(), d1.data_ptr(), ctypes.byref(p), None, qz.data_ptr(), None,
                                    side.cuda_stream) == aidw.OK

    call()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        call()
    for _ in range(3):
        z.mul_(1.5).add_(0.125)
        torch.cuda.synchronize()
        qz.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        got = qz.clone()
        call()
        torch.cuda.synchronize()
        assert torch.equal(got, qz)


@pytest.mark.parametrize("occupancy", [0.6, 2.0, 40.0])
@pytest.mark.parametrize("kind", ["uniform", "lattice", "piles", "one_place"])
@pytest.mark.parametrize("n,m", [(1, 3), (10, 1), (1000, 257), (1024, 7168), (4096, 4096), (8000, 192), (8191, 1)])
def test_small_grid_matches_the_large_build(n, m, kind, occupancy):
    """The one-workgroup build against the banded one: the same data with the queries repeated until they
    are too many for it must give the same arrays, and every query the same neighbours."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1601_05904_amd as aidw
    aidw.load(build_if_missing=False)
    rng = np.random.default_rng(n + m)
    p, q = rng.random((n, 2)), rng.random((m, 2))
    if kind == "lattice":
        p = np.floor(p * 64) / 64
    elif kind == "piles":  # a few cells with hundreds of points
        p[: n * 3 // 4] = 0.3 + 1e-4 * p[: n * 3 // 4]
    elif kind == "one_place":
        p[:] = 0.5
    x, y, qx, qy = (torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda() for a in
                    (p[:, 0], p[:, 1], q[:, 0], q[:, 1]))
    z = torch.rand(n, device="cuda") + 0.5
    k = min(n, 10)
    prm = aidw.Params(k=k, occupancy=occupancy, area=1.0)
    times = 8193 // m + 1
    many = [a.repeat(times) for a in (qx, qy)]
    got, want = [], []
    for out, qs in ((got, (qx, qy)), (want, many)):
        grid = aidw.build_grid(x, y, *qs, prm)
        out.append(grid.describe())
        out.extend(t.clone() for t in grid.arrays())
        grid.close()
    assert got[0] == want[0]
    for a, b in zip(got[1:], want[1:]):
        assert torch.equal(a, b)
    r = aidw.run(x, y, z, qx, qy, prm, want_alpha=True, want_robs=True)
    r_many = aidw.run(x, y, z, *many, prm, want_alpha=True, want_robs=True)
    assert torch.equal(r[1], r_many[1][:m]) and torch.equal(r[2], r_many[2][:m])


def test_captured_memory_is_not_shared():
    """The memory of a captured call belongs to its graph: no later call takes it, on another stream or its own, it
    survives aidw_release_cached_memory, and a second capture without a call between takes it again."""
    import ctypes
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1601_05904_amd as aidw
    lib = aidw.load(build_if_missing=False)
    n = m = 200000
    rng = np.random.default_rng(3)
    x, y, z = (torch.from_numpy(a).cuda() for a in rng.random((3, n)).astype(np.float32))
    qx, qy = (torch.from_numpy(a).cuda() for a in rng.random((2, m)).astype(np.float32))
    grid = aidw.build_grid(x, y, qx, qy, aidw.Params(k=10))
    r_obs, d1, _ = aidw.knn(grid, qx, qy, 10)
    p = aidw.Params(k=10, area=grid.describe()["area"])._c()
    grid.close()
    side, other = torch.cuda.Stream(), torch.cuda.Stream()

    def call(out, stream):
        assert lib.aidw_interpolate(x.data_ptr(), y.data_ptr(), z.data_ptr(), n, qx.data_ptr(), qy.data_ptr(), m,
                                    r_obs.data_ptr(), d1.data_ptr(), ctypes.byref(p), None, out.data_ptr(), None,
                                    stream.cuda_stream) == aidw.OK
        torch.cuda.synchronize()

    def taken(f):
        """Device memory that f takes beyond what is cached (the moments alone are some 30 MB)."""
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info()[0]
        f()
        torch.cuda.synchronize()
        return before - torch.cuda.mem_get_info()[0]

    outs = [torch.empty(m, device="cuda") for _ in range(4)]
    torch.cuda.synchronize()
    aidw.release_cached_memory()
    used = taken(lambda: call(outs[0], side))
    assert used > 30 << 20
    graphs = [torch.cuda.CUDAGraph() for _ in range(2)]

    def capture(graph, out):
        torch.cuda.synchronize()
        with torch.cuda.graph(graph, stream=side):
            assert lib.aidw_interpolate(x.data_ptr(), y.data_ptr(), z.data_ptr(), n, qx.data_ptr(), qy.data_ptr(), m,
                                        r_obs.data_ptr(), d1.data_ptr(), ctypes.byref(p), None, out.data_ptr(), None,
                                        side.cuda_stream) == aidw.OK

    for graph, out in zip(graphs, outs):
        capture(graph, out)
    assert taken(lambda: call(outs[2], other)) > used // 2
    assert taken(lambda: call(outs[3], other)) == 0
    assert taken(lambda: aidw.release_cached_memory()) <= -(used // 2)
    assert taken(lambda: call(outs[3], side)) > used // 2
    aidw.release_cached_memory()
    for _ in range(3):
        z.mul_(1.5).add_(0.125)
        for o in outs:
            o.zero_()
        torch.cuda.synchronize()
        for graph in graphs:
            graph.replay()
            torch.cuda.synchronize()
        call(outs[2], other)
        call(outs[3], side)
        assert all(torch.equal(outs[0], o) for o in outs[1:])
