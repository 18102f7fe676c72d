"""Plans whose hierarchically summed jobs turn out off, or have no room for their moments."""
import numpy as np
import pytest

from paper_1601_05904_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def T():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1601_05904_amd as aidw
    aidw.load(build_if_missing=False)
    return torch


def job(T, n, m, seed, kind="even", levels=(1, 2, 3, 4, 5)):
    import paper_1601_05904_amd as aidw
    import paper_1601_05904_amd.batch as B
    ds = W.make(n, m, 10, seed, "uniform", 8)
    x, y, z = ds.x.copy(), ds.y.copy(), ds.z.copy()
    if kind == "dense":
        x[:30000], y[:30000] = W.quantise(0.5 + 1e-4 * np.random.default_rng(seed).random((2, 30000)))
    elif kind == "huge":
        z *= np.float32(1e33)
    return B.Job(*(T.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).to("cuda") for a in (x, y, z, ds.qx, ds.qy)),
                 params=aidw.Params(k=10, levels=levels))


def alone(T, jb, split, q=1):
    """The job by itself with every pair evaluated in `split` data ranges."""
    import paper_1601_05904_amd as aidw
    aidw.set_interp_config(q, split, -1)
    try:
        return aidw.run(jb.x, jb.y, jb.z, jb.qx, jb.qy, jb.params)
    finally:
        aidw.set_interp_config(0, 0, -1)


@pytest.mark.parametrize("q", [1, 2])
@pytest.mark.parametrize("split_points", [0, 4096])
@pytest.mark.parametrize("kinds", [("dense",), ("even", "huge", "dense"), ("even", "even")])
def test_off_is_the_pair_kernel(T, kinds, split_points, q):
    """A job that turns out off has the bits of every pair evaluated in the plan's data ranges, among jobs that are
    summed hierarchically and one too small for it; graph replays included."""
    import paper_1601_05904_amd.batch as B
    n, m = 61440, 40000  # 15 ranges of 4096 points
    jobs = [job(T, 3000, 700, 30)] + [job(T, n, m, 31 + i, kind) for i, kind in enumerate(kinds)]
    jobs.append(job(T, n, m, 40, kinds[-1], (0.5, 1.25, 2.5, 3.5, 7.5)))
    plan = B.Plan(jobs, B.Config(q=q, split_points=split_points, use_graph=1))
    side = T.cuda.Stream()
    T.cuda.synchronize()
    for _ in range(3):
        plan.run(side)
        T.cuda.synchronize()
        for i, kind in enumerate(("small",) + kinds + kinds[-1:]):
            split = 1 if split_points == 0 or kind == "small" else 15
            assert T.equal(plan.qz[i], alone(T, jobs[i], split, q)) == (kind != "even"), (i, kind)
        for jb in jobs:
            jb.z.mul_(1.5)
        T.cuda.synchronize()
    plan.close()


def test_no_room_for_the_moments(T, monkeypatch):
    """A plan whose workspace fits only without the moments evaluates every pair."""
    import paper_1601_05904_amd as aidw
    import paper_1601_05904_amd.batch as B
    n, m = 61440, 40000
    jobs = [job(T, n, m, 50 + i) for i in range(2)]
    config = B.Config(split_points=4096)
    full = B.Plan(jobs, config)
    full_bytes = full.describe()["workspace_bytes"]
    full.close()
    # an 80-byte record of a point (its moments and its share of a pool) is left out of the limit
    monkeypatch.setenv("AIDW_FAULT", "alloc:%d" % (full_bytes - 80 * 2 * n))
    plan = B.Plan(jobs, config)
    assert plan.describe()["workspace_bytes"] < full_bytes - 80 * 2 * n
    plan.run()
    T.cuda.synchronize()
    monkeypatch.setenv("AIDW_FAULT", "alloc:1024")
    with pytest.raises(aidw.AidwError):
        B.Plan(jobs, config)
    monkeypatch.delenv("AIDW_FAULT")
    for i, jb in enumerate(jobs):
        assert T.equal(plan.qz[i], alone(T, jb, 15))
    plan.close()
