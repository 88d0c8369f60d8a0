"""Totals of 3-d FP64 sims are the same bit for bit alone (neighbour lists) and
in a pool (neighbour masks): list tiles of two transfer tiles along each axis,
with the second missing at the edge of the grid, and of one, with at most and
with more particles than the workgroup has threads."""
import numpy as np
import pytest

from paper_2204_03756_amd import workloads as W

pytestmark = pytest.mark.gpu

from gpu_helpers import load_mt, say  # noqa: E402


@pytest.fixture(scope="module")
def mt():
    return load_mt()


# (particles, box, species, axis of the two transfer tiles (None: one), particles in the first tile's cells)
CASES = [(899, [18.1, 5.3, 13.1], 1, 0, 0), (9001, [20.8, 20.8, 20.8], 3, 0, 0), (1411, [8.8, 12.6, 22.8], 3, 0, 420),
         (1189, [14.7, 10.7, 8.0], 1, 1, 0), (1267, [19.0, 5.2, 15.0], 3, 1, 0), (1155, [8.4, 16.9, 10.2], 1, 2, 0),
         (1189, [8.8, 7.2, 23.5], 3, 2, 0), (1051, [20.4, 7.1, 10.6], 1, None, 0), (1101, [13.3, 15.8, 11.6], 3, None, 560)]


@pytest.mark.parametrize("d_rw", [0.3, 0.0])
@pytest.mark.parametrize("n,hi,ns,axis,first", CASES)
def test_totals_alone_equal_the_pools(mt, monkeypatch, n, hi, ns, axis, first, d_rw):
    monkeypatch.setenv("MTPT_MIN_TILES", "1")
    rng = np.random.Generator(np.random.Philox(20230105 + n))
    psi = 1.1
    p = W.Params(dim=3, n=n, lo=[0.0] * 3, hi=hi, d_rw=d_rw, d_mt=psi * psi / 3.6, dt=0.1, psi=psi, seed=5, n_species=ns,
                 k_react=1.0 if ns == 3 else 0.0, precision=W.FP64)
    plan = mt.mtpt_plan(p)
    x, m = rng.random((n, 3)) * hi, rng.random((ns, n))
    x[:first] = rng.random((first, 3)) * (np.array(plan["tile"]) * psi)
    two = [k for k in range(3) if plan["tile"][k] != plan["ttile"][k]]
    assert plan["lists"] and two == ([] if axis is None else [axis])
    say(f"  totals n={n} ns={ns} tile {plan['tile']} of {plan['ttile']} d_rw={d_rw}")
    alloc = mt.TorchAllocator("cuda:0")
    with mt.Sim(p, x, m, allocator=alloc) as sim:
        assert mt.mtpt_sim_plan(sim.h)["lists"]
        sim.step(3)
        alone, masses = sim.stats(), sim.masses()
    pool = mt.mtpt_pool_create(0, 1, None, alloc)
    try:
        t = mt.mtpt_pool_admit(pool, p, x, m, 3)
        for _ in range(3):
            mt.mtpt_pool_tick(pool)
        pooled = mt.mtpt_pool_stats(pool, t)
        assert np.array_equal(mt.mtpt_pool_result(pool, t, n, ns), masses)
    finally:
        mt.mtpt_pool_destroy(pool)
    assert pooled == alone
