"""Totals of 3-d FP64 sims are the same bit for bit alone (neighbour lists) and
in a pool (neighbour masks): list tiles of two transfer tiles along each axis,
with the second missing at the edge of the grid, and of one, with at most and
with more particles than the workgroup has threads."""
import numpy as np
import pytest

from paper_2204_03756_amd import workloads as W

pytestmark = pytest.mark.gpu

from gpu_helpers import TOL, load_mt, normwise, say  # noqa: E402


@pytest.fixture(scope="module")
def mt():
    return load_mt()


# (particles, box, species, axis of the two transfer tiles (None: one), particles in the first tile's cells)
CASES = [(1311, [19.3, 13.9, 8.3], 1, 0, 0), (9001, [20.8, 20.8, 20.8], 3, 2, 0), (1411, [8.8, 12.6, 22.8], 3, 0, 420),
         (1303, [21.4, 11.0, 11.9], 1, 1, 0), (1267, [19.0, 5.2, 15.0], 3, 1, 0), (1155, [8.4, 16.9, 10.2], 1, 2, 0),
         (1317, [19.0, 6.4, 13.9], 3, 0, 0), (13707, [32.6, 23.7, 24.7], 3, 2, 0), (5301, [18.2, 43.3, 9.7], 3, 1, 0),
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


@pytest.mark.parametrize("d_rw", [0.3, 0.0])
@pytest.mark.parametrize("plume", [False, True])
def test_sums_that_the_ordinary_place_has_no_room_for(mt, oracle, monkeypatch, plume, d_rw):
    """Partial sums in the pid buffer that is free between two place passes (a
    static sim's second one), finalized by the scatter launch: with lists and,
    where the particles crowd together, with masks, alone and in a pool, read
    after every step and at the end only."""
    monkeypatch.setenv("MTPT_MIN_TILES", "1")
    rng = np.random.Generator(np.random.Philox(20230123))
    n, hi, psi = 13707, np.array([32.6, 23.7, 24.7]), 1.1
    p = W.Params(dim=3, n=n, lo=[0.0] * 3, hi=list(hi), d_rw=d_rw, d_mt=psi * psi / 3.6, dt=0.1, psi=psi, seed=6,
                 n_species=3, k_react=1.0, precision=W.FP64)
    x, m = rng.random((n, 3)) * hi, rng.random((3, n))
    if plume:
        x = np.clip(hi / 2 + hi / 6 * rng.standard_normal((n, 3)), 0.0, hi)
    say(f"  sums in the spare pids plume={plume} d_rw={d_rw}")
    alloc = mt.TorchAllocator("cuda:0")
    got = []
    for chunks in ([1] * 6, [6], [2, 3, 1]):
        with mt.Sim(p, x, m, allocator=alloc) as sim:
            assert mt.mtpt_sim_plan(sim.h)["lists"] != plume
            for k in chunks:
                sim.step(k)
                st = sim.stats()
            got.append((st, sim.masses(), sim.positions()))
    pool = mt.mtpt_pool_create(0, 1, None, alloc)
    try:
        t = mt.mtpt_pool_admit(pool, p, x, m, 6)
        for _ in range(6):
            mt.mtpt_pool_tick(pool)
        pooled = mt.mtpt_pool_stats(pool, t)
        assert np.array_equal(mt.mtpt_pool_result(pool, t, n, 3), got[0][1])
    finally:
        mt.mtpt_pool_destroy(pool)
    ref = oracle.run(p, x, m, 6)
    for st, masses, pos in got:
        assert st == pooled and st["pairs_total"] == int(ref.pairs.sum())
        assert np.array_equal(masses, got[0][1]) and np.array_equal(pos, ref.x)
        assert normwise(masses, ref.m) <= TOL[W.FP64]
        assert np.all(np.abs(np.array(st["mass_total"]) - ref.totals[-1]) <= TOL[W.FP64] * ref.totals[-1])
