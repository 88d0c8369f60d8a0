"""Which 3-d FP64 sims take neighbour lists, and that their results do not
depend on it: even particles do (a cube, a slab four cells thick, static ones,
a few particles with more neighbours than a list holds, a tile beyond the LDS),
crowded ones and those that a drift gathers at the walls take the masks."""
import numpy as np
import pytest

from paper_2204_03756_amd import workloads as W

pytestmark = pytest.mark.gpu

from gpu_helpers import TOL, load_mt, normwise, say  # noqa: E402

PSI = 1.1


@pytest.fixture(scope="module")
def mt():
    return load_mt()


def _params(n, hi, ns, d_rw=0.3, vel=(0.0, 0.0, 0.0)):
    return W.Params(dim=3, n=n, lo=[0.0] * 3, hi=hi, d_rw=d_rw, d_mt=PSI * PSI / 3.6, dt=0.1, psi=PSI, seed=5,
                    n_species=ns, k_react=1.0 if ns == 3 else 0.0, precision=W.FP64, vel=list(vel))


@pytest.mark.parametrize("ns", [1, 3])
@pytest.mark.parametrize("kind,lists", [("uniform", True), ("slab", True), ("static", True), ("few", True),
                                        ("plume", False), ("clump", False), ("drift", False)])
def test_variant_and_results(mt, oracle, monkeypatch, kind, lists, ns):
    rng = np.random.Generator(np.random.Philox(20230111))
    n, hi = (30_001, [31.0] * 3) if kind in ("few", "clump") else (5003, [33.0, 33.0, 4.6]) if kind == "slab" else \
        (9001, [20.8] * 3)
    p = _params(n, hi, ns, 0.0 if kind == "static" else 0.3, (0.4, 0.0, 0.0) if kind == "drift" else (0.0, 0.0, 0.0))
    x, m = rng.random((n, 3)) * hi, rng.random((ns, n))
    if kind == "plume":
        x = np.clip(10.4 + 4.0 * rng.standard_normal((n, 3)), 0.0, 20.8)
    if kind in ("few", "clump"):        # 18 of 30001 past a list's length; 60 close together
        k = 18 if kind == "few" else 60
        x[:k] = 15.0 + 0.5 * rng.random((k, 3))
    got = []
    for tiles, expect in (("1", lists), ("1000000", False)):   # a million: one cell a tile, masks
        monkeypatch.setenv("MTPT_MIN_TILES", tiles)
        assert mt.mtpt_plan(p)["lists"] == (tiles == "1" and kind != "drift")
        say(f"  list choice {kind} ns={ns} min tiles {tiles}")
        with mt.Sim(p, x, m, allocator=mt.TorchAllocator("cuda:0")) as sim:
            assert mt.mtpt_sim_plan(sim.h)["lists"] == expect
            sim.step(2)
            sim.stats()
            sim.step(1)
            hot = [sim.step_neighbors(0), sim.step_neighbors(1)]
            got.append((sim.masses(), sim.positions(), sim.stats(), hot))
    ref = oracle.run(p, x, m, 3)
    orow, ocol = oracle.neighbors(ref.x, PSI, "kdtree")
    assert np.array_equal(got[0][0], got[1][0])
    for gm, gx, st, hot in got:
        assert np.array_equal(gx, ref.x) and st["pairs_total"] == int(ref.pairs.sum())
        assert normwise(gm, ref.m) <= TOL[W.FP64]
        assert np.all(np.abs(np.array(st["mass_total"][:ns]) - ref.totals[-1, :ns]) <= TOL[W.FP64] * ref.totals[-1, :ns])
        for row, col in hot:
            assert np.array_equal(row, orow) and np.array_equal(col, ocol)


def test_a_tile_beyond_the_lds(mt):
    """560 particles in the middle of one tile of a million: it is scanned from
    global memory, its particles have no lists, and the sim keeps them."""
    rng = np.random.Generator(np.random.Philox(20230112))
    n, side = 1_000_001, 100.0
    p = _params(n, [side] * 3, 1)
    plan = mt.mtpt_plan(p)
    cell = side / int(side / (PSI * (1 + 1e-6)))
    mid = (np.array(plan["tile"]) * 3.5) * cell
    x, m = rng.random((n, 3)) * side, rng.random((1, n))
    x[:560] = mid + 2.5 * cell * rng.uniform(-1, 1, (560, 3))
    say(f"  a tile beyond the LDS, tiles {plan['tile']}")
    alloc = mt.TorchAllocator("cuda:0")
    with mt.Sim(p, x, m, allocator=alloc) as sim:
        assert mt.mtpt_sim_plan(sim.h)["lists"]
        sim.step(2)
        alone, masses = sim.stats(), sim.masses()
    pool = mt.mtpt_pool_create(0, 1, None, alloc)
    try:
        t = mt.mtpt_pool_admit(pool, p, x, m, 2)
        for _ in range(2):
            mt.mtpt_pool_tick(pool)
        assert mt.mtpt_pool_stats(pool, t) == alone
        assert np.array_equal(mt.mtpt_pool_result(pool, t, n, 1), masses)
    finally:
        mt.mtpt_pool_destroy(pool)
