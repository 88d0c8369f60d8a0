"""The neighbour-list variant of the 3-d FP64 passes against the mask variant
bit for bit and against the oracle: uniform particles (lists of every length,
ragged tiles), a cluster (lists too long for the packing, tiles beyond the
LDS), a slab one cell thick, static sims, one and three species."""
import numpy as np
import pytest

from paper_2204_03756_amd import workloads as W

pytestmark = pytest.mark.gpu

from gpu_helpers import TOL, load_mt, normwise, say  # noqa: E402


@pytest.fixture(scope="module")
def mt():
    return load_mt()


def _case(kind, ns):
    rng = np.random.Generator(np.random.Philox(20221223))
    n, hi, psi, d_rw = 9001, [20.8, 20.8, 20.8], 1.1, 0.3
    if kind == "slab":
        n, hi = 5003, [70.0, 70.0, 1.0]
    x = rng.random((n, 3)) * hi
    if kind == "cluster":               # a blob of 15 to 60 neighbours, and one of ~2000 in two cells
        x[:1500] = np.clip([6.0, 6.0, 6.0] + 1.3 * rng.standard_normal((1500, 3)), 0.0, 20.8)
        x[1500:3500] = np.clip([15.0, 15.0, 15.0] + 0.7 * rng.standard_normal((2000, 3)), 0.0, 20.8)
    if kind == "static":
        d_rw = 0.0
    p = W.Params(dim=3, n=n, lo=[0.0] * 3, hi=hi, d_rw=d_rw, d_mt=psi * psi / 3.6, dt=0.1, psi=psi, seed=5,
                 n_species=ns, k_react=1.0 if ns == 3 else 0.0, precision=W.FP64)
    return W.Workload(kind, p, x, rng.random((ns, n)), 3, {})


@pytest.mark.parametrize("ns", [1, 3])
@pytest.mark.parametrize("kind", ["uniform", "cluster", "slab", "static"])
def test_lists_equal_masks(mt, oracle, monkeypatch, kind, ns):
    w = _case(kind, ns)
    p = w.params
    got = []
    for tiles in ("1", "1000000"):       # at least 1 tile: lists; a million: one cell a tile, masks
        monkeypatch.setenv("MTPT_MIN_TILES", tiles)
        say(f"  lists {kind} ns={ns} min tiles {tiles}")
        with mt.Sim(p, w.x0, w.m0, allocator=mt.TorchAllocator("cuda:0")) as sim:
            sim.step(2)
            sim.stats()
            sim.step(1)
            hot = [sim.step_neighbors(0), sim.step_neighbors(1)]
            got.append((sim.masses(), sim.positions(), sim.stats()["pairs_total"], hot))
    ref = oracle.run(p, w.x0, w.m0, 3)
    orow, ocol = oracle.neighbors(ref.x, p.psi, "kdtree")
    assert np.array_equal(got[0][0], got[1][0])
    for m, x, pairs, hot in got:
        assert np.array_equal(x, ref.x) and pairs == int(ref.pairs.sum())
        assert normwise(m, ref.m) <= TOL[W.FP64]
        for row, col in hot:
            assert np.array_equal(row, orow) and np.array_equal(col, ocol)
