"""3-d sims whose rule for few tiles gives them more tiles than the memory of
their pair counts holds: the counts then lie behind the tiles' mass sums.  One and
three species, more and fewer tiles than set-up blocks, a sim with neighbour
lists; counters and totals after every read against the oracle."""
import numpy as np
import pytest

from paper_2204_03756_amd import workloads as W

pytestmark = pytest.mark.gpu

from gpu_helpers import TOL, load_mt, normwise, say  # noqa: E402


@pytest.fixture(scope="module")
def mt():
    return load_mt()


# (particles, per unit of volume, species, precision, row-sum tiles, transfer tiles, lists); in
# waves of particles the row-sum tiles were 256, 320, 256, 256 and 280
CASES = [(63_709, 1.0, 1, W.FP64, 400, 400, False), (63_709, 1.0, 3, W.FP64, 400, 360, False),
         (63_709, 1.0, 3, W.FP32W_FP64ACC, 400, 360, False), (75_177, 1.0, 1, W.FP32_KAHAN, 264, 264, False),
         (75_177, 0.5, 3, W.FP64, 336, 336, True)]


@pytest.mark.parametrize("d_rw", [0.5, 0.0])
@pytest.mark.parametrize("n,density,ns,prec,tiles,ttiles,lists", CASES)
def test_counters_and_totals(mt, oracle, n, density, ns, prec, tiles, ttiles, lists, d_rw):
    rng = np.random.Generator(np.random.Philox(20230117))
    side = (n / density) ** (1 / 3)
    p = W.Params(dim=3, n=n, lo=[0.0] * 3, hi=[side] * 3, d_rw=d_rw, d_mt=0.5, dt=0.1, seed=11, n_species=ns,
                 precision=prec)
    x, m = rng.random((n, 3)) * side, rng.random((ns, n))
    say(f"  pair room n={n} ns={ns} precision={prec} d_rw={d_rw}")
    with mt.Sim(p, x, m, allocator=mt.TorchAllocator("cuda:0")) as sim:
        plan = mt.mtpt_sim_plan(sim.h)
        assert (plan["tiles"], plan["ttiles"], plan["lists"]) == (tiles, ttiles, lists)
        sim.step(1)
        first = sim.stats()
        sim.step(2)
        last, got = sim.stats(), sim.masses()
    ref = oracle.run(p, x, m, 3)
    assert first["pairs_last"] == int(ref.pairs[0])
    assert last["pairs_total"] == int(ref.pairs.sum()) and last["pairs_last"] == int(ref.pairs[2])
    assert normwise(got, ref.m) <= TOL[prec]
    want = got.sum(axis=1)               # FP64 sums of the exported masses, any order
    assert np.all(np.abs(np.asarray(last["mass_total"])[:ns] - want) <= 1e-12 * np.abs(want))
