"""3-d sims of few tiles, whose per-tile pair counts lie behind the mass sums
(one species) or whose shapes stay those of more tiles (three species): the
counters and totals of every step against the oracle, read in between and not."""
import numpy as np
import pytest

from paper_2204_03756_amd import workloads as W

pytestmark = pytest.mark.gpu

from gpu_helpers import TOL, load_mt, normwise, say  # noqa: E402


@pytest.fixture(scope="module")
def mt():
    return load_mt()


@pytest.mark.parametrize("d_rw", [0.5, 0.0])
@pytest.mark.parametrize("ns,prec", [(1, W.FP64), (3, W.FP64), (1, W.FP32_KAHAN), (3, W.FP32W_FP64ACC)])
def test_counters_and_totals(mt, oracle, ns, prec, d_rw):
    rng = np.random.Generator(np.random.Philox(20221229))
    n = 54_401
    side = (n / 4.4766) ** (1 / 3)
    p = W.Params(dim=3, n=n, lo=[0.0] * 3, hi=[side] * 3, d_rw=d_rw, d_mt=0.5, dt=0.1, seed=11, n_species=ns,
                 precision=prec)
    x, m = rng.random((n, 3)) * side, rng.random((ns, n))
    say(f"  few tiles ns={ns} precision={prec} d_rw={d_rw}")
    with mt.Sim(p, x, m, allocator=mt.TorchAllocator("cuda:0")) as sim:
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
