"""The cutoff test of the row-sum pass where FP32 cannot decide it.

Jittered lattices whose spacing divides psi: a large part of the pairs lies
within 1e-5 relative of psi^2, on either side, so nearly every chunk of 32
candidates of every wave meets the band that only the FP64 test decides.
Spacing psi gives short rows (scanned whole), psi / 2 long ones (trimmed to
each particle's x-window); the sizes leave ragged last groups of candidates,
last waves and last tiles.
"""
import numpy as np
import pytest

from paper_2204_03756_amd import workloads as W

pytestmark = pytest.mark.gpu

from gpu_helpers import PREC_NAMES, TOL, load_mt, normwise, say  # noqa: E402


@pytest.fixture(scope="module")
def mt():
    return load_mt()


@pytest.mark.parametrize("prec", [W.FP64, W.FP32W_FP64ACC, W.FP32_KAHAN])
@pytest.mark.parametrize("shape,psi", [((41, 29), 1.0), ((41, 29), 2.0), ((13, 12, 11), 1.0), ((13, 12, 11), 2.0)])
def test_pairs_at_the_cutoff(mt, oracle, shape, psi, prec):
    """Sec. 3, Eq. (1): pair count, the transfer pass's pairs and the masses
    of one step equal the oracle's."""
    dim = len(shape)
    rng = np.random.Generator(np.random.Philox(20221209 + dim))
    g = np.stack(np.meshgrid(*[np.arange(1.0, k + 1.0) for k in shape], indexing="ij"), -1).reshape(-1, dim)
    # steps of 2^-18: exact in FP32 up to 64, at most 7.6e-6 relative in r^2 each
    x = g + rng.integers(-1, 2, size=g.shape) * 2.0 ** -18
    m = rng.random((1, len(x)))
    hi = [k + 2.0 for k in shape] + [0.0] * (3 - dim)
    p = W.Params(dim=dim, n=len(x), lo=[0.0] * 3, hi=hi, d_rw=0.0, d_mt=psi * psi / 3.6, dt=0.1, beta=0.5, psi=psi,
                 precision=prec)
    say(f"  cutoff ties {shape} psi={psi} {PREC_NAMES[prec]}")
    with mt.Sim(p, x, m, allocator=mt.TorchAllocator("cuda:0")) as sim:
        sim.step(1)
        got, st, (row, col) = sim.masses(), sim.stats(), sim.step_neighbors(1)
    ref = oracle.run(p, x, m, 1)
    orow, ocol = oracle.neighbors(x, psi, "brute")
    d = np.repeat(np.arange(len(x)), np.diff(orow))
    q = ((x[d] - x[ocol]) ** 2).sum(axis=1) / psi ** 2
    assert np.mean((q > 1 - 1e-5) & (d != ocol)) > 0.05      # the case tests what it says
    assert st["pairs_last"] == int(ref.pairs[-1])
    assert np.array_equal(row, orow) and np.array_equal(col, ocol)
    assert normwise(got, ref.m) <= TOL[prec]
