"""The input checks that several host threads share report the first fault, and
large uploads and exports (pinned, in chunks, in several threads) move every
value."""
import ctypes as C

import numpy as np
import pytest

from paper_2204_03756_amd import mtpt, workloads as W


def _params(n, dim, ns, prec=W.FP64):
    return W.Params(dim=dim, n=n, lo=[0.0] * 3, hi=[1.0] * dim + [0.0] * (3 - dim), d_rw=0.0, d_mt=1e-6, dt=0.1,
                    n_species=ns, precision=prec)


@pytest.mark.parametrize("bad,message", [
    ({"x": [(399_999, 1), (70_001, 2), (300_000, 0)]}, "particle 70001 coordinate 2 = 1.5 outside [0, 1]"),
    ({"x": [(0, 0), (399_999, 2)]}, "particle 0 coordinate 0 = 1.5 outside [0, 1]"),
    ({"m": [(2, 0), (1, 399_999), (1, 200_000)]}, "mass 600000 is not finite"),
    ({"m": [(0, 5)], "x": [(399_999, 2)]}, "particle 399999 coordinate 2 = 1.5 outside [0, 1]"),
])
def test_first_fault_is_reported(bad, message):
    lib = mtpt.load()
    n = 400_000                              # several threads' worth
    x, m = np.full((n, 3), 0.25), np.ones((3, n))
    for i, k in bad.get("x", []):
        x[i, k] = 1.5
    for c, i in bad.get("m", []):
        m[c, i] = np.nan
    p, h = mtpt.make_params(_params(n, 3, 3)), C.c_void_p()
    rc = lib.mtpt_create(C.byref(p), x.ctypes.data_as(mtpt._f64p), m.ctypes.data_as(mtpt._f64p), None, None,
                         C.byref(h))
    assert rc == mtpt.MTPT_E_ARG and not h.value
    assert lib.mtpt_last_error().decode() == message


@pytest.mark.parametrize("i,k,c,j", [(0, 0, 2, 1_499_999), (187_500, 2, 1, 187_499), (1_499_999, 1, 0, 749_999)])
def test_first_fault_of_several_threads(i, k, c, j):
    """67 MiB of inputs: eight ranges, faults at their edges and in more than one."""
    lib = mtpt.load()
    n = 1_500_000
    x, m = np.full((n, 3), 0.25), np.ones((3, n))
    p = mtpt.make_params(_params(n, 3, 3))

    def create():
        h = C.c_void_p()
        rc = lib.mtpt_create(C.byref(p), x.ctypes.data_as(mtpt._f64p), m.ctypes.data_as(mtpt._f64p), None, None,
                             C.byref(h))
        assert rc == mtpt.MTPT_E_ARG and not h.value
        return lib.mtpt_last_error().decode()

    m[c, j] = m[2, n - 1] = np.inf
    assert create() == f"mass {c * n + j} is not finite"
    x[i, k] = x[n - 1, 2] = -0.5
    assert create() == f"particle {i} coordinate {k} = -0.5 outside [0, 1]"


@pytest.mark.gpu
@pytest.mark.parametrize("n,dim,ns,prec", [(2_800_001, 3, 3, W.FP64), (4_200_003, 2, 1, W.FP64),
                                           (2_900_003, 3, 1, W.FP32_KAHAN), (70_001, 2, 3, W.FP32W_FP64ACC)])
def test_what_goes_in_comes_out(n, dim, ns, prec):
    """No step taken: masses and positions as given (rounded to FP32 where
    they are FP32 state), below and above the threaded export's 64 MiB, with
    a ragged last chunk."""
    rng = np.random.Generator(np.random.Philox(20221217))
    x, m = rng.random((n, dim)), rng.random((ns, n))
    print(f"  in and out n={n} dim={dim} ns={ns} prec={prec}", flush=True)
    with mtpt.Sim(_params(n, dim, ns, prec), x, m, allocator=mtpt.TorchAllocator("cuda:0")) as sim:
        gm, gx = sim.masses(), sim.positions()
    assert np.array_equal(gx, x if prec == W.FP64 else x.astype(np.float32))
    assert np.array_equal(gm, m.astype(np.float32) if prec == W.FP32_KAHAN else m)
