"""The input checks above 64 MiB of inputs, where several host threads share
them: the first fault is reported, positions before masses, whichever range
holds it."""
import ctypes as C

import numpy as np
import pytest

from paper_2204_03756_amd import mtpt, workloads as W

N = 1_500_000                                # 67 MiB: eight ranges of 187500 particles


@pytest.mark.parametrize("bad,message", [
    ({"x": [(N - 1, 1), (262_501, 2), (1_125_000, 0)]}, "particle 262501 coordinate 2 = 1.5 outside [0, 1]"),
    ({"x": [(0, 0), (N - 1, 2)]}, "particle 0 coordinate 0 = 1.5 outside [0, 1]"),
    ({"m": [(2, 0), (1, N - 1), (1, 750_000)]}, f"mass {N + 750_000} is not finite"),
    ({"m": [(0, 5)], "x": [(N - 1, 2)]}, f"particle {N - 1} coordinate 2 = 1.5 outside [0, 1]"),
])
def test_first_fault_is_reported(bad, message):
    lib = mtpt.load()
    x, m = np.full((N, 3), 0.25), np.ones((3, N))
    for i, k in bad.get("x", []):
        x[i, k] = 1.5
    for c, i in bad.get("m", []):
        m[c, i] = np.nan
    p = mtpt.make_params(W.Params(dim=3, n=N, lo=[0.0] * 3, hi=[1.0] * 3, d_rw=0.0, d_mt=1e-6, dt=0.1, n_species=3,
                                  precision=W.FP64))
    h = C.c_void_p()
    rc = lib.mtpt_create(C.byref(p), x.ctypes.data_as(mtpt._f64p), m.ctypes.data_as(mtpt._f64p), None, None, C.byref(h))
    assert rc == mtpt.MTPT_E_ARG and not h.value
    assert lib.mtpt_last_error().decode() == message
