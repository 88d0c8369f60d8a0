"""The library's host side on a device that does nothing (helpers/fakehip.c,
preloaded in a process of its own; no GPU): which HIP calls an entry point
makes, and what it does when one of them fails."""
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def fakehip(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("fakehip") / "libfakehip.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", so, os.path.join(HERE, "helpers", "fakehip.c")], check=True)
    return so


PRELUDE = """
import ctypes as C, sys
sys.path.insert(0, {root!r})
import numpy as np
from paper_2204_03756_amd import mtpt, workloads as W
fake = C.CDLL({so!r})
calls = lambda name: fake.fakehip_calls(name.encode())
def params(n, dim=3, ns=1):
    return W.Params(dim=dim, n=n, lo=[0.0] * 3, hi=[1.0] * dim + [0.0] * (3 - dim), d_rw=1e-4, d_mt=1e-6, dt=0.1,
                    n_species=ns)
"""


def _run(so, body, fail=None):
    env = dict(os.environ)
    env["LD_PRELOAD"] = ":".join(v for v in (env.get("LD_PRELOAD"), so) if v)
    if fail:
        env["FAKEHIP_FAIL"] = fail
    src = PRELUDE.format(root=os.path.dirname(HERE), so=so) + body + "\nprint('as expected')\n"
    r = subprocess.run([sys.executable, "-c", src], env=env, capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "as expected" in r.stdout, r.stderr[-2000:]


def test_exports_free_no_pinned_memory(fakehip):
    """hipHostFree waits for the whole device: neither a pool's result of 64 MiB
    nor a sim's masses may call it, and what was pinned is given back once the
    last sim or pool is destroyed."""
    _run(fakehip, """
n = (64 << 20) // 24 + 1
x, m = np.full((n, 3), 0.5), np.ones((3, n))
pool = mtpt.mtpt_pool_create(1 << 40, 2)
t = [mtpt.mtpt_pool_admit(pool, params(n, ns=3), x, m, 1) for _ in range(2)]
mtpt.mtpt_pool_tick(pool)
before = calls("hipHostFree"), calls("hipHostMalloc")
for k in t:
    mtpt.mtpt_pool_result(pool, k, n, 3)
sim = mtpt.mtpt_create(params(n, ns=3), x, m)
for _ in range(3):
    mtpt.mtpt_masses(sim, n, 3)
    mtpt.mtpt_positions(sim, n, 3)
assert calls("hipHostFree") == before[0], calls("hipHostFree") - before[0]
assert calls("hipHostMalloc") == before[1] + 1
mtpt.mtpt_pool_destroy(pool)
mtpt.mtpt_masses(sim, n, 3)
assert calls("hipHostMalloc") == before[1] + 1
mtpt.mtpt_destroy(sim)
assert calls("hipHostFree") == calls("hipHostMalloc")
sim = mtpt.mtpt_create(params(n, ns=3), x, m)
mtpt.mtpt_masses(sim, n, 3)
mtpt.mtpt_destroy(sim)
assert calls("hipHostFree") == calls("hipHostMalloc") == before[1] + 2
""")


def test_exports_of_several_threads(fakehip):
    """Four threads export at once: two have a ring, none waits for another's."""
    _run(fakehip, """
import threading
n = (64 << 20) // 8 + 12345
sims = [mtpt.mtpt_create(params(n, dim=2), np.full((n, 2), 0.5), np.ones((1, n))) for _ in range(4)]
def export(s):
    for _ in range(3):
        assert mtpt.mtpt_masses(s, n, 1).shape == (1, n)
threads = [threading.Thread(target=export, args=(s,)) for s in sims]
[t.start() for t in threads]
[t.join() for t in threads]
assert 1 <= calls("hipHostMalloc") <= 2 and calls("hipHostFree") == 0
for s in sims:
    mtpt.mtpt_destroy(s)
assert calls("hipHostFree") == calls("hipHostMalloc")
""")


def test_exports_without_a_ring(fakehip):
    """No pinned memory to be had: the plain copy, and the next export tries again."""
    _run(fakehip, """
n = (64 << 20) // 8 + 1
sim = mtpt.mtpt_create(params(n, dim=2), np.full((n, 2), 0.5), np.ones((1, n)))
a = mtpt.mtpt_masses(sim, n, 1)
assert calls("hipHostMalloc") == 1
b = mtpt.mtpt_masses(sim, n, 1)
assert calls("hipHostMalloc") == 2 and a.shape == b.shape
mtpt.mtpt_destroy(sim)
assert calls("hipHostFree") == 1
""", fail="hipHostMalloc:1")


@pytest.mark.parametrize("failing,created", [(0, 1), (1, 0), (2, 0), (3, 1)])
def test_a_pool_needs_two_streams_and_takes_a_third(fakehip, failing, created):
    """The third stream, the 3-d sims' lane, is not needed: without it the pool
    steps every sim on the first.  Every stream made is destroyed."""
    _run(fakehip, f"""
try:
    pool = mtpt.mtpt_pool_create(1 << 30, 4)
except mtpt.MtptError as e:
    assert not {created} and e.code == mtpt.MTPT_E_DEVICE
else:
    assert {created}
    n = 1000
    t = [mtpt.mtpt_pool_admit(pool, params(n, dim=d), np.full((n, d), 0.5), np.ones((1, n)), 2) for d in (2, 3, 2, 3)]
    assert [mtpt.mtpt_pool_tick(pool) for _ in range(2)] == [0, 4]
    assert all(mtpt.mtpt_pool_done(pool, k) for k in t)
    for k in t:
        mtpt.mtpt_pool_result(pool, k, n, 1)
    mtpt.mtpt_pool_destroy(pool)
assert calls("hipStreamDestroy") == calls("hipStreamCreateWithFlags") - {1 if failing else 0}
""", fail=f"hipStreamCreateWithFlags:{failing}" if failing else None)
