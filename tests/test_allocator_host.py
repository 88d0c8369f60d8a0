"""The binding keeps an allocator alive as long as the library may call into it:
until the sim or the pool that was created with it is destroyed (no GPU: a
library that hands out handles stands in)."""
import ctypes as C
import gc
import weakref

import numpy as np
import pytest

from paper_2204_03756_amd import mtpt, serve, workloads as W


class _Library:
    def __init__(self):
        self.next = 0x1000
        self.live = set()

    def _new(self, *args):
        self.next += 16
        self.live.add(self.next)
        args[-1]._obj.value = self.next
        return mtpt.MTPT_OK

    def _end(self, handle):
        self.live.discard(handle.value if isinstance(handle, C.c_void_p) else handle)
        return mtpt.MTPT_OK

    mtpt_create = mtpt_pool_create = _new
    mtpt_destroy = mtpt_pool_destroy = _end


class _Allocator:
    struct = mtpt.mtpt_allocator()


def _sim(alloc):
    p = W.Params(dim=2, n=2, lo=[0.0] * 3, hi=[1.0, 1.0, 0.0], d_rw=0.0, d_mt=1.0, dt=0.1)
    return mtpt.mtpt_create(p, np.zeros((2, 2)), np.zeros((1, 2)), None, alloc)


@pytest.mark.parametrize("create,destroy", [
    (_sim, mtpt.mtpt_destroy),
    (lambda a: mtpt.mtpt_pool_create(0, 4, None, a), mtpt.mtpt_pool_destroy),
    (lambda a: serve.PoolBackend(allocator=a), lambda b: b.close()),
])
def test_a_temporary_allocator_outlives_its_handle(monkeypatch, create, destroy):
    lib = _Library()
    monkeypatch.setattr(mtpt, "load", lambda: lib)
    alloc = _Allocator()
    gone = weakref.ref(alloc)
    handles = [create(alloc), create(alloc)]
    del alloc
    gc.collect()
    assert gone() is not None and len(lib.live) == 2
    destroy(handles.pop())
    gc.collect()
    assert gone() is not None
    destroy(handles.pop())
    gc.collect()
    assert gone() is None and not lib.live
