"""The pool's two lanes (2-d and 3-d sims on a stream each) against one stream
of the caller's: the same results bit for bit, for mixes that leave a lane
empty, that admit into a lane while the other runs, and that end at different
ticks."""
import numpy as np
import pytest

from paper_2204_03756_amd import workloads as W

pytestmark = pytest.mark.gpu

from gpu_helpers import load_mt, say  # noqa: E402


@pytest.fixture(scope="module")
def mt():
    return load_mt()


@pytest.mark.parametrize("dims", [(2, 2, 2), (3, 3), (2, 3, 2, 3, 3), (3, 2)])
def test_lanes_equal_one_stream(mt, dims):
    import torch
    from paper_2204_03756_amd import serve

    def request(k, dim):
        rng = np.random.Generator(np.random.Philox(20221213 + k))
        n = 1500 + 701 * k
        L = n ** (1.0 / dim)
        p = W.Params(dim=dim, n=n, lo=[0.0] * 3, hi=[L] * dim + [0.0] * (3 - dim), d_rw=0.5 if k % 3 else 0.0, d_mt=0.5,
                     dt=0.1, seed=77 + k, precision=k % 3)
        return W.Request(k, 0.0, p, rng.random((n, dim)) * L, rng.random((1, n)), 3 + 2 * k)

    reqs = [request(k, d) for k, d in enumerate(dims)]
    say(f"  lanes {dims}")
    got = []
    alloc = mt.TorchAllocator("cuda:0")      # the library calls into it: it outlives the pools
    for stream in (None, torch.cuda.Stream()):
        be = serve.PoolBackend(max_slots=2, allocator=alloc,
                               stream=stream.cuda_stream if stream is not None else None)
        rep = serve.serve(be, reqs)          # two slots: admitted as others finish
        be.close()
        assert not rep.rejected
        got.append([(rep.outcomes[r.rid].masses, rep.outcomes[r.rid].pairs_total) for r in reqs])
    for (a, pa), (b, pb) in zip(*got):
        assert np.array_equal(a, b) and pa == pb
