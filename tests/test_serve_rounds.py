"""The serving executor's rounds: several requests go out as one batch, a lone one as a
single call on the same stream; a refused call raises."""
import contextlib
import types

import pytest

from paper_2402_09481_amd.serve import GpuExecutor, Request


class Calls:
    def __init__(self, rc=0):
        self.rc, self.log = rc, []

    def batch(self, jobs, stream=None):
        self.log.append(("batch", [(j["kind"], j["n"], j["m"], j["seed_order"], j["z"]) for j in jobs], stream))
        return self.rc, [self.rc] * len(jobs)

    def extract(self, kind, x, y, n, m, z=None, seed_order="paper", stream=None, check=True):
        assert not check
        self.log.append(("extract", [(kind, n, m, seed_order, z)], stream))
        return self.rc, z


def executor(ctx):
    ex = GpuExecutor.__new__(GpuExecutor)
    event = types.SimpleNamespace(record=lambda s: None, query=lambda: True)
    ex.torch = types.SimpleNamespace(int64=None, empty=lambda n, dtype, device: ("z", n),
                                     cuda=types.SimpleNamespace(stream=lambda s: contextlib.nullcontext(), Event=lambda: event))
    ex.ctx, ex.streams, ex.free = ctx, ["s0", "s1"], [0, 1]
    return ex


@pytest.mark.parametrize("count", [1, 2, 5])
def test_rounds(count):
    ctx = Calls()
    ex = executor(ctx)
    reqs = [Request(rid=i, t_arrival=0.0, kind="toeplitz", n=1000 + i, m=100 + 64 * i, seed_order="linear") for i in range(count)]
    h = ex.submit(reqs)
    want = [("toeplitz", r.n, r.m, "linear", ("z", (r.m + 63) >> 6)) for r in reqs]
    assert ctx.log == [("extract" if count == 1 else "batch", want, "s1")]
    assert ex.free == [0] and ex.done(h)
    ex.release(h)
    assert ex.free == [0, 1]


@pytest.mark.parametrize("count", [1, 2])
def test_a_refused_round_raises(count):
    ex = executor(Calls(rc=-4))
    with pytest.raises(RuntimeError):
        ex.submit([Request(rid=i, t_arrival=0.0, kind="toeplitz", n=1000, m=100) for i in range(count)])
