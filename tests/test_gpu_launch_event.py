"""A single call's workspace goes back to the context's pool with an event that the
call's last launch completes. Calls that alternate between two streams of one context,
with nothing awaited in between, may take each other's workspace only after that
event: every output must equal the one of the same call made alone. The forms end
with different launches: the GF(2)[t] path's inverse rows, the transform's last
inverse pass, its parity transpose (64-bit field), its fold (circulant) and the Von
Neumann extractor's last kernel. A captured stream records the event instead."""
import pytest

import workloads as W
from gpu_helpers import show_case, to_dev, to_host

pytestmark = pytest.mark.gpu

FORMS = [("toeplitz", 300007, 150003, {}), ("toeplitz", (1 << 20) + 77, 1 << 19, {}), ("dodis", 1048589, 500000, {}),
         ("circulant", 65586, 65586, {}), ("toeplitz", 40000, 39999, {"single_transform": True}),
         ("von_neumann", 1000003, 0, {})]
CALLS = 24


def _inputs(kind, n, m, seed):
    g = W.rng(seed)
    x = W.bernoulli_bits(g, n, 0.4)
    if kind == "von_neumann":
        return to_dev(x), None
    bits = {"toeplitz": n + m - 1, "circulant": n + 1, "dodis": n}[kind]
    return to_dev(x), to_dev(W.bernoulli_bits(g, bits, 0.5))


def _call(ctx, kind, n, m, kw, x, y, z, stream=None):
    if kind == "von_neumann":
        ctx.von_neumann(x, n, z=z[0], m_out=z[1], stream=stream)
    else:
        ctx.extract(kind, x, y, n, m, z=z[0], stream=stream, **kw)


def _outputs(kind, n, m, count):
    import torch
    words = W.nwords(n // 2 if kind == "von_neumann" else m)
    return [(torch.zeros(words, dtype=torch.int64, device="cuda"), torch.zeros(1, dtype=torch.int64, device="cuda"))
            for _ in range(count)]


@pytest.mark.parametrize("kind,n,m,kw", FORMS, ids=lambda v: str(v) if not isinstance(v, dict) else "")
def test_alternating_streams(kind, n, m, kw):
    import torch

    import paper_2402_09481_amd as P
    show_case("alternating streams", kind, n, m, kw)
    ctx = P.Context(0)
    ins = [_inputs(kind, n, m, 700 + i) for i in range(3)]
    want, got = _outputs(kind, n, m, 3), _outputs(kind, n, m, CALLS)
    for (x, y), z in zip(ins, want):
        _call(ctx, kind, n, m, kw, x, y, z)
        torch.cuda.synchronize()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    for i in range(CALLS):
        x, y = ins[i % 3]
        _call(ctx, kind, n, m, kw, x, y, got[i], stream=streams[(i // 2) % 2])
    torch.cuda.synchronize()
    for i in range(CALLS):
        assert (to_host(got[i][0]) == to_host(want[i % 3][0])).all(), i
        assert int(got[i][1].item()) == int(want[i % 3][1].item()), i


def test_captured_stream():
    import torch

    import paper_2402_09481_amd as P
    kind, n, m, kw = FORMS[1]
    show_case("captured stream", kind, n, m)
    ctx = P.Context(0)
    (x, y), (x2, y2) = _inputs(kind, n, m, 710), _inputs(kind, n, m, 711)
    want, got = _outputs(kind, n, m, 2), _outputs(kind, n, m, 1)[0]
    stream = torch.cuda.Stream()
    for a, b, z in ((x, y, want[0]), (x2, y2, want[1])):
        _call(ctx, kind, n, m, kw, a, b, z, stream=stream)
        torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        _call(ctx, kind, n, m, kw, x, y, got, stream=stream)
    for a, b, z in ((x.clone(), y.clone(), want[0]), (x2, y2, want[1]), (x.clone(), y.clone(), want[0])):
        x.copy_(a)
        y.copy_(b)
        got[0].zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert (to_host(got[0]) == to_host(z[0])).all()
