"""Batches of members with several groups of outputs (m > 2^25, products of groups through the
workgroup table), beside shorter ones, directly and from graphs: two batches in turn whose
launches differ in the transforms back over rows alone. Every output against one
transform of the same call; and the few members that share a transform's launches."""
import numpy as np
import pytest

import oracle
import workloads as W
from gpu_helpers import show_case, to_dev, to_host

pytestmark = pytest.mark.gpu

B = 1 << 14


@pytest.fixture(scope="module")
def ctx():
    import paper_2402_09481_amd as P
    c = P.Context(0)
    yield c
    c.close()


def _jobs(ctx, shapes, seed):
    import torch
    jobs, want = [], []
    for i, (n, m) in enumerate(shapes):
        x = W.bernoulli_bits_device(n, 0.4, seed + 2 * i)
        y = W.bernoulli_bits_device(n + m - 1, 0.5, seed + 2 * i + 1)
        jobs.append({"kind": "toeplitz", "n": n, "m": m, "x": x, "y": y,
                     "z": torch.empty(W.nwords(m), dtype=torch.int64, device="cuda")})
        want.append(ctx.extract("toeplitz", x, y, n, m, sync=True, single_transform=True))
    return jobs, want


@pytest.mark.parametrize("graph", [False, True])
@pytest.mark.parametrize("first,second", [
    ([(100679680, 66994176), (100663296, 67108864), (100663296, 67108864)],
     [(100663296, 67239936), (100663296, 67239936), (100663296, 66846720)]),
    ([(5144 * B, 4065 * B), (7501 * B, 1894 * B), (6897 * B, 5313 * B)],
     [(8828 * B, 6257 * B), (5037 * B, 642 * B), (5673 * B, 4376 * B)]),
    ([(8193 * B + 7, 2049 * B - 1), (4097 * B, 4097 * B - 9), (300007, 100003), (5000, 2500)],
     [(70000, 30000), (2049 * B, 2048 * B + 1), (1 << 22, 1 << 21), (1 << 22, 1 << 20)]),
])
def test_groups_of_outputs(ctx, first, second, graph):
    import torch
    batches = [_jobs(ctx, first, 100), _jobs(ctx, second, 200)]
    for k in (0, 1, 0, 1, 1, 0):
        jobs, want = batches[k]
        for j in jobs:
            j["z"].fill_(-1)
        show_case("groups", [(j["n"], j["m"]) for j in jobs], graph)
        rc, errs = ctx.batch(jobs, sync=True, graph=graph)
        assert rc == 0 and not any(errs)
        for j, w in zip(jobs, want):
            assert torch.equal(j["z"], w), (j["n"], j["m"])


@pytest.mark.parametrize("graph", [False, True])
@pytest.mark.parametrize("kind,n,m,count", [("toeplitz", 21299, 10649, 2), ("toeplitz", 65536, 65536, 8), ("dodis", 65587, 60000, 3),
                                            ("circulant", 16420, 16420, 5)])
def test_few_members_of_one_length(ctx, kind, n, m, count, graph):
    import torch
    jobs, want = [], []
    for i in range(count):
        g = W.rng(31 * i + n)
        x = W.bernoulli_bits(g, n, 0.4)
        y = W.bernoulli_bits(g, {"toeplitz": n + m - 1, "circulant": n + 1, "dodis": n}[kind], 0.5)
        if kind == "dodis":
            x[0] = (int(x[0]) | 1) & ~2
        jobs.append({"kind": kind, "n": n, "m": m, "x": to_dev(x), "y": to_dev(y),
                     "z": torch.full((W.nwords(m),), -1, dtype=torch.int64, device="cuda")})
        want.append(oracle.extract_product(kind, x, y, n, m, "paper")[1])
    show_case("few", kind, n, m, count, graph)
    for _ in range(3):
        ctx.profile(True)
        rc, errs = ctx.batch(jobs, sync=True, graph=graph)
        labels = [lab for lab, _ in ctx.profile_read()]
        ctx.profile(False)
        assert rc == 0 and not any(errs)
        assert graph or (any(lab.startswith("strided") for lab in labels) and "gf2_fwd" not in labels), labels
        for j, w in zip(jobs, want):
            assert np.array_equal(to_host(j["z"]), w)
            j["z"].fill_(-1)
