"""The batch's job array: the native module fills it with the same bytes as the
Python loop for every ordinary form of job, leaves every other form to that loop, and
the loop's errors are unchanged."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _arrays(jobs):
    import paper_2402_09481_amd as P
    from paper_2402_09481_amd import _lib
    a, b = (P.ExtJob * len(jobs))(), (P.ExtJob * len(jobs))()
    ok = _lib.marshal().fill(jobs, ctypes.addressof(a))
    P.Context._fill_jobs(jobs, b)
    return ok, bytes(a), bytes(b)


def test_native_and_python_arrays_are_the_same():
    import torch
    g = np.random.default_rng(3)
    pool = torch.zeros(1 << 14, dtype=torch.int64, device="cuda")
    st = torch.zeros(64, dtype=torch.int32, device="cuda")
    jobs = []
    for i in range(200):
        n = int(g.integers(1, 60000))
        j = {"kind": ("toeplitz", "circulant", "dodis")[i % 3], "n": n, "m": int(g.integers(1, n + 1)),
             "x": pool[i:], "y": pool[2 * i:].view(torch.uint64) if i % 2 else pool, "z": pool[i:12000]}
        if i % 4 == 1:
            j["seed_order"] = "linear" if i % 8 == 1 else "paper"
        if i % 5 == 2:
            j["single_transform"] = bool(i % 2)
        if i % 3 == 1:
            j["status"] = st[i % 60:] if i % 2 else None
        jobs.append(j)
    jobs.append({"kind": "toeplitz", "n": 5, "m": 9, "x": pool[:0], "y": pool[:0], "z": pool[:0]})  # the library's to reject
    ok, a, b = _arrays(jobs)
    assert ok and a == b
    par = torch.nn.Parameter(pool, requires_grad=False)
    ok, a, b = _arrays([dict(jobs[0], x=par)])
    assert ok and a == b
    # forms the native module leaves to the loop
    for change in ({"n": np.int64(640)}, {"single_transform": 1}, {"kind": np.str_("dodis")}):
        ok, a, b = _arrays([dict(dict(jobs[0], n=640, m=64), **change)])
        assert not ok


def test_bad_jobs_raise_as_before():
    import torch

    import paper_2402_09481_amd as P
    w = torch.zeros(64, dtype=torch.int64, device="cuda")
    good = {"kind": "toeplitz", "n": 1000, "m": 500, "x": w, "y": w, "z": w}
    c = P.Context(0)
    for change, err in (({"kind": "other"}, ValueError), ({"x": w.cpu()}, TypeError), ({"y": w[::2]}, ValueError),
                        ({"z": w[:3]}, ValueError), ({"x": w.view(torch.int32)}, TypeError),
                        ({"status": w}, TypeError), ({"n": None}, TypeError)):
        with pytest.raises(err):
            c.batch([good, dict(good, **change)])
    bad = dict(good)
    del bad["x"]
    with pytest.raises(KeyError):
        c.batch([bad])
    assert c.batch([dict(good, m=2000)]) == (P.EXT_EINVAL, [P.EXT_EINVAL])
    c.close()
