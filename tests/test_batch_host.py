"""Batches on the CPU: the C-ABI's own host code (csrc/abi.cpp) on a model of the HIP
calls (tests/abi_host), every launch checked for the workgroups of every job. A graph
recorded for one batch is replayed only for batches of the same launches."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
PKG = os.path.join(os.path.dirname(HERE), "paper_2402_09481_amd")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
GRAPH = 4
B = 1 << 14


class Result:
    pass


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    out = str(tmp_path_factory.mktemp("abi") / "abi_host.so")
    # (-Bsymbolic: the model's HIP calls, not the runtime's)
    subprocess.check_call([HIPCC, "--offload-arch=gfx950", "--offload-host-only", "-x", "hip", "-O1", "-std=c++17", "-shared", "-fPIC",
                           "-Wno-unused-value", "-Wno-unused-result", os.path.join(HERE, "abi_host", "abi_host.cpp"), "-o", out,
                           "-Wl,-Bsymbolic", "-L" + PKG, "-Wl,-rpath," + PKG, "-l:libextractor.so"])
    L = ctypes.CDLL(out)
    L.host_ctx.restype = ctypes.c_void_p
    L.host_ctx.argtypes = [ctypes.c_size_t, ctypes.c_int]
    L.host_ctx_free.argtypes = [ctypes.c_void_p]
    L.host_batch.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_size_t, ctypes.c_uint32] + [ctypes.c_void_p] * 4 + \
        [ctypes.c_char_p, ctypes.c_size_t]
    return L


@pytest.fixture
def context(lib):
    made = []

    def make(budget=256 << 30, gf2=True):
        made.append(lib.host_ctx(budget, int(gf2)))
        return made[-1]
    yield make
    for c in made:
        lib.host_ctx_free(c)


def run(lib, c, jobs, graph=False):
    """jobs: (kind, n, m) rows"""
    a = np.ascontiguousarray(jobs, np.uint64)
    r = Result()
    faults, done, threads, leased = ctypes.c_int(), ctypes.c_size_t(), ctypes.c_uint64(), ctypes.c_size_t()
    labels = ctypes.create_string_buffer(1 << 13)
    r.rc = lib.host_batch(c, a.ctypes.data, len(a), GRAPH if graph else 0, ctypes.byref(faults), ctypes.byref(done),
                          ctypes.byref(threads), ctypes.byref(leased), labels, len(labels))
    r.faults, r.done, r.threads, r.leased = faults.value, done.value, threads.value, leased.value
    r.labels = labels.value.decode().split()
    return r


def toeplitz(*shapes):
    return [(0, n, m) for n, m in shapes]


# batches of three whose launches differ in the transforms back over rows alone
ALIKE = [
    (toeplitz((100679680, 66994176), (100663296, 67108864), (100663296, 67108864)),
     toeplitz((100663296, 67239936), (100663296, 67239936), (100663296, 66846720))),
    (toeplitz(*((n * B, m * B) for n, m in ((5144, 4065), (7501, 1894), (6897, 5313)))),
     toeplitz(*((n * B, m * B) for n, m in ((8828, 6257), (5037, 642), (5673, 4376))))),
]


@pytest.mark.parametrize("first,second", [(p[i], p[1 - i]) for p in ALIKE for i in (0, 1)])
def test_replays_of_batches_with_nearly_the_same_launches(lib, context, first, second):
    c = context()
    for jobs in (first, second, first):
        r = run(lib, c, jobs, graph=True)
        assert r.rc == 0 and r.faults == 0 and r.done == len(jobs), (r.rc, r.faults, r.done)


@pytest.mark.parametrize("graph", [False, True])
def test_every_workgroup_of_mixed_batches(lib, context, graph):
    """Every step, number of rows and number of groups, many batches through one context."""
    c = context()
    g = np.random.default_rng(7)
    for _ in range(40):
        count = int(g.integers(1, 7))
        jobs = []
        for _ in range(count):
            n = int(2 ** g.uniform(3, 27.5))
            jobs.append((0, n, max(1, int(n * 2 ** g.uniform(-5, 0)))))
        r = run(lib, c, jobs, graph)
        assert r.rc == 0 and r.faults == 0, jobs
        assert r.done == count or "strided" in r.labels or "small" in r.labels, jobs


def test_launches_stay_within_a_grid(lib, context):
    """A launch holds fewer than 2^32 threads, however many short members a batch has: 524,289
    members of 8192 output bits are 2^23 + 16 workgroups of 512 threads."""
    r = run(lib, context(), np.tile(np.array([0, 8192, 8192], np.uint64), ((1 << 19) + 1, 1)))
    assert r.rc == 0 and r.faults == 0 and r.done == (1 << 19) + 1
    assert r.threads < 1 << 32


def _classes(lo, hi, count):
    """as many members of every transform length as fill a workspace of about `count` of the largest"""
    return toeplitz(*((1 << (lg - 1), 1 << (lg - 2)) for lg in range(lo, hi) for _ in range(count << (hi - 1 - lg))))


@pytest.mark.parametrize("graph", [False, True])
@pytest.mark.parametrize("name,jobs", [
    ("short", toeplitz(*[(8192, 8192)] * 4096)),
    ("one class", toeplitz(*[(1 << 18, 1 << 17)] * 64)),
    ("classes", _classes(15, 29, 1)),
    ("long inputs, short outputs", toeplitz(*[(n, 64) for n in range(1 << 15, 1 << 20, 1 << 13)])),
])
def test_a_budget_that_held_the_transforms_holds_the_batch(lib, context, name, jobs, graph):
    """Workspace and descriptors of the members on their transforms: as much is enough on any route."""
    r = run(lib, context(gf2=False), jobs, graph)
    assert r.rc == 0 and r.done == 0
    c = context(budget=r.leased)
    for _ in range(2):
        r = run(lib, c, jobs, graph)
        assert r.rc == 0 and r.faults == 0, (name, r.rc)
    r = run(lib, context(budget=r.leased // 2), jobs, graph)  # (less may be enough, or is refused)
    assert r.rc in (0, -4)


@pytest.mark.parametrize("graph", [False, True])
@pytest.mark.parametrize("jobs,transform", [
    ([(21299, 10649)] * 2, True),
    ([(21299, 10649)] * 8, True),
    ([(21299, 10649)] * 9, False),
    ([(65536, 65536)] * 8, True),
    ([(131072, 131072)] * 4, True),
    ([(131072, 131072)] * 5, False),                # more than 2^20 coefficients
    ([(340787, 170393)] * 2, True),
    ([(524288, 524288)] * 2, False),
    ([(85196, 5324)] * 2, False),                   # (as transforms two pieces each)
    ([(21299, 10649), (42598, 21299)], False),      # two transform lengths
    ([(85196, 42598)] * 2 + [(1 << 21, 1 << 20)], False),  # beside a member of the other route
    ([(85196, 42598)] * 2 + [(4096, 2048)] * 3, True),     # beside short members
    ([(85196, 42598)], False),
])
def test_few_members_of_one_length_share_a_transform(lib, context, jobs, transform, graph):
    """Two to eight members of one transform length, 2^20 coefficients together at most."""
    r = run(lib, context(), toeplitz(*jobs), graph)
    assert r.rc == 0 and r.faults == 0
    short = sum(n + m - 1 <= 1 << 14 for n, m in jobs)
    assert ("strided" in r.labels, "fwd" in r.labels) == (transform, not transform), r.labels
    assert r.done == (short if transform else len(jobs))


def test_the_event_behind_a_workspace(lib, context):
    """An event without a system fence, carried by the last launch, only where the workspace's last
    call is still running: a call that comes after a wait records an ordinary one."""
    c = context()
    lib.host_release_event.argtypes = [ctypes.c_void_p, ctypes.c_int, ctypes.c_int]
    got = [lib.host_release_event(c, *s) for s in ((0, 0), (0, 0), (1, 0), (1, 0), (0, 0), (1, 1), (0, 1), (1, 0), (2, 0))]
    assert got == [0, 0, 1, 1, 0, 0, 0, 1, 0]
