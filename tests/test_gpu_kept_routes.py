"""The routes that default calls of ordinary sizes no longer take, each run on purpose and
known by its launches' labels: piece schedules over the lazy field, 3*2^30+1 and the 64-bit
field, the persistent launch of single-workgroup transforms, and the one-pass Von
Neumann form. They serve plans that a caller sets, one-transform calls, larger shapes and
longer inputs."""
import os

import numpy as np
import pytest

import oracle
import test_gpu_batch
import test_gpu_vn
import workloads as W
from gpu_helpers import gpu_extract, show_case, to_dev, to_host

pytestmark = pytest.mark.gpu


def _context(**env):
    import paper_2402_09481_amd as P
    os.environ.update(env)
    try:
        return P.Context(0)
    finally:
        for k in env:
            del os.environ[k]


@pytest.fixture(scope="module")
def transforms():
    """a context on the transforms: their own line between one transform and two pieces, named"""
    c = _context(EXT_SPLIT_MIN_LG="25")
    yield c
    c.close()


def _labels(ctx, fn):
    import torch
    ctx.profile(True)
    out = fn()
    torch.cuda.synchronize()
    labels = [lab for lab, _ in ctx.profile_read()]
    ctx.profile(False)
    assert not any(lab.startswith("gf2") for lab in labels), labels
    return out, labels


def _pieces(labels, field, count):
    """the products of all pieces but the first, which are added before the one inverse"""
    prod = [lab for lab in labels if lab.startswith("contig[%s" % field) and ("mode=3" in lab or "mode=4" in lab)]
    first = [lab for lab in labels if lab.startswith("contig[%s" % field) and "mode=2" in lab]
    assert (len(prod), len(first)) == (count - 1, 1), labels


@pytest.mark.parametrize("kind,n,m,order", [
    ("toeplitz", 1 << 24, 1 << 23, "paper"),   # one transform of 2^25 over the lazy field, halved
    ("toeplitz", (1 << 26) - 333, (1 << 25) - 7, "linear"),
    ("dodis", None, 1 << 24, "paper"),        # n: the next prime >= 2^26 - 2^20 with primitive root 2
    ("circulant", None, (1 << 24) + 5, "paper"),
])
def test_two_pieces_over_the_lazy_field(transforms, kind, n, m, order):
    if n is None:
        p = oracle.next_na((1 << 26) - (1 << 20))
        n = p if kind == "dodis" else p - 1
    g = W.rng(n ^ m)
    x = W.bernoulli_bits(g, n, 0.45)
    y = W.bernoulli_bits(g, {"toeplitz": n + m - 1, "circulant": n + 1, "dodis": n}[kind], 0.5)
    show_case("lazy two-piece", kind, n, m, order)
    (code, z), labels = _labels(transforms, lambda: gpu_extract(transforms, kind, x, y, n, m, order))
    assert code == 0 and np.array_equal(z, oracle.extract_product(kind, x, y, n, m, order)[1])
    _pieces(labels, "lz", 2)


def test_a_caller_set_plan_keeps_the_pieces():
    """ext_tune_set of the one transform's class: the call runs that class's piece schedule."""
    c = _context()
    n, m = 1 << 24, 1 << 23  # 2^25, halved
    x = W.bernoulli_bits_device(n, 0.4, 3)
    y = W.bernoulli_bits_device(n + m - 1, 0.5, 4)
    want = c.extract("toeplitz", x, y, n, m, sync=True)
    c.tune_set(32, 25, [9, 8, 8])
    z, labels = _labels(c, lambda: c.extract("toeplitz", x, y, n, m, sync=True))
    assert np.array_equal(to_host(z), to_host(want))
    _pieces(labels, "lz", 2)
    c.close()


@pytest.mark.parametrize("graph", [False, True])
def test_batch_of_pieces_and_small_transforms(transforms, graph):
    run = lambda: test_gpu_batch.test_batch_with_lazy_two_piece_jobs(transforms, graph)
    if graph:
        return run()
    _, labels = _labels(transforms, run)
    assert "small_persist" in labels
    assert any(lab.startswith("contig[lz") and "mode=2" in lab for lab in labels), labels


@pytest.mark.parametrize("graph", [False, True])
def test_batch_of_every_transform_length(transforms, graph):
    run = lambda: test_gpu_batch.test_batch_matches_oracle_and_single(transforms, graph)
    if graph:
        run()
        return test_gpu_batch.test_batch_replay_with_new_inputs(transforms)
    assert "small_persist" in _labels(transforms, run)[1]


@pytest.mark.parametrize("kind,n,m,field,count", [
    ("toeplitz", 1 << 30, 1 << 29, "p0", 2),                    # halves of 2^30 over 3*2^30+1
    ("circulant", 1_738_000_138, 23_998_262, "p0", 2),
    ("toeplitz", 6_500_000_000, 581_294_933, "u64", 5),         # pieces of 2^31 over the 64-bit field
])
def test_large_piece_schedules_equal_the_default_route(transforms, kind, n, m, field, count):
    import torch

    import paper_2402_09481_amd as P
    show_case("pieces at size", kind, n, m)
    x = W.bernoulli_bits_device(n, 0.4, 11)
    y = W.bernoulli_bits_device(n + m - 1 if kind == "toeplitz" else n + 1, 0.5, 12)
    a, labels = _labels(transforms, lambda: transforms.extract(kind, x, y, n, m, sync=True))
    _pieces(labels, field, count)
    c = P.Context(0)
    b = c.extract(kind, x, y, n, m, sync=True)
    assert torch.equal(a, b)
    c.close()
    transforms.trim()
    del x, y, a, b
    torch.cuda.empty_cache()


@pytest.fixture(scope="module")
def one_pass():
    c = _context(EXT_VN_ONE_PASS="1")
    yield c
    c.close()


@pytest.mark.parametrize("kind", ["iid", "half", "biased", "alternating", "sparse", "bursts"])
def test_von_neumann_in_one_pass(one_pass, kind):
    _, labels = _labels(one_pass, lambda: test_gpu_vn.test_parity_sizes(one_pass, kind))
    assert set(labels) == {"vn_zero", "vn_main", "vn_fix"}


def test_von_neumann_in_one_pass_paper_shape_and_tails(one_pass):
    test_gpu_vn.test_many_tiles_paper_shape(one_pass)
    test_gpu_vn.test_degenerate_and_tails(one_pass)
    test_gpu_vn.test_sync_and_errors(one_pass)
