"""The GF(2)[t] path at the sizes where it can go wrong, every output bit against
the oracle's product (or, beyond the oracle's time, against one number-theoretic
transform of the same call): block edges (rows of 2^14 bits), the change from
term-by-term products to transforms over rows, each number of rows a transform runs
on, groups of rows in the input alone and in both directions; all kinds and seed orders,
the shortest and longest outputs, biased and degenerate inputs."""
import numpy as np
import pytest

import oracle
import workloads as W
from gpu_helpers import gpu_extract, show_case, to_dev, to_host

pytestmark = pytest.mark.gpu

B = 1 << 14


@pytest.fixture(scope="module")
def ctx():
    import paper_2402_09481_amd as P
    c = P.Context(0)
    yield c
    c.close()


def _labels(ctx, fn):
    import torch
    ctx.profile(True)
    out = fn()
    torch.cuda.synchronize()
    labels = [lab for lab, _ in ctx.profile_read()]
    ctx.profile(False)
    return out, labels


def _batch_of_one(ctx, kind, x, y, n, m, order):
    import torch
    z = torch.full((W.nwords(m),), -1, dtype=torch.int64, device="cuda")
    rc, errs = ctx.batch([{"kind": kind, "n": n, "m": m, "x": to_dev(x), "y": to_dev(y), "z": z, "seed_order": order}],
                         sync=True)
    assert rc == 0 and errs == [0]
    return to_host(z)


def _inputs(kind, n, m, seed):
    g = W.rng(seed)
    x = W.bernoulli_bits(g, n, 0.4)
    if kind == "dodis":
        x[0] = (int(x[0]) | 1) & ~2
    return x, W.bernoulli_bits(g, {"toeplitz": n + m - 1, "circulant": n + 1, "dodis": n}[kind], 0.5)


def _check(ctx, kind, n, m, order, rows):
    """rows: whether the products run by a transform over rows"""
    x, y = _inputs(kind, n, m, n + m)
    show_case("gf2", kind, n, m, order)
    if n + m > (1 << 20):
        (code, z), labels = _labels(ctx, lambda: gpu_extract(ctx, kind, x, y, n, m, order))
        assert code == 0
    else:  # (alone, these run the transform)
        z, labels = _labels(ctx, lambda: _batch_of_one(ctx, kind, x, y, n, m, order))
    steps = ["gf2_rows_fwd", "gf2_rows_inv"] if rows else ["gf2_mul"]
    assert [lab for lab in labels if lab != "gf2_rows_prod"] == ["gf2_fwd"] + steps + ["gf2_inv"], labels
    rc, ref = oracle.extract_product(kind, x, y, n, m, order)
    assert rc == 0 and np.array_equal(z, ref), (kind, n, m, order)


@pytest.mark.parametrize("batch", [False, True])
def test_bit_by_bit(ctx, batch):
    """Short extractions: word and workgroup edges (4 and 16 output words), the longest input
    and the most work that the kernel takes alone, and the longest in a batch."""
    shapes = [(n, m) for n in (1, 2, 31, 32, 33, 63, 64, 65, 127, 129, 2048, 4096, 8191, 8192)
              for m in sorted({1, n // 2 or 1, n})]
    shapes += [(16383, 2)] + ([] if batch else [(131072, 32768), (65537, 65535), (16420, 9000), (131071, 1)])
    for n, m in shapes:
        kinds = [("toeplitz", "paper"), ("toeplitz", "linear")]
        kinds += [("dodis", "paper")] if n > 3 and oracle.is_na_prime(n) else []
        kinds += [("circulant", "paper")] if oracle.is_na_prime(n + 1) else []
        for kind, order in kinds:
            x, y = _inputs(kind, n, m, n + m)
            show_case("gf2 bits", kind, n, m, order, batch)
            if batch:
                z, labels = _labels(ctx, lambda: _batch_of_one(ctx, kind, x, y, n, m, order))
            else:
                (code, z), labels = _labels(ctx, lambda: gpu_extract(ctx, kind, x, y, n, m, order))
                assert code == 0
            assert labels == ["gf2_bits"], labels
            rc, ref = oracle.extract_product(kind, x, y, n, m, order)
            assert rc == 0 and np.array_equal(z, ref), (kind, n, m, order)


@pytest.mark.parametrize("order", ["paper", "linear"])
@pytest.mark.parametrize("n,m", [(B, 2), (B, B), (B + 1, B), (2 * B - 1, B + 1), (2 * B, 1), (2 * B, 2 * B), (5 * B + 31, 3 * B - 33),
                                 (17 * B + 1, 16 * B), (300007, 100003), (128 * B, 96 * B)])
def test_products_term_by_term(ctx, n, m, order):
    _check(ctx, "toeplitz", n, m, order, rows=False)


@pytest.mark.parametrize("n,m,order", [
    (111 * B, 111 * B, "paper"),              # the fewest products: 2^8 rows
    (129 * B - 5, 128 * B, "linear"),         # 2^8 rows exactly
    (130 * B, 128 * B - 1, "paper"),          # 2^9
    (400 * B + 77, 200 * B + 1, "linear"),    # 2^10
    (700 * B, 330 * B + 5, "paper"),          # 2^11
    (1600 * B + 1, 900 * B, "linear"),        # 2^12
    (4000 * B, 90 * B - 3, "paper"),          # 2^12, a short output
    (5000 * B + 9, 700 * B, "linear"),        # two groups of the input
])
def test_products_by_a_transform_over_rows(ctx, n, m, order):
    _check(ctx, "toeplitz", n, m, order, rows=True)


@pytest.mark.parametrize("nx,nz", [(2, 2), (3, 2), (4, 4), (5, 3), (6, 5)])
def test_sums_of_products_of_groups(ctx, nx, nz):
    """Groups of 2048 rows, whose products are summed four groups of the output at a time, the
    next turn's input fetched ahead: the fewest turns, and tiles that are not full."""
    _check(ctx, "toeplitz", (2048 * (nx - 1) + 1) * B - 3, (2048 * (nz - 1) + 1) * B - 7, "paper", rows=True)


@pytest.mark.parametrize("kind,n,m", [("dodis", 16421, 9000), ("dodis", 65587, 65587), ("circulant", 16420, 16420),
                                      ("circulant", 65586, 30001), ("dodis", 1048589, 1 << 19),
                                      ("circulant", 3145748, 3145748)])
def test_periodic_seeds(ctx, kind, n, m):
    if kind == "circulant" and not oracle.is_na_prime(n + 1):
        n = oracle.next_na(n) - 1
        m = min(n, m)
    px, pz = -(-(n + (kind == "circulant")) // B), -(-m // B)
    _check(ctx, kind, n, m, "paper", rows=px * pz > 12288)


def test_degenerate_inputs(ctx):
    for n in (5, 4099, 65587, 1048589):
        y = W.bernoulli_bits(W.rng(3), n, 0.5)
        for x in (np.zeros(W.nwords(n), np.uint64), W.mask_tail(np.full(W.nwords(n), ~np.uint64(0)), n)):
            code, z = gpu_extract(ctx, "dodis", x, y, n, n // 2)
            assert code == oracle.EDEGENERATE and not z.any()


def test_groups_in_both_directions_equal_one_transform(ctx):
    """More than 2^11 output rows: groups of the input and of the output."""
    import torch
    for n, m, order in (((1 << 26) + 12345, (1 << 25) + (1 << 14) + 1, "paper"), ((1 << 27) - 1, (1 << 26) + 3, "linear")):
        x = W.bernoulli_bits_device(n, 0.4, 5)
        y = W.bernoulli_bits_device(n + m - 1, 0.5, 6)
        show_case("gf2 groups", n, m, order)
        a, labels = _labels(ctx, lambda: ctx.extract("toeplitz", x, y, n, m, seed_order=order, sync=True))
        assert "gf2_rows_inv" in labels
        b = ctx.extract("toeplitz", x, y, n, m, seed_order=order, sync=True, single_transform=True)
        assert torch.equal(a, b), (n, m, order)


def test_a_plan_set_by_the_caller_keeps_the_transform(ctx):
    """ext_tune_set on a context makes that size class run the plan it names; removing the
    plan, or a plan read from a table, does not."""
    import paper_2402_09481_amd as P
    c = P.Context(0)
    n, m = 1000003, 500001  # transform 2^21
    x, y = _inputs("toeplitz", n, m, 1)
    ref = oracle.extract_product("toeplitz", x, y, n, m)[1]
    for plan, word in ((None, "gf2_fwd"), ([9, 12], "contig"), (None, "gf2_fwd")):
        c.tune_set(32, 21, plan)
        (code, z), labels = _labels(c, lambda: gpu_extract(c, "toeplitz", x, y, n, m))
        assert code == 0 and np.array_equal(z, ref)
        assert any(lab.startswith(word) for lab in labels), labels
    c.close()
