"""Von Neumann in two passes: tiles of 2^18 input bits that share output words. A shared
word is completed from the next tile's first 64 words, or, where they hold too few
differing pairs, by every tile that has a part of it, up to more than 64 tiles apart;
and the line beyond which one pass is taken."""
import numpy as np
import pytest

import oracle
import workloads as W
from gpu_helpers import show_case, to_dev, to_host

pytestmark = pytest.mark.gpu

TILE = 1 << 18
AHEAD = 64 * 64
LINE = 3 << 29


def _run(ctx, x, n):
    import torch
    z = torch.full((W.nwords(n // 2) + 1,), -1, dtype=torch.int64, device="cuda")
    z, m_out = ctx.von_neumann(x, n, z=z)
    torch.cuda.synchronize()
    return z, int(m_out.item())


def _place(bits, g, start, count):
    """count differing pairs from pair position start on, of random first bits."""
    a = g.integers(0, 2, size=count).astype(np.uint8)
    bits[start:start + 2 * count:2] = a
    bits[start + 1:start + 2 * count:2] = a ^ 1


# (tiles, [(tile, offset in bits, differing pairs)]): what the first 64 words of the next
# tile hold against what the word lacks, words over several tiles, owners far behind
LAYOUTS = [
    (2, [(0, 10, 40), (1, 0, 24), (1, AHEAD, 50)]),
    (2, [(0, 10, 40), (1, 0, 23), (1, AHEAD, 50)]),
    (2, [(0, 10, 40), (1, AHEAD - 2 * 24, 24), (1, AHEAD + 100, 7)]),
    (2, [(0, 10, 64), (1, AHEAD, 5)]),
    (4, [(0, TILE - 20, 10), (1, 6, 3), (2, 50, 4), (3, 8, 200)]),
    (5, [(0, 0, 70), (2, AHEAD + 2, 30), (4, 0, 28)]),
    (70, [(0, 4, 5), (67, 4, 3), (69, 1000, 90)]),
    (70, [(0, 4, 100), (65, 2, 28), (66, 2, 1)]),
    (131, [(1, 4, 1), (130, 4, 1)]),
    (131, [(0, 0, 300), (130, TILE - 2, 1)]),
]


@pytest.mark.parametrize("tiles,parts", LAYOUTS, ids=range(len(LAYOUTS)))
@pytest.mark.parametrize("cut", [0, 1, 130])
def test_shared_words(tiles, parts, cut):
    import paper_2402_09481_amd as P
    n = tiles * TILE - cut
    g = W.rng(900 + tiles + cut)
    bits = np.zeros(tiles * TILE, np.uint8)
    for t, at, count in parts:
        _place(bits, g, t * TILE + at, count)
    x = W.pack_bits(bits[:n])
    show_case("von_neumann shared words", n, parts)
    code, want, m = oracle.von_neumann(x, n)
    assert code == 0
    z, got = _run(P.Context(0), to_dev(x), n)
    assert got == m
    zh = to_host(z)
    assert np.array_equal(zh[:W.nwords(m)], want)
    assert np.all(zh[W.nwords(m):] == np.uint64((1 << 64) - 1))


def test_one_pass_beyond_the_line():
    # the same bits, and a pair more: the outputs agree but for the last pair's bit
    import torch

    import paper_2402_09481_amd as P
    ctx = P.Context(0)
    show_case("von_neumann line", LINE)
    x = W.bernoulli_bits_device(LINE + 64, 0.25, 41)
    x[-1] = (x[-1] & ~3) | 1
    za, ma = _run(ctx, x, LINE)
    zb, mb = _run(ctx, x, LINE + 2)
    assert mb == ma + 1
    full = ma // 64
    assert torch.equal(za[:full], zb[:full])
    last = int(zb[full].item()) & ((1 << 64) - 1)
    assert last >> (ma % 64) == 1
    assert (last ^ (1 << (ma % 64))) == (int(za[full].item()) & ((1 << 64) - 1) if ma % 64 else 0)
