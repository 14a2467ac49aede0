"""The GF(2)[t] path's host-compilable parts (csrc/gf2.h, csrc/gf2_steps.h) on the CPU: the
field against a polynomial model of the tower, the subspace polynomials, the
linear forms behind a product by a constant, the runs read from the packed strings over
all their forms (both seed orders, reversed and periodic strings, every kind of edge;
no word outside a string is read), and the basis-change layers, in their three
directions, against the defining polynomial division."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CXX = shutil.which("g++") or shutil.which("clang++") or "/opt/rocm/llvm/bin/clang++"


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("gf2") / "gf2_host.so")
    subprocess.check_call([CXX, "-O1", "-std=c++17", "-shared", "-fPIC", "-I", os.path.join(HERE, "gf2_host"), "-o", out,
                           os.path.join(HERE, "gf2_host", "gf2_host.cpp")])
    L = ctypes.CDLL(out)
    u64 = ctypes.c_uint64
    L.gf2_run.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_void_p, u64, u64, u64, u64, u64, ctypes.c_int64,
                          ctypes.c_void_p]
    for f in (L.gf2_mul, L.gf2_subspace):
        f.restype = ctypes.c_uint32
    return L


def monomials(a, b, level=4):
    """Product of the tower's elements by multiplying out monomials and reducing x_k^2 =
    x_k + x_0 .. x_(k-1) (x_0^2 = x_0 + 1)."""
    def mono(i, j):  # product of two monomials as a set of monomials
        both = i & j
        if not both:
            return {i | j}
        k = both.bit_length() - 1
        i2, j2 = i & ~(1 << k), j & ~(1 << k)
        out = set()
        for t in ((1 << k), (1 << k) - 1):  # x_k, x_0 .. x_(k-1)
            for r in mono(i2, j2):
                out ^= mono(r, t)
        return out
    acc = 0
    for i in range(1 << level):
        if (a >> i) & 1:
            for j in range(1 << level):
                if (b >> j) & 1:
                    for r in mono(i, j):
                        acc ^= 1 << r
    return acc


def test_field_and_subspace_polynomials(lib):
    g = np.random.default_rng(1)
    vals = [0, 1, 2, 3, 0x8000, 0xFFFF] + [int(v) for v in g.integers(0, 1 << 16, 12)]
    for a in vals:
        for b in vals[::3]:
            assert lib.gf2_mul(a, b) == monomials(a, b), (a, b)
    for i in range(16):
        assert lib.gf2_subspace(i, 1 << i) == 1
        for j in range(16):
            v = lib.gf2_subspace(i, 1 << j)
            assert v.bit_length() == max(0, j - i + 1)
    w = (ctypes.c_uint32 * 3)()
    w2 = (ctypes.c_uint32 * 3)()
    w3 = (ctypes.c_uint32 * 3)()
    for a in vals:  # the forms are linear, and determine the constant
        for b in vals:
            lib.gf2_forms(a, w)
            lib.gf2_forms(b, w2)
            lib.gf2_forms(a ^ b, w3)
            assert [x ^ y for x, y in zip(w, w2)] == list(w3)
        lib.gf2_forms(a, w)
        assert ((w[0] & 3) | ((w[0] >> 3) & 3) << 2) == (a & 15)


def _words(bits):
    pad = np.zeros(-(-len(bits) // 64) * 64, np.uint8)
    pad[:len(bits)] = bits
    return np.packbits(pad, bitorder="little").view(np.uint64).copy()


@pytest.mark.parametrize("single", [0, 1])
@pytest.mark.parametrize("form", ["prefix", "reversed", "reversed-short", "seed-linear", "seed-paper", "seed-periodic"])
def test_runs_of_the_packed_strings(lib, form, single):
    g = np.random.default_rng(len(form))
    for n in [520, 1000, 4097, 16385] + [1, 2, 5, 31, 33, 70] * single:
        if n == 1 and form == "reversed-short":
            continue
        for m in sorted({1, min(33, n), n // 2 or 1, n}):
            N = n + m - 1
            if form.startswith("seed"):
                P = N if form != "seed-periodic" else n
                rot = m % N if form == "seed-paper" else 0
                src = g.integers(0, 2, P).astype(np.uint8)
                full = np.array([src[(k + rot) % P] for k in range(N)], np.uint8)
                args = (1, 1, P, n - 1, N, rot, P)
            elif form == "prefix":
                src = g.integers(0, 2, n).astype(np.uint8)
                full = src
                args = (0, 0, n, 0, 0, 0, 0)
            else:  # the input reversed; short: its generator has one more position, a zero
                ln = n if form == "reversed" else n - 1
                src = g.integers(0, 2, ln).astype(np.uint8)
                full = np.concatenate([np.zeros(n - ln, np.uint8), src[::-1]])
                args = (0, 2, ln, n, n, 0, 0)
            seed, mode, ln, a, NN, rot, P = args
            w = _words(src)
            # bits past the string's end are garbage for the library to ignore
            if len(src) % 64:
                w[-1] |= np.uint64(0xFFFFFFFFFFFFFFFF) << np.uint64(len(src) % 64)
            out = np.zeros(16, np.uint32)
            edges = [-17000, -513, -512, -511, -33, -1, 0, 1, 31, 32, len(full) - 513, len(full) - 512, len(full) - 511,
                     len(full) - 1, len(full), len(full) + 40000] + [int(v) for v in g.integers(-600, len(full) + 600, 24)]
            if form == "seed-paper":
                edges += [N - rot - 300, N - rot - 512, N - rot]
            for pos in edges:
                if not seed:
                    pos = max(0, pos) & ~31  # input runs start at multiples of the run
                bad = lib.gf2_run(single, seed, mode, w.ctypes.data, ln, a, NN, rot, P, pos, out.ctypes.data)
                got = np.unpackbits(out.view(np.uint8), bitorder="little")
                want = np.array([full[k] if 0 <= k < len(full) else 0 for k in range(pos, pos + 512)], np.uint8)
                assert bad == 0, (form, n, m, pos)
                assert np.array_equal(got, want), (form, n, m, pos)


def _taylor(a, k, side):
    """The layers d = 2^j, h = 2^(k+j) (j from the top) on a whole array of 2^K rows, one row
    at a time: division by x^h + x^d, its transposed inverse in reversed order, its
    transpose."""
    K = len(a).bit_length() - 1
    a = list(a)
    ops = []
    for j in range(K - k - 1, -1, -1):
        h, d = 1 << (k + j), 1 << j
        for base in range(0, len(a), 2 * h):
            for i in range(base + 2 * h - 1, base + h - 1, -1):
                ops.append((i - (h - d), i))
    if side == 0:
        for dst, src in ops:
            a[dst] ^= a[src]
    elif side == 1:
        L = len(a) - 1
        for dst, src in ops:
            a[L - src] ^= a[L - dst]
    else:
        for dst, src in reversed(ops):
            a[src] ^= a[dst]
    return a


@pytest.mark.parametrize("side", [0, 1, 2])
def test_taylor_layers(lib, side):
    g = np.random.default_rng(7)
    for k, r in [(4, 4), (8, 1), (8, 2), (8, 3), (8, 4)]:
        a = g.integers(0, 1 << 32, 1 << (k + r), dtype=np.uint32)
        b = a.copy()
        assert lib.gf2_classes(side, k, r, b.ctypes.data_as(ctypes.c_void_p)) == 0
        assert list(b) == _taylor([int(v) for v in a], k, side), (k, r)

    def basis(a, side):  # the whole basis change of 2^K units, recursively
        K = len(a).bit_length() - 1
        if K <= 1:
            return a
        k = 1
        while 2 * k < K:
            k *= 2
        if side != 2:
            a = _taylor(a, k, side)
        hi = [a[x::1 << k] for x in range(1 << k)]
        hi = [basis(v, side) for v in hi]
        a = [hi[i & ((1 << k) - 1)][i >> k] for i in range(len(a))]
        for q in range(0, len(a), 1 << k):
            a[q:q + (1 << k)] = basis(a[q:q + (1 << k)], side)
        return _taylor(a, k, side) if side == 2 else a

    for r in (2, 3, 4):
        a = g.integers(0, 1 << 32, 1 << r, dtype=np.uint32)
        b = a.copy()
        assert lib.gf2_units(side, r, b.ctypes.data_as(ctypes.c_void_p)) == 0
        assert list(b) == basis([int(v) for v in a], side), r
