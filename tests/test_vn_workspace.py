"""The Von Neumann workspace holds the arrays of both forms of the extraction, for every tile
size that the one-pass kernel is built with (csrc/vonneumann.hip: VN_WORDS_PER_THREAD)."""
import ctypes
import os
import subprocess

import pytest

PKG = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2402_09481_amd")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


class Pair(ctypes.Structure):
    _fields_ = [("head", ctypes.c_uint64), ("count", ctypes.c_uint64)]


@pytest.mark.parametrize("words", [2, 8, 16])
def test_workspace_holds_both_forms(words, tmp_path):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    out = str(tmp_path / "vn.so")
    subprocess.check_call([HIPCC, "--offload-arch=gfx950", "-O1", "-std=c++17", "-shared", "-fPIC", "-Xclang", "-target-feature",
                           "-Xclang", "-packed-fp32-ops", "-Wno-unused-value", "-DVN_WORDS_PER_THREAD=%d" % words,
                           os.path.join(PKG, "csrc", "vonneumann.hip"), "-o", out, "-Wl,-Bsymbolic", "-L" + PKG,
                           "-Wl,-rpath," + PKG, "-l:libextractor.so"])
    L = ctypes.CDLL(out)
    u64 = ctypes.c_uint64
    size, two, pair = L._ZN3ext18vn_workspace_bytesEm, L._ZN3ext11vn_two_passEm, L._ZN3ext12vn_pair_workEPcm
    size.restype, size.argtypes = ctypes.c_size_t, [u64]
    two.restype, two.argtypes = ctypes.c_bool, [u64]
    pair.restype, pair.argtypes = Pair, [u64, u64]
    for n in [2, 64, 4096 * 64, 4096 * 64 + 2, 5 * 10**8, 3 << 29, (3 << 29) + 2, 1 << 33]:
        tiles = -(-(-(-n // 64)) // (1024 * words))
        assert size(n) >= 24 * tiles + 8  # the one pass: three arrays of a word a tile, and two counters
        if two(n):
            w = pair(0, n)
            tiles = -(-(-(-n // 64)) // 4096)
            assert w.head == 0 and w.count == 8 * tiles and size(n) >= w.count + 4 * tiles, (n, size(n))
    assert two(3 << 29) and not two((3 << 29) + 2)
