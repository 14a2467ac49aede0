"""The calls whose speed is followed: what users of the extractors run, through
the package's public entry points.

The listed cases span the smallest single call (a few thousand bits, where
latency and launches count) to the paper's privacy-amplification sizes, the
three convolution extractors, both Toeplitz seed orders, the allocation-free
call, a graph-replayed batch, a serving round and the Von Neumann extractor.
``draw`` gives further cases of the same ranges. Inputs are packed 64-bit words
on the GPU, as every caller holds them; a call writes into an output buffer that
the caller keeps.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

import paper_2402_09481_amd as P

DEV = "cuda"

QKD_N, QKD_M = 1_738_000_000, 41_378_264  # the paper's QKD privacy-amplification example


def listed():
    return [
        # the smallest ordinary call: one block of a few thousand bits through the
        # paper's interface, which waits for the result
        {"name": "toeplitz_4096", "family": "single", "kind": "toeplitz", "n": 4096, "m": 2048, "order": "linear",
         "p": 16, "sync": True},
        # a short privacy-amplification block with the circulant extractor, ragged sizes
        {"name": "circulant_16420", "family": "single", "kind": "circulant", "n": 16420, "m": 9000, "order": "paper",
         "p": 13},
        # an ordinary block of a few 10^5 bits, odd lengths
        {"name": "toeplitz_300007", "family": "single", "kind": "toeplitz", "n": 300007, "m": 100003,
         "order": "paper", "p": 13},
        # the two-source workload: n the first admissible prime from 2^20, biased input
        {"name": "dodis_1048589", "family": "single", "kind": "dodis", "n": 1048589, "m": 1 << 19, "order": "paper",
         "p": 10},
        # a tight loop that may not allocate, near the largest shape it admits
        {"name": "toeplitz_noalloc_2p21", "family": "noalloc", "kind": "toeplitz", "n": (1 << 21) + 1234,
         "m": (1 << 20) + 7, "order": "paper", "p": 13},
        # a mid-size block, as the larger served requests
        {"name": "toeplitz_2p24", "family": "single", "kind": "toeplitz", "n": 1 << 24, "m": 1 << 23,
         "order": "linear", "p": 16},
        # the paper's QKD example with the improved circulant extractor (padded raw key)
        {"name": "qkd_circulant", "family": "single", "kind": "circulant", "n": 1_738_000_138, "m": 23_998_262,
         "order": "paper", "p": 16},
        # the large Toeplitz workload with the library's default plan
        {"name": "toeplitz_2p30", "family": "single", "kind": "toeplitz", "n": 1 << 30, "m": 1 << 29,
         "order": "paper", "p": 13},
        # the same as one number-theoretic transform over the 64-bit prime (the benchmark's headline)
        {"name": "toeplitz_2p30_one_transform", "family": "single", "kind": "toeplitz", "n": 1 << 30, "m": 1 << 29,
         "order": "paper", "p": 13, "single_transform": True},
        # thousands of independent blocks of uneven length, the signature replayed as a graph
        {"name": "batch_4096", "family": "batch", "count": 4096, "lo": 10.0, "hi": 22.0, "sizes": 3, "rule": "half",
         "graph": True},
        # one admission round of the serving loop: Toeplitz requests of mixed sizes, no graph
        {"name": "serving_round_64", "family": "batch", "count": 64, "lo": 12.0, "hi": 26.0, "sizes": 4,
         "rule": "serve", "graph": False},
        # the paper's largest Von Neumann input, min-entropy half its length
        {"name": "von_neumann_5e8", "family": "vn", "n": 500_000_000, "p": 75},
    ]


def draw(rng: random.Random):
    """One more case of the listed ranges, without a name."""
    def size(lo, hi):
        return int(2.0 ** rng.uniform(lo, hi))

    family = rng.choices(["single", "noalloc", "batch", "vn"], [6, 1, 2, 1])[0]
    if family == "vn":
        return {"family": "vn", "n": size(12, 31), "p": 75}
    if family == "batch":
        rule = rng.choice(["half", "serve"])
        if rule == "half":
            return {"family": "batch", "count": size(4, 10), "lo": 10.0, "hi": round(rng.uniform(14, 22), 2),
                    "sizes": rng.randrange(1 << 30), "rule": "half", "graph": rng.random() < 0.7}
        return {"family": "batch", "count": size(1, 6), "lo": 12.0, "hi": round(rng.uniform(18, 26), 2),
                "sizes": rng.randrange(1 << 30), "rule": "serve", "graph": False}
    kind = rng.choice(["toeplitz", "toeplitz", "circulant", "dodis"]) if family == "single" else "toeplitz"
    n = size(8, 29) if family == "single" else size(8, 21)
    if kind == "circulant":
        n = P.next_na_set(n + 1) - 1
    elif kind == "dodis":
        n = P.next_na_set(n)
    m = max(1, min(n, int(n * 2.0 ** rng.uniform(-6, 0)))) if rng.random() < 0.5 else n // 2
    order = rng.choice(["paper", "linear"]) if kind == "toeplitz" else "paper"
    return {"family": family, "kind": kind, "n": n, "m": m, "order": order, "p": rng.choice([10, 13, 16]),
            "sync": rng.random() < 0.3}


# ------------------------------------------------------------------ inputs

def _seed_bits(kind, n, m):
    return {"toeplitz": n + m - 1, "circulant": n + 1, "dodis": n}[kind]


def _words(g, nwords):
    return torch.randint(-(1 << 63), (1 << 63) - 1, (nwords,), generator=g, device=DEV, dtype=torch.int64)


def _mask_tail(w, nbits):
    if nbits & 63:
        w[-1] &= (1 << (nbits & 63)) - 1
    return w


def _biased(g, nbits, num, lg):
    """nbits packed bits, each one with probability num / 2^lg (one random word per digit)."""
    nw = P.words(nbits)
    out = None
    for d in range(lg):
        if not (num >> d) & 1 and out is None:
            continue
        r = _words(g, nw)
        if out is None:
            out = r
        elif (num >> d) & 1:
            out |= r
        else:
            out &= r
    return _mask_tail(out, nbits)


def _jobs(case):
    """(kind, n, m) of every job of a batch, from the case alone."""
    rng = random.Random(case["sizes"])
    out = []
    for _ in range(case["count"]):
        n = int(2.0 ** rng.uniform(case["lo"], case["hi"]))
        if case["rule"] == "half":
            if rng.random() < 0.5:
                n = P.next_na_set(n + 1) - 1
                out.append(("circulant", n, n // 2))
            else:
                out.append(("toeplitz", n, n // 2))
        else:
            out.append(("toeplitz", n, rng.randint(-(-n // 4), n // 2)))
    return out


def prepare(case, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    ctx = P.default_context(torch.cuda.current_device())
    fam = case["family"]
    if fam == "vn":
        n = case["n"]
        return {"case": case, "ctx": ctx, "x": _biased(g, n, case["p"], 8),
                "z": torch.zeros(max(1, P.words(n // 2)), dtype=torch.int64, device=DEV),
                "m_out": torch.zeros(1, dtype=torch.int64, device=DEV)}
    if fam == "batch":
        shapes = _jobs(case)
        if case["rule"] == "serve":  # inputs are slices of a resident pool, seeds a few resident strings
            top = max(n for _, n, _ in shapes)
            pool = _words(g, 2 * P.words(top))
            seeds = [_words(g, P.words(2 * top)) for _ in range(4)]
            rng = random.Random(int(seed))
            xs = []
            for _, n, _ in shapes:
                off = rng.randrange(pool.numel() - P.words(n) + 1)
                xs.append(pool[off:off + P.words(n)])
            ys = [seeds[rng.randrange(4)][:P.words(n + m - 1)] for _, n, m in shapes]
        else:
            sx = [P.words(n) for _, n, _ in shapes]
            sy = [P.words(_seed_bits(*s)) for s in shapes]
            xs = list(torch.split(_biased(g, 64 * sum(sx), 11, 5), sx))
            ys = list(torch.split(_words(g, sum(sy)), sy))
        zall = torch.zeros(sum(P.words(m) for _, _, m in shapes), dtype=torch.int64, device=DEV)
        zs = list(torch.split(zall, [P.words(m) for _, _, m in shapes]))
        jobs = [{"kind": k, "n": n, "m": m, "x": x, "y": y, "z": z} for (k, n, m), x, y, z in zip(shapes, xs, ys, zs)]
        return {"case": case, "ctx": ctx, "jobs": jobs, "zall": zall}
    n, m = case["n"], case["m"]
    if case.get("name") == "qkd_circulant":  # the raw key, padded with zeros
        x = torch.zeros(P.words(n), dtype=torch.int64, device=DEV)
        x[:P.words(QKD_N)] = _biased(g, QKD_N, case["p"], 5)
    else:
        x = _biased(g, n, case["p"], 5)
    y = _mask_tail(_words(g, P.words(_seed_bits(case["kind"], n, m))), _seed_bits(case["kind"], n, m))
    if case["kind"] == "dodis":
        x[0] = (x[0] | 1) & ~2  # neither all zeros nor all ones
    cls = {"toeplitz": P.Toeplitz, "circulant": P.Circulant, "dodis": P.Dodis}[case["kind"]]
    return {"case": case, "ctx": ctx, "x": x, "y": y, "ext": cls(n, m, seed_order=case["order"], context=ctx),
            "z": torch.zeros(P.words(m), dtype=torch.int64, device=DEV)}


def run(state):
    case, ctx = state["case"], state["ctx"]
    fam = case["family"]
    if fam == "vn":
        z, m_out = ctx.von_neumann(state["x"], case["n"], z=state["z"], m_out=state["m_out"])
        return z, m_out
    if fam == "batch":
        rc, errs = ctx.batch(state["jobs"], graph=case["graph"])
        if rc != 0:
            raise RuntimeError("batch: %d %s" % (rc, [e for e in errs if e][:4]))
        return state["zall"]  # every job's output, one after another
    if fam == "noalloc":
        return ctx.extract("toeplitz", state["x"], state["y"], case["n"], case["m"], z=state["z"],
                           seed_order=case["order"], no_alloc=True)
    if case.get("single_transform"):
        return ctx.extract(case["kind"], state["x"], state["y"], case["n"], case["m"], z=state["z"],
                           seed_order=case["order"], single_transform=True)
    return state["ext"].extract(state["x"], state["y"], z=state["z"], sync=bool(case.get("sync")))


def work(case):
    """Bytes: the packed input and seed read once, the packed output written once. The
    arithmetic is on bits and has no floating-point operations."""
    fam = case["family"]
    if fam == "vn":
        p = case["p"] / 256.0
        return {"bytes": int(case["n"] / 8 * (1 + p * (1 - p))), "flops": 0}
    shapes = _jobs(case) if fam == "batch" else [(case["kind"], case["n"], case["m"])]
    return {"bytes": 8 * sum(P.words(n) + P.words(_seed_bits(k, n, m)) + P.words(m) for k, n, m in shapes),
            "flops": 0}


# ------------------------------------------------------------------ the same outputs from plain torch

def _unpack(w, nbits):
    sh = torch.arange(64, device=w.device, dtype=torch.int64)
    return ((w.view(-1, 1) >> sh) & 1).to(torch.uint8).view(-1)[:nbits]


def _pack(bits, nwords):
    b = torch.zeros(nwords * 64, dtype=torch.int64, device=bits.device)
    b[:bits.numel()] = bits.to(torch.int64)
    sh = torch.arange(64, device=bits.device, dtype=torch.int64)
    return (b.view(-1, 64) << sh).sum(1)


def _toeplitz_linear(x, s, n, m):
    """z_i = sum_j s_(i-j+n-1) x_j mod 2, by a real convolution in 64 bits."""
    L = 1 << max(1, math.ceil(math.log2(n + m - 1)))
    fx = torch.fft.rfft(x.to(torch.float64), n=L)
    fx *= torch.fft.rfft(s.to(torch.float64), n=L)
    c = torch.fft.irfft(fx, n=L)[n - 1:n + m - 1]
    return torch.round(c).to(torch.int64) & 1


def _exact_job(kind, n, m, order, x, y):
    xb, yb = _unpack(x, n), _unpack(y, _seed_bits(kind, n, m))
    if kind == "toeplitz":
        s = yb if order == "linear" else torch.roll(yb, -m)  # s_k = y_((k + m) mod N)
    else:
        if kind == "circulant":
            xb, n = torch.cat([xb, xb.new_zeros(1)]), n + 1
        xb = xb.flip(0)
        s = torch.cat([yb, yb[:m - 1]])
    return _pack(_toeplitz_linear(xb, s, n, m), P.words(m))


def exact(case, seed):
    fam = case["family"]
    shapes = _jobs(case) if fam == "batch" else None
    if fam == "batch":
        if sum(n for _, n, _ in shapes) > 1 << 29 or max(n for _, n, _ in shapes) > 1 << 26:
            return None
    elif case["n"] > (1 << 29 if fam == "vn" else 1 << 26):
        return None
    st = prepare(case, seed)
    if fam == "vn":
        n = case["n"]
        z = torch.zeros_like(st["z"])
        bits = torch.cat([_unpack(c, 64 * c.numel()) for c in torch.split(st["x"], 1 << 20)])[:n // 2 * 2].view(-1, 2)
        kept = bits[:, 0][bits[:, 0] != bits[:, 1]]
        del bits
        step = 1 << 26
        for i in range(0, kept.numel(), step):
            part = kept[i:i + step]
            z[i >> 6:(i >> 6) + P.words(part.numel())] = _pack(part, P.words(part.numel()))
        return z, torch.tensor([kept.numel()], dtype=torch.int64, device=z.device)
    if fam == "batch":
        return torch.cat([_exact_job(j["kind"], j["n"], j["m"], "paper", j["x"], j["y"]) for j in st["jobs"]])
    return _exact_job(case["kind"], case["n"], case["m"], case["order"], st["x"], st["y"])
