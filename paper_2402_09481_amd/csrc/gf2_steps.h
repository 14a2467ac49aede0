// The index maps and register steps of the GF(2)[t] kernels that the CPU tests compile as
// they are: reading runs of the packed inputs, and the Taylor layers of the basis
// change over rows.
#pragma once
#include <stdint.h>

#include "kernels.h"

#if defined(__HIPCC__)
#define GF2_FN __device__ __forceinline__
#else
#define GF2_FN inline
#endif

namespace ext {
namespace gf2 {

using u32 = uint32_t;

#if defined(__HIPCC__)
GF2_FN u32 load_word(const u32 *p) { return *(const __attribute__((address_space(1))) u32 *)p; }
GF2_FN u32 funnel(u32 hi, u32 lo, int sh) { return __builtin_amdgcn_alignbit(hi, lo, sh); }
GF2_FN u32 bit_reverse(u32 v) { return __brev(v); }
#else
u32 load_word(const u32 *p);  // (the test's, which checks the address)
GF2_FN u32 funnel(u32 hi, u32 lo, int sh) { return (u32)((((uint64_t)hi << 32) | lo) >> sh); }
GF2_FN u32 bit_reverse(u32 v) {
    u32 r = 0;
    for (int b = 0; b < 32; ++b) r |= ((v >> b) & 1u) << (31 - b);
    return r;
}
#endif

enum Side { T_FWD = 0, T_SEED = 1, T_OUT = 2 };

// bits pos .. pos + 31 (any sign) of a string of len >= 1 bits, zero outside it
GF2_FN u32 clip_word(const uint64_t *bits, uint64_t len, int64_t pos) {
    if (pos >= (int64_t)len || pos <= -32) return 0u;
    const u32 *b = (const u32 *)bits;
    const int64_t w = pos >> 5, last = (int64_t)((len + 31) >> 5) - 1;
    const u32 lo = w >= 0 ? load_word(b + w) : 0u, hi = w < last ? load_word(b + w + 1) : 0u;
    const u32 v = funnel(hi, lo, (int)(pos & 31));
    const int64_t left = (int64_t)len - pos;
    return left < 32 ? v & ((1u << left) - 1u) : v;
}

// positions i .. i + 31 (i >= 0) of the input x' (PREFIX or REV), zero outside it
GF2_FN u32 input_word(const Emb &e, int64_t i) {
    if (e.mode == EMB_PREFIX) return clip_word(e.bits, e.len, i);
    const u32 v = bit_reverse(clip_word(e.bits, e.len, (int64_t)e.N - 32 - i));
    const int64_t left = (int64_t)e.a - i;
    return left >= 32 ? v : left <= 0 ? 0u : v & ((1u << left) - 1u);
}

// seed positions k .. k + 31 (s_k = bit (k + rot) mod P for 0 <= k < N, zero outside); P may
// be as small as 1
GF2_FN u32 seed_word(const Emb &e, int64_t k) {
    const int64_t N = (int64_t)e.N, P = (int64_t)e.P;
    if (k >= N || k <= -32) return 0u;
    int64_t r = k + (int64_t)e.rot;
    while (r < 0) r += P;
    while (r >= P) r -= P;
    u32 v = 0u;
    for (int64_t at = r; at > r - 32 - P && at > -32; at -= P) v |= clip_word(e.bits, e.P, at);
    if (k < 0) v &= ~0u << (int)(-k);
    if (N - k < 32) v &= (1u << (N - k)) - 1u;
    return v;
}

// The 16 words from bit pos (any sign) of a string of len >= 1 bits, ORed into v; bits
// outside the string are zero and no word outside it is read.
GF2_FN void clip_run(u32 *v, const uint64_t *bits, uint64_t len, int64_t pos) {
    const u32 *b = (const u32 *)bits;
    const int64_t w0 = pos >> 5, last = (int64_t)((len + 31) >> 5) - 1;
    const int sh = (int)(pos & 31);
    // word w0 + k (0 <= k <= 16) exists for k0 <= k <= k1
    const int k0 = w0 >= 0 ? 0 : (int)(w0 < -16 ? 17 : -w0);
    const int k1 = last < w0 ? -1 : (int)(last - w0 > 16 ? 16 : last - w0);
    const u32 tail = (len & 31) ? (1u << (len & 31)) - 1u : ~0u;
    const u32 *base = k0 <= k1 ? b + w0 : b;
    u32 w[17];
#pragma unroll
    for (int k = 0; k < 17; ++k) {
        const int c = k0 <= k1 ? (k < k0 ? k0 : k > k1 ? k1 : k) : 0;
        w[k] = load_word(base + c);
    }
#pragma unroll
    for (int k = 0; k < 17; ++k) {
        if (w0 + k == last) w[k] &= tail;
        if (k < k0 || k > k1) w[k] = 0u;
    }
#pragma unroll
    for (int k = 0; k < 16; ++k) v[k] |= funnel(w[k + 1], w[k], sh);
}

// clears the bits of the run at position p that lie outside positions 0 .. n - 1
GF2_FN void keep_positions(u32 *v, int64_t p, int64_t n) {
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        const int64_t q = p + 32 * k, left = n - q;
        u32 m = left >= 32 ? ~0u : left <= 0 ? 0u : (1u << left) - 1u;
        if (q < 0) m &= q <= -32 ? 0u : ~0u << (int)(-q);
        v[k] &= m;
    }
}

GF2_FN void reverse_run(u32 *v) {
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const u32 a = bit_reverse(v[k]), b = bit_reverse(v[15 - k]);
        v[k] = b;
        v[15 - k] = a;
    }
}

// positions i .. i + 511 of the input x' (PREFIX or REV), zero outside it
GF2_FN void input_run(u32 *v, const Emb &e, int64_t i) {
    if (e.mode == EMB_PREFIX) {
        clip_run(v, e.bits, e.len, i);
    } else {
        clip_run(v, e.bits, e.len, (int64_t)e.N - 512 - i);
        reverse_run(v);
        keep_positions(v, i, (int64_t)e.a);
    }
}

// seed positions k .. k + 511 (s_k = bit (k + rot) mod P for 0 <= k < N, zero outside)
GF2_FN void seed_run(u32 *v, const Emb &e, int64_t k) {
    const int64_t P = (int64_t)e.P;
    int64_t r = k + (int64_t)e.rot;
    if (r < 0) r += P;
    while (r >= P) r -= P;
    clip_run(v, e.bits, e.P, r);
    clip_run(v, e.bits, e.P, r - P);
    keep_positions(v, k, (int64_t)e.N);
}

// Taylor layers on 2^R units a[0 ..] of a thread (the basis change of 2^R rows, R <= 4)
template <int SIDE, int HL, int DL, int UL, int N>
GF2_FN void taylor_units(u32 *a) {  // blocks of 2h units of 2^UL entries
    constexpr int U = 1 << UL, h = 1 << HL, d = 1 << DL;
#pragma unroll
    for (int base = 0; base < N; base += 2 * h * U)
#pragma unroll
        for (int x = 0; x < U; ++x) {
            u32 *L = a + base + x, *H = L + h * U;
            if constexpr (SIDE == T_FWD) {
#pragma unroll
                for (int t = 0; t < d; ++t) H[t * U] ^= H[(h - d + t) * U];
#pragma unroll
                for (int u = d; u < h; ++u) L[u * U] ^= H[(u - d) * U];
            } else if constexpr (SIDE == T_SEED) {
#pragma unroll
                for (int u = 0; u < d; ++u) L[u * U] ^= L[(h - d + u) * U];
#pragma unroll
                for (int u = d; u < h; ++u) L[u * U] ^= H[(u - d) * U];
            } else {
#pragma unroll
                for (int t = 0; t < h - d; ++t) H[t * U] ^= L[(t + d) * U];
#pragma unroll
                for (int t = 0; t < d; ++t) H[(h - d + t) * U] ^= H[t * U];
            }
        }
}
template <int SIDE, int R>
GF2_FN void basis_units(u32 *a) {
    constexpr int N = 1 << R;
    if constexpr (R == 2) {
        taylor_units<SIDE, 1, 0, 0, N>(a);
    } else if constexpr (R == 3) {  // bit 2 against bits 1, 0; then within bits 1, 0
        if constexpr (SIDE != T_OUT) {
            taylor_units<SIDE, 2, 0, 0, N>(a);
            taylor_units<SIDE, 1, 0, 0, N>(a);
        } else {
            taylor_units<SIDE, 1, 0, 0, N>(a);
            taylor_units<SIDE, 2, 0, 0, N>(a);
        }
    } else if constexpr (R == 4) {
        if constexpr (SIDE != T_OUT) {
            taylor_units<SIDE, 3, 1, 0, N>(a);
            taylor_units<SIDE, 2, 0, 0, N>(a);
            taylor_units<SIDE, 1, 0, 2, N>(a);
            taylor_units<SIDE, 1, 0, 0, N>(a);
        } else {
            taylor_units<SIDE, 1, 0, 0, N>(a);
            taylor_units<SIDE, 1, 0, 2, N>(a);
            taylor_units<SIDE, 2, 0, 0, N>(a);
            taylor_units<SIDE, 3, 1, 0, N>(a);
        }
    }
}

// R layers that write 2^(K+R) rows in terms of x^(2^K) + x: rows rho + q (2^K - 1) form
// classes of their own (rho < 2^K - 1; q < 2^R, and q = 2^R, 2^R + 1 where those lie
// inside). Row q of a class lies in the 2^K-row block q if q <= rho and in q - 1 after that
// (the last row of all, q = 17 of class 0 for K = R = 4, in block 15), whose bit b says whether
// layer b adds it to row q - 2^b. (T_SEED: the mirrored rows, the sums the
// other way round; T_OUT: that in reverse.) get / put: row -> word.
template <int SIDE, int K, int R, class Get, class Put>
GF2_FN void taylor_classes(int rho, Get &&get, Put &&put) {
    constexpr int N = 1 << R, STEP = (1 << K) - 1, ROWS = 1 << (K + R);
    constexpr int TOP = N > STEP ? N + 1 : N;  // the largest q of any class
    static_assert((TOP + 1) * STEP >= ROWS, "no class is longer");
    u32 a[TOP + 1];
    auto row = [&](int q) {
        const int i = rho + q * STEP;
        return SIDE == T_SEED ? ROWS - 1 - i : i;
    };
    const bool extra = rho + N * STEP < ROWS, extra2 = TOP > N && rho == 0;
#pragma unroll
    for (int q = 0; q < N; ++q) a[q] = get(row(q));
    a[N] = extra ? get(row(N)) : 0u;
    if constexpr (TOP > N) a[TOP] = extra2 ? get(row(TOP)) : 0u;
    auto op = [&](int b, int q) {
        if (q < (1 << b)) return;
        const bool in = (q >> b) & 1, in1 = ((q - 1) >> b) & 1;
        const u32 past = rho < q ? ~0u : 0u;  // row q lies in block q - 1
        u32 m = in && in1 ? ~0u : in1 ? past : in ? ~past : 0u;
        if (q == N) m = extra ? ~0u : 0u;     // (block N - 1)
        if (q > N) m = extra2 ? ~0u : 0u;
        if (SIDE == T_FWD) a[q - (1 << b)] ^= a[q] & m;
        else a[q] ^= a[q - (1 << b)] & m;
    };
    if constexpr (SIDE != T_OUT) {
#pragma unroll
        for (int b = R - 1; b >= 0; --b)
#pragma unroll
            for (int q = TOP; q >= 1; --q) op(b, q);
    } else {
#pragma unroll
        for (int b = 0; b < R; ++b)
#pragma unroll
            for (int q = 1; q <= TOP; ++q) op(b, q);
    }
#pragma unroll
    for (int q = 0; q < N; ++q) put(row(q), a[q]);
    if (extra) put(row(N), a[N]);
    if (extra2) put(row(TOP), a[TOP]);
}

}  // namespace gf2
}  // namespace ext
