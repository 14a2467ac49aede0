// Extraction as a product over GF(2)[t] by additive FFTs (gf2.h: field and jobs).
//
// A Toeplitz extraction needs the middle part of the product of the input and
// the seed. That product is the transpose of an ordinary one: with T the
// transform (evaluation) of a row of 2B bits, an output block is
//     T^t ( T(x block) * (T^-1)^t (seed window) )
// where * is the product of field elements, so that a row of 2B bits serves a
// window of 2B - 1 seed bits, B input bits and B output bits, with no wrap-around
// to undo. Writing covectors by their coordinates in the basis dual to the bit basis
// makes both transposes additive FFTs of the same form: T^-t is T on the
// bit-reversed order with every twiddle c replaced by c + 1, and T^t runs T's
// stages backwards on (g0, g1) -> (g0 + g1, c (g0 + g1) + g1).
//
// T (2^15 bits, index bits 14 .. 0): a change to the basis of products of subspace
// polynomials (XORs only, "Taylor" layers below), then one stage per index bit,
// from bit 14 down. Because the coefficients are bits, it is enough to evaluate
// at one point of every orbit of squaring: the index bits 14, 13, 11 and 7 are not
// split into two points but extend the field (GF(2) to 4, 16, 256 and 2^16), the
// other eleven are. All data stay in bit planes: the four extending index bits
// number a value's 16 bits, and a word holds 32 values of one bit.
//
// k_gf2_fwd, k_gf2_inv: a row is held by 32 lanes of a wave, 32 words each, all of
// its stages in registers: index bits move between register number, lane and
// position in the word by permlane swaps, DPP moves and shifts, and only the
// change of layout between the Taylor layers goes through LDS.
#include "gf2.h"

#include <type_traits>

#include "gf2_steps.h"
#include "launch.h"

namespace ext {
using namespace gf2;
namespace {

template <int I, int N, class F>
__device__ __forceinline__ void unroll(F &&f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>());
        unroll<I + 1, N>(f);
    }
}

// s_i(v_j)
constexpr u32 TW(int i, int j) { return subspace_poly(i, 1u << j); }

// ------------------------------------------------------------------ products by a constant, in bit planes

// bit K of x as a mask of 32 equal bits. The instruction is spelled out: from the
// builtin the compiler makes a compare and a select, two instructions more.
template <int K>
__device__ __forceinline__ u32 bit_mask(u32 x) {
    u32 m;
    asm("v_bfe_i32 %0, %1, %2, 1" : "=v"(m) : "v"(x), "n"(K));
    return m;
}

// acc ^ (a & m) as the one instruction it is (left to the compiler the sums are
// regrouped into more of them); a compile-time m (0 or all ones) folds
template <class Fm>
__device__ __forceinline__ u32 and_xor(u32 acc, u32 a, u32 m) {
    if constexpr (Fm::CONSTANT) return acc ^ (a & m);
    else return __builtin_amdgcn_bitop3_b32(acc, a, m, 0x78);
}

// the same on moved bits: w ^ (t & m), m a literal
__device__ __forceinline__ u32 xor_masked(u32 w, u32 t, u32 m) { return __builtin_amdgcn_bitop3_b32(w, t, m, 0x78); }

// The steps of a row stay in order: without these the scheduler overlaps them at the
// price of spilled registers.
__device__ __forceinline__ void step_end() { __builtin_amdgcn_sched_barrier(0); }

// The values exist here: keeps the compiler from moving a row's last steps behind the
// branch that follows, their operands spilled.
__device__ __forceinline__ void pin(u32 *v) {
#pragma unroll
    for (int t = 0; t < 32; ++t) asm volatile("" : "+v"(v[t]));
}

// Providers of the constant's forms as planes: get<H, L, K>() is form (L, K) of the
// H-th 8-bit part (gf2.h: forms81).
template <u32 C>
struct ConstForms {  // known at compile time: the product becomes a fixed XOR network
    static constexpr bool CONSTANT = true;
    static constexpr Forms f = forms81(C);
    template <int H, int L, int K>
    __device__ __forceinline__ u32 get() const {
        return (f.w[H] >> (L * 9 + K)) & 1 ? ~0u : 0u;
    }
};
struct LaneForms {  // one constant per lane
    static constexpr bool CONSTANT = false;
    u32 w[3];
    template <int H, int L, int K>
    __device__ __forceinline__ u32 get() const {
        return bit_mask<L * 9 + K>(w[H]);
    }
};
// one constant per lane, plus s_I(v_j) for the word's positions with the index bits j =
// 5, 4, .. above I set (stage I inside the word: word bit I + k holds index bit
// I + k + 1)
constexpr u32 word_bit_mask(int b) {
    return b == 0 ? 0xAAAAAAAAu : b == 1 ? 0xCCCCCCCCu : b == 2 ? 0xF0F0F0F0u : b == 3 ? 0xFF00FF00u : 0xFFFF0000u;
}
template <int I>
struct WordForms {
    static constexpr bool CONSTANT = false;
    u32 w[3];
    static constexpr u32 pattern(int h, int bit) {
        u32 p = 0;
        for (int wb = I; wb < 5; ++wb)
            if ((forms81(TW(I, wb + 1)).w[h] >> bit) & 1) p ^= word_bit_mask(wb);
        return p;
    }
    template <int H, int L, int K>
    __device__ __forceinline__ u32 get() const {
        constexpr u32 p = pattern(H, L * 9 + K);  // (constant expression)
        const u32 m = bit_mask<L * 9 + K>(w[H]);
        return p ? m ^ p : m;
    }
};

// acc += a * b over the field of 16
template <int H, int L, class Fm>
__device__ __forceinline__ void mul4(u32 *c, const u32 *a, const Fm &f) {
    const u32 b0 = f.template get<H, L, 0>(), b1 = f.template get<H, L, 1>(), b01 = f.template get<H, L, 2>();
    c[0] = and_xor<Fm>(c[0], a[0], b0);
    c[1] = and_xor<Fm>(c[1], a[0], b1);
    c[0] = and_xor<Fm>(c[0], a[1], b1);
    c[1] = and_xor<Fm>(c[1], a[1], b01);
    const u32 b2 = f.template get<H, L, 3>(), b3 = f.template get<H, L, 4>(), b23 = f.template get<H, L, 5>();
    c[2] = and_xor<Fm>(c[2], a[0], b2);
    c[3] = and_xor<Fm>(c[3], a[0], b3);
    c[2] = and_xor<Fm>(c[2], a[1], b3);
    c[3] = and_xor<Fm>(c[3], a[1], b23);
    c[0] = and_xor<Fm>(c[0], a[2], b3);
    c[1] = and_xor<Fm>(c[1], a[2], b23);
    c[0] = and_xor<Fm>(c[0], a[3], b23);
    c[1] = and_xor<Fm>(c[1], a[3], b2);
    const u32 b02 = f.template get<H, L, 6>(), b13 = f.template get<H, L, 7>(), bs = f.template get<H, L, 8>();
    c[2] = and_xor<Fm>(c[2], a[2], b02);
    c[3] = and_xor<Fm>(c[3], a[2], b13);
    c[2] = and_xor<Fm>(c[2], a[3], b13);
    c[3] = and_xor<Fm>(c[3], a[3], bs);
}

// c += a * b over the field of 256
template <int H, class Fm>
__device__ __forceinline__ void mul8(u32 *c, const u32 *a, const Fm &f) {
    u32 p[4] = {0, 0, 0, 0};
    mul4<H, 0>(p, a, f);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        c[i] ^= p[i];
        c[4 + i] ^= p[i];
    }
    const u32 s[4] = {a[0] ^ a[4], a[1] ^ a[5], a[2] ^ a[6], a[3] ^ a[7]};
    mul4<H, 1>(c + 4, s, f);
    mul4<H, 2>(c, a + 4, f);
}

// c += a * b over the field of 2^16, in three parts
template <class Fm>
__device__ __forceinline__ void mul16_low(u32 *c, const u32 *a, const Fm &f) {
    u32 p[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    mul8<0>(p, a, f);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        c[i] ^= p[i];
        c[8 + i] ^= p[i];
    }
}
template <class Fm>
__device__ __forceinline__ void mul16_sum(u32 *c, const u32 *a, const Fm &f) {
    u32 s[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) s[i] = a[i] ^ a[8 + i];
    mul8<1>(c + 8, s, f);
}
template <class Fm>
__device__ __forceinline__ void mul16(u32 *c, const u32 *a, const Fm &f) {
    mul16_low(c, a, f);
    step_end();
    mul16_sum(c, a, f);
    step_end();
    mul8<2>(c, a + 8, f);
    step_end();
}

// ------------------------------------------------------------------ moving index bits

__device__ __forceinline__ u32 bperm(int lane4, u32 v) { return (u32)__builtin_amdgcn_ds_bpermute(lane4, (int)v); }

// exchange register-number bit RB with lane bit LB
template <int RB, int LB>
__device__ __forceinline__ void swap_lane(u32 *v) {
#pragma unroll
    for (int t = 0; t < 32; ++t) {
        if (t & (1 << RB)) continue;
        u32 &a = v[t], &b = v[t | (1 << RB)];
        if constexpr (LB == 5) {
            const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
            a = r[0];
            b = r[1];
        } else if constexpr (LB == 4) {
            const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
            a = r[0];
            b = r[1];
        } else if constexpr (LB == 3 || LB == 2) {
            // row_shr / row_shl by 8 or 4 into the upper / lower banks
            constexpr int up = LB == 3 ? 0xc : 0xa;
            const u32 na = (u32)__builtin_amdgcn_update_dpp((int)a, (int)b, 0x110 + (1 << LB), 0xf, up, false);
            b = (u32)__builtin_amdgcn_update_dpp((int)b, (int)a, 0x100 + (1 << LB), 0xf, up ^ 0xf, false);
            a = na;
        } else {
            static_assert(LB == 1, "lane bit 0 is the row of the wave");
            const bool hi = (threadIdx.x >> 1) & 1;
            const u32 pa = (u32)__builtin_amdgcn_update_dpp(0, (int)a, 0x4E, 0xf, 0xf, true);
            const u32 pb = (u32)__builtin_amdgcn_update_dpp(0, (int)b, 0x4E, 0xf, 0xf, true);
            a = hi ? pb : a;
            b = hi ? b : pa;
        }
    }
}

// exchange register-number bit RB with word bit WB
template <int RB, int WB>
__device__ __forceinline__ void swap_word(u32 *v) {
    constexpr u32 hi = word_bit_mask(WB), lo = ~hi;
#pragma unroll
    for (int t = 0; t < 32; ++t) {
        if (t & (1 << RB)) continue;
        const u32 a = v[t], b = v[t | (1 << RB)];
        v[t] = (a & lo) | ((b << (1 << WB)) & hi);
        v[t | (1 << RB)] = ((a >> (1 << WB)) & lo) | (b & hi);
    }
}

// ------------------------------------------------------------------ Taylor layers
//
// One layer writes a polynomial's blocks of 2h coefficients in terms of
// x^h + x^d: with L, H a block's halves,
//   T_FWD: H[t] += H[h - d + t] (t < d), then L[u] += H[u - d] (u >= d)
//   T_SEED (the transposed inverse in reversed order): L[u] += the concatenation
//          of L and H at u + h - d
//   T_OUT (the transpose): H[t] += L[t + d] (t < h - d), then H[h - d + t] += H[t] (t < d)
// Layers: index bits 8..14 against the lower eight (7 layers, d = 2^6 .. 1 bits),
// then within bits 8..14 and within the lower eight likewise.
// halves of NW words L = v[l0 ..], H = v[h0 ..], d = D bits, all in one thread
template <int SIDE, int NW, int D>
__device__ __forceinline__ void taylor_words(u32 *v, int l0, int h0) {
    constexpr int DW = D / 32, DB = D % 32;
    static_assert(DW == 0 || DB == 0, "whole words or less than one");
    u32 *L = v + l0, *H = v + h0;
    if constexpr (SIDE == T_FWD) {
        if constexpr (DW > 0) {
#pragma unroll
            for (int t = 0; t < DW; ++t) H[t] ^= H[NW - DW + t];
#pragma unroll
            for (int u = DW; u < NW; ++u) L[u] ^= H[u - DW];
        } else {
            H[0] ^= H[NW - 1] >> (32 - DB);
            L[0] ^= H[0] << DB;
#pragma unroll
            for (int u = 1; u < NW; ++u) L[u] ^= __builtin_amdgcn_alignbit(H[u], H[u - 1], 32 - DB);
        }
    } else if constexpr (SIDE == T_SEED) {
        if constexpr (DW > 0) {
#pragma unroll
            for (int u = 0; u < DW; ++u) L[u] ^= L[NW - DW + u];
#pragma unroll
            for (int u = DW; u < NW; ++u) L[u] ^= H[u - DW];
        } else {
            L[0] ^= __builtin_amdgcn_alignbit(H[0], L[NW - 1], 32 - DB);
#pragma unroll
            for (int u = 1; u < NW; ++u) L[u] ^= __builtin_amdgcn_alignbit(H[u], H[u - 1], 32 - DB);
        }
    } else {
        if constexpr (DW > 0) {
#pragma unroll
            for (int t = 0; t < NW - DW; ++t) H[t] ^= L[t + DW];
#pragma unroll
            for (int t = 0; t < DW; ++t) H[NW - DW + t] ^= H[t];
        } else {
#pragma unroll
            for (int t = 0; t + 1 < NW; ++t) H[t] ^= __builtin_amdgcn_alignbit(L[t + 1], L[t], DB);
            H[NW - 1] ^= L[NW - 1] >> DB;
            H[NW - 1] ^= H[0] << (32 - DB);
        }
    }
}

// halves of h = HB bits inside every word
constexpr u32 repeat_mask(int lo, int hi, int period) {  // bits lo .. hi - 1 of every period
    u32 m = 0;
    for (int b = 0; b < 32; ++b)
        if (b % period >= lo && b % period < hi) m |= 1u << b;
    return m;
}
template <int SIDE, int HB, int D>
__device__ __forceinline__ void taylor_in_word(u32 *v) {
    constexpr int S = HB - D;
    constexpr u32 h_low = repeat_mask(HB, HB + D, 2 * HB), l_high = repeat_mask(D, HB, 2 * HB),
                  l_all = repeat_mask(0, HB, 2 * HB), h_rest = repeat_mask(HB, 2 * HB - D, 2 * HB),
                  h_high = repeat_mask(2 * HB - D, 2 * HB, 2 * HB);
#pragma unroll
    for (int t = 0; t < 32; ++t) {
        u32 w = v[t];
        if constexpr (SIDE == T_FWD) {
            w = xor_masked(w, w >> S, h_low);
            w = xor_masked(w, w >> S, l_high);
        } else if constexpr (SIDE == T_SEED) {
            w = xor_masked(w, w >> S, l_all);
        } else {
            w = xor_masked(w, w << S, h_rest);
            w = xor_masked(w, w << S, h_high);
        }
        v[t] = w;
    }
}

// The layers of bits 9..14 against the lower eight: register bit 4 holds the layer's
// index bit P, registers 0..15 are 16 consecutive words, and the 2^(P-9) runs of 16
// words of a half lie in the lanes whose rotated number rho (lane bits 5, 1, 2, 3, 4 from
// the lowest) differs in its low P - 9 bits.
template <int SIDE, int P>
__device__ __forceinline__ void taylor_runs(u32 *v) {
    constexpr int D = 1 << (P - 8), NB = P - 9, DW = D / 32, DB = D % 32;
    constexpr u32 M = (1u << NB) - 1;
    const u32 lane = threadIdx.x & 63, rho = (lane >> 5) | (lane & 0x1e);
    const u32 to = SIDE == T_OUT ? (rho + 1) & M : (rho - 1) & M;
    const u32 nr = (rho & ~M) | to;
    const int nb = (int)(((lane & 1) | (nr & 0x1e) | ((nr & 1) << 5)) << 2);
    // first run of its half (T_OUT: last run)
    const bool edge = (rho & M) == (SIDE == T_OUT ? M : 0u);
    u32 *L = v, *H = v + 16;
    if constexpr (SIDE != T_OUT) {
        u32 carry[DW > 0 ? DW : 1];
        constexpr int NC = DW > 0 ? DW : 1;
#pragma unroll
        for (int k = 0; k < NC; ++k) {
            const u32 c = bperm(nb, H[16 - NC + k]);
            if constexpr (SIDE == T_FWD) {
                const u32 fix = edge ? c : 0u;
                if constexpr (DW > 0) H[k] ^= fix;
                else H[0] ^= fix >> (32 - DB);
                carry[k] = edge ? 0u : c;
            } else {
                const u32 lc = bperm(nb, L[16 - NC + k]);
                carry[k] = edge ? lc : c;
            }
        }
        if constexpr (DW > 0) {
#pragma unroll
            for (int u = 15; u >= DW; --u) L[u] ^= H[u - DW];
#pragma unroll
            for (int u = 0; u < DW; ++u) L[u] ^= carry[u];
        } else {
#pragma unroll
            for (int u = 15; u >= 1; --u) L[u] ^= __builtin_amdgcn_alignbit(H[u], H[u - 1], 32 - DB);
            L[0] ^= __builtin_amdgcn_alignbit(H[0], carry[0], 32 - DB);
        }
    } else {
        constexpr int NC = DW > 0 ? DW : 1;
        u32 carry[NC];
#pragma unroll
        for (int k = 0; k < NC; ++k) {
            const u32 c = bperm(nb, L[k]);
            carry[k] = edge ? 0u : c;
        }
        if constexpr (DW > 0) {
#pragma unroll
            for (int u = 0; u < 16; ++u) H[u] ^= u + DW < 16 ? L[u + DW] : carry[u + DW - 16];
        } else {
#pragma unroll
            for (int u = 0; u < 16; ++u) H[u] ^= __builtin_amdgcn_alignbit(u < 15 ? L[u + 1] : carry[0], L[u], DB);
        }
#pragma unroll
        for (int k = 0; k < NC; ++k) {
            const u32 c = bperm(nb, H[k]);  // the first run's lowest words, updated
            const u32 fix = edge ? c : 0u;
            if constexpr (DW > 0) H[16 - DW + k] ^= fix;
            else H[15] ^= fix << (32 - DB);
        }
    }
}

// registers only: blocks of 2h units, a unit 2^UL consecutive register numbers
template <int SIDE, int UL, int HL, int DL>
__device__ __forceinline__ void taylor_regs(u32 *v) {
    constexpr int U = 1 << UL, h = 1 << HL, d = 1 << DL;
#pragma unroll
    for (int base = 0; base < 32; base += 2 * h * U)
#pragma unroll
        for (int x = 0; x < U; ++x) {
            auto L = [&](int u) -> u32 & { return v[base + u * U + x]; };
            auto H = [&](int u) -> u32 & { return v[base + (h + u) * U + x]; };
            if constexpr (SIDE == T_FWD) {
#pragma unroll
                for (int t = 0; t < d; ++t) H(t) ^= H(h - d + t);
#pragma unroll
                for (int u = d; u < h; ++u) L(u) ^= H(u - d);
            } else if constexpr (SIDE == T_SEED) {
#pragma unroll
                for (int u = 0; u < d; ++u) L(u) ^= L(h - d + u);
#pragma unroll
                for (int u = d; u < h; ++u) L(u) ^= H(u - d);
            } else {
#pragma unroll
                for (int t = 0; t < h - d; ++t) H(t) ^= L(t + d);
#pragma unroll
                for (int t = 0; t < d; ++t) H(h - d + t) ^= H(t);
            }
        }
}

// Pair bit: register bit PB; the half's units are ordered by register bits PB - 1 .. TB,
// then by the lane bits 5 (and, LANES == 2, 4); d = one unit, lower register bits run
// in parallel.
template <int SIDE, int PB, int TB, int LANES>
__device__ __forceinline__ void taylor_lanes(u32 *v) {
    constexpr int U = 1 << TB, NT = 1 << (PB - TB);
    const u32 lane = threadIdx.x & 63;
    const u32 ord = LANES == 2 ? lane >> 4 : lane >> 5;  // 0 .. 2^LANES - 1, bit 5 first
    constexpr u32 M = (1u << LANES) - 1;
    const u32 no = (SIDE == T_OUT ? ord + 1 : ord - 1) & M;
    const int nb = (int)((LANES == 2 ? (lane & 15) | no << 4 : (lane & 31) | no << 5) << 2);
    const bool first = ord == 0, last = ord == M;
#pragma unroll
    for (int base = 0; base < 32; base += 2 << PB)
#pragma unroll
        for (int x = 0; x < U; ++x) {
            auto L = [&](int t) -> u32 & { return v[base + t * U + x]; };
            auto H = [&](int t) -> u32 & { return v[base + (1 << PB) + t * U + x]; };
            if constexpr (SIDE != T_OUT) {
                if constexpr (SIDE == T_FWD) {
                    const u32 f = bperm(nb, H(NT - 1));
                    H(0) ^= first ? f : 0u;
                }
                u32 y[NT];
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    const u32 prev = t ? H(t ? t - 1 : 0) : (SIDE == T_SEED ? L(NT - 1) : 0u);
                    y[t] = bperm(nb, last ? prev : H(t));
                }
#pragma unroll
                for (int t = 0; t < NT; ++t) L(t) ^= y[t];
            } else {
                u32 y[NT];
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    const u32 next = t + 1 < NT ? L(t + 1 < NT ? t + 1 : 0) : 0u;
                    y[t] = bperm(nb, first ? next : L(t));
                }
#pragma unroll
                for (int t = 0; t < NT; ++t) H(t) ^= y[t];
                const u32 f = bperm(nb, H(0));
                H(NT - 1) ^= last ? f : 0u;
            }
        }
}

// the layers within the lower eight index bits: registers 0..2 of the number are
// index bits 5..7, the word holds bits 0..4
template <int SIDE>
__device__ __forceinline__ void taylor_low(u32 *v) {
    auto words = [&](auto nw, auto d) {
        constexpr int NW = decltype(nw)::value, D = decltype(d)::value;
#pragma unroll
        for (int b = 0; b < 32; b += 2 * NW) taylor_words<SIDE, NW, D>(v, b, b + NW);
    };
#define IC(x) std::integral_constant<int, x>()
    if constexpr (SIDE != T_OUT) {
        words(IC(4), IC(8));
        step_end();
        words(IC(2), IC(4));
        step_end();
        words(IC(1), IC(2));
        step_end();
        taylor_in_word<SIDE, 16, 1>(v);
        step_end();
        words(IC(4), IC(32));   // within index bits 4..7
        step_end();
        words(IC(2), IC(16));
        step_end();
        words(IC(4), IC(64));
        step_end();
        words(IC(1), IC(16));
        step_end();
        taylor_in_word<SIDE, 8, 2>(v);  // within index bits 0..3
        step_end();
        taylor_in_word<SIDE, 4, 1>(v);
        step_end();
        taylor_in_word<SIDE, 8, 4>(v);
        step_end();
        taylor_in_word<SIDE, 2, 1>(v);
        step_end();
    } else {
        taylor_in_word<SIDE, 2, 1>(v);
        step_end();
        taylor_in_word<SIDE, 8, 4>(v);
        step_end();
        taylor_in_word<SIDE, 4, 1>(v);
        step_end();
        taylor_in_word<SIDE, 8, 2>(v);
        step_end();
        words(IC(1), IC(16));
        step_end();
        words(IC(4), IC(64));
        step_end();
        words(IC(2), IC(16));
        step_end();
        words(IC(4), IC(32));
        step_end();
        taylor_in_word<SIDE, 16, 1>(v);
        step_end();
        words(IC(1), IC(2));
        step_end();
        words(IC(2), IC(4));
        step_end();
        words(IC(4), IC(8));
        step_end();
    }
#undef IC
}

// ------------------------------------------------------------------ the stages of a row
//
// Register number bits 4, 3, 1 hold the index bits 14, 13, 11 and, from stage 7 on,
// bit 2 holds index bit 7: the value's bit number is (b4, b3, b1, b2) from the lowest.
__device__ constexpr int vreg(int e) { return (e & 1) << 4 | (e & 2) << 2 | (e & 4) >> 1 | (e & 8) >> 1; }

// f0 += c f1 over 2^BITS elements (f: the constant's forms), planes at registers r0 +
// vreg(e), r1 + vreg(e)
template <int BITS, class Fm>
__device__ __forceinline__ void madd(u32 *v, int r0, int r1, const Fm &f) {
    u32 c[BITS < 4 ? 4 : BITS], a[BITS < 4 ? 4 : BITS];
#pragma unroll
    for (int e = 0; e < (BITS < 4 ? 4 : BITS); ++e) {
        c[e] = e < BITS ? v[r0 + vreg(e)] : 0u;
        a[e] = e < BITS ? v[r1 + vreg(e)] : 0u;
    }
    if constexpr (BITS <= 4)
        mul4<0, 0>(c, a, f);
    else if constexpr (BITS == 8)
        mul8<0>(c, a, f);
    else
        mul16(c, a, f);
#pragma unroll
    for (int e = 0; e < BITS; ++e) v[r0 + vreg(e)] = c[e];
}

// the lanes' constants of stage I: s_I of the point bits held by the wave (base) and
// by the lane bits 5, 4, 3, 2, 1 (J5 .. J1: their index bits, 0: none)
struct LaneBits {
    u32 m5, m4, m3, m2, m1;
};
template <int I, int NW, int J5, int J4, int J3 = 0, int J2 = 0, int J1 = 0>
__device__ __forceinline__ void lane_forms(u32 *w, const LaneBits &b, u32 plus_one) {
    unroll<0, NW>([&](auto h) {
        constexpr u32 c15 = forms81(TW(I, 15)).w[h], c5 = forms81(TW(I, J5)).w[h], c4 = forms81(TW(I, J4)).w[h],
                      c3 = J3 ? forms81(TW(I, J3)).w[h] : 0u, c2 = J2 ? forms81(TW(I, J2)).w[h] : 0u,
                      c1 = J1 ? forms81(TW(I, J1)).w[h] : 0u, one = forms81(1).w[h];
        u32 x = c15 ^ (one & plus_one) ^ (b.m5 & c5) ^ (b.m4 & c4);
        if constexpr (J3 > 0) x ^= b.m3 & c3;
        if constexpr (J2 > 0) x ^= b.m2 & c2;
        if constexpr (J1 > 0) x ^= b.m1 & c1;
        w[h] = x;
    });
}

// A stage on the pairs (f0, f1): forward f0 += c f1, f1 += f0; backwards (the
// transpose) f0 += f1, f1 += c f0. Extending stages (EXTEND): forward f0 += c' f1;
// backwards (f0, f1) <- (f1, f0 + (c' + 1) f1). plus_one: all ones for the seed's transform, whose
// twiddles are c + 1 (added here where c is a compile-time constant).
template <int BITS, bool INV, bool EXTEND, class Fm>
__device__ __forceinline__ void stage(u32 *v, int r0, int r1, const Fm &f, u32 plus_one = 0u) {
    if constexpr (!INV) {
#pragma unroll
        for (int e = 0; e < BITS; ++e) v[r0 + vreg(e)] ^= v[r1 + vreg(e)] & plus_one;
        madd<BITS>(v, r0, r1, f);
        if constexpr (!EXTEND) {
#pragma unroll
            for (int e = 0; e < BITS; ++e) v[r1 + vreg(e)] ^= v[r0 + vreg(e)];
        }
    } else if constexpr (!EXTEND) {
#pragma unroll
        for (int e = 0; e < BITS; ++e) v[r0 + vreg(e)] ^= v[r1 + vreg(e)];
        madd<BITS>(v, r1, r0, f);
    } else {
        madd<BITS>(v, r0, r1, f);
#pragma unroll
        for (int e = 0; e < BITS; ++e) {
            const u32 lo = v[r0 + vreg(e)], hi = v[r1 + vreg(e)];
            v[r0 + vreg(e)] = hi;
            v[r1 + vreg(e)] = lo ^ hi;
        }
    }
}

// Stage 4 .. 0: inside the word
template <int I, bool INV>
__device__ __forceinline__ void word_stage(u32 *v, const LaneBits &lb, u32 plus_one) {
    WordForms<I> f;
    lane_forms<I, 3, 12, 10, 9, 8, 6>(f.w, lb, plus_one);
    if constexpr (!INV) swap_word<0, I>(v);
    stage<16, INV, false>(v, 0, 1, f);
    if constexpr (INV) swap_word<0, I>(v);
}

__device__ __forceinline__ LaneBits lane_bits() {
    const u32 lane = threadIdx.x & 63;
    return LaneBits{bit_mask<5>(lane), bit_mask<4>(lane), bit_mask<3>(lane), bit_mask<2>(lane), bit_mask<1>(lane)};
}

// stages 14 .. 10, whose constants are known: register bits 4..0 are index bits 14..10
template <bool INV>
__device__ __forceinline__ void stages_high(u32 *v, u32 plus_one) {
    auto s14 = [&] {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            u32 &f0 = v[r], &f1 = v[r + 16];
            constexpr u32 c14 = TW(14, 15), c = (c14 & 1) ? ~0u : 0u;
            if constexpr (!INV) {
                f0 ^= f1 & (c ^ plus_one);
            } else {
                const u32 lo = f0, hi = f1;
                f0 = hi;
                f1 = lo ^ (hi & ~c);
            }
        }
    };
    auto s13 = [&] {
        unroll<0, 8>([&](auto r) { stage<2, INV, true>(v, r, r + 8, ConstForms<(TW(13, 15) & 3)>(), plus_one); });
    };
    auto s12 = [&] {
        unroll<0, 4>([&](auto r) { stage<4, INV, false>(v, r, r + 4, ConstForms<TW(12, 15)>(), plus_one); });
    };
    auto s11 = [&] {
        unroll<0, 4>([&](auto q) {  // q bit 1: index bit 12 (register bit 2), q bit 0: index bit 10
            constexpr int r = (q & 2) << 1 | (q & 1);
            stage<4, INV, true>(v, r, r + 2, ConstForms<((TW(11, 15) ^ ((q & 2) ? TW(11, 12) : 0)) & 15)>(), plus_one);
        });
    };
    auto s10 = [&] {
        unroll<0, 2>([&](auto q) {
            constexpr int r = q << 2;
            stage<8, INV, false>(v, r, r + 1, ConstForms<(TW(10, 15) ^ (q ? TW(10, 12) : 0))>(), plus_one);
        });
    };
    if constexpr (!INV) {
        s14();
        step_end();
        s13();
        step_end();
        s12();
        step_end();
        s11();
        step_end();
        s10();
        step_end();
    } else {
        s10();
        step_end();
        s11();
        step_end();
        s12();
        step_end();
        s13();
        step_end();
        s14();
        step_end();
    }
}

// stages 9 .. 0. On entry (forward) lane bits 5..1 are index bits 9..5; afterwards
// index bits 12, 10, 9, 8, 6, register bit 0 index bit 0, word bits 4..0 index bits 5..1.
template <bool INV>
__device__ __forceinline__ void stages_low(u32 *v, const LaneBits &lb, u32 plus_one) {
    auto s9 = [&] {
        LaneForms f;
        lane_forms<9, 1, 12, 10>(f.w, lb, plus_one);
        unroll<0, 2>([&](auto q) { stage<8, INV, false>(v, q, q + 4, f); });
    };
    auto s8 = [&] {
        LaneForms f, g;
        lane_forms<8, 1, 12, 10>(f.w, lb, plus_one);
        constexpr u32 c9 = forms81(TW(8, 9)).w[0];
        g.w[0] = f.w[0] ^ c9;
        stage<8, INV, false>(v, 0, 1, f);
        stage<8, INV, false>(v, 4, 5, g);
    };
    auto s7 = [&] {
        // the extending stage's constant without its leading bit 8 (forms27 of the low byte)
        LaneForms f, g;
        constexpr u32 c15 = forms27(TW(7, 15) & 255), c12 = forms27(TW(7, 12) & 255), c10 = forms27(TW(7, 10) & 255),
                      c9 = forms27(TW(7, 9) & 255), c8 = forms27(TW(7, 8) & 255), c1 = forms27(1);
        f.w[0] = c15 ^ (c1 & plus_one) ^ (lb.m5 & c12) ^ (lb.m4 & c10) ^ (lb.m3 & c9);
        g.w[0] = f.w[0] ^ c8;
        stage<8, INV, true>(v, 0, 4, f);
        stage<8, INV, true>(v, 1, 5, g);
    };
    auto s6 = [&] {
        LaneForms f;
        lane_forms<6, 3, 12, 10, 9, 8>(f.w, lb, plus_one);
        stage<16, INV, false>(v, 0, 1, f);
    };
    auto s5 = [&] {
        LaneForms f;
        lane_forms<5, 3, 12, 10, 9, 8, 6>(f.w, lb, plus_one);
        stage<16, INV, false>(v, 0, 1, f);
    };
    // within index bits 8 and 9 (register bits 0 and 2)
    auto t89 = [&] {
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int r = (q & 1) << 1 | (q & 6) << 2;
            u32 &a0 = v[r], &a1 = v[r + 1], &a2 = v[r + 4], &a3 = v[r + 5];
            if constexpr (!INV) {  // T_FWD: a2 += a3, a1 += a2; T_SEED: a0 += a1, a1 += a2
                a2 ^= a3 & ~plus_one;
                a0 ^= a1 & plus_one;
                a1 ^= a2;
            } else {
                a2 ^= a1;
                a3 ^= a2;
            }
        }
    };
    if constexpr (!INV) {
        swap_lane<2, 5>(v);
        step_end();
        swap_lane<0, 4>(v);
        step_end();
        t89();
        step_end();
        s9();
        step_end();
        s8();
        step_end();
        swap_lane<2, 3>(v);
        step_end();
        s7();
        step_end();
        swap_lane<0, 2>(v);
        step_end();
        s6();
        step_end();
        swap_lane<0, 1>(v);
        step_end();
        s5();
        step_end();
        word_stage<4, INV>(v, lb, plus_one);
        step_end();
        word_stage<3, INV>(v, lb, plus_one);
        step_end();
        word_stage<2, INV>(v, lb, plus_one);
        step_end();
        word_stage<1, INV>(v, lb, plus_one);
        step_end();
        word_stage<0, INV>(v, lb, plus_one);
        step_end();
    } else {
        word_stage<0, INV>(v, lb, plus_one);
        step_end();
        word_stage<1, INV>(v, lb, plus_one);
        step_end();
        word_stage<2, INV>(v, lb, plus_one);
        step_end();
        word_stage<3, INV>(v, lb, plus_one);
        step_end();
        word_stage<4, INV>(v, lb, plus_one);
        step_end();
        s5();
        step_end();
        swap_lane<0, 1>(v);
        step_end();
        s6();
        step_end();
        swap_lane<0, 2>(v);
        step_end();
        s7();
        step_end();
        swap_lane<2, 3>(v);
        step_end();
        s8();
        step_end();
        s9();
        step_end();
        t89();
        step_end();
        swap_lane<0, 4>(v);
        step_end();
        swap_lane<2, 5>(v);
        step_end();
    }
}

// ------------------------------------------------------------------ change of basis

constexpr int RUN_PITCH = 36;                    // words from one run of 32 to the next in LDS
constexpr int ROW_LDS = 32 * RUN_PITCH + 16;     // words of one row (the two rows of a wave on other banks)
constexpr int FWD_WAVES = 4;                     // waves of a workgroup

// The Taylor layers on a row whose lane rho holds words 16 rho .. of each half (register
// bit 4: index bit 14), leaving index bits 14..10 in the register number and 9..5 in
// lane bits 5..1 (all but the layer within bits 8 and 9, which stages_low runs).
template <int SIDE>
__device__ __forceinline__ void to_stages(u32 *v, u32 *lds) {
    const u32 lane = threadIdx.x & 63, rho = (lane >> 5) | (lane & 0x1e);
    taylor_runs<SIDE, 14>(v);
    step_end();
    swap_lane<4, 4>(v);
    step_end();
    taylor_runs<SIDE, 13>(v);
    step_end();
    swap_lane<4, 3>(v);
    step_end();
    taylor_runs<SIDE, 12>(v);
    step_end();
    swap_lane<4, 2>(v);
    step_end();
    taylor_runs<SIDE, 11>(v);
    step_end();
    swap_lane<4, 1>(v);
    step_end();
    taylor_runs<SIDE, 10>(v);
    step_end();
    swap_lane<4, 5>(v);
    step_end();
    taylor_words<SIDE, 16, 2>(v, 0, 16);
    step_end();
    taylor_words<SIDE, 8, 1>(v, 0, 8);
    step_end();
    taylor_words<SIDE, 8, 1>(v, 16, 24);
    step_end();
    taylor_low<SIDE>(v);
    step_end();
    u32 *row = lds + (lane & 1) * ROW_LDS;
#pragma unroll
    for (int t = 0; t < 32; t += 4) *(uint4 *)(row + rho * RUN_PITCH + t) = make_uint4(v[t], v[t + 1], v[t + 2], v[t + 3]);
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int t = 0; t < 32; ++t) v[t] = row[t * RUN_PITCH + (lane >> 1)];
    taylor_regs<SIDE, 0, 4, 0>(v);          // bit 14 against bits 13..10
    step_end();
    taylor_lanes<SIDE, 3, 0, 1>(v);         // bit 13 against bits 12..9
    step_end();
    taylor_lanes<SIDE, 2, 0, 2>(v);         // bit 12 against bits 11..8
    step_end();
    taylor_regs<SIDE, 2, 2, 0>(v);          // within bits 14..12
    step_end();
    taylor_regs<SIDE, 2, 1, 0>(v);
    step_end();
    taylor_lanes<SIDE, 1, 0, 1>(v);         // within bits 11..8
    step_end();
    taylor_lanes<SIDE, 0, 0, 2>(v);
    step_end();
    taylor_regs<SIDE, 0, 1, 0>(v);
    step_end();
}

// The transpose, backwards; index bit 14 = 0 (registers 0..15) is the output half, whose
// word 16 rho + t is register t.
__device__ __forceinline__ void from_stages(u32 *v, u32 *lds) {
    constexpr int SIDE = T_OUT;
    const u32 lane = threadIdx.x & 63, rho = (lane >> 5) | (lane & 0x1e);
    taylor_regs<SIDE, 0, 1, 0>(v);
    step_end();
    taylor_lanes<SIDE, 0, 0, 2>(v);
    step_end();
    taylor_lanes<SIDE, 1, 0, 1>(v);
    step_end();
    taylor_regs<SIDE, 2, 1, 0>(v);
    step_end();
    taylor_regs<SIDE, 2, 2, 0>(v);
    step_end();
    taylor_lanes<SIDE, 2, 0, 2>(v);
    step_end();
    taylor_lanes<SIDE, 3, 0, 1>(v);
    step_end();
    taylor_regs<SIDE, 0, 4, 0>(v);
    step_end();
    u32 *row = lds + (lane & 1) * ROW_LDS;
#pragma unroll
    for (int t = 0; t < 32; ++t) row[t * RUN_PITCH + (lane >> 1)] = v[t];
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int t = 0; t < 32; t += 4) {
        const uint4 q = *(const uint4 *)(row + rho * RUN_PITCH + t);
        v[t] = q.x;
        v[t + 1] = q.y;
        v[t + 2] = q.z;
        v[t + 3] = q.w;
    }
    taylor_low<SIDE>(v);
    step_end();
    taylor_words<SIDE, 8, 1>(v, 0, 8);
    step_end();
    taylor_words<SIDE, 8, 1>(v, 16, 24);
    step_end();
    taylor_words<SIDE, 16, 2>(v, 0, 16);
    step_end();
    swap_lane<4, 5>(v);
    step_end();
    taylor_runs<SIDE, 10>(v);
    step_end();
    swap_lane<4, 1>(v);
    step_end();
    taylor_runs<SIDE, 11>(v);
    step_end();
    swap_lane<4, 2>(v);
    step_end();
    taylor_runs<SIDE, 12>(v);
    step_end();
    swap_lane<4, 3>(v);
    step_end();
    taylor_runs<SIDE, 13>(v);
    step_end();
    swap_lane<4, 4>(v);
    step_end();
    // (the layer of bit 14 changes only the half that is not output)
}

// ------------------------------------------------------------------ reading the packed inputs

typedef u32 u32x4 __attribute__((ext_vector_type(4), aligned(4)));

// 16 words from bit src, which with the 511 after it lies inside the string
__device__ __forceinline__ void load_run(u32 *v, const uint64_t *bits, uint64_t src) {
    const u32 *b = (const u32 *)bits + (src >> 5);
    const int sh = (int)(src & 31);
    u32 w[17];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const u32x4 q = *(const __attribute__((address_space(1))) u32x4 *)(b + 4 * k);
        w[4 * k] = q.x;
        w[4 * k + 1] = q.y;
        w[4 * k + 2] = q.z;
        w[4 * k + 3] = q.w;
    }
    w[16] = *(const __attribute__((address_space(1))) u32 *)(b + (sh ? 16 : 15));
#pragma unroll
    for (int k = 0; k < 16; ++k) v[k] = __builtin_amdgcn_alignbit(w[k + 1], w[k], sh);
}

// ------------------------------------------------------------------ kernels

// Whether the Dodis input has no one bit or no zero bit (the flags' parts: JobDev::flags)
constexpr u32 PARTS_MAX = 31;
__device__ inline bool degenerate(const Gf2Job &J) {
    if (!J.degen_n) return false;
    const u32 parts = J.flags[0] < PARTS_MAX ? J.flags[0] : PARTS_MAX;
    u32 one_ = 0, zero_ = 0;
    for (u32 g = 0; g < parts; ++g) {
        one_ |= J.flags[2 + 2 * g];
        zero_ |= J.flags[3 + 2 * g];
    }
    return one_ == 0 || zero_ == 0;
}

// part g of the check: words [g c, (g+1) c) of the input
__device__ inline void degen_part(const Gf2Job &J, u32 g, u32 *red) {
    if (threadIdx.x < 2) red[threadIdx.x] = 0;
    __syncthreads();
    const uint64_t nw = (J.degen_n + 63) >> 6, chunk = (nw + PARTS_MAX - 1) / PARTS_MAX;
    const uint64_t w0 = (uint64_t)g * chunk, w1 = w0 + chunk < nw ? w0 + chunk : nw;
    const uint64_t tail = (J.degen_n & 63) ? ((1ull << (J.degen_n & 63)) - 1) : ~0ull;
    u32 one_ = 0, zero_ = 0;
#pragma unroll 4
    for (uint64_t w = w0 + threadIdx.x; w < w1; w += 64 * FWD_WAVES) {
        const uint64_t x = J.ex.bits[w], mk = w + 1 < nw ? ~0ull : tail;
        one_ |= (x & mk) != 0;
        zero_ |= (~x & mk) != 0;
    }
    if (one_) atomicOr(&red[0], 1u);
    if (zero_) atomicOr(&red[1], 1u);
    __syncthreads();
    if (threadIdx.x < 2) J.flags[2 + 2 * g + threadIdx.x] = red[threadIdx.x];
    if (g == 0 && threadIdx.x == 0) J.flags[0] = PARTS_MAX;
}

// Forward transforms: workgroup `wg` of the job takes 8 rows, two to a wave: the input's px
// rows (an odd count padded by an idle one), then the ps seed windows; the workgroups
// after those run the Dodis check. tab: per workgroup its job and its number within
// the job (nullptr: the one job). Bound by instruction issue: 5361 instructions a wave of
// two rows, 17.8 us where each SIMD has one wave (a lone wave issues one in 7 clocks: n =
// 2^20) and 660 us for the 163839 rows of n = 2^30, m = 2^29, 98% of what their mix can
// issue (3.6 clocks each: shifts, masks, moves between lanes and operands in scalar
// registers take four, swaps between lanes eight, the rest two and a half). 113 registers
// hold four waves a SIMD; five or six waves spill 59 or 125 registers.
__global__ void __launch_bounds__(64 * FWD_WAVES) __attribute__((amdgpu_waves_per_eu(4))) k_gf2_fwd(const Gf2Job *jobs, Gf2Job one, const uint2 *tab) {
    __shared__ __align__(16) u32 lds_all[FWD_WAVES * 2 * ROW_LDS];
    const uint2 tw = tab ? tab[blockIdx.x] : make_uint2(0, blockIdx.x);
    const Gf2Job &J = jobs ? jobs[tw.x] : one;
    const u32 pxe = (J.px + 1) & ~1u, rows = pxe + J.ps, row_wgs = (rows + 2 * FWD_WAVES - 1) / (2 * FWD_WAVES);
    if (tw.y >= row_wgs) {
        degen_part(J, tw.y - row_wgs, lds_all);
        return;
    }
    const u32 wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    u32 *lds = lds_all + wave * 2 * ROW_LDS;
    const u32 row0 = (tw.y * FWD_WAVES + wave) * 2;
    if (row0 >= rows) return;  // (waves of a workgroup do not meet again)
    const bool seed = row0 >= pxe;
    const u32 r = row0 + (lane & 1) - (seed ? pxe : 0u);
    const bool valid = r < (seed ? J.ps : J.px);
    const u32 rho = (lane >> 5) | (lane & 0x1e);

    // this lane's runs: words 16 rho .. of the row's lower half and, for a seed
    // window, of its upper half
    u32 v[32];
    {
        const Emb &e = seed ? J.ey : J.ex;
        const int64_t B = BLOCK_BITS;
        int64_t p0 = (int64_t)r * B + rho * 512;
        if (seed) p0 += (int64_t)J.n - B - 1 - (int64_t)(J.px - 1) * B;
        bool fast;
        uint64_t s0 = 0, s1 = 0;
        if (!seed) {
            if (e.mode == EMB_PREFIX) {
                fast = p0 + 512 <= (int64_t)e.len;
                s0 = (uint64_t)p0;
            } else {
                const int64_t low = (int64_t)e.N - 512 - p0;
                fast = low >= 0 && low + 512 <= (int64_t)e.len && p0 + 512 <= (int64_t)e.a;
                s0 = (uint64_t)low;
            }
        } else {
            const int64_t P = (int64_t)e.P, p1 = p0 + B;
            int64_t r0 = p0 + (int64_t)e.rot, r1 = p1 + (int64_t)e.rot;
            while (r0 >= P) r0 -= P;
            while (r1 >= P) r1 -= P;
            fast = p0 >= 0 && p1 + 512 <= (int64_t)e.N && r0 + 512 <= P && r1 + 512 <= P;
            s0 = (uint64_t)r0;
            s1 = (uint64_t)r1;
        }
#pragma unroll
        for (int k = 0; k < 32; ++k) v[k] = 0u;
        if (__all(fast && valid)) {
            load_run(v, e.bits, s0);
            if (!seed && e.mode != EMB_PREFIX) reverse_run(v);
            if (seed) load_run(v + 16, e.bits, s1);
        } else if (valid) {  // at an edge of the strings
            if (seed) {
                seed_run(v, e, p0);
                seed_run(v + 16, e, p0 + B);
            } else {
                input_run(v, e, p0);
            }
        }
    }
    const u32 plus_one = seed ? ~0u : 0u;
    if (seed)
        to_stages<T_SEED>(v, lds);
    else
        to_stages<T_FWD>(v, lds);
    stages_high<false>(v, plus_one);
    stages_low<false>(v, lane_bits(), plus_one);
    pin(v);
    if (!valid) return;
    u32 *out = (seed ? J.S : J.X) + (uint64_t)r * J.rs;
    const uint64_t ss = seed ? J.s_ss : J.x_ss;
#pragma unroll
    for (int b0 = 0; b0 < 2; ++b0)
#pragma unroll
        for (int g = 0; g < 4; ++g)
            *(uint4 *)(out + (b0 * 32 + (lane >> 1)) * ss + g * 4) =
                make_uint4(v[b0 + vreg(4 * g)], v[b0 + vreg(4 * g + 1)], v[b0 + vreg(4 * g + 2)], v[b0 + vreg(4 * g + 3)]);
}

// The planes of a variable factor, its forms made as they are needed.
struct PlaneForms {
    static constexpr bool CONSTANT = false;
    const u32 *y;
    template <int H, int I>
    __device__ __forceinline__ u32 plane() const {  // bit I of lo, lo + hi or x0x1x2 hi
        if constexpr (H == 0) return y[I];
        if constexpr (H == 1) return y[I] ^ y[8 + I];
        u32 z = 0;
        unroll<0, 8>([&](auto k) {
            constexpr u32 p = fmul(1u << k, 0x80, 3);
            if constexpr ((p >> I) & 1) z ^= y[8 + k];
        });
        return z;
    }
    template <int H, int L, int I>
    __device__ __forceinline__ u32 part() const {  // bit I of that half's lo, lo + hi or x0x1 hi
        if constexpr (L == 0) return plane<H, I>();
        if constexpr (L == 1) return plane<H, I>() ^ plane<H, 4 + I>();
        u32 z = 0;
        unroll<0, 4>([&](auto k) {
            constexpr u32 p = fmul(1u << k, 8, 2);
            if constexpr ((p >> I) & 1) z ^= plane<H, 4 + k>();
        });
        return z;
    }
    template <int H, int L, int K>
    __device__ __forceinline__ u32 get() const {
        if constexpr (K == 0) return part<H, L, 0>();
        else if constexpr (K == 1) return part<H, L, 1>();
        else if constexpr (K == 2) return part<H, L, 0>() ^ part<H, L, 1>();
        else if constexpr (K == 3) return part<H, L, 2>();
        else if constexpr (K == 4) return part<H, L, 3>();
        else if constexpr (K == 5) return part<H, L, 2>() ^ part<H, L, 3>();
        else if constexpr (K == 6) return part<H, L, 0>() ^ part<H, L, 2>();
        else if constexpr (K == 7) return part<H, L, 1>() ^ part<H, L, 3>();
        else return part<H, L, 0>() ^ part<H, L, 1>() ^ part<H, L, 2>() ^ part<H, L, 3>();
    }
};

// the 16 planes of a slice
__device__ __forceinline__ void load_slice(u32 *x, const u32 *slice) {
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        const u32x4 q = *(const __attribute__((address_space(1))) u32x4 *)(slice + g * 4);
        x[4 * g] = q.x;
        x[4 * g + 1] = q.y;
        x[4 * g + 2] = q.z;
        x[4 * g + 3] = q.w;
    }
}

// Product rows: G[split][r] = sum of X_q S_(r-q+px-1) over the split's q. A wave takes
// every (8 splits)-th q, a lane 32 values of the row; the eight waves' sums meet in LDS.
// About 260 instructions a product; latency at one call's sizes (6 us at n = 2^20, m =
// 2^19, 13 us at n = 2^21, m = 2^20), instruction issue in a batch.
constexpr int MUL_WAVES = 8;
__global__ void __launch_bounds__(64 * MUL_WAVES) k_gf2_mul(const Gf2Job *jobs, Gf2Job one, const uint2 *tab) {
    __shared__ __align__(16) u32 part[MUL_WAVES * ROW_WORDS];
    const uint2 tw = tab ? tab[blockIdx.x] : make_uint2(0, blockIdx.x);
    const Gf2Job &J = jobs ? jobs[tw.x] : one;
    const u32 wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const u32 r = tw.y / J.splits, split = tw.y % J.splits, px = J.px;
    u32 acc[16] = {};
    for (u32 q = split * MUL_WAVES + wave; q < px; q += MUL_WAVES * J.splits) {
        u32 x[16], y[16];
        load_slice(x, J.X + (uint64_t)q * ROW_WORDS + lane * 16);
        load_slice(y, J.S + (uint64_t)(r + px - 1 - q) * ROW_WORDS + lane * 16);
        mul16(acc, x, PlaneForms{y});
    }
#pragma unroll
    for (int g = 0; g < 4; ++g)
        *(uint4 *)(part + wave * ROW_WORDS + g * 256 + lane * 4) =
            make_uint4(acc[4 * g], acc[4 * g + 1], acc[4 * g + 2], acc[4 * g + 3]);
    __syncthreads();
    u32 *out = J.G + ((uint64_t)split * J.pz + r) * ROW_WORDS;
#pragma unroll
    for (u32 i = threadIdx.x; i < ROW_WORDS; i += 64 * MUL_WAVES) {  // word i of the row: slice i / 16, plane i % 16
        u32 s = 0;
#pragma unroll
        for (int w = 0; w < MUL_WAVES; ++w) s ^= part[w * ROW_WORDS + (i & 12) * 64 + (i >> 4) * 4 + (i & 3)];
        out[i] = s;
    }
}


// ------------------------------------------------------------------ transforms over rows
//
// The product rows G_r = sum_q X_q S_(r-q+px-1) are, value by value, a Toeplitz product
// over the field of 2^16: the same transposed product as within a row, by additive
// FFTs over 2^P rows (all 2^P points of the subspace W_P; nothing extends the field here).
// A workgroup runs one slice (32 values of every row) through the whole transform: a
// thread holds four rows of it in registers, two stages at a time. The row bits in
// register number, lane and wave change by LDS between waves (a quarter of
// the planes at a time) and by permlane swaps and DPP moves within one. Stage i's
// twiddles lie in the span of v_0 .. v_(P-1-i): the first stages multiply by elements of
// 16 or 256 only. The Taylor layers run in LDS, 16 or 17 rows of a plane to a thread.

template <int P>
struct Rows {
    static constexpr int ROWS = 1 << P, NT = ROWS / 4, WAVES = NT / 64;
    // eight planes, in two arrays of four; a pad of four words per 16 rows
    static constexpr int PITCH = 16 * 4 + 4, HALF = ROWS / 16 * PITCH, LDS_WORDS = 2 * HALF;
    __device__ static __forceinline__ int at(int row) { return row * 4 + (row >> 4) * 4; }
};

// Forms of one constant per wave, in scalar registers.
struct WaveForms {
    static constexpr bool CONSTANT = false;
    u32 w[3];
    template <int H, int L, int K>
    __device__ __forceinline__ u32 get() const {
        return (u32)__builtin_amdgcn_sbfe((int)w[H], L * 9 + K, 1);
    }
};

// c += a b with b in the subfield of 2^BITS elements
template <int BITS, class Fm>
__device__ __forceinline__ void mul_sub(u32 *c, const u32 *a, const Fm &f) {
    if constexpr (BITS == 4) {
#pragma unroll
        for (int g = 0; g < 4; ++g) mul4<0, 0>(c + 4 * g, a + 4 * g, f);
    } else if constexpr (BITS == 8) {
#pragma unroll
        for (int g = 0; g < 2; ++g) mul8<0>(c + 8 * g, a + 8 * g, f);
    } else {
        mul16(c, a, f);
    }
}
template <int BITS, bool INV, class Fm>
__device__ __forceinline__ void row_butterfly(u32 *f0, u32 *f1, const Fm &f) {
    if constexpr (!INV) {
        mul_sub<BITS>(f0, f1, f);
#pragma unroll
        for (int e = 0; e < 16; ++e) f1[e] ^= f0[e];
    } else {
#pragma unroll
        for (int e = 0; e < 16; ++e) f0[e] ^= f1[e];
        mul_sub<BITS>(f1, f0, f);
    }
}
// Two products by one constant, leaf by leaf, so that they share its masks (nine at a
// time: the masks of a whole product kept for the other would spill).
template <int H, class Fm>
__device__ __forceinline__ void mul8_two(u32 *c, const u32 *a, u32 *d, const u32 *b, const Fm &f) {
    u32 p[4] = {0, 0, 0, 0}, q[4] = {0, 0, 0, 0};
    mul4<H, 0>(p, a, f);
    mul4<H, 0>(q, b, f);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        c[i] ^= p[i];
        c[4 + i] ^= p[i];
        d[i] ^= q[i];
        d[4 + i] ^= q[i];
    }
    step_end();
    const u32 s[4] = {a[0] ^ a[4], a[1] ^ a[5], a[2] ^ a[6], a[3] ^ a[7]};
    const u32 t[4] = {b[0] ^ b[4], b[1] ^ b[5], b[2] ^ b[6], b[3] ^ b[7]};
    mul4<H, 1>(c + 4, s, f);
    mul4<H, 1>(d + 4, t, f);
    step_end();
    mul4<H, 2>(c, a + 4, f);
    mul4<H, 2>(d, b + 4, f);
    step_end();
}
template <int BITS, class Fm>
__device__ __forceinline__ void mul_sub_two(u32 *c, const u32 *a, u32 *d, const u32 *b, const Fm &f) {
    if constexpr (BITS == 4) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            mul4<0, 0>(c + 4 * g, a + 4 * g, f);
            mul4<0, 0>(d + 4 * g, b + 4 * g, f);
        }
    } else if constexpr (BITS == 8) {
        mul8_two<0>(c, a, d, b, f);
        mul8_two<0>(c + 8, a + 8, d + 8, b + 8, f);
    } else {
        u32 p[8] = {0, 0, 0, 0, 0, 0, 0, 0}, q[8] = {0, 0, 0, 0, 0, 0, 0, 0};
        mul8_two<0>(p, a, q, b, f);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            c[i] ^= p[i];
            c[8 + i] ^= p[i];
            d[i] ^= q[i];
            d[8 + i] ^= q[i];
        }
        step_end();
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            p[i] = a[i] ^ a[8 + i];
            q[i] = b[i] ^ b[8 + i];
        }
        mul8_two<1>(c + 8, p, d + 8, q, f);
        mul8_two<2>(c, a + 8, d, b + 8, f);
    }
}
template <int BITS, bool INV, class Fm>
__device__ __forceinline__ void row_butterfly_two(u32 *f0, u32 *f1, u32 *g0, u32 *g1, const Fm &f) {
    if constexpr (!INV) {
        mul_sub_two<BITS>(f0, f1, g0, g1, f);
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            f1[e] ^= f0[e];
            g1[e] ^= g0[e];
        }
    } else {
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            f0[e] ^= f1[e];
            g0[e] ^= g1[e];
        }
        mul_sub_two<BITS>(f1, f0, g1, g0, f);
    }
}
constexpr int stage_bits(int i) { return i >= 8 ? 4 : i >= 4 ? 8 : 16; }  // of 2^12 rows; fewer rows need no more

// The stages of row bits HI = 2k + 1 and 2k, held in the register number (rows 0..3: bits
// (HI, HI - 1)). wave: the row bits from 8 up that the wave number holds, as bits of the
// row number; lane_row: those of the lane.
template <int HI, bool INV, bool DO_HI, bool DO_LO, bool LANES>
__device__ __forceinline__ void row_round(u32 *v, u32 wave_row, u32 lane_row, u32 plus_one) {
    using Fm = typename std::conditional<LANES, LaneForms, WaveForms>::type;
    auto forms = [&](auto stage) {
        constexpr int I = stage;
        Fm f;
        unroll<0, (stage_bits(I) + 7) / 8 == 2 ? 3 : 1>([&](auto h) {
            constexpr u32 one = forms81(1).w[h];
            u32 x = one & plus_one;
            unroll<HI + 1, ROWS_LG_MAX>([&](auto j) {
                constexpr u32 c = forms81(TW(I, j)).w[h];
                if (LANES && j < 8) x ^= bit_mask<j>(lane_row) & c;
                else x ^= (u32)__builtin_amdgcn_sbfe((int)wave_row, j, 1) & c;
            });
            f.w[h] = x;
        });
        return f;
    };
    auto hi = [&] {
        if constexpr (DO_HI) {
            const Fm f = forms(std::integral_constant<int, HI>());
            row_butterfly_two<stage_bits(HI), INV>(v, v + 32, v + 16, v + 48, f);
            step_end();
        }
    };
    auto lo = [&] {
        if constexpr (DO_LO) {
            Fm f = forms(std::integral_constant<int, HI - 1>());
            row_butterfly<stage_bits(HI - 1), INV>(v, v + 16, f);
            step_end();
            unroll<0, stage_bits(HI - 1) == 16 ? 3 : 1>([&](auto h) {
                constexpr u32 c = forms81(TW(HI - 1, HI)).w[h];
                f.w[h] ^= c;
            });
            row_butterfly<stage_bits(HI - 1), INV>(v + 32, v + 48, f);
            step_end();
        }
    };
    if constexpr (!INV) {
        hi();
        lo();
    } else {
        lo();
        hi();
    }
}

// exchange row (register) bit RB of v[64] with lane bit LB
template <int RB, int LB>
__device__ __forceinline__ void swap_row_lane(u32 *v) {
#pragma unroll
    for (int t = 0; t < 64; ++t) {
        if (t & (16 << RB)) continue;
        u32 &a = v[t], &b = v[t | (16 << RB)];
        if constexpr (LB == 5) {
            const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
            a = r[0];
            b = r[1];
        } else if constexpr (LB == 4) {
            const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
            a = r[0];
            b = r[1];
        } else if constexpr (LB == 3 || LB == 2) {
            constexpr int up = LB == 3 ? 0xc : 0xa;
            const u32 na = (u32)__builtin_amdgcn_update_dpp((int)a, (int)b, 0x110 + (1 << LB), 0xf, up, false);
            b = (u32)__builtin_amdgcn_update_dpp((int)b, (int)a, 0x100 + (1 << LB), 0xf, up ^ 0xf, false);
            a = na;
        } else {
            constexpr int perm = LB == 1 ? 0x4E : 0xB1;  // lanes exchanged in pairs 0-2, 1-3 or 0-1, 2-3
            const bool up = (threadIdx.x >> LB) & 1;
            const u32 pa = (u32)__builtin_amdgcn_update_dpp(0, (int)a, perm, 0xf, 0xf, true);
            const u32 pb = (u32)__builtin_amdgcn_update_dpp(0, (int)b, perm, 0xf, 0xf, true);
            a = up ? pb : a;
            b = up ? b : pa;
        }
    }
}

// The basis change of 2^P rows of eight planes in LDS, two planes to a thread. (The thread's
// number is hidden from the optimizer at every step: it would otherwise keep the
// addresses of all steps, for all planes, in registers, and spill.)
template <int SIDE, int P>
__device__ __forceinline__ void rows_basis(u32 *lds) {
    using Rw = Rows<P>;
    auto thread = [](int &pl, int &u) {  // plane, and u < ROWS / 16
        int t = threadIdx.x;
        asm volatile("" : "+v"(t));
        pl = t & 3;
        u = t >> 2;
    };
    // 2^R rows from word `at` on, `pitch` words apart
    auto units = [&](auto rr, u32 *at, auto pitch) {
        constexpr int R = decltype(rr)::value, D = decltype(pitch)::value;
        u32 a[1 << R], c[1 << R];
#pragma unroll
        for (int k = 0; k < (1 << R); ++k) a[k] = at[k * D];
#pragma unroll
        for (int k = 0; k < (1 << R); ++k) c[k] = at[k * D + Rw::HALF];
        basis_units<SIDE, R>(a);
        basis_units<SIDE, R>(c);
#pragma unroll
        for (int k = 0; k < (1 << R); ++k) at[k * D] = a[k];
#pragma unroll
        for (int k = 0; k < (1 << R); ++k) at[k * D + Rw::HALF] = c[k];
    };
#define IC(x) std::integral_constant<int, x>()
    constexpr int R = P - 8;  // bits above the lower eight
    auto classes = [&](auto kk, auto rr, int rho, u32 *base) {
#pragma unroll 1
        for (int h = 0; h < 2; ++h, base += Rw::HALF)
            taylor_classes<SIDE, decltype(kk)::value, decltype(rr)::value>(
                rho, [&](int row) { return base[Rw::at(row)]; }, [&](int row, u32 w) { base[Rw::at(row)] = w; });
    };
    auto top = [&] {  // those bits against the lower eight
        if constexpr (R > 0) {
            __syncthreads();
            int pl, u;
            thread(pl, u);
            for (int rho = u; rho < 255; rho += Rw::ROWS / 16) classes(IC(8), IC(R), rho, lds + pl);
        }
    };
    auto high = [&] {  // within them
        if constexpr (R > 1) {
            __syncthreads();
            int pl, u;
            thread(pl, u);
            for (int base = u; base < 256; base += Rw::ROWS / 16)
                units(IC(R), lds + Rw::at(base) + pl, IC(Rw::PITCH * 16));
        }
    };
    auto low_classes = [&] {  // bits 7..4 against 3..0
        __syncthreads();
        int pl, u;
        thread(pl, u);
        if ((u & 15) < 15) classes(IC(4), IC(4), u & 15, lds + (u >> 4) * 16 * Rw::PITCH + pl);
    };
    auto mid = [&] {
        __syncthreads();
        int pl, u;
        thread(pl, u);
        units(IC(4), lds + Rw::at((u >> 4) * 256 + (u & 15)) + pl, IC(Rw::PITCH));
    };
    auto low = [&] {
        __syncthreads();
        int pl, u;
        thread(pl, u);
        units(IC(4), lds + u * Rw::PITCH + pl, IC(4));
    };
#undef IC
    if constexpr (SIDE != T_OUT) {
        top();
        high();
        low_classes();
        mid();
        low();
    } else {
        low();
        mid();
        low_classes();
        high();
        top();
    }
    __syncthreads();
}

// Moves v from rows row_out(b) to rows row_in(b) of this thread (b < 4), half of the planes at
// a time; step(lds) runs in between on the rows of eight planes.
template <int P, class Out, class In, class Step>
__device__ __forceinline__ void rows_exchange(u32 *v, u32 *lds, Out &&row_out, In &&row_in, Step &&step) {
    using Rw = Rows<P>;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const u32 *q = v + b * 16 + 8 * c + 4 * h;
                *(uint4 *)(lds + Rw::at(row_out(b)) + h * Rw::HALF) = make_uint4(q[0], q[1], q[2], q[3]);
            }
        step(lds);
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const uint4 q = *(const uint4 *)(lds + Rw::at(row_in(b)) + h * Rw::HALF);
                v[b * 16 + 8 * c + 4 * h] = q.x;
                v[b * 16 + 8 * c + 4 * h + 1] = q.y;
                v[b * 16 + 8 * c + 4 * h + 2] = q.z;
                v[b * 16 + 8 * c + 4 * h + 3] = q.w;
            }
        __syncthreads();
    }
}

// Row of register row b when the register number holds row bits HI and HI - 1, the lanes
// row bits 5..0 (or the lower six without them) and the waves the rest.
template <int P, int HI>
__device__ __forceinline__ int row_at(int b) {
    const int t = threadIdx.x;  // the row number without bits HI, HI - 1
    const int low = t & ((1 << (HI - 1)) - 1), high = t >> (HI - 1);
    return low | b << (HI - 1) | high << (HI + 1);
}

// first layout: register bits = row bits P - 1, P - 2
template <int P, bool INV>
__device__ __forceinline__ void rows_stages(u32 *v, u32 *lds, u32 plus_one) {
    const u32 lane = threadIdx.x & 63;
    const u32 wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    auto sync = [](u32 *) { __syncthreads(); };
    // register row bits (HI, HI - 1) in rounds 11/10, 9/8, 7/6, 5/4, 3/2, 1/0; an odd P starts
    // with the upper bit alone (the first round has no row bits above it)
    auto ex = [&](auto from, auto to) {
        rows_exchange<P>(v, lds, [](int b) { return row_at<P, decltype(from)::value>(b); },
                         [](int b) { return row_at<P, decltype(to)::value>(b); }, sync);
    };
#define IC(x) std::integral_constant<int, x>()
    // rows held before round HI: for HI >= 9 the wave number's bits that lie above HI
    auto wave_above = [&](int hi) { return (u32)((threadIdx.x >> 6 << 6) >> (hi - 1)) << (hi + 1); };
    auto r11 = [&] { row_round<11, INV, true, true, false>(v, 0u, 0u, plus_one); };
    auto r10 = [&] { row_round<10, INV, true, false, false>(v, 0u, 0u, plus_one); };
    auto r9 = [&] {
        row_round<9, INV, true, true, false>(v, __builtin_amdgcn_readfirstlane(wave_above(9)), 0u, plus_one);
    };
    auto r8 = [&] { row_round<8, INV, true, false, false>(v, 0u, 0u, plus_one); };
    auto r7 = [&] { row_round<7, INV, true, true, false>(v, wave << 8, 0u, plus_one); };
    auto r5 = [&] { row_round<5, INV, true, true, true>(v, wave << 8, lane << 2, plus_one); };
    auto r3 = [&] { row_round<3, INV, true, true, true>(v, wave << 8, lane << 2, plus_one); };
    auto r1 = [&] { row_round<1, INV, true, true, true>(v, wave << 8, lane << 2, plus_one); };
    static_assert(P >= ROWS_LG_MIN && P <= ROWS_LG_MAX, "rows");
    if constexpr (!INV) {
        if constexpr (P == 12) {
            r11();
            ex(IC(11), IC(9));
        }
        if constexpr (P == 11) {
            r10();
            ex(IC(10), IC(9));
        }
        if constexpr (P >= 10) {
            r9();
            ex(IC(9), IC(7));
        }
        if constexpr (P == 9) {
            r8();
            ex(IC(8), IC(7));
        }
        r7();
        swap_row_lane<1, 5>(v);
        swap_row_lane<0, 4>(v);
        r5();
        swap_row_lane<1, 3>(v);
        swap_row_lane<0, 2>(v);
        r3();
        swap_row_lane<1, 1>(v);
        swap_row_lane<0, 0>(v);
        r1();
    } else {
        r1();
        swap_row_lane<0, 0>(v);
        swap_row_lane<1, 1>(v);
        r3();
        swap_row_lane<0, 2>(v);
        swap_row_lane<1, 3>(v);
        r5();
        swap_row_lane<0, 4>(v);
        swap_row_lane<1, 5>(v);
        r7();
        if constexpr (P == 9) {
            ex(IC(7), IC(8));
            r8();
        }
        if constexpr (P >= 10) {
            ex(IC(7), IC(9));
            r9();
        }
        if constexpr (P == 11) {
            ex(IC(9), IC(10));
            r10();
        }
        if constexpr (P == 12) {
            ex(IC(9), IC(11));
            r11();
        }
    }
#undef IC
}

// XB, SB and PB hold the 2^P rows of a slice as the threads of k_gf2_rows_fwd and _inv
// have them: wave by wave, the b-th row of its 64 lanes (b < 4), four words of a lane
// beside those of the next, so that every load and store of a wave is one piece of
// 1 KB. (The products are row by row: any order serves.) Words of a row's 64 lanes:
constexpr u32 UNIT = 64 * 16;
__device__ __forceinline__ u32 unit_at(u32 thread) { return (thread >> 6) * 4 * UNIT + (thread & 63) * 4; }
__device__ __forceinline__ void load_unit(u32 *x, const u32 *p) {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const u32x4 q = *(const __attribute__((address_space(1))) u32x4 *)(p + c * 256);
        x[4 * c] = q.x;
        x[4 * c + 1] = q.y;
        x[4 * c + 2] = q.z;
        x[4 * c + 3] = q.w;
    }
}
// From LDS, where a wave's unit keeps its order (p: this lane's first words).
__device__ __forceinline__ void read_unit(u32 *x, const u32 *p) {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const uint4 q = *(const uint4 *)(p + c * 256);
        x[4 * c] = q.x;
        x[4 * c + 1] = q.y;
        x[4 * c + 2] = q.z;
        x[4 * c + 3] = q.w;
    }
}
// Four words of every lane to LDS, the wave's 1 KB from `to` on, without registers.
__device__ __forceinline__ void load_to_lds(const u32 *from, u32 *to) {
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)from,
                                     (__attribute__((address_space(3))) void *)to, 16, 0, 0);
}
constexpr int WAIT_LOADS = 0x0f70;  // s_waitcnt vmcnt(0), the other counters as they are
__device__ __forceinline__ void store_unit(u32 *p, const u32 *x) {
#pragma unroll
    for (int c = 0; c < 4; ++c) *(uint4 *)(p + c * 256) = make_uint4(x[4 * c], x[4 * c + 1], x[4 * c + 2], x[4 * c + 3]);
}

// Forward: workgroup = slice of a group of X (its hx rows, zeros above) or of a window of
// S (its hx + hz - 1 rows, at the top of the 2^P). With P = 12 one workgroup fills a CU's
// registers and LDS: 5056 workgroups (n = 2^30, m = 2^29) take 1170 us, 59 us a round,
// of which the 7150 instructions a wave (3.1 clocks each) are 40 and the 256 KB in and out
// the rest, hardly overlapped. The larger P is still the cheaper: half of it would double the sums of
// products.
template <int P>
__global__ void __launch_bounds__(Rows<P>::NT) __attribute__((amdgpu_waves_per_eu(P == 12 ? 4 : 1)))
k_gf2_rows_fwd(const Gf2Job *jobs, Gf2Job one, const uint2 *tab) {
    using Rw = Rows<P>;
    __shared__ __align__(16) u32 lds[Rw::LDS_WORDS];
    const uint2 tw = tab ? tab[blockIdx.x] : make_uint2(0, blockIdx.x);
    const Gf2Job &J = jobs ? jobs[tw.x] : one;
    const u32 sl = tw.y % SLICES, blk = tw.y / SLICES;
    const bool seed = blk >= J.nx;
    const u32 g = seed ? blk - J.nx : blk;
    // rows first .. last - 1 of the transform come from rows src + (row - first)
    int first, last;
    uint64_t src;
    if (!seed) {
        first = 0;
        const u32 left = J.px - g * J.hx;
        last = (int)(left < J.hx ? left : J.hx);
        src = (uint64_t)g * J.hx;
    } else {
        // window of group difference g - (nx - 1): seed rows from (g - nx + 1) h - (hx - 1), which is
        // row 0 of S for the difference -(nx - 1) when px is a multiple of hx
        const int64_t h = J.nz > 1 ? (int64_t)J.hz : (int64_t)J.hx;
        const int64_t lo = ((int64_t)g - (int64_t)(J.nx - 1)) * h - (int64_t)(J.hx - 1) + (int64_t)(J.px - 1);
        first = Rw::ROWS - (int)(J.hx + J.hz - 1);
        last = Rw::ROWS;
        // the windows' rows outside 0 .. ps - 1 meet only zero rows of X or unused rows of z
        int64_t s0 = lo, skip = s0 < 0 ? -s0 : 0;
        first += (int)skip;
        s0 += skip;
        const int64_t end = s0 + (last - first);
        if (end > (int64_t)J.ps) last -= (int)(end - (int64_t)J.ps);
        src = (uint64_t)s0;
    }
    const u32 *in = (seed ? J.S + sl * J.s_ss : J.X + sl * J.x_ss) + src * J.rs;
    u32 v[64];
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        const int row = row_at<P, P - 1>(b);
        if (row >= first && row < last) {
            load_slice(v + 16 * b, in + (uint64_t)(row - first) * J.rs);
        } else {
#pragma unroll
            for (int e = 0; e < 16; ++e) v[16 * b + e] = 0u;
        }
    }
    auto own = [](int b) { return row_at<P, P - 1>(b); };
    if (seed)
        rows_exchange<P>(v, lds, own, own, [](u32 *l) { rows_basis<T_SEED, P>(l); });
    else
        rows_exchange<P>(v, lds, own, own, [](u32 *l) { rows_basis<T_FWD, P>(l); });
    rows_stages<P, false>(v, lds, seed ? ~0u : 0u);
    // register rows are now rows 4 tid + b
    u32 *out = (seed ? J.SB : J.XB) + ((uint64_t)(g * SLICES + sl) << (P + 4)) + unit_at(threadIdx.x);
#pragma unroll
    for (int b = 0; b < 4; ++b) store_unit(out + b * UNIT, v + 16 * b);
}

// Sums of products of groups (more than one group of the input): a thread takes one row of
// a slice in TG groups of z, whose seed windows it keeps in registers: the next input
// group needs one new window, and the others shifted by one group. With TG = 4 the
// registers hold two waves a SIMD (one wave alone issues an instruction in 5 clocks, two
// in 2 each) and no operand ahead of its use, so the next input group's row and window
// come straight into LDS while this one's products run. n = 2^30, m = 2^29 (32 groups by
// 16): 1250 -> 640 us, of which the layout of the rows gave 120, the loads ahead 150 and
// the second wave 340; the instructions alone are 450 us (2.5 clocks each). Two turns ahead: 1005 against
// 978 us before the second wave. TG = 1 (one group of z) reads 64 bytes for every product
// and runs at 4.2 TB/s.
template <int TG>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(TG > 1 ? 2 : 4))) k_gf2_rows_prod(const Gf2Job *jobs, Gf2Job one, const uint2 *tab) {
    constexpr bool AHEAD = TG > 1;
    __shared__ __align__(16) u32 lds[AHEAD ? 2 * 4 * 2 * UNIT : 4];  // two turns, four waves, row and window
    const uint2 tw = tab ? tab[blockIdx.x] : make_uint2(0, blockIdx.x);
    const Gf2Job &J = jobs ? jobs[tw.x] : one;
    const u32 lg = J.rows_lg + 6;  // rows of all slices of a group: 2^lg, in 2^(lg - 8) workgroups
    const u32 nz = J.nz, nx = J.nx;
    // the tiles of z that read the same rows run side by side on one XCD (workgroups go to
    // the eight XCDs in turn)
    const u32 tiles = (nz + TG - 1) / TG, turn = tw.y >> 3;
    const u32 g0 = turn % tiles * TG;
    const u32 wave = (u32)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const uint64_t at = ((uint64_t)(turn / tiles * 8 + (tw.y & 7)) * 4 + wave) * UNIT + lane * 4;
    const u32 *const XB = J.XB + at, *const SB = J.SB + at;
    u32 acc[TG][16] = {}, s[TG][16];
    // windows g0 + t + nx - 1 - q; before q = 0, those of t >= 1 in their places for t - 1
#pragma unroll
    for (int t = 1; t < TG; ++t) {
        const u32 w = g0 + t + nx - 1;
        load_unit(s[t - 1], SB + ((uint64_t)(w < nx + nz - 1 ? w : nx + nz - 2) << (lg + 4)));
    }
    auto place = [&](u32 q) { return lds + ((q & 1) * 4 + wave) * 2 * UNIT; };
    auto fetch = [&](u32 q) {
        const u32 *x = XB + ((uint64_t)q << (lg + 4)), *w = SB + ((uint64_t)(g0 + nx - 1 - q) << (lg + 4));
        u32 *to = place(q);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            load_to_lds(x + c * 256, to + c * 256);
            load_to_lds(w + c * 256, to + UNIT + c * 256);
        }
    };
    if constexpr (AHEAD) fetch(0);
    for (u32 q0 = 0; q0 < nx; q0 += TG) {
#pragma unroll
        for (int i = 0; i < TG; ++i) {  // (window of t at q0 + i: place (t - i - 1) mod TG)
            const u32 q = q0 + i;
            if (q >= nx) break;
            u32 x[16];
            if constexpr (AHEAD) {
                // a wave reads only what it fetched itself; the other turn's place was read before
                // the products of the turn before
                __builtin_amdgcn_s_waitcnt(WAIT_LOADS);
                const u32 *from = place(q) + lane * 4;
                read_unit(x, from);
                read_unit(s[(2 * TG - i - 1) % TG], from + UNIT);
                // (read before the next fetch is begun, or the read would wait for that one)
#pragma unroll
                for (int k = 0; k < 16; ++k) asm volatile("" : "+v"(x[k]), "+v"(s[(2 * TG - i - 1) % TG][k]) : : "memory");
                if (q + 1 < nx) fetch(q + 1);
                step_end();
            } else {
                load_unit(x, XB + ((uint64_t)q << (lg + 4)));
                load_unit(s[(2 * TG - i - 1) % TG], SB + ((uint64_t)(g0 + nx - 1 - q) << (lg + 4)));
            }
            // one 8-bit part of x for all windows, then the next: a third of its forms at a time
            const PlaneForms f{x};
#pragma unroll
            for (int t = 0; t < TG; ++t) {
                mul16_low(acc[t], s[(2 * TG + t - i - 1) % TG], f);
                step_end();
            }
#pragma unroll
            for (int t = 0; t < TG; ++t) {
                mul16_sum(acc[t], s[(2 * TG + t - i - 1) % TG], f);
                step_end();
            }
#pragma unroll
            for (int t = 0; t < TG; ++t) {
                mul8<2>(acc[t], s[(2 * TG + t - i - 1) % TG] + 8, f);
                step_end();
            }
        }
    }
#pragma unroll
    for (int t = 0; t < TG; ++t) {
        if (g0 + t >= nz) break;
        store_unit(J.PB + ((uint64_t)(g0 + t) << (lg + 4)) + at, acc[t]);
    }
}

// Backwards: workgroup = slice of a group of z: its product (or, with several groups of the
// input, the sum that k_gf2_rows_prod left), the transform back, and its rows (in reverse
// order) to G. Bound like k_gf2_rows_fwd: 245 us for 1024 workgroups of P = 12.
template <int P>
__global__ void __launch_bounds__(Rows<P>::NT) __attribute__((amdgpu_waves_per_eu(P == 12 ? 4 : 1)))
k_gf2_rows_inv(const Gf2Job *jobs, Gf2Job one, const uint2 *tab) {
    using Rw = Rows<P>;
    __shared__ __align__(16) u32 lds[Rw::LDS_WORDS];
    const uint2 tw = tab ? tab[blockIdx.x] : make_uint2(0, blockIdx.x);
    const Gf2Job &J = jobs ? jobs[tw.x] : one;
    // slices side by side on one XCD (workgroups go to the eight in turn): the 64-byte halves
    // of a line of G meet in its L2
    const u32 r0 = tw.y % SLICES, sl = (r0 & 7) * 8 + (r0 >> 3), g = tw.y / SLICES;
    u32 v[64];
    const uint64_t at = ((uint64_t)(g * SLICES + sl) << (P + 4)) + unit_at(threadIdx.x);
    if (J.nx > 1) {
#pragma unroll
        for (int b = 0; b < 4; ++b) load_unit(v + 16 * b, J.PB + at + b * UNIT);
    } else {  // (then nz is 1 as well)
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            u32 a[16], c[16];
            load_unit(a, J.XB + at + b * UNIT);
            load_unit(c, J.SB + at + b * UNIT);
#pragma unroll
            for (int e = 0; e < 16; ++e) v[16 * b + e] = 0u;
            mul16(v + 16 * b, a, PlaneForms{c});
            step_end();
        }
    }
    rows_stages<P, true>(v, lds, 0u);
    auto own = [](int b) { return row_at<P, P - 1>(b); };
    rows_exchange<P>(v, lds, own, own, [](u32 *l) { rows_basis<T_OUT, P>(l); });
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        const u32 row = (u32)own(b);
        const u32 r = g * J.hz + J.hz - 1 - row;  // (row < hz)
        if (row < J.hz && r < J.pz) {
            u32 *out = J.G + (uint64_t)r * ROW_WORDS + sl * 16;
#pragma unroll
            for (int k = 0; k < 16; k += 4)
                *(uint4 *)(out + k) = make_uint4(v[16 * b + k], v[16 * b + k + 1], v[16 * b + k + 2], v[16 * b + k + 3]);
        }
    }
}

// Backwards transforms of the product rows and the output bits: 8 rows to a workgroup,
// two to a wave. Output block r is in reverse order: position i of the row is z bit
// r B + B - 1 - i. Bound like k_gf2_fwd: 15.4 us with one wave a SIMD, 140 us for the 32768
// rows of n = 2^30, m = 2^29.
__global__ void __launch_bounds__(64 * FWD_WAVES) __attribute__((amdgpu_waves_per_eu(4))) k_gf2_inv(const Gf2Job *jobs, Gf2Job one, const uint2 *tab) {
    __shared__ __align__(16) u32 lds_all[FWD_WAVES * 2 * ROW_LDS];
    const uint2 tw = tab ? tab[blockIdx.x] : make_uint2(0, blockIdx.x);
    const Gf2Job &J = jobs ? jobs[tw.x] : one;
    const u32 wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    u32 *lds = lds_all + wave * 2 * ROW_LDS;
    const u32 r = (tw.y * FWD_WAVES + wave) * 2 + (lane & 1);
    if ((r & ~1u) >= J.pz) return;
    const bool valid = r < J.pz;
    u32 v[32];
#pragma unroll
    for (int t = 0; t < 32; ++t) v[t] = 0u;
    for (u32 s = 0; s < J.splits; ++s) {
        const u32 *row = J.G + ((uint64_t)s * J.pz + (valid ? r : 0u)) * ROW_WORDS;
#pragma unroll
        for (int b0 = 0; b0 < 2; ++b0)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const u32x4 q =
                    *(const __attribute__((address_space(1))) u32x4 *)(row + (b0 * 32 + (lane >> 1)) * 16 + g * 4);
                v[b0 + vreg(4 * g)] ^= q.x;
                v[b0 + vreg(4 * g + 1)] ^= q.y;
                v[b0 + vreg(4 * g + 2)] ^= q.z;
                v[b0 + vreg(4 * g + 3)] ^= q.w;
            }
    }
    stages_low<true>(v, lane_bits(), 0u);
    stages_high<true>(v, 0u);
    from_stages(v, lds);
    pin(v);
    const bool degen = degenerate(J);
    if (r == 0 && lane == 0 && J.status) *J.status = degen ? -3 : 0;
    if (!valid) return;
    const u32 rho = (lane >> 5) | (lane & 0x1e);
    const uint64_t w0 = (uint64_t)r * (BLOCK_BITS / 32) + 496 - 16 * rho;  // first output word of the lane
    const uint64_t zwords = ((J.m + 63) >> 6) << 1;
    u32 *z = (u32 *)J.z;
    u32 o[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) o[k] = degen ? 0u : __brev(v[15 - k]);
    if ((w0 + 16) * 32 <= J.m) {
#pragma unroll
        for (int k = 0; k < 16; k += 4) {
            const u32x4 q = {o[k], o[k + 1], o[k + 2], o[k + 3]};
            *(__attribute__((address_space(1))) u32x4 *)(z + w0 + k) = q;
        }
    } else {
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const uint64_t p = (w0 + k) * 32;
            if (w0 + k < zwords) {
                const u32 w = p >= J.m ? 0u : J.m - p < 32 ? o[k] & ((1u << (J.m - p)) - 1u) : o[k];
                z[w0 + k] = w;
            }
        }
    }
}

// ------------------------------------------------------------------ short extractions, bit by bit
//
// Up to BITS_MAX_WORDS input words the defining sum itself is the fastest way to a result: for
// every input bit one funnel shift gives the 32 seed bits that meet a word of 32
// outputs, and one AND-XOR adds them: 3 instructions (with the bit's mask) for 32
// products, no passes and no workspace. A workgroup takes OW output words and the
// whole input; a lane takes one output word and a share of the input words (the seed
// window of the next input word is the last one's, moved by a word). Circulant n = 16420,
// m = 9000: 6.2 us a call, where the transform's five launches took 26; Toeplitz n = 4096,
// m = 2048, with the wait for it, 32.2 -> 17 us.
constexpr int BITS_NT = 512;

template <int OW>
__global__ void __launch_bounds__(BITS_NT) k_gf2_bits(const Gf2Job *jobs, Gf2Job one, const uint2 *tab) {
    constexpr int SUB = 64 / OW, SHARES = BITS_NT / 64 * SUB;
    __shared__ u32 xw[BITS_MAX_WORDS], sw[BITS_MAX_WORDS + OW + 1];
    __shared__ u32 part[BITS_NT / 64][OW];
    __shared__ u32 seen[2];
    const uint2 tw = tab ? tab[blockIdx.x] : make_uint2(0, blockIdx.x);
    const Gf2Job &J = jobs ? jobs[tw.x] : one;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n = (int)J.n, V = (n + 31) >> 5, w0 = (int)tw.y * OW;
    // input words, and seed word t: positions 32 (w0 - V + 1 + t) + n - 32 ..
    u32 one_ = 0, zero_ = 0;
    if (tid < 2) seen[tid] = 0;
    for (int v = tid; v < V; v += BITS_NT) {
        const u32 x = input_word(J.ex, (int64_t)v * 32);
        const u32 valid = n - v * 32 >= 32 ? ~0u : (1u << (n - v * 32)) - 1u;
        one_ |= x;
        zero_ |= ~x & valid;
        xw[v] = x;
    }
    for (int t = tid; t < V + OW; t += BITS_NT) sw[t] = seed_word(J.ey, (int64_t)(w0 - V + 1 + t) * 32 + n - 32);
    __syncthreads();
    if (J.degen_n) {  // (the input words hold exactly the Dodis input's bits)
        if (one_) atomicOr(&seen[0], 1u);
        if (zero_) atomicOr(&seen[1], 1u);
    }
    const int w = lane % OW, share = wave * SUB + lane / OW, chunk = (V + SHARES - 1) / SHARES;
    const int v0 = share * chunk, v1 = v0 + chunk < V ? v0 + chunk : V;
    u32 acc0 = 0, acc1 = 0;
    if (v0 < v1) {
        u32 hi = sw[w + V - v0];
        for (int v = v0; v < v1; ++v) {
            const u32 lo = sw[w + V - 1 - v], x = xw[v];
            unroll<0, 16>([&](auto b) {
                acc0 = __builtin_amdgcn_bitop3_b32(acc0, __builtin_amdgcn_alignbit(hi, lo, 31 - 2 * b),
                                                   bit_mask<2 * b>(x), 0x78);
                acc1 = __builtin_amdgcn_bitop3_b32(acc1, __builtin_amdgcn_alignbit(hi, lo, 30 - 2 * b),
                                                   bit_mask<2 * b + 1>(x), 0x78);
            });
            hi = lo;
        }
    }
    u32 acc = acc0 ^ acc1;
#pragma unroll
    for (int o = OW; o < 64; o <<= 1) acc ^= bperm((lane ^ o) << 2, acc);
    if (lane < OW) part[wave][lane] = acc;
    __syncthreads();
    const bool degen = J.degen_n && (seen[0] == 0 || seen[1] == 0);
    if (tid < OW) {
        u32 z = 0;
#pragma unroll
        for (int k = 0; k < BITS_NT / 64; ++k) z ^= part[k][tid];
        const int zw = w0 + tid, m = (int)J.m, left = m - zw * 32;
        if (degen || left <= 0) z = 0;
        else if (left < 32) z &= (1u << left) - 1u;
        if (zw < ((m + 63) >> 6) << 1) ((u32 *)J.z)[zw] = z;
    }
    if (tw.y == 0 && tid == 0 && J.status) *J.status = degen ? -3 : 0;
}

}  // namespace

// (few workgroups of many lanes' work for a launch of its own; wider ones, which read the
// input less often, where many jobs share it)
constexpr int BITS_OW_ONE = 4, BITS_OW_MANY = 16;
uint32_t gf2_bits_workgroups(const Gf2Job &j, bool many) {
    const uint32_t ow = many ? BITS_OW_MANY : BITS_OW_ONE, words = (uint32_t)((j.m + 63) >> 6) << 1;
    return (words + ow - 1) / ow;
}
hipError_t launch_gf2_bits(uint32_t wgs, const Gf2Job *jobs, const Gf2Job &one, const uint2 *tab, hipStream_t s) {
    if (jobs) return launch_k(k_gf2_bits<BITS_OW_MANY>, dim3(wgs), dim3(BITS_NT), 0, s, jobs, one, tab);
    return launch_k(k_gf2_bits<BITS_OW_ONE>, dim3(wgs), dim3(BITS_NT), 0, s, jobs, one, tab);
}

uint32_t gf2_fwd_workgroups(const Gf2Job &j) {
    const uint32_t rows = ((j.px + 1) & ~1u) + j.ps;
    return (rows + 2 * FWD_WAVES - 1) / (2 * FWD_WAVES) + (j.degen_n ? PARTS_MAX : 0);
}
uint32_t gf2_mul_workgroups(const Gf2Job &j) { return j.pz * j.splits; }
uint32_t gf2_rows_fwd_workgroups(const Gf2Job &j) { return (2 * j.nx + j.nz - 1) * SLICES; }
// (four groups of z to a thread where there are that many)
uint32_t gf2_rows_prod_workgroups(const Gf2Job &j) {
    if (j.nx <= 1) return 0;
    return (j.nz > 1 ? (j.nz + 3) / 4 : 1) * (SLICES << (j.rows_lg - 8));
}
hipError_t launch_gf2_rows_prod(bool one_group, uint32_t wgs, const Gf2Job *jobs, const Gf2Job &one, const uint2 *tab,
                                hipStream_t s) {
    if (one_group) return launch_k(k_gf2_rows_prod<1>, dim3(wgs), dim3(256), 0, s, jobs, one, tab);
    return launch_k(k_gf2_rows_prod<4>, dim3(wgs), dim3(256), 0, s, jobs, one, tab);
}
uint32_t gf2_rows_inv_workgroups(const Gf2Job &j) { return j.nz * SLICES; }
uint32_t gf2_inv_workgroups(const Gf2Job &j) { return (j.pz + 2 * FWD_WAVES - 1) / (2 * FWD_WAVES); }

hipError_t launch_gf2_fwd(uint32_t wgs, const Gf2Job *jobs, const Gf2Job &one, const uint2 *tab, hipStream_t s) {
    return launch_k(k_gf2_fwd, dim3(wgs), dim3(64 * FWD_WAVES), 0, s, jobs, one, tab);
}
hipError_t launch_gf2_mul(uint32_t wgs, const Gf2Job *jobs, const Gf2Job &one, const uint2 *tab, hipStream_t s) {
    return launch_k(k_gf2_mul, dim3(wgs), dim3(64 * MUL_WAVES), 0, s, jobs, one, tab);
}
#define ROWS_CASE(K, P) case P: return launch_k(K<P>, dim3(wgs), dim3(Rows<P>::NT), 0, s, jobs, one, tab)
hipError_t launch_gf2_rows_fwd(int rows_lg, uint32_t wgs, const Gf2Job *jobs, const Gf2Job &one, const uint2 *tab,
                               hipStream_t s) {
    switch (rows_lg) {
        ROWS_CASE(k_gf2_rows_fwd, 8);
        ROWS_CASE(k_gf2_rows_fwd, 9);
        ROWS_CASE(k_gf2_rows_fwd, 10);
        ROWS_CASE(k_gf2_rows_fwd, 11);
        ROWS_CASE(k_gf2_rows_fwd, 12);
    }
    return hipErrorInvalidValue;
}
hipError_t launch_gf2_rows_inv(int rows_lg, uint32_t wgs, const Gf2Job *jobs, const Gf2Job &one, const uint2 *tab,
                               hipStream_t s) {
    switch (rows_lg) {
        ROWS_CASE(k_gf2_rows_inv, 8);
        ROWS_CASE(k_gf2_rows_inv, 9);
        ROWS_CASE(k_gf2_rows_inv, 10);
        ROWS_CASE(k_gf2_rows_inv, 11);
        ROWS_CASE(k_gf2_rows_inv, 12);
    }
    return hipErrorInvalidValue;
}
#undef ROWS_CASE
hipError_t launch_gf2_inv(uint32_t wgs, const Gf2Job *jobs, const Gf2Job &one, const uint2 *tab, hipStream_t s) {
    return launch_k(k_gf2_inv, dim3(wgs), dim3(64 * FWD_WAVES), 0, s, jobs, one, tab);
}

}  // namespace ext
