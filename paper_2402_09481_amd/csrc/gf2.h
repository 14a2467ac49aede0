// The binary field of the GF(2)[t] transforms and their job descriptors.
//
// The extractors' output is a Toeplitz product over GF(2),
// z_i = XOR_j s_(i-j+n-1) x_j: part of a product of two polynomials over GF(2).
// The transforms here evaluate those polynomials over the field of 2^16
// elements (an additive FFT over the chain of subspaces W_i spanned by the first
// i basis elements), so that one field element stands for 16 coefficients where
// the number-theoretic transforms take a 32- or 64-bit word for each.
//
// Field: the tower GF(2)[x0]/(x0^2+x0+1), [x1]/(x1^2+x1+x0),
// [x2]/(x2^2+x2+x0x1), [x3]/(x3^2+x3+x0x1x2); bit e of an element is the
// coefficient of the product of those x_k whose bit k is set in e. Its bit basis
// v_0, v_1, ... (v_j: bit j alone) spans the subspaces W_i, whose vanishing
// polynomials s_0(x) = x, s_(i+1)(x) = s_i(x)^2 + s_i(x) have coefficients in GF(2)
// and satisfy s_i(v_i) = 1.
#pragma once
#include <stdint.h>

#include "kernels.h"

namespace ext {
namespace gf2 {

// product in the subfield of 2^(2^l) elements
constexpr uint32_t fmul(uint32_t a, uint32_t b, int l = 4) {
    if (l == 0) return a & b;
    const int h = 1 << (l - 1);
    const uint32_t m = (1u << h) - 1;
    const uint32_t a0 = a & m, a1 = a >> h, b0 = b & m, b1 = b >> h;
    const uint32_t p0 = fmul(a0, b0, l - 1), p2 = fmul(a1, b1, l - 1), p1 = fmul(a0 ^ a1, b0 ^ b1, l - 1);
    return (p0 ^ fmul(p2, 1u << (h - 1), l - 1)) | ((p1 ^ p0) << h);
}
// s_i(v)
constexpr uint32_t subspace_poly(int i, uint32_t v) {
    for (int k = 0; k < i; ++k) v = fmul(v, v) ^ v;
    return v;
}

// A multiplication by c is carried out in bit planes: a product of two
// elements of 16 is 16 AND-XORs of planes with nine linear forms of the constant's
// four bits, b0 b1 b0+b1 | b2 b3 b2+b3 | b0+b2 b1+b3 and their sum; one level up, three
// such products (by lo, lo + hi and the level's constant times hi), and once
// more for 16 bits. forms27 holds the 27 bits for an 8-bit constant, and
// Forms the 81 bits for a 16-bit one; both are linear in the constant.
constexpr uint32_t forms9(uint32_t b) {
    const uint32_t b0 = b & 1, b1 = (b >> 1) & 1, b2 = (b >> 2) & 1, b3 = (b >> 3) & 1;
    return b0 | b1 << 1 | (b0 ^ b1) << 2 | b2 << 3 | b3 << 4 | (b2 ^ b3) << 5 | (b0 ^ b2) << 6 | (b1 ^ b3) << 7 |
           (b0 ^ b1 ^ b2 ^ b3) << 8;
}
constexpr uint32_t forms27(uint32_t b) {
    const uint32_t lo = b & 15, hi = (b >> 4) & 15;
    return forms9(lo) | forms9(lo ^ hi) << 9 | forms9(fmul(hi, 8, 2)) << 18;
}
struct Forms {
    uint32_t w[3];
};
constexpr Forms forms81(uint32_t c) {
    const uint32_t lo = c & 255, hi = (c >> 8) & 255;
    return Forms{{forms27(lo), forms27(lo ^ hi), forms27(fmul(hi, 0x80, 3))}};
}
constexpr Forms operator^(const Forms &a, const Forms &b) {
    return Forms{{a.w[0] ^ b.w[0], a.w[1] ^ b.w[1], a.w[2] ^ b.w[2]}};
}

// Blocks: the input is cut into rows of B bits, a row's transform has 2B bits:
// 64 slices of 16 words, one word (32 values) for each of the 16 planes.
constexpr int ROW_LG = 15;
constexpr uint32_t BLOCK_BITS = 1u << (ROW_LG - 1);
constexpr uint32_t ROW_WORDS = 1u << (ROW_LG - 5);
constexpr uint32_t SLICES = 64;

// Input words of the longest extraction that the bit-by-bit kernel takes.
constexpr int BITS_MAX_WORDS = 4096;

// Rows of a transform over rows: 2^ROWS_LG_MIN .. 2^ROWS_LG_MAX.
constexpr int ROWS_LG_MIN = 8, ROWS_LG_MAX = 12;

}  // namespace gf2

// One extraction on the GF(2)[t] path, in the Toeplitz form
// z_i = XOR_j s_(i-j+n-1) x'_j (Dodis and Circulant: x' the reversed input,
// s the periodic seed): x' in px rows of B bits, z in pz rows, and the ps = px + pz - 1
// seed windows of 2B - 1 bits that lie B bits apart. The product rows are
// G_r = sum_q X_q S_(r-q+px-1).
//   direct (rows_lg = 0): the sums term by term.
//   by a transform over 2^rows_lg rows: x' in nx groups of hx rows, z in nz groups of
//   hz rows (hx + hz - 1 <= 2^rows_lg, and hx = hz unless nz = 1); XB and SB hold the
//   transformed groups and the transformed nx + nz - 1 windows of hx + hz - 1 rows, PB
//   (nx > 1) the nz groups' sums of products.
// Word (row r, slice s, plane e) of X and S is at r * rs + s * ss + e.
struct Gf2Job {
    Emb ex, ey;
    uint32_t *X, *S, *G;
    uint32_t *XB, *SB, *PB;
    uint64_t *z;
    int32_t *status;
    uint32_t *flags;      // degenerate check (JobDev::flags)
    uint64_t n, m;
    uint64_t degen_n;
    uint64_t x_ss, s_ss;  // ss of X and S
    uint32_t rs;
    uint32_t px, ps, pz;
    uint32_t splits;      // direct: G is the sum of `splits` arrays of pz rows
    uint32_t rows_lg, hx, hz, nx, nz;
};

// Workgroups of a job in each launch, and the launches: jobs and tab are device
// arrays (tab: for every workgroup its job and its number within the job), or both
// nullptr to run `one`.
uint32_t gf2_bits_workgroups(const Gf2Job &j, bool many);  // the whole extraction bit by bit (many: in a batch)
uint32_t gf2_fwd_workgroups(const Gf2Job &j);
uint32_t gf2_mul_workgroups(const Gf2Job &j);       // direct
uint32_t gf2_rows_fwd_workgroups(const Gf2Job &j);  // rows_lg > 0: transforms of X and S over rows,
uint32_t gf2_rows_prod_workgroups(const Gf2Job &j);  // sums of products (none when nx = 1)
uint32_t gf2_rows_inv_workgroups(const Gf2Job &j);   // transforms back (nx = 1: products first)
uint32_t gf2_inv_workgroups(const Gf2Job &j);
hipError_t launch_gf2_bits(uint32_t wgs, const Gf2Job *jobs, const Gf2Job &one, const uint2 *tab, hipStream_t s);
hipError_t launch_gf2_fwd(uint32_t wgs, const Gf2Job *jobs, const Gf2Job &one, const uint2 *tab, hipStream_t s);
hipError_t launch_gf2_mul(uint32_t wgs, const Gf2Job *jobs, const Gf2Job &one, const uint2 *tab, hipStream_t s);
// (every job of a launch has the given rows_lg)
hipError_t launch_gf2_rows_fwd(int rows_lg, uint32_t wgs, const Gf2Job *jobs, const Gf2Job &one, const uint2 *tab,
                               hipStream_t s);
hipError_t launch_gf2_rows_prod(bool one_group, uint32_t wgs, const Gf2Job *jobs, const Gf2Job &one, const uint2 *tab,
                                hipStream_t s);  // one_group: every job's nz is 1, or none's
hipError_t launch_gf2_rows_inv(int rows_lg, uint32_t wgs, const Gf2Job *jobs, const Gf2Job &one, const uint2 *tab,
                               hipStream_t s);
hipError_t launch_gf2_inv(uint32_t wgs, const Gf2Job *jobs, const Gf2Job &one, const uint2 *tab, hipStream_t s);

}  // namespace ext
