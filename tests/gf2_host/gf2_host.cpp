// CPU build of the GF(2)[t] path's index maps, basis-change layers and field constants
// (csrc/gf2.h, csrc/gf2_steps.h) for tests/test_gf2_host.py.
#include "../../paper_2402_09481_amd/csrc/gf2.h"
#include "../../paper_2402_09481_amd/csrc/gf2_steps.h"

static const uint32_t *g_lo, *g_hi;
static int g_bad;
namespace ext {
namespace gf2 {
u32 load_word(const u32 *p) {  // every word the kernels would read lies inside the string
    if (p < g_lo || p >= g_hi) {
        ++g_bad;
        return 0xDEADBEEFu;
    }
    return *p;
}
}  // namespace gf2
}  // namespace ext
using namespace ext;

extern "C" {
uint32_t gf2_mul(uint32_t a, uint32_t b) { return gf2::fmul(a, b); }
uint32_t gf2_subspace(int i, uint32_t v) { return gf2::subspace_poly(i, v); }
void gf2_forms(uint32_t c, uint32_t *w) {
    const gf2::Forms f = gf2::forms81(c);
    for (int i = 0; i < 3; ++i) w[i] = f.w[i];
}
// 16 words of the input (seed = 0) or the seed from position pos, read as one run or word
// by word; returns the reads outside the string's dwords
int gf2_run(int single, int seed, int mode, const uint64_t *bits, uint64_t len, uint64_t a, uint64_t N, uint64_t rot, uint64_t P,
            int64_t pos, uint32_t *out) {
    const Emb e{bits, len, a, N, rot, P, (uint32_t)mode, 0};
    g_lo = (const uint32_t *)bits;
    g_hi = g_lo + ((seed ? P : len) + 31) / 32;
    g_bad = 0;
    for (int k = 0; k < 16; ++k) out[k] = 0;
    for (int k = 0; single && k < 16; ++k) out[k] = seed ? gf2::seed_word(e, pos + 32 * k) : gf2::input_word(e, pos + 32 * k);
    if (!single && seed) gf2::seed_run(out, e, pos);
    if (!single && !seed) gf2::input_run(out, e, pos);
    return g_bad;
}
}

template <int SIDE, int K, int R>
static void classes(uint32_t *rows) {
    for (int rho = 0; rho < (1 << K) - 1; ++rho)
        gf2::taylor_classes<SIDE, K, R>(
            rho, [&](int r) { return rows[r]; }, [&](int r, uint32_t w) { rows[r] = w; });
}
template <int SIDE>
static int classes_side(int k, int r, uint32_t *rows) {
    if (k == 4 && r == 4) return classes<SIDE, 4, 4>(rows), 0;
    if (k != 8) return 1;
    if (r == 1) return classes<SIDE, 8, 1>(rows), 0;
    if (r == 2) return classes<SIDE, 8, 2>(rows), 0;
    if (r == 3) return classes<SIDE, 8, 3>(rows), 0;
    if (r == 4) return classes<SIDE, 8, 4>(rows), 0;
    return 1;
}
template <int SIDE>
static int units_side(int r, uint32_t *rows) {
    if (r == 2) return gf2::basis_units<SIDE, 2>(rows), 0;
    if (r == 3) return gf2::basis_units<SIDE, 3>(rows), 0;
    if (r == 4) return gf2::basis_units<SIDE, 4>(rows), 0;
    return 1;
}
extern "C" {
int gf2_classes(int side, int k, int r, uint32_t *rows) {
    return side == 0 ? classes_side<gf2::T_FWD>(k, r, rows)
           : side == 1 ? classes_side<gf2::T_SEED>(k, r, rows)
                       : classes_side<gf2::T_OUT>(k, r, rows);
}
int gf2_units(int side, int r, uint32_t *rows) {
    return side == 0 ? units_side<gf2::T_FWD>(r, rows)
           : side == 1 ? units_side<gf2::T_SEED>(r, rows)
                       : units_side<gf2::T_OUT>(r, rows);
}
}
