// Von Neumann extractor on gfx950 (section "Von Neumann": output bit j is
// x_{2j} when x_{2j} != x_{2j+1} and nothing otherwise; Alg. 3 walks the pairs
// in order and appends).
//
// The output is a stream compaction of the input's pairs. Up to VN_TWO_MAX input bits
// it takes two passes over the input:
//
//   k_vn_count one workgroup per tile of VP_TILE_W words: its count of differing pairs.
//   k_vn_pack  sums the counts before its tile, compresses the tile and writes it.
//
// and beyond, where the second reading would come from HBM, one pass:
//
//   k_vn_zero  clears the tile states and the tile ticket counter.
//   k_vn_main  one workgroup per tile of VN_TILE_W input words, in the order
//              of a ticket counter. The tile is loaded coalesced and its
//              aggregate (its count of differing pairs) published at once; its
//              output offset comes from a decoupled look-back over the states
//              of the tiles before it (aggregate, then inclusive prefix, one
//              64-bit word each), whose first poll goes out with the aggregate
//              and is answered while the tile is compressed. The tile is staged
//              in LDS, each thread takes VN_WPT consecutive words and compresses
//              each (per byte a 256-entry table: the bits kept from its four
//              pairs), and the per-thread counts are scanned to assemble the
//              tile's bits in LDS at tile-local positions. They are written out
//              shifted onto the output's 64-bit word grid: words wholly inside
//              the tile's range straight to z, the first and last partial words
//              to side arrays.
//   k_vn_fix   one thread per tile: the partial words. The tile holding a word's
//              first output bit ORs in the parts of the tiles that follow it
//              inside that word and stores it; the last thread writes the output
//              length and the status.
//
// Every wait in the look-back is bounded: past VN_SPIN_LIMIT polls a tile
// publishes an error state (which the tiles after it pass on) and the status
// reports EXT_EDEVICE instead of hanging.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/extractor.h"
#include "launch.h"

namespace ext {
namespace {

#ifndef VN_WORDS_PER_THREAD
#define VN_WORDS_PER_THREAD 8
#endif
// Tiles of 8192 words (1024 threads x 8 words; 73 KiB of LDS, two workgroups
// per CU): measured against 4096-word tiles of 256 x 16, 0.444 -> 0.424 ms at
// n = 2^33 and 0.049 -> 0.036 ms at n = 5*10^8 (half the workgroups to launch
// and look back over, twice the waves per CU).
constexpr int VN_NT = 1024;
constexpr int VN_WPT = VN_WORDS_PER_THREAD;       // consecutive input words per thread
constexpr int VN_TILE_W = VN_NT * VN_WPT;         // words per tile
constexpr int VN_RAW = VN_TILE_W + VN_NT;         // padded LDS words (one pad word per thread's run)
constexpr int VN_OBUF = VN_TILE_W / 2 + 2;        // output words of one tile, on the global grid
static_assert(VN_OBUF <= VN_RAW, "output buffer aliases the input tile");
static_assert(VN_WPT >= 2 && VN_WPT <= 32, "words per thread");
static_assert(VN_NT >= 256 && VN_NT <= 1024 && VN_NT % 64 == 0, "the byte table is filled by the first 256 threads");

// Two passes up to here: the second pass reads the input from the 256 MB last-level
// cache as long as it is kept there. One pass against two, us a call back to back: n =
// 10^6 15.5 / 10.2, 2^27 19.6 / 11.9, 5*10^8 41.6 / 30.6, 2^30 65.3 / 55.3, 3*2^29 89.2 /
// 80.5, 2^31 122 / 121, 3*2^30 174 / 213.
constexpr uint64_t VN_TWO_MAX = 3ull << 29;
constexpr uint64_t ST_AGG = 1ull << 62, ST_PREFIX = 2ull << 62, ST_ERR = 3ull << 62;
constexpr uint64_t ST_VAL = (1ull << 62) - 1;
constexpr uint32_t VN_SPIN_LIMIT = 1u << 22;
constexpr int VN_LB = 4;  // look-back states polled per lane per round trip

__device__ __forceinline__ uint64_t load_state(const uint64_t *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void store_state(uint64_t *p, uint64_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ uint64_t wave_sum(uint64_t v) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

// Byte b holds four pairs (bits 2j, 2j+1, j < 4): the kept bits, packed.
__device__ __forceinline__ uint32_t byte_entry(uint32_t b) {
    uint32_t out = 0, k = 0;
    for (int j = 0; j < 4; ++j) {
        uint32_t a = (b >> (2 * j)) & 1u, c = (b >> (2 * j + 1)) & 1u;
        if (a != c) out |= a << k++;
    }
    return out;
}

// One input word: the kept bits (<= 32, packed from bit 0) and their count.
__device__ __forceinline__ uint32_t vn_word(uint64_t v, const uint8_t *tab, uint32_t &cnt) {
    const uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32);
    const uint32_t dlo = (lo ^ (lo >> 1)) & 0x55555555u, dhi = (hi ^ (hi >> 1)) & 0x55555555u;
    uint32_t out = tab[lo & 255u];
    out |= (uint32_t)tab[(lo >> 8) & 255u] << __popc(dlo & 0xffu);
    out |= (uint32_t)tab[(lo >> 16) & 255u] << __popc(dlo & 0xffffu);
    out |= (uint32_t)tab[lo >> 24] << __popc(dlo & 0xffffffu);
    const uint32_t a = __popc(dlo);
    out |= (uint32_t)tab[hi & 255u] << a;
    out |= (uint32_t)tab[(hi >> 8) & 255u] << (a + __popc(dhi & 0xffu));
    out |= (uint32_t)tab[(hi >> 16) & 255u] << (a + __popc(dhi & 0xffffu));
    out |= (uint32_t)tab[hi >> 24] << (a + __popc(dhi & 0xffffffu));
    cnt = a + __popc(dhi);
    return out;
}

__device__ __forceinline__ int raw_index(int w) { return w + w / VN_WPT; }

__global__ void k_vn_zero(VnWork w, uint64_t T) {
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < T) w.state[i] = 0;
    if (i < 2) w.counter[i] = 0;
}

// Input words of tile t in the coalesced order (word k * VN_NT + tid of the tile
// in pre[k]). The loads are the same instructions for every tile, from addresses
// clamped into x (tiles at or past T read word 0): no branch, so a wave's later
// waits can count exactly which loads are still in flight. Words past the pairs
// are zeroed before the tile is used (mask_tile).
__device__ __forceinline__ void load_tile(const uint64_t *__restrict__ x, uint64_t nwords, uint32_t t, uint32_t T,
                                          int tid, uint64_t (&pre)[VN_WPT]) {
    const uint64_t base = (uint64_t)t * VN_TILE_W;
#pragma unroll
    for (int k = 0; k < VN_WPT; ++k) {
        const uint64_t gi = base + k * VN_NT + tid;
        const uint64_t idx = t < T ? (gi < nwords ? gi : nwords - 1) : 0;
        pre[k] = x[idx];
    }
}

// Zero the words of pre past the pairs (only the tile holding the last input
// word has any).
__device__ __forceinline__ void mask_tile(uint64_t (&pre)[VN_WPT], uint64_t nwords, uint64_t last_mask, uint32_t t,
                                          int tid) {
    const uint64_t base = (uint64_t)t * VN_TILE_W;
    if (base + VN_TILE_W < nwords) return;
#pragma unroll
    for (int k = 0; k < VN_WPT; ++k) {
        const uint64_t gi = base + k * VN_NT + tid;
        if (gi >= nwords) pre[k] = 0;
        if (gi == nwords - 1) pre[k] &= last_mask;
    }
}

// Pairs of a word whose bits differ.
__device__ __forceinline__ uint32_t pairs_differing(uint64_t v) {
    return (uint32_t)__popcll((v ^ (v >> 1)) & 0x5555555555555555ull);
}

__device__ __forceinline__ uint32_t wave_sum32(uint32_t v) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

// Look-back state of the control wave. A poll reads VN_LB states per lane:
// lane l, slot k holds tile j - 64 k with j = t - 1 - l for the first window,
// so one round trip covers the 64 VN_LB nearest tiles; tiles before tile 0
// count as a zero prefix.
struct LookBack {
    uint64_t s[VN_LB];
    int64_t j;
    uint64_t excl;
    uint32_t spins;
    bool err;
};

enum LbStep { LB_DONE, LB_WAIT, LB_NEXT };

__device__ __forceinline__ void lb_load(LookBack &b, const VnWork &w) {
#pragma unroll
    for (int k = 0; k < VN_LB; ++k) b.s[k] = b.j - 64 * k >= 0 ? load_state(&w.state[b.j - 64 * k]) : ST_PREFIX;
}

// Re-read the states that were not yet published.
__device__ __forceinline__ void lb_repoll(LookBack &b, const VnWork &w) {
#pragma unroll
    for (int k = 0; k < VN_LB; ++k)
        if ((b.s[k] >> 62) == 0) b.s[k] = load_state(&w.state[b.j - 64 * k]);
}

// One look at the current window: DONE when the exclusive prefix is known (or
// on error), WAIT when a nearer tile has published nothing yet, NEXT when the
// whole window holds aggregates only (their sum is taken and the window moves
// back; its states are requested).
__device__ __forceinline__ LbStep lb_step(LookBack &b, int lane, const VnWork &w) {
    uint32_t d = 64 * VN_LB;  // distance (lane + 64 k) of the nearest tile with a prefix
#pragma unroll
    for (int k = VN_LB - 1; k >= 0; --k) {
        const uint64_t pm = __ballot((b.s[k] >> 62) == 2);
        if (pm) d = 64 * k + (__ffsll((unsigned long long)pm) - 1);
    }
    bool waiting = false;
#pragma unroll
    for (int k = 0; k < VN_LB; ++k) waiting |= __ballot((b.s[k] >> 62) == 0 && (uint32_t)(lane + 64 * k) < d) != 0;
    if (waiting) {
        if (++b.spins > VN_SPIN_LIMIT) {
            b.err = true;
            return LB_DONE;
        }
        return LB_WAIT;
    }
    uint64_t part = 0;
    bool bad = false;
#pragma unroll
    for (int k = 0; k < VN_LB; ++k) {
        if ((uint32_t)(lane + 64 * k) <= d) {  // d = window size: the whole window
            part += b.s[k] & ST_VAL;
            bad |= (b.s[k] >> 62) == 3;
        }
    }
    if (__ballot(bad) != 0) {
        b.err = true;
        return LB_DONE;
    }
    b.excl += wave_sum(part);
    if (d < 64 * VN_LB) return LB_DONE;
    b.j -= 64 * VN_LB;
    lb_load(b, w);
    return LB_NEXT;
}

// One workgroup per tile. The tile index comes from a ticket counter, so every
// tile before this one belongs to a workgroup that is already running: the
// look-back waits only on work that is under way. The tile's aggregate is
// published as soon as the tile is loaded and the first look-back poll goes out
// with it; the look-back is finished (by wave 0) after the words are
// compressed, and the bits are assembled at tile-local positions and shifted
// onto the output's word grid as they are written.
__global__ __launch_bounds__(VN_NT) void k_vn_main(const uint64_t *__restrict__ x, uint64_t nwords, uint64_t last_mask,
                                                   uint64_t *__restrict__ z, uint64_t zcap, VnWork w, uint32_t T) {
    __shared__ uint64_t raw[VN_RAW];
    __shared__ uint8_t tab[256];
    __shared__ uint32_t wsum[VN_NT / 64];
    __shared__ uint32_t wagg[VN_NT / 64];
    __shared__ uint32_t sh_ticket;
    __shared__ uint64_t sh_excl;
    uint64_t *obuf = raw;  // tile-local output words, once every thread holds its input words
    constexpr int NW = VN_NT / 64;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform in a wave: scalar branches
    if (tid == 0) sh_ticket = atomicAdd(w.counter, 1u);
    if (tid < 256) tab[tid] = (uint8_t)byte_entry((uint32_t)tid);
    __syncthreads();
    const uint32_t t = sh_ticket;

    // load the tile (coalesced), count its differing pairs (a sum, so the order
    // of the words does not matter) and stage it in LDS
    {
        uint64_t pre[VN_WPT];
        load_tile(x, nwords, t, T, tid, pre);
        mask_tile(pre, nwords, last_mask, t, tid);
        uint32_t c = 0;
#pragma unroll
        for (int k = 0; k < VN_WPT; ++k) {
            c += pairs_differing(pre[k]);
            raw[raw_index(k * VN_NT + tid)] = pre[k];
        }
        c = wave_sum32(c);
        if (lane == 0) wagg[wave] = c;
    }
    __syncthreads();
    uint32_t agg = 0;
#pragma unroll
    for (int v = 0; v < NW; ++v) agg += wagg[v];

    // wave 0: publish the aggregate and send the first poll
    LookBack b;
    if (wave == 0) {
        b.excl = 0;
        b.spins = 0;
        b.err = false;
        if (lane == 0) store_state(&w.state[t], (t == 0 ? ST_PREFIX : ST_AGG) | agg);
        if (t != 0) {
            b.j = (int64_t)t - 1 - lane;
            lb_load(b, w);
        }
    }

    // this thread's VN_WPT consecutive words
    uint32_t out[VN_WPT], cnt[VN_WPT];
    uint32_t total = 0;
#pragma unroll
    for (int i = 0; i < VN_WPT; ++i) {
        out[i] = vn_word(raw[tid * (VN_WPT + 1) + i], tab, cnt[i]);
        // materialise the packed word here, so its eight table values are not
        // kept live until the assembly below
        asm volatile("" : "+v"(out[i]), "+v"(cnt[i]));
        total += cnt[i];
    }
    // workgroup scan of the per-thread counts
    uint32_t incl = total;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t v = __shfl_up(incl, o);
        if (lane >= o) incl += v;
    }
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();  // raw is free; the wave sums are visible
    uint32_t before = 0;
#pragma unroll
    for (int v = 0; v < NW; ++v) before += v < wave ? wsum[v] : 0u;
    const uint32_t pos0 = before + incl - total;  // this thread's first bit within the tile
    for (int i = tid; i < VN_OBUF; i += VN_NT) obuf[i] = 0;

    // wave 0: finish the look-back
    if (wave == 0) {
        if (t != 0) {
            for (;;) {
                const LbStep r = lb_step(b, lane, w);
                if (r == LB_DONE) break;
                if (r == LB_WAIT) {
                    __builtin_amdgcn_s_sleep(2);
                    lb_repoll(b, w);
                }
            }
            if (lane == 0) {
                store_state(&w.state[t], (b.err ? ST_ERR : ST_PREFIX) | ((b.excl + agg) & ST_VAL));
                if (b.err) atomicOr(&w.counter[1], 1u);
            }
        }
        if (lane == 0) sh_excl = b.excl;
    }
    __syncthreads();

    // this thread's bits at tile-local positions (local word q = tile bits 64 q ..)
    {
        uint32_t wi = pos0 >> 6, sh = pos0 & 63;
        uint64_t cur = 0;
#pragma unroll
        for (int i = 0; i < VN_WPT; ++i) {
            cur |= (uint64_t)out[i] << sh;
            if (sh + cnt[i] >= 64) {  // then sh >= 32: the carry shift is in [1, 32]
                atomicOr((unsigned long long *)&obuf[wi < VN_OBUF ? wi : VN_OBUF - 1], (unsigned long long)cur);
                ++wi;
                cur = (uint64_t)out[i] >> (64 - sh);
            }
            sh = (sh + cnt[i]) & 63;
        }
        if (sh) atomicOr((unsigned long long *)&obuf[wi < VN_OBUF ? wi : VN_OBUF - 1], (unsigned long long)cur);
    }
    __syncthreads();

    // the tile's bits start at global bit E: shift them onto the 64-bit word grid
    const uint64_t E = sh_excl;
    if (agg != 0) {
        const uint64_t g0 = E >> 6;
        const uint32_t sft = (uint32_t)(E & 63);
        const uint32_t nq = (uint32_t)((sft + agg + 63) >> 6);
        const bool head = sft != 0, tail = ((E + agg) & 63) != 0;
        for (uint32_t q = tid; q < nq && q < VN_OBUF; q += VN_NT) {
            uint64_t v = obuf[q];
            if (sft) v = (v << sft) | (q ? obuf[q - 1] >> (64 - sft) : 0);
            const bool first = q == 0 && head, last = q == nq - 1 && tail;
            if (first) w.pf[t] = v;
            if (last) w.pl[t] = v;
            if (!first && !last && g0 + q < zcap) z[g0 + q] = v;
        }
    }
}

__global__ void k_vn_fix(VnWork w, uint64_t T, uint64_t *__restrict__ z, uint64_t zcap, uint64_t *m_out,
                         int32_t *status) {
    const uint64_t t = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= T) return;
    const uint64_t incl = w.state[t] & ST_VAL;
    const uint64_t E = t ? (w.state[t - 1] & ST_VAL) : 0;
    if (t == T - 1) {
        if (m_out) *m_out = incl;
        if (status) *status = w.counter[1] ? EXT_EDEVICE : (incl ? EXT_OK : EXT_EDEGENERATE);
    }
    if (incl <= E || (incl & 63) == 0) return;  // empty tile, or its range ends on a word boundary
    const uint64_t ql = (incl - 1) >> 6;
    if ((ql << 6) < E) return;  // the word's first bit belongs to an earlier tile
    uint64_t v = w.pl[t];
    const uint64_t end = (ql << 6) + 64;
    for (uint64_t u = t + 1; u < T; ++u) {
        const uint64_t Eu = w.state[u - 1] & ST_VAL;
        if (Eu >= end) break;
        const uint64_t iu = w.state[u] & ST_VAL;
        if (iu == Eu) continue;
        v |= w.pf[u];
        if (iu >= end) break;
    }
    if (ql < zcap) z[ql] = v;
}

// ---------------------------------------------------------------- two passes (up to VN_TWO_MAX bits)

// k_vn_count leaves every tile's count of differing pairs and its first 64 kept bits.
// k_vn_pack sums the counts before its tile itself: no ticket, no look-back, no tile
// waits for another, and the tile's place in z is known before its bits are assembled,
// so they go straight onto the output's word grid, two input words at a time. An output
// word that tiles share is stored by the one it begins in, from the first bits of the
// tiles after it. (Where tiles met in the workspace by atomics instead, with the counts
// in the same lines, that took 17 us.) A thread's eight words are loaded from where they
// are (64 bytes a lane: the second half of a line comes from the L1), not staged through
// LDS. At n = 5*10^8 (62.5 MB in, 41% of the pairs kept) the call takes 30.6 us, and 41.6
// in one pass: the count 11 us, the cache's 6 TB/s; the packing 19 us, of which 6.5 go to
// the byte table's reads and shifts and the rest to loads and stores over two rounds of
// workgroups that are not full. Tiles of 256 threads x 16 words or 1024 x 4: 3 and 5 us
// more.
constexpr int VP_NT = 512;
constexpr int VP_WPT = 8;
constexpr int VP_TILE_W = VP_NT * VP_WPT;
constexpr int VP_OBUF = VP_TILE_W / 2 + 3;
constexpr int VP_NW = VP_NT / 64;

// Inclusive sums over a wave, in six dependent adds that read other lanes directly.
__device__ __forceinline__ uint32_t wave_scan32(uint32_t v) {
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false);  // row_shr:1, 2, 4, 8
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false);  // row_bcast:15 to rows 1, 3
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false);  // row_bcast:31 to rows 2, 3
    return v;
}
__device__ __forceinline__ uint32_t last_lane(uint32_t v) { return (uint32_t)__builtin_amdgcn_readlane((int)v, 63); }

typedef uint64_t WordPair __attribute__((ext_vector_type(2), aligned(8)));

// The eight consecutive words of thread tid in tile t; words past the pairs read as 0.
__device__ __forceinline__ void load_eight(const uint64_t *__restrict__ x, uint64_t nwords, uint64_t last_mask,
                                           uint32_t t, int tid, uint64_t (&v)[VP_WPT]) {
    const uint64_t base = (uint64_t)t * VP_TILE_W + VP_WPT * tid;
    if ((uint64_t)(t + 1) * VP_TILE_W < nwords) {
#pragma unroll
        for (int k = 0; k < VP_WPT; k += 2) {
            const WordPair p = *(const WordPair *)(x + base + k);
            v[k] = p.x;
            v[k + 1] = p.y;
        }
        return;
    }
#pragma unroll
    for (int k = 0; k < VP_WPT; ++k) {
        v[k] = base + k < nwords ? x[base + k] : 0;
        if (base + k == nwords - 1) v[k] &= last_mask;
    }
}

__global__ __launch_bounds__(VP_NT) void k_vn_count(const uint64_t *__restrict__ x, uint64_t nwords,
                                                    uint64_t last_mask, VnPairWork w) {
    __shared__ uint32_t wsum[VP_NW];
    __shared__ uint64_t head;
    __shared__ uint8_t tab[256];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    uint64_t v[VP_WPT];
    load_eight(x, nwords, last_mask, blockIdx.x, tid, v);
    if (tid < 256) tab[tid] = (uint8_t)byte_entry((uint32_t)tid);
    if (tid == 0) head = 0;
    uint32_t mine = 0;
#pragma unroll
    for (int k = 0; k < VP_WPT; ++k) mine += pairs_differing(v[k]);
    const uint32_t incl = wave_scan32(mine);
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    uint32_t sum = 0, pos = incl - mine;
#pragma unroll
    for (int k = 0; k < VP_NW; ++k) {
        pos += k < wave ? wsum[k] : 0u;
        sum += wsum[k];
    }
    if (mine && pos < 64) {
#pragma unroll
        for (int k = 0; k < VP_WPT; ++k) {
            uint32_t c;
            const uint32_t bits = vn_word(v[k], tab, c);
            if (c && pos < 64) atomicOr((unsigned long long *)&head, (unsigned long long)bits << pos);
            pos += c;
        }
    }
    __syncthreads();
    if (tid == 0) {
        w.count[blockIdx.x] = sum;
        w.head[blockIdx.x] = head;
    }
}

__global__ __launch_bounds__(VP_NT) void k_vn_pack(const uint64_t *__restrict__ x, uint64_t nwords,
                                                   uint64_t last_mask, uint64_t *__restrict__ z, uint64_t zcap,
                                                   VnPairWork w, uint32_t T, uint64_t *m_out, int32_t *status) {
    __shared__ uint64_t obuf[VP_OBUF];
    __shared__ uint8_t tab[256];
    __shared__ uint32_t wsum[VP_NW], wbefore[VP_NW], wtotal[VP_NW];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t t = blockIdx.x;
    uint64_t v[VP_WPT];
    load_eight(x, nwords, last_mask, t, tid, v);
    uint32_t before = 0, total = 0;
    for (uint32_t i0 = tid; i0 < T; i0 += 4 * VP_NT) {  // four loads in flight
        uint32_t c[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) c[k] = i0 + k * VP_NT < T ? w.count[i0 + k * VP_NT] : 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            total += c[k];
            before += i0 + k * VP_NT < t ? c[k] : 0;
        }
    }
    // wave 1: the 64 tiles after this one
    uint32_t u = t + 1 + lane, next = 0;
    uint64_t head = 0;
    if (wave == 1 && u < T) {
        next = w.count[u];
        head = w.head[u];
    }
    if (tid < 256) tab[tid] = (uint8_t)byte_entry((uint32_t)tid);
    for (int i = tid; i < VP_OBUF; i += VP_NT) obuf[i] = 0;
    __syncthreads();

    uint64_t kept[VP_WPT / 2];  // the bits kept from two words each
    uint32_t cnt[VP_WPT / 2], mine = 0;
#pragma unroll
    for (int i = 0; i < VP_WPT / 2; ++i) {
        uint32_t c0, c1;
        const uint32_t lo = vn_word(v[2 * i], tab, c0), hi = vn_word(v[2 * i + 1], tab, c1);
        kept[i] = lo | (uint64_t)hi << c0;
        cnt[i] = c0 + c1;
        asm volatile("" : "+v"(kept[i]), "+v"(cnt[i]));  // packed here, not at the assembly
        mine += cnt[i];
    }
    const uint32_t incl = wave_scan32(mine);
    before = wave_scan32(before);
    total = wave_scan32(total);
    if (lane == 63) {
        wsum[wave] = incl;
        wbefore[wave] = before;
        wtotal[wave] = total;
    }
    __syncthreads();
    uint32_t agg = 0, pos = incl - mine;
    before = total = 0;
#pragma unroll
    for (int k = 0; k < VP_NW; ++k) {
        pos += k < wave ? wsum[k] : 0u;
        agg += wsum[k];
        before += wbefore[k];
        total += wtotal[k];
    }
    if (t == 0 && tid == 0) {
        *m_out = total;
        if (status) *status = total ? EXT_OK : EXT_EDEGENERATE;
    }
    if (agg == 0) return;

    const uint32_t sft = before & 63;  // the tile's first bit in its first output word
    uint32_t p = sft + pos;
#pragma unroll
    for (int i = 0; i < VP_WPT / 2; ++i) {
        const uint32_t wi = p >> 6, sh = p & 63;
        // (nothing is ORed where nothing is kept: with few differing pairs all lanes
        // would take turns at one word)
        if (cnt[i]) atomicOr((unsigned long long *)&obuf[wi], (unsigned long long)(kept[i] << sh));
        if (sh + cnt[i] > 64) atomicOr((unsigned long long *)&obuf[wi + 1], (unsigned long long)(kept[i] >> (64 - sh)));
        p += cnt[i];
    }
    __syncthreads();
    // this tile's words: from the first one that begins in it to the last
    const uint64_t q0 = before >> 6;
    const uint32_t end = sft + agg, nq = (end + 63) >> 6;
    const bool tail = (end & 63) != 0;  // the last word is not full
    for (uint32_t q = tid + (sft != 0); q < nq - tail; q += VP_NT)
        if (q0 + q < zcap) z[q0 + q] = obuf[q];
    if (wave == 1 && tail && (nq > 1 || sft == 0)) {
        const uint64_t q = q0 + nq - 1;
        const uint32_t left = total - (uint32_t)(q << 6) < 64 ? total - (uint32_t)(q << 6) : 64;  // bits of the word
        uint32_t has = end & 63;
        uint64_t part = 0;
        while (has < left) {  // (at the last tile has = left: each turn looks at tiles that are there)
            next = next < 64 ? next : 64;
            const uint32_t sum = wave_scan32(next), at = has + sum - next;
            if (at < 64) part |= head << at;
            has += last_lane(sum);
            if (has >= left) break;
            u += 64;
            next = u < T ? w.count[u] : 0;
            head = u < T ? w.head[u] : 0;
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) part |= __shfl_xor(part, o);
        if (lane == 0 && q < zcap) z[q] = obuf[nq - 1] | part;
    }
}

}  // namespace

namespace {
struct VnInput {
    uint64_t nwords;     // words that hold pairs
    uint64_t last_mask;  // the pairs' bits in the last of them
};
VnInput vn_input(uint64_t n) {
    const uint64_t nb = n & ~1ull;
    return VnInput{(nb + 63) >> 6, (nb & 63) ? ((1ull << (nb & 63)) - 1) : ~0ull};
}
uint64_t vn_pair_tiles(uint64_t n) { return (vn_input(n).nwords + VP_TILE_W - 1) / VP_TILE_W; }
}  // namespace

uint64_t vn_tiles(uint64_t n) { return (vn_input(n).nwords + VN_TILE_W - 1) / VN_TILE_W; }

// room for either form: the one pass has three words a tile and its counters, the two passes
// 12 bytes for each of their (smaller) tiles
size_t vn_workspace_bytes(uint64_t n) {
    const uint64_t pairs = vn_two_pass(n) ? vn_pair_tiles(n) * (sizeof(uint64_t) + sizeof(uint32_t)) : 0;
    const uint64_t one = 3 * vn_tiles(n) * 8;
    return (size_t)((one > pairs ? one : pairs) + 256);
}

VnPairWork vn_pair_work(char *ws, uint64_t n) {
    VnPairWork w;
    w.head = (uint64_t *)ws;
    w.count = (uint32_t *)(w.head + vn_pair_tiles(n));
    return w;
}

VnWork vn_work(char *ws, uint64_t n) {
    const uint64_t T = vn_tiles(n);
    VnWork w;
    w.state = (uint64_t *)ws;
    w.pf = w.state + T;
    w.pl = w.pf + T;
    w.counter = (uint32_t *)(w.pl + T);
    return w;
}

bool vn_two_pass(uint64_t n) { return n <= VN_TWO_MAX; }

hipError_t launch_vn_count(const uint64_t *x, uint64_t n, const VnPairWork &w, hipStream_t s) {
    const VnInput in = vn_input(n);
    return launch_k(k_vn_count, dim3((unsigned)vn_pair_tiles(n)), dim3(VP_NT), 0, s, x, in.nwords, in.last_mask, w);
}

hipError_t launch_vn_pack(const uint64_t *x, uint64_t n, uint64_t *z, uint64_t zcap, const VnPairWork &w,
                          uint64_t *m_out, int32_t *status, hipStream_t s) {
    const VnInput in = vn_input(n);
    const uint64_t T = vn_pair_tiles(n);
    return launch_k(k_vn_pack, dim3((unsigned)T), dim3(VP_NT), 0, s, x, in.nwords, in.last_mask, z, zcap, w, (uint32_t)T,
                    m_out, status);
}

hipError_t launch_vn_zero(const VnWork &w, uint64_t n, hipStream_t s) {
    const uint64_t T = vn_tiles(n);
    const uint64_t items = T > 2 ? T : 2;
    return launch_k(k_vn_zero, dim3((unsigned)((items + 255) / 256)), dim3(256), 0, s, w, T);
}

hipError_t launch_vn_main(const uint64_t *x, uint64_t n, uint64_t *z, uint64_t zcap, const VnWork &w, hipStream_t s) {
    const uint64_t T = vn_tiles(n);
    const VnInput in = vn_input(n);
    return launch_k(k_vn_main, dim3((unsigned)T), dim3(VN_NT), 0, s, x, in.nwords, in.last_mask, z, zcap, w, (uint32_t)T);
}

hipError_t launch_vn_fix(const VnWork &w, uint64_t n, uint64_t *z, uint64_t zcap, uint64_t *m_out, int32_t *status,
                         hipStream_t s) {
    const uint64_t T = vn_tiles(n);
    return launch_k(k_vn_fix, dim3((unsigned)((T + 255) / 256)), dim3(256), 0, s, w, T, z, zcap, m_out, status);
}

}  // namespace ext
