// Exact selection of the k-th largest delta magnitude of a block, shared by
// the TIES merge kernel (per selected unit) and the catalog kernel that
// stores every unit's threshold (k_index.hip).
//
// Magnitudes are compared as fp32 bit patterns with the sign cleared (the
// same order as the values, since they are not negative).  The window is the
// binade of the block maximum and the three binades below it, keyed by
// |d| >> KS (exponent and MB mantissa bits): NBIN bins, each with NC copies
// so that lanes holding equal values (frequent in bf16 deltas) update
// different words.  No magnitude lies above the window.  The low half of a
// counter counts the bin's elements, the high half the ones above the bin's
// floor (low bits not zero).
#pragma once

#include "device_common.h"

namespace mp {

namespace ties {
constexpr int MB = 7;           // mantissa bits in a window key
constexpr int NC = 2;           // copies of each window bin (lanes spread over them)
constexpr int KS = 23 - MB;     // pattern bits below a key
constexpr int NBIN = 4 << MB;   // window bins: four binades
constexpr int NB = NBIN * NC;   // words per histogram row
constexpr int LG = 3;           // log2 of a bin's bytes (4 NC)
static_assert((4 * NC) == (1 << LG), "a bin's bytes");
enum : uint32_t { DONE = 0u, LIST = 1u, RADIX = 2u };
}  // namespace ties


struct Cut {
    uint32_t found, bin, rank, count, aux;  // wave-uniform
    uint32_t total;                         // elements counted in the whole histogram (window walks)
};

// Wave-level, all lanes: the bin of the window histogram h (NBIN bins of NC
// = 2 words) where the count from the top first reaches k.  A bin's count is
// the low 16 bits of its words' sum, aux the high half's.  rank = k minus the
// count above the bin.  The whole row (at most 65,535 elements) is read at
// once, 16 consecutive bytes per lane and read (conflict-free), and the four
// quarter rows' lane sums are prefix-summed two to a register, so the walk
// costs one LDS latency and one chain of seven adds wherever the cut lies;
// quarter after quarter it was up to four of each, on the critical path of
// every unit.
__device__ inline Cut wave_find_window(const uint32_t* __restrict__ h, uint32_t k, int lane)
{
    using namespace ties;
    static_assert(NC == 2 && NB == 4 * 256, "four reads of 64 lanes x 4 words cover the row");
    uint32_t hi[4], lo[4], s[4];  // the lane's two bins of each quarter (hi above lo), their counts
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const uint4 raw = *reinterpret_cast<const uint4*>(h + NB - 4 - 4 * (j * 64 + lane));
        hi[j] = raw.z + raw.w;
        lo[j] = raw.x + raw.y;
        s[j] = (hi[j] + lo[j]) & 0xffffu;
    }
    const uint32_t i01 = wave_incl_sum(s[0] | (s[1] << 16)), i23 = wave_incl_sum(s[2] | (s[3] << 16));
    const uint32_t t01 = (uint32_t)__builtin_amdgcn_readlane((int)i01, 63);
    const uint32_t t23 = (uint32_t)__builtin_amdgcn_readlane((int)i23, 63);
    const uint32_t c0 = t01 & 0xffffu, c1 = c0 + (t01 >> 16), c2 = c1 + (t23 & 0xffffu), c3 = c2 + (t23 >> 16);
    Cut r{0u, 0u, 0u, 0u, 0u, c3};
    if (k > c3)
        return r;
    // the quarter holding the cut (wave-uniform), and the lane's bins there
    uint32_t above, incl, sj, hj, lj, q;
    if (k <= c1) {
        const bool f = k <= c0;
        q = f ? 0u : 1u;
        above = f ? 0u : c0;
        incl = f ? (i01 & 0xffffu) : (i01 >> 16);
        sj = f ? s[0] : s[1];
        hj = f ? hi[0] : hi[1];
        lj = f ? lo[0] : lo[1];
    } else {
        const bool f = k <= c2;
        q = f ? 2u : 3u;
        above = f ? c1 : c2;
        incl = f ? (i23 & 0xffffu) : (i23 >> 16);
        sj = f ? s[2] : s[3];
        hj = f ? hi[2] : hi[3];
        lj = f ? lo[2] : lo[3];
    }
    const uint32_t before = above + incl - sj;
    const unsigned long long bal = __ballot(before < k && k <= before + sj);
    const int src = __ffsll((long long)bal) - 1;  // exactly one lane
    const uint32_t hb = (uint32_t)__builtin_amdgcn_readlane((int)hj, src);
    const uint32_t lb = (uint32_t)__builtin_amdgcn_readlane((int)lj, src);
    const uint32_t bf = (uint32_t)__builtin_amdgcn_readlane((int)before, src);
    const uint32_t hc = hb & 0xffffu;
    const bool up = bf + hc >= k;  // the cut lies in the lane's upper bin
    const uint32_t w = up ? hb : lb;
    r.found = 1u;
    r.bin = (uint32_t)(NBIN - 1) - 2u * (q * 64u + (uint32_t)src) - (up ? 0u : 1u);
    r.rank = k - bf - (up ? 0u : hc);
    r.count = w & 0xffffu;
    r.aux = w >> 16;
    return r;
}

// Wave-level, all lanes: as above over one-word bins (a radix digit's
// counters), walking downward from bin `top` in rounds of 256.
__device__ inline Cut wave_find_from_top(const uint32_t* __restrict__ h, int top, uint32_t k, int lane)
{
    Cut r{0u, 0u, 0u, 0u, 0u, 0u};
    uint32_t above = 0;
    for (int hi = top | 3; hi >= 0; hi -= 256) {
        const int g4 = hi - 4 * lane - 3;  // multiple of 4: the lane's words are g4 .. g4+3
        uint4 raw = make_uint4(0u, 0u, 0u, 0u);
        if (g4 >= 0)
            raw = *reinterpret_cast<const uint4*>(h + g4);
        const uint32_t bw[4] = {raw.w, raw.z, raw.y, raw.x};  // highest bin first
        const uint32_t s = raw.x + raw.y + raw.z + raw.w;
        const uint32_t incl = wave_incl_sum(s);
        const uint32_t before = above + incl - s;  // count in the bins above this lane's
        const bool hit = before < k && k <= above + incl;
        const unsigned long long bal = __ballot(hit);
        if (bal) {
            uint32_t c = before, bin = 0u, cnt = 0u;
            bool got = false;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (!got && (c + bw[q] >= k || q == 3)) {
                    got = true;
                    bin = (uint32_t)(g4 + 3 - q);
                    cnt = bw[q];
                } else if (!got) {
                    c += bw[q];
                }
            }
            const int src = __ffsll((long long)bal) - 1;
            r.found = 1u;
            r.bin = (uint32_t)__builtin_amdgcn_readlane((int)bin, src);
            r.rank = (uint32_t)__builtin_amdgcn_readlane((int)(k - c), src);
            r.count = (uint32_t)__builtin_amdgcn_readlane((int)cnt, src);
            return r;
        }
        above += (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
    }
    return r;
}

// Sum over the lanes of a wave (wave-uniform result).
__device__ inline uint32_t wave_sum_u32(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_readlane((int)wave_incl_sum(v), 63);
}


// Wave-level: the r-th largest of the n patterns in `list`, all of which
// share the key (pattern >> KS); the low bits are fixed from the top down.
// Up to 64 patterns sit one per lane in a register, and each bit then
// costs one compare: the count is the popcount of its lane mask.
__device__ inline uint32_t wave_select_list(const uint32_t* __restrict__ list, uint32_t n, uint32_t key,
                                            uint32_t r, int lane)
{
    uint32_t pref = key << ties::KS;
    if (n <= 64u) {
        const uint32_t v = ((uint32_t)lane < n) ? list[lane] : 0u;  // 0 lies below every candidate
        // wave-uniform values, kept in scalar registers
        uint32_t sp = (uint32_t)__builtin_amdgcn_readfirstlane((int)pref);
        const uint32_t sr = (uint32_t)__builtin_amdgcn_readfirstlane((int)r);
#pragma unroll
        for (int bit = ties::KS - 1; bit >= 0; --bit) {
            const uint32_t cand = sp | (1u << bit);
            if ((uint32_t)__popcll(__ballot(v >= cand)) >= sr)
                sp = cand;
        }
        return sp;
    }
#pragma unroll 1
    for (int bit = ties::KS - 1; bit >= 0; --bit) {
        const uint32_t cand = pref | (1u << bit);
        uint32_t c = 0u;
        for (uint32_t i = (uint32_t)lane; i < n; i += 64u)
            c += (list[i] >= cand) ? 1u : 0u;
        if (wave_sum_u32(c) >= r)
            pref = cand;
    }
    return pref;
}


// The LDS operations of one wave take effect in program order; this keeps
// the compiler from reordering them across a hand-off between lanes.
__device__ inline void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Adds one element to the window histogram.  base + koff + (key << LG) is
// the byte address of the lane's copy of the element's bin (koff holds the
// row's offset from base, the lane's copy and -wb bins; see window_koff).
// Nothing lies above the window, so one test against the window's floor
// pattern selects the elements to count.  MAG: bits is a magnitude pattern
// (sign cleared; compared as an integer); otherwise a signed fp32 pattern
// whose magnitude is compared (NaN is never counted).  inc is the counter
// increment: its low half-word must hold 1; its high half-word is set to 1
// when the element lies above its bin's floor (low bits not zero).
template <bool MAG>
__device__ inline void window_add(char* base, uint32_t bits, uint32_t floor_bits, uint32_t koff, uint32_t& inc)
{
    using namespace ties;
    const bool in = MAG ? bits >= floor_bits : fabsf(__uint_as_float(bits)) >= __uint_as_float(floor_bits);
    // the address and increment are formed in every lane (one instruction
    // each either way), so inc flows from element to element unmerged
    static_assert(KS == 16, "the low bits are the low half-word");
    uint32_t key, boff;
    asm("v_bfe_u32 %0, %1, %2, %3" : "=v"(key) : "v"(bits), "i"(KS), "i"(31 - KS));
    asm("v_lshl_add_u32 %0, %1, %2, %3" : "=v"(boff) : "v"(key), "i"(LG), "v"(koff));
    // high half-word of inc = min(low half-word of bits, 1); low half-word kept
    asm("v_min_u32_sdwa %0, %1, 1 dst_sel:WORD_1 dst_unused:UNUSED_PRESERVE src0_sel:WORD_0 src1_sel:DWORD"
        : "+v"(inc) : "v"(bits));
    if (in)
        atomicAdd(reinterpret_cast<uint32_t*>(base + boff), inc);
}

// window_add on signed patterns for one wave's row: the address is one 16-bit
// multiply-add on the pattern's high half-word.  Modulo 2^16 the sign and the
// exponent's top bits fall away, and every row lies within the first 64 KiB
// past base.  boff is the address register, passed on from element to element:
// its high half-word must hold 0.  The loop is bound by vector-ALU issue;
// one instruction of ten less took the catalog of 80M fp32 elements (blocks of
// 1024, K = 6) from 342 to 327 us and that of explicit bf16 deltas (1.5M units)
// from 2196 to 1884-2015 us.  The workgroup-wide trim (k_merge_ties) is faster
// with the two-instruction form (2515 against 2551 us).
__device__ inline void window_add16(char* base, uint32_t bits, uint32_t floor_bits, uint32_t koff, uint32_t& inc,
                                    uint32_t& boff)
{
    using namespace ties;
    const bool in = fabsf(__uint_as_float(bits)) >= __uint_as_float(floor_bits);
    static_assert(KS == 16, "the key and the low bits are half-words");
    asm("v_mad_u16 %0, %1, %2, %3 op_sel:[1,0,0,0]" : "+v"(boff) : "v"(bits), "i"(1 << LG), "v"(koff));
    asm("v_min_u32_sdwa %0, %1, 1 dst_sel:WORD_1 dst_unused:UNUSED_PRESERVE src0_sel:WORD_0 src1_sel:DWORD"
        : "+v"(inc) : "v"(bits));
    if (in)
        atomicAdd(reinterpret_cast<uint32_t*>(base + boff), inc);
}

// Floor pattern of the window whose bin 0 has key wb (everything at or
// above it lies in the window).
__device__ inline uint32_t window_floor(int wb)
{
    return (uint32_t)(wb > 0 ? wb : 0) << ties::KS;
}

// Key of bin 0 of the window anchored at the block maximum's pattern: the
// top bin holds the last key of the maximum's binade.
__host__ __device__ constexpr int window_base(uint32_t bmax)
{
    using namespace ties;
    return (int)((bmax >> 23) << MB) + (1 << MB) - NBIN;
}

// Byte offset term of window_add for the lane's copy, given the key wb of bin
// 0: key kk goes to ((kk - wb) * NC + (lane % NC)) * 4.  It wraps (for normal
// floats it is close to 2^32), so it is only ever added to another 32-bit
// offset, never to a pointer.
__host__ __device__ constexpr uint32_t window_koff_at(int wb, int lane)
{
    using namespace ties;
    return (uint32_t)(lane & (NC - 1)) * 4u - (uint32_t)wb * (uint32_t)(4 * NC);
}
__device__ inline uint32_t window_koff(uint32_t bmax, int lane, int* wb_out)
{
    *wb_out = window_base(bmax);
    return window_koff_at(*wb_out, lane);
}

// Byte offset in the histogram row of a magnitude pattern of the window: the
// sum wraps back into the row.
__host__ __device__ constexpr uint32_t window_off(uint32_t mg, uint32_t koff)
{
    using namespace ties;
    return ((mg >> KS) << LG) + koff;
}
// first and last word of the row, at both ends of the range of patterns
static_assert(window_off(0x7f800000u, window_koff_at(window_base(0x7f800000u), 1)) ==
                  (ties::NBIN - (1u << ties::MB)) * 4u * ties::NC + 4u, "infinity: the top binade's first bin");
static_assert(window_off(0x3fffffffu, window_koff_at(window_base(0x3f800000u), ties::NC - 1)) == ties::NB * 4u - 4u,
              "the last key of the maximum's binade: the row's last word");
static_assert(window_off((uint32_t)window_base(0x3f800000u) << ties::KS, window_koff_at(window_base(0x3f800000u), 0)) ==
                  0u, "the window's floor: the row's first word");
static_assert(window_off(0u, window_koff_at(window_base(1u), 0)) == (ties::NBIN - (1u << ties::MB)) * 4u * ties::NC,
              "subnormals: the window reaches below zero, zero starts its top binade");

// |x|'s pattern, formed where it is used: the rare fallbacks below do not
// keep a second copy of the values (the compiler would otherwise share one
// between them).
__device__ inline uint32_t mag_bits(float x)
{
    uint32_t r;
    asm volatile("v_and_b32 %0, 0x7fffffff, %1" : "=v"(r) : "v"(x));
    return r;
}

// max(m, |a|, |b|) in one instruction.  Written out because the compiler,
// unable to tell that these values are canonical, otherwise quiets each one
// with a v_max_f32 of its own before comparing (1.75 instructions per value
// instead of 0.5).
__device__ inline float max3_abs(float m, float a, float b)
{
    float r;
    asm("v_max3_f32 %0, %1, |%2|, |%3|" : "=v"(r) : "v"(m), "v"(a), "v"(b));
    return r;
}

// Wave-level, all lanes: exact k-th largest magnitude pattern (multiplicity
// counted) of the E values each lane holds in d (NaN is not ordered: keep
// it out), 1 <= k <= the number of values that are not padding; padding
// values are zeros, which cannot change the k largest.  The wave-private
// LDS row of NB words starts row_off bytes after base.
//
// guess (wave-uniform) is a magnitude pattern expected at or below the
// answer, 0 for none.  The histogram then first counts only the values at or
// above the floor of guess's bin: the bins from there up are exact, so a cut
// found among them is the answer, and one not found means the answer lies
// lower, when the whole window is counted again.  A good guess leaves most
// values out of the LDS atomics (and their bank conflicts).
template <int E>
__device__ inline uint32_t wave_kth_largest(char* base, int row_off, const float (&d)[E], uint32_t k, int lane,
                                            uint32_t guess = 0u)
{
    using namespace ties;
    uint32_t* __restrict__ h = reinterpret_cast<uint32_t*>(base + row_off);
    float mxf = 0.0f;
#pragma unroll
    for (int e = 0; e < E; e += 2)  // pairs: one three-way maximum each
        mxf = max3_abs(mxf, d[e], d[e + 1]);
    const uint32_t bmax = wave_max_u32(__float_as_uint(mxf));
    if (bmax == 0u)
        return 0u;  // all zero
    int wb;
    const uint32_t koff = window_koff(bmax, lane, &wb) + (uint32_t)row_off;
    const uint32_t wfloor = window_floor(wb);
    uint32_t flo = (guess > wfloor) ? (guess >> KS) << KS : wfloor;
    Cut c;
#pragma unroll 1
    for (;;) {
#pragma unroll
        for (int q = 0; q < NB / 256; ++q)
            *reinterpret_cast<uint4*>(&h[4 * (q * 64 + lane)]) = make_uint4(0u, 0u, 0u, 0u);
        wave_lds_sync();
        uint32_t inc = 1u, boff = 0u;
#pragma unroll
        for (int e = 0; e < E; ++e)
            window_add16(base, __float_as_uint(d[e]), flo, koff, inc, boff);
        wave_lds_sync();
        c = wave_find_window(h, k, lane);
        if (c.found || flo == wfloor)
            break;
        flo = wfloor;  // below the guess: count the whole window
        wave_lds_sync();
    }
    if (!c.found) {
        // The k-th largest lies below the window (high densities, deltas that
        // mostly round to zero): windows further down, each anchored at the
        // largest magnitude below the last one.  Every step goes down at
        // least four binades and stops at zero.  A NaN is in no window: units
        // that hold one go to the radix select, where it ranks above infinity.
        bool nan = false;
#pragma unroll
        for (int e = 0; e < E; ++e)
            nan |= mag_bits(d[e]) > 0x7f800000u;
        uint32_t r = k - c.total, below = wfloor;
#pragma unroll 1
        while (!__any(nan)) {
            uint32_t mx = 0u;
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const uint32_t mg = mag_bits(d[e]);
                mx = max(mx, mg < below ? mg : 0u);
            }
            mx = wave_max_u32(mx);
            if (mx == 0u)
                return 0u;  // only zeros are left
            const uint32_t ko = window_koff(mx, lane, &wb) + (uint32_t)row_off;
            const uint32_t fl = window_floor(wb);
            wave_lds_sync();
#pragma unroll
            for (int q = 0; q < NB / 256; ++q)
                *reinterpret_cast<uint4*>(&h[4 * (q * 64 + lane)]) = make_uint4(0u, 0u, 0u, 0u);
            wave_lds_sync();
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const uint32_t mg = mag_bits(d[e]);
                const uint32_t at = window_off(mg, ko);  // in 32 bits: ko wraps
                if (mg >= fl && mg < below)
                    atomicAdd(reinterpret_cast<uint32_t*>(base + at), (mg & ((1u << KS) - 1u)) != 0u ? 0x10001u : 1u);
            }
            wave_lds_sync();
            c = wave_find_window(h, r, lane);
            if (c.found)
                break;
            r -= c.total;
            below = fl;
        }
    }
    if (c.found) {
        if (c.aux < c.rank)
            return (uint32_t)(wb + (int)c.bin) << KS;  // the rank-th largest of the bin is its floor
        // list the bin's values, then fix their low bits one at a time
        const uint32_t key = (uint32_t)(wb + (int)c.bin);
        wave_lds_sync();
        uint32_t n = 0u;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const uint32_t mg = mag_bits(d[e]);
            const bool in = (mg >> KS) == key;
            const unsigned long long bal = __ballot(in);
            // position: n plus the lanes below this one that list a value
            const uint32_t pos =
                __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, n));
            const uint32_t nn = n + (uint32_t)__popcll(bal);  // wave-uniform: one bound test for all lanes
            if (in && nn <= (uint32_t)NB)
                h[pos] = mg;
            n = nn;
        }
        wave_lds_sync();
        if (n <= (uint32_t)NB)
            return wave_select_list(h, n, key, c.rank, lane);
    }
    // exact radix select over all values, from bit 30 down in digits of WD
    // bits (the row holds 2^WD counters): 30..20, 19..9, 8..0 for a row of
    // 2048 words
    constexpr int WD = (NB >= 2048) ? 11 : (NB >= 1024) ? 10 : 9;
    constexpr int NL = (31 + WD - 1) / WD;
    uint32_t pref = 0u, r = k;
#pragma unroll 1
    for (int lv = 0; lv < NL; ++lv) {
        const int top_bit = 31 - lv * WD;  // one past the digit's highest bit
        const int sh = (top_bit - WD > 0) ? top_bit - WD : 0;
        const int wd = top_bit - sh;
        wave_lds_sync();
#pragma unroll
        for (int q = 0; q < NB / 256; ++q)
            *reinterpret_cast<uint4*>(&h[4 * (q * 64 + lane)]) = make_uint4(0u, 0u, 0u, 0u);
        wave_lds_sync();
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const uint32_t mg = mag_bits(d[e]);
            const uint32_t hi = (lv == 0) ? 0u : (mg >> (sh + wd));
            if (hi == pref)
                atomicAdd(&h[(mg >> sh) & ((1u << wd) - 1u)], 1u);
        }
        wave_lds_sync();
        const Cut c = wave_find_from_top(h, (1 << wd) - 1, r, lane);
        pref = (pref << wd) | c.bin;
        r = c.rank;
    }
    return pref;
}

}  // namespace mp
