// TIES trim thresholds at tensor scope: for expert i and tensor t, the k-th
// largest |d| over the tensor's zero-completed masked deltas (unselected
// blocks count as zeros and are never read), k = min(n_t, ceil(rho n_t)).
// This is the per-tensor variant of Appendix A.1's trim; merges then use
// the per-unit threshold kernel with each unit taking its tensor's value.
//
// Two exact routes.  The bracket route reads the selected blocks once, after
// a sample of about a 32nd of them:
//   k_tt_sample   (twice) histograms a slice of every selected block, first
//                 of bits 30..20, then of the range that the first kept;
//   k_tt_bracket  (twice) one wave per (expert, tensor) pair turns the sample
//                 histogram into a bracket [lo, hi) of patterns around the
//                 k-th largest, five standard deviations of the sample's rank
//                 to either side;
//   k_tt_scan     the full pass: counts the elements at or above hi, counts
//                 the bracket's elements in 256 bins (512 in fp32, if that
//                 is a bin per pattern), and lists those of them
//                 that do not equal their bin's floor (coarse bf16 deltas repeat
//                 a few floors millions of times; those need no listing);
//   k_tt_pick     one workgroup per pair: the bin that holds the k-th largest;
//                 it is the bin's floor, or one of the listed elements.
// Nothing depends on the sample being right: a pair whose k-th largest lies
// outside its bracket, or whose list overflows, is left to the second route
// (in the second case from the bin on: each digit pass fixes up to 11 of the
// bin's at most 23 open bits, and skips the pair once it is resolved).
// The full pass is bound by memory (base and selected experts once, 1.46 ms of
// the 1.5B-parameter case against 4.5 ms for three digit passes).
//
// The radix route is an exact MSD select on the 31-bit magnitude patterns,
// three digit passes (bits 30..20, 19..9, 8..0) over the selected blocks.  It
// takes whole layouts with blocks over 4096 elements or without room for the
// lists, and the pairs that the first route left (the host, which waits for the
// call anyway, sees their number and launches it only then):
//   k_tt_hist     one workgroup per (run of consecutive blocks of one
//                 tensor, expert): LDS histogram of the digit of the
//                 elements that match the prefix fixed so far, nonzero bins
//                 added to the pair's global histogram.  Each XCD takes a
//                 contiguous range of (run, expert) pairs with the expert
//                 fastest, so the K workgroups of a run read its base
//                 blocks through one L2;
//   k_tt_resolve  one wave per (expert, tensor) pair: the bin holding the
//                 k-th largest fixes the digit and the remaining rank.  In
//                 the first pass, k = 0 gives all ones (nothing kept) and
//                 fewer than k selected elements give 0 (the k-th largest
//                 is a completed zero);
//   k_tt_expand   tau[g*K + i] = the pair's threshold for every unit.
// State per pair (uint4): {prefix, remaining rank, done, tau, or the bits of
// the prefix until done}; the entry after
// the pairs' holds {error, pairs left by the first route, 0, 0}.  The bracket
// route adds per pair {lo, hi - lo, bin shift, sampled elements above hi} and
// {selected elements, elements above hi, listed, 0}.
#include <algorithm>
#include <cmath>

#include "device_common.h"
#include "mp_internal.h"
#include "ties_select.h"

namespace mp {

namespace {

constexpr int kTT = 256;
constexpr int kDigBins = 2048;  // 11-bit digits (the last pass uses 9 bits)
// Digit-pass workgroups: the first pass counts every element, and equal
// top digits are common, so its histogram has four copies of each bin
// (lane l adds to copy l mod 4) in 512-thread workgroups (32 KiB of LDS, 32
// waves per CU); later passes count only the prefix's elements, with two
// copies in 256-thread workgroups.  On the Qwen2.5-1.5B-shaped family at
// B = 25/50/100%, thresholds and merge: 4.29-4.34 / 6.51-6.55 / 11.07-11.22
// ms; 4.14 / 6.42 / 12.32 ms with the later passes' form throughout, 4.39 /
// 6.52 / 10.92 ms with the first's.
constexpr int kTH0 = 512, kCop0 = 4;
constexpr int kTH = 256, kCop = 2;

// The lowest bit of the next digit, with `open` bits of the pattern left: from
// 31, the digits 30..20, 19..9 and 8..0.
__device__ inline int tt_shift(int open) { return open > 11 ? open - 11 : 0; }

__global__ __launch_bounds__(kTT) void k_tt_zero(uint32_t* __restrict__ p, int64_t n)
{
    for (int64_t q = (int64_t)blockIdx.x * kTT + threadIdx.x; q < n; q += (int64_t)gridDim.x * kTT)
        p[q] = 0u;
}

template <int DT, bool DELTA, int kTH, int kCopies>
__global__ __launch_bounds__(kTH) void k_tt_hist(const void* __restrict__ base, ExpertPtrs ex, int K,
                                                  const uint4* __restrict__ chunks,
                                                  const uint64_t* __restrict__ boff,
                                                  const uint32_t* __restrict__ blen,
                                                  const uint32_t* __restrict__ mask,
                                                  const uint4* __restrict__ state, int T,
                                                  uint32_t* __restrict__ hist, uint32_t n_pairs, uint32_t per_xcd)
{
    constexpr int V = Fmt<DT>::V;
    __shared__ __align__(16) uint32_t h[kDigBins * kCopies];  // h[bin * kCopies + copy]
    static_assert(kCopies == 1 || kCopies == 2 || kCopies == 4, "a bin's copies are one LDS read");
    // workgroup id -> (run, expert): XCD x = id mod 8 takes pairs
    // x*per_xcd .. in order
    const uint32_t pr = (blockIdx.x & 7u) * per_xcd + (blockIdx.x >> 3);
    if (pr >= n_pairs)
        return;
    const uint4 ch = chunks[pr / (uint32_t)K];
    const int i = (int)(pr % (uint32_t)K);
    const uint32_t t = ch.z;
    const uint4 st = state[(size_t)i * T + t];
    if (st.z != 0u)  // this pair's threshold is already known
        return;
    const int tid = threadIdx.x;
    // nothing to count when the expert has no selected block in the run
    static_assert(kMaxRunBlocks <= kTH, "a thread per block of a run");
    if (!__syncthreads_or(tid < (int)(ch.y - ch.x) && ((mask[ch.x + (uint32_t)tid] >> i) & 1u)))
        return;
    for (int q = tid; q < kDigBins * kCopies / 4; q += kTH)
        reinterpret_cast<uint4*>(h)[q] = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
    const uint32_t cp = (uint32_t)(tid % kCopies);
    const int hsh = 31 - (int)st.w, sh = tt_shift(hsh);  // the bits above the digit must match the prefix
    const uint32_t dmask = (1u << (hsh - sh)) - 1u;
    const uint32_t prefix = st.x;
    for (uint32_t g = ch.x; g < ch.y; ++g) {
        if (!((mask[g] >> i) & 1u))
            continue;
        const uint64_t off = boff[g];
        const uint32_t nch = blen[g] / V;
        const uint4* pe = chunk_ptr(ex.p[i], off, Fmt<DT>::esize);
        const uint4* pb = chunk_ptr(base, off, Fmt<DT>::esize);
        // two chunks per thread in flight (a 4096-element bf16 block is
        // exactly two)
        for (uint32_t c0 = tid; c0 < nch; c0 += 2 * kTH) {
            uint4 re[2], rb[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const uint32_t c = c0 + (uint32_t)(u * kTH);
                re[u] = c < nch ? ld16s(pe + c) : make_uint4(0u, 0u, 0u, 0u);
                rb[u] = (!DELTA && c < nch) ? pb[c] : make_uint4(0u, 0u, 0u, 0u);  // cached: the run's other experts read it too
            }
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                if (c0 + (uint32_t)(u * kTH) >= nch)
                    continue;
                float fe[V], fb[V];
                Fmt<DT>::unpack(re[u], fe);
                if (!DELTA)
                    Fmt<DT>::unpack(rb[u], fb);
#pragma unroll
                for (int v = 0; v < V; ++v) {
                    const float d = DELTA ? fe[v] : fe[v] - fb[v];
                    const uint32_t mg = __float_as_uint(d) & 0x7fffffffu;
                    if ((mg >> hsh) == prefix)
                        atomicAdd(&h[((mg >> sh) & dmask) * kCopies + cp], 1u);
                }
            }
        }
    }
    __syncthreads();
    uint32_t* out = hist + ((size_t)i * T + t) * kDigBins;
    for (int q = tid; q < kDigBins; q += kTH) {
        uint32_t v;
        if constexpr (kCopies == 4) {
            const uint4 w = reinterpret_cast<const uint4*>(h)[q];
            v = w.x + w.y + w.z + w.w;
        } else if constexpr (kCopies == 2) {
            const uint2 w = reinterpret_cast<const uint2*>(h)[q];
            v = w.x + w.y;
        } else {
            v = h[q];
        }
        if (v != 0u)
            atomicAdd(&out[q], v);
    }
}

__global__ __launch_bounds__(kTT) void k_tt_resolve(uint4* __restrict__ state, const uint32_t* __restrict__ hist,
                                                     const uint64_t* __restrict__ tnumel, int K, int T,
                                                     double density, uint32_t* __restrict__ err,
                                                     int force_no_cut)
{
    const int lane = threadIdx.x & 63;
    const int64_t q = (int64_t)blockIdx.x * (kTT / 64) + (threadIdx.x >> 6);
    if (q >= (int64_t)K * T)
        return;
    const int t = (int)(q % T);
    uint4 st = state[q];
    if (st.z != 0u)
        return;
    const uint32_t* h = hist + (size_t)q * kDigBins;
    const int open = 31 - (int)st.w, wd = open - tt_shift(open);
    constexpr int per = kDigBins / 64;  // lane l holds bins [l*per, (l+1)*per) (a narrower digit leaves the top ones 0)
    uint32_t c[per];
    uint32_t mine = 0u;
#pragma unroll
    for (int j = 0; j < per; ++j) {
        c[j] = h[lane * per + j];
        mine += c[j];
    }
    // count in the bins above this lane's range (suffix over higher lanes)
    uint32_t incl = mine;  // inclusive sum over lanes >= lane
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t y = __shfl_down(incl, (unsigned)off);
        if (lane + off < 64)
            incl += y;
    }
    const uint32_t total = __shfl(incl, 0);
    uint32_t rank = st.y;
    if (st.w == 0u) {  // the first digit
        const uint64_t n = tnumel[t];
        const double kk = ceil(density * (double)n);
        const uint64_t k = (kk >= (double)n) ? n : (uint64_t)kk;
        if (k == 0u || (uint64_t)total < k) {
            if (lane == 0)
                state[q] = make_uint4(0u, 0u, 1u, k == 0u ? 0xffffffffu : 0u);
            return;
        }
        rank = (uint32_t)k;
    }
    const uint32_t above = incl - mine;  // elements in bins of higher lanes
    int bin = -1;
    uint32_t before = 0u;
    if (above < rank && incl >= rank) {  // the k-th largest is in this lane's range
        uint32_t acc = above;
#pragma unroll
        for (int j = per - 1; j >= 0; --j) {
            if (bin < 0 && acc + c[j] >= rank) {
                bin = lane * per + j;
                before = acc;
            }
            acc += c[j];
        }
    }
    unsigned long long bal = __ballot(bin >= 0);
    if (force_no_cut && q == 0)
        bal = 0ull;  // test hook: pair 0 takes the error path
    if (bal == 0ull) {  // cannot happen: the prefix's elements hold the rank-th largest
        if (lane == 0) {
            state[q] = make_uint4(st.x, 0u, 1u, 0u);
            err[0] = 1u;  // the host reports an internal error
        }
        return;
    }
    const int src = __ffsll((long long)bal) - 1;
    bin = __shfl(bin, src);
    before = __shfl(before, src);
    if (lane == 0) {
        st.x = (st.x << wd) | (uint32_t)bin;
        st.y = rank - before;
        st.w += (uint32_t)wd;
        if (wd == open) {
            st.z = 1u;
            st.w = st.x;
        }
        state[q] = st;
    }
}

// ---------------------------------------------------------------- bracket route
constexpr int kSampleShare = 32;          // the sample: a 32nd of every block
constexpr uint32_t kSampleRuns = 8;       // runs per sampling workgroup
constexpr uint32_t kSmallTensor = 8192u;  // a pair's list has room for so many elements at least
// Bins of the full pass: up to 256 of four copies, or for an fp32 bracket of up
// to 512 patterns one bin each of two copies (nothing is off its bin's floor
// then: a quantised expert's repeated magnitude needs no list).  Not in bf16,
// whose repeated magnitudes end in zero bits and are on a floor already.  Two
// experts of 128M fp32 deltas of one magnitude, in tensors of 64M: 0.45 ms, 33.9
// with 256 bins and a list (0.91 by three digit passes alone).
constexpr int kScanBins = 512, kScanWords = 1024;
// Words of the workgroup's list (with the bins 18 KiB: eight workgroups a CU).
// Up to so many selected elements a pair lists every one; beyond, listing all
// overflows it into the pair's list, one atomic round trip after another (list
// all up to 8,192 / up to here: 64M bf16 elements x 2 experts in tensors of
// 8,192, all selected, density 0.2 / 0.5, 1015 / 1024 us against 454 / 443).
constexpr uint32_t kScanList = 3584u;
// Words of an average pair's room from which its list counts as long (tensors
// of about 200,000 elements; see k_tt_pick).
constexpr uint64_t kPickLong = 24576u;

// A pair's list is words tlist[t] .. tlist[t + 1] of its expert's lwords (see
// ties_tensor_room); a pair that needs more takes the radix route.
__device__ inline uint32_t* tt_list(uint32_t* list, int i, uint32_t lwords, const uint32_t* tlist, uint32_t t)
{
    return list + (uint64_t)i * lwords + tlist[t];
}

// Adds a workgroup's nonzero sample bins to the pair's histogram and clears them.
__device__ inline void tt_flush_sample(uint32_t* h, uint32_t* __restrict__ out)
{
    __syncthreads();
    for (int q = (int)threadIdx.x; q < kDigBins; q += kTT) {
        const uint32_t v = h[q];
        if (v != 0u) {
            atomicAdd(&out[q], v);
            h[q] = 0u;
        }
    }
    __syncthreads();
}

// Sample pass LV (0: bits 30..20 of every sampled element, and the pair's
// selected elements; 1: the bracket's elements by (pattern - lo) >> shift).
// One workgroup per expert and kSampleRuns consecutive runs; from block g of
// a run it takes the (g mod kSampleShare)-th slice of segc 16-byte chunks, so the
// slices visit every part of a tensor's blocks.
template <int DT, bool DELTA, int LV>
__global__ __launch_bounds__(kTT) void k_tt_sample(const void* __restrict__ base, ExpertPtrs ex, int K,
                                                   const uint4* __restrict__ chunks,
                                                   const uint64_t* __restrict__ boff,
                                                   const uint32_t* __restrict__ blen,
                                                   const uint32_t* __restrict__ mask, uint32_t n_runs, int T,
                                                   uint32_t run_blocks, uint32_t segc,
                                                   const uint4* __restrict__ state,
                                                   const uint4* __restrict__ br, uint32_t* __restrict__ hist,
                                                   uint4* __restrict__ cnt)
{
    constexpr int V = Fmt<DT>::V;
    __shared__ uint32_t h[kDigBins];
    // the K experts of a group of runs on one XCD (id mod 8), one after another
    const uint32_t pos = blockIdx.x >> 3;
    const int i = (int)(pos % (uint32_t)K);
    const uint32_t r0 = (pos / (uint32_t)K * 8u + (blockIdx.x & 7u)) * kSampleRuns, r1 = min(r0 + kSampleRuns, n_runs);
    if (r0 >= n_runs)
        return;
    const uint32_t tid = threadIdx.x;
    for (int q = (int)tid; q < kDigBins; q += kTT)
        h[q] = 0u;
    __syncthreads();
    // (run, share of its slices) pairs in order, kAhead of them loaded at once:
    // one at a time the pass was a chain of latencies
    constexpr uint32_t kAhead = 4u;
    const uint32_t nq = (run_blocks * segc + kTT - 1u) / kTT, steps = (r1 - r0) * nq;
    uint32_t cur = 0xffffffffu;  // the tensor whose counts h holds
    for (uint32_t x0 = 0u; x0 < steps; x0 += kAhead) {
        uint4 ch[kAhead], re[kAhead], rb[kAhead];
        uint32_t n[kAhead];
        bool in[kAhead];
#pragma unroll
        for (uint32_t a = 0u; a < kAhead; ++a) {
            const uint32_t x = min(x0 + a, steps - 1u);
            ch[a] = chunks[r0 + x / nq];
            const uint32_t q = x % nq * kTT + tid, nb = ch[a].y - ch[a].x;  // at most run_blocks
            const uint32_t g = min(ch[a].x + q / segc, ch[a].y - 1u), nch = blen[g] / V;
            uint32_t c = (g % kSampleShare) * segc + q % segc;
            if (nch <= (g % kSampleShare) * segc)
                c = q % segc;  // a short block without that slice: its first one
            in[a] = x0 + a < steps && q < nb * segc && ((mask[g] >> i) & 1u) && c < nch;
            const uint64_t off = boff[g];
            re[a] = rb[a] = make_uint4(0u, 0u, 0u, 0u);
            if (in[a]) {
                re[a] = chunk_ptr(ex.p[i], off, Fmt<DT>::esize)[c];
                if (!DELTA)
                    rb[a] = chunk_ptr(base, off, Fmt<DT>::esize)[c];
            }
            if (LV == 0)  // the run's selected elements, counted with its first share
                n[a] = x0 + a < steps && x % nq == 0u && tid < nb && ((mask[ch[a].x + tid] >> i) & 1u)
                           ? blen[ch[a].x + tid]
                           : 0u;
        }
#pragma unroll
        for (uint32_t a = 0u; a < kAhead; ++a) {
            if (x0 + a >= steps)
                break;
            const size_t pq = (size_t)i * T + ch[a].z;
            if (cur != ch[a].z && cur != 0xffffffffu)
                tt_flush_sample(h, hist + ((size_t)i * T + cur) * kDigBins);
            cur = ch[a].z;
            if (LV == 0) {
                const uint32_t sum = (uint32_t)__builtin_amdgcn_readlane((int)wave_incl_sum(n[a]), 63);
                if ((tid & 63u) == 0u && sum != 0u)
                    atomicAdd(&cnt[pq].x, sum);
            }
            uint32_t lo = 0u, width = 0x80000000u, sh = 20u;
            if (LV == 1) {
                const uint4 st = state[pq];
                if (st.z != 0u || st.y == 0u)  // decided, or every element is listed
                    continue;
                const uint4 b = br[pq];
                lo = b.x;
                width = b.y;
                sh = b.z;
            }
            if (in[a]) {
                float fe[V], fb[V];
                Fmt<DT>::unpack(re[a], fe);
                if (!DELTA)
                    Fmt<DT>::unpack(rb[a], fb);
#pragma unroll
                for (int v = 0; v < V; ++v) {
                    const uint32_t mg = __float_as_uint(DELTA ? fe[v] : fe[v] - fb[v]) & 0x7fffffffu;
                    if (LV == 0 || mg - lo < width)
                        atomicAdd(&h[(mg - lo) >> sh], 1u);
                }
            }
        }
    }
    if (cur != 0xffffffffu)
        tt_flush_sample(h, hist + ((size_t)i * T + cur) * kDigBins);
}

// The smallest shift that leaves the patterns [lo, hi) at most `bins` bins
// (ALIGNED: bins of whole multiples of 2^shift, else counted from lo).
__device__ inline uint32_t tt_shift_for(uint32_t lo, uint32_t hi, uint32_t bins, bool aligned)
{
    uint32_t s = 0u;
    while ((aligned ? ((hi - 1u) >> s) - (lo >> s) : (hi - 1u - lo) >> s) >= bins)
        ++s;
    return s;
}

// One wave per pair after sample pass LV: narrows the pair's bracket (a pair of
// at most kScanList selected elements keeps the whole range: state.y, the
// sampled elements, stays 0 and every element is listed) and clears its
// histogram.  Pass 0 also ends the pairs that keep nothing
// (k = 0: all ones) or whose k-th largest is a completed zero (fewer than k
// elements selected: 0).  Brackets of up to `single` patterns get a bin each.
template <int LV>
__global__ __launch_bounds__(kTT) void k_tt_bracket(uint4* __restrict__ state, uint4* __restrict__ br,
                                                    const uint4* __restrict__ cnt, uint32_t* __restrict__ hist,
                                                    const uint64_t* __restrict__ tnumel, int K, int T, double density,
                                                    uint32_t single)
{
    constexpr int per = kDigBins / 64;
    const int lane = threadIdx.x & 63;
    const int64_t q = (int64_t)blockIdx.x * (kTT / 64) + (threadIdx.x >> 6);
    if (q >= (int64_t)K * T)
        return;
    const uint64_t n = tnumel[q % T];
    const double kk = ceil(density * (double)n);
    const uint64_t k = (kk >= (double)n) ? n : (uint64_t)kk;
    const uint32_t N = cnt[q].x;
    uint32_t* h = hist + (size_t)q * kDigBins;
    if (LV == 1 && state[q].z != 0u)
        return;
    if (LV == 0 && (k == 0u || (uint64_t)N < k)) {
        if (lane == 0)
            state[q] = make_uint4(0u, 0u, 1u, k == 0u ? 0xffffffffu : 0u);
        return;
    }
    // the histogram, for pairs that the sample decides: read, and cleared for
    // the next pass (pass 1 leaves the full pass its bins only)
    const bool sampled = LV == 0 ? N > kScanList : state[q].y != 0u;
    uint32_t c[per] = {}, mine = 0u;
    if (sampled) {
#pragma unroll
        for (int j = 0; j < per; j += 4) {
            const uint4 v = reinterpret_cast<const uint4*>(h + lane * per)[j / 4];
            c[j] = v.x;
            c[j + 1] = v.y;
            c[j + 2] = v.z;
            c[j + 3] = v.w;
            mine += v.x + v.y + v.z + v.w;
        }
    }
    uint4 b = LV == 0 ? make_uint4(0u, 0x80000000u, 20u, 0u) : br[q];
    const uint32_t incl0 = wave_incl_sum(mine);
    const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)incl0, 63);
    const uint32_t above = total - incl0;  // samples in the bins of higher lanes
    // the sampled elements (level 1 counts only the bracket's; the pair's
    // sampled total travels in state.y)
    const uint32_t ns = LV == 0 ? total : state[q].y;
    uint32_t lo = b.x, hi = b.x + b.y, sab = b.w;  // hi: 2^31 at most
    if (ns >= 64u) {
        const double f = (double)ns / (double)N, p = (double)k / (double)N;
        const double rs = (double)k * f, m = 5.0 * sqrt(rs * (1.0 - p)) + 8.0;
        // ranks counted from the top of the bracket
        const double rhi = rs - m - (double)b.w, rlo = rs + m - (double)b.w;
        int bhi = -1, blo = -1;  // the bins that hold them, if any
        uint32_t ahi = 0u, acc = above;
#pragma unroll
        for (int j = per - 1; j >= 0; --j) {
            const double before = (double)acc, after = (double)(acc + c[j]);
            if (rhi >= 1.0 && before < rhi && rhi <= after) {
                bhi = lane * per + j;
                ahi = acc;
            }
            if (rlo >= 1.0 && before < rlo && rlo <= after)
                blo = lane * per + j;
            acc += c[j];
        }
        const unsigned long long mh = __ballot(bhi >= 0), ml = __ballot(blo >= 0);
        if (mh != 0ull) {  // otherwise the bracket keeps its top
            const int src = __ffsll((long long)mh) - 1;
            hi = min(hi, b.x + (((uint32_t)__shfl(bhi, src) + 1u) << b.z));
            sab += __shfl(ahi, src);
        }
        if (ml != 0ull)  // otherwise it keeps its bottom
            lo = b.x + ((uint32_t)__shfl(blo, __ffsll((long long)ml) - 1) << b.z);
    }
    if (lane == 0) {
        const uint32_t s = LV == 0           ? tt_shift_for(lo, hi, kDigBins, false)
                           : hi - lo <= single ? 0u
                                             : tt_shift_for(lo, hi, kScanWords / 4, true);
        br[q] = make_uint4(lo, hi - lo, s, sab);
        if (LV == 0)
            state[q].y = ns;
    }
    // clear for the next pass, once every lane's bins have been used
    if (LV == 1) {
        static_assert(kScanBins == 2 * 64 * 4, "eight bins a lane, or four");
        reinterpret_cast<uint4*>(h)[lane] = make_uint4(0u, 0u, 0u, 0u);
        if (single != 0u)
            reinterpret_cast<uint4*>(h)[64 + lane] = make_uint4(0u, 0u, 0u, 0u);
    } else if (sampled) {
#pragma unroll
        for (int j = 0; j < per / 4; ++j)
            reinterpret_cast<uint4*>(h)[j * 64 + lane] = make_uint4(0u, 0u, 0u, 0u);
    }
}

// The full pass.  One workgroup per (run, expert) in k_tt_hist's order.  Per
// element two compares and a subtraction; the bracket's elements add to the
// bins (four copies) and, off their bin's floor, to the workgroup's list,
// which is appended to the pair's at the end (entries past the LDS list go
// there directly; a thread that finds the pair's room used up lists nothing
// more, for the pair is left to the radix route: going on, the elements queue up
// at the pair's counter).  No workgroup asks beforehand whether the list is full:
// reading the counter that the others add to made ordinary fp32 tensors of 64M
// 17% slower (409 -> 476 us).
template <int DT, bool DELTA>
__global__ __launch_bounds__(kTT) void k_tt_scan(const void* __restrict__ base, ExpertPtrs ex, int K,
                                                 const uint4* __restrict__ chunks, const uint64_t* __restrict__ boff,
                                                 const uint32_t* __restrict__ blen, const uint32_t* __restrict__ mask,
                                                 const uint4* __restrict__ state, const uint4* __restrict__ br, int T,
                                                 uint32_t* __restrict__ hist, uint4* __restrict__ cnt,
                                                 uint32_t* __restrict__ list, const uint32_t* __restrict__ tlist,
                                                 uint32_t lwords, uint32_t cpb, uint32_t n_pairs, uint32_t per_xcd)
{
    constexpr int V = Fmt<DT>::V;
    __shared__ __align__(16) uint32_t h[kScanWords];
    __shared__ uint32_t lst[kScanList];
    __shared__ uint32_t s_n, s_at, s_above, s_over;
    __shared__ unsigned long long s_sel[kTT / 64];  // the run's selected blocks
    const uint32_t pr = (blockIdx.x & 7u) * per_xcd + (blockIdx.x >> 3);
    if (pr >= n_pairs)
        return;
    const uint4 ch = chunks[pr / (uint32_t)K];
    const int i = (int)(pr % (uint32_t)K);
    const size_t pq = (size_t)i * T + ch.z;
    if (state[pq].z != 0u)
        return;
    const int tid = threadIdx.x;
    static_assert(kMaxRunBlocks <= kTT, "a thread per block of a run");
    const bool selected = tid < (int)(ch.y - ch.x) && ((mask[ch.x + (uint32_t)tid] >> i) & 1u);
    const unsigned long long sel = __ballot(selected);
    if ((tid & 63) == 0)
        s_sel[tid >> 6] = sel;
    if (!__syncthreads_or(selected))
        return;
    const uint4 b = br[pq];
    const uint32_t lo = b.x, width = b.y, sh = b.z, b0 = lo >> sh, hi = lo + width;
    uint32_t low = (1u << sh) - 1u;  // 0 once the thread knows that the list is full
    uint32_t* const glist = tt_list(list, i, lwords, tlist, ch.z);
    const uint32_t cap = tlist[ch.z + 1u] - tlist[ch.z];
    for (int q = tid; q < kScanWords; q += kTT)
        h[q] = 0u;
    if (tid == 0) {
        s_n = 0u;
        s_above = 0u;
        s_over = 0u;
    }
    __syncthreads();
    const uint32_t nb = ((hi - 1u) >> sh) - b0 + 1u;  // bins in use
    const uint32_t cl = DT == 0 && nb > (uint32_t)kScanWords / 4u ? 1u : 2u;  // log2 of their copies
    const uint32_t cp = (uint32_t)tid & ((1u << cl) - 1u);
    uint32_t above = 0u;
    // one chunk's elements
    auto take = [&](const uint4& e16, const uint4& b16) {
        float fe[V], fb[V];
        Fmt<DT>::unpack(e16, fe);
        if (!DELTA)
            Fmt<DT>::unpack(b16, fb);
#pragma unroll
        for (int v = 0; v < V; ++v) {
            const uint32_t mg = __float_as_uint(DELTA ? fe[v] : fe[v] - fb[v]) & 0x7fffffffu;
            above += mg >= hi ? 1u : 0u;
            if (mg - lo < width) {
                atomicAdd(&h[(((mg >> sh) - b0) << cl) + cp], 1u);
                if ((mg & low) != 0u) {
                    const uint32_t at = atomicAdd(&s_n, 1u);
                    if (at < kScanList) {
                        lst[at] = mg;
                    } else {
                        const uint32_t to = atomicAdd(&cnt[pq].z, 1u);
                        if (to < cap)
                            glist[to] = mg;
                        else
                            s_over = 1u;
                        low = s_over == 0u ? low : 0u;
                    }
                }
            }
        }
    };
    if (cpb >= 2u * kTT) {  // blocks that give every thread two chunks, one after another
        for (uint32_t g = ch.x; g < ch.y; ++g) {
            if (!((mask[g] >> i) & 1u))
                continue;
            const uint64_t off = boff[g];
            const uint32_t nch = blen[g] / V;
            const uint4* pe = chunk_ptr(ex.p[i], off, Fmt<DT>::esize);
            const uint4* pb = chunk_ptr(base, off, Fmt<DT>::esize);
            for (uint32_t c0 = tid; c0 < nch; c0 += 2 * kTT) {
                uint4 re[2], rb[2];
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const uint32_t c = c0 + (uint32_t)(u * kTT);
                    re[u] = c < nch ? ld16s(pe + c) : make_uint4(0u, 0u, 0u, 0u);
                    rb[u] = (!DELTA && c < nch) ? pb[c] : make_uint4(0u, 0u, 0u, 0u);  // cached: the run's other experts read it too
                }
#pragma unroll
                for (int u = 0; u < 2; ++u)
                    if (c0 + (uint32_t)(u * kTT) < nch)
                        take(re[u], rb[u]);
            }
        }
    } else {
        // short blocks: the run is one contiguous range of chunks, shared out
        // without regard to blocks (one block at a time leaves three quarters
        // of the threads without a chunk at 512 bf16 elements)
        const uint64_t off = boff[ch.x];
        const uint32_t nch = (ch.y - 1u - ch.x) * cpb + blen[ch.y - 1u] / V;
        const uint4* pe = chunk_ptr(ex.p[i], off, Fmt<DT>::esize);
        const uint4* pb = chunk_ptr(base, off, Fmt<DT>::esize);
        for (uint32_t c0 = tid; c0 < nch; c0 += 2 * kTT) {
            uint4 re[2], rb[2];
            bool in[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const uint32_t c = c0 + (uint32_t)(u * kTT), j = c / cpb;
                in[u] = c < nch && ((s_sel[j / 64u % (kTT / 64)] >> (j % 64u)) & 1ull);
                re[u] = in[u] ? ld16s(pe + c) : make_uint4(0u, 0u, 0u, 0u);
                rb[u] = (!DELTA && in[u]) ? pb[c] : make_uint4(0u, 0u, 0u, 0u);
            }
#pragma unroll
            for (int u = 0; u < 2; ++u)
                if (in[u])
                    take(re[u], rb[u]);
        }
    }
    above = (uint32_t)__builtin_amdgcn_readlane((int)wave_incl_sum(above), 63);
    if ((tid & 63) == 0)
        atomicAdd(&s_above, above);
    __syncthreads();
    const uint32_t n = min(s_n, kScanList);
    if (tid == 0) {
        s_at = n != 0u ? atomicAdd(&cnt[pq].z, n) : 0u;
        if (s_above != 0u)
            atomicAdd(&cnt[pq].y, s_above);
    }
    uint32_t* out = hist + pq * kDigBins;
    for (uint32_t q = (uint32_t)tid; q < nb; q += kTT) {
        uint32_t v;
        if (cl == 2u) {
            const uint4 w = reinterpret_cast<const uint4*>(h)[q];
            v = w.x + w.y + w.z + w.w;
        } else {
            const uint2 w = reinterpret_cast<const uint2*>(h)[q];
            v = w.x + w.y;
        }
        if (v != 0u)
            atomicAdd(&out[q], v);
    }
    __syncthreads();
    const uint32_t at = s_at;
    for (uint32_t q = (uint32_t)tid; q < n; q += kTT)
        if (at + q < cap)
            glist[at + q] = lst[q];
}

// One workgroup per pair after the full pass (see the top of the file).  The
// list is read once for patterns whose bin leaves at most 11 bits open, and
// once more per further 11 bits; four independent loads a thread hide the
// latency that bounds it.  kPick threads: 1024 for long lists, 256 for short
// ones, which are bound by the barriers and by the workgroups in flight (the
// call, 256 / 1024 threads, us: 2 fp32 experts of 128M elements in tensors of
// 4M, density 0.2, 420 / 392, of 393,216 440 / 431, of 98,304 624 / 628; of 64M in
// bf16 in tensors of 16,384, a quarter selected, density 0.05, 281 / 385).
template <int kPick>
__global__ __launch_bounds__(kPick) void k_tt_pick(uint4* __restrict__ state, const uint4* __restrict__ br,
                                                   const uint4* __restrict__ cnt, const uint32_t* __restrict__ hist,
                                                   uint32_t* __restrict__ list,
                                                   const uint32_t* __restrict__ tlist, uint32_t lwords,
                                                   const uint64_t* __restrict__ tnumel, int T, double density,
                                                   uint32_t* __restrict__ left)
{
    __shared__ __align__(16) uint32_t h[kDigBins];
    __shared__ uint32_t s_bin, s_rank, s_cnt, s_ok;
    const size_t q = blockIdx.x;
    if (state[q].z != 0u)
        return;
    const int tid = threadIdx.x, lane = tid & 63;
    const int t = (int)(q % (size_t)T);
    const uint64_t n = tnumel[t];
    const double kk = ceil(density * (double)n);
    const uint32_t k = (uint32_t)((kk >= (double)n) ? n : (uint64_t)kk);
    const uint4 b = br[q], ct = cnt[q];
    const uint32_t nl = ct.z;
    const uint32_t* __restrict__ L = tt_list(list, (int)(q / (size_t)T), lwords, tlist, (uint32_t)t);
    // only a bracket of a bin per pattern uses (and has cleared) more than 256
    const int bins = b.z == 0u && b.y > (uint32_t)kScanWords / 4u ? kScanBins : kScanWords / 4;
    for (int x = tid; x < bins; x += kPick)
        h[x] = hist[q * kDigBins + (size_t)x];
    __syncthreads();
    if (tid < 64) {
        Cut c{0u, 0u, 0u, 0u, 0u, 0u};
        if (k > ct.y)
            c = wave_find_from_top(h, bins - 1, k - ct.y, lane);
        if (tid == 0) {
            s_ok = c.found;
            s_bin = c.bin;
            s_rank = c.rank;
            s_cnt = c.count;
        }
    }
    __syncthreads();
    if (s_ok == 0u) {  // outside the bracket
        if (tid == 0) {
            state[q] = make_uint4(0u, 0u, 0u, 0u);
            atomicAdd(left, 1u);
        }
        return;
    }
    uint32_t sb = b.z, pref = (b.x >> b.z) + s_bin, rank = s_rank;
    if (sb != 0u && nl > tlist[t + 1] - tlist[t]) {  // the list overflowed: the bin is known, its bits are open
        if (tid == 0) {
            state[q] = make_uint4(pref, rank, 0u, 31u - sb);
            atomicAdd(left, 1u);
        }
        return;
    }
    bool first = true;
    while (sb != 0u) {
        const uint32_t wd = min(sb, 11u), up = sb;
        sb -= wd;
        __syncthreads();
        for (int x = tid; x < kDigBins; x += kPick)
            h[x] = 0u;
        if (tid == 0)
            s_cnt = 0u;
        __syncthreads();
        const uint32_t dm = (1u << wd) - 1u;
        uint32_t mine = 0u;
        for (uint32_t a = (uint32_t)tid; a < nl; a += 4u * kPick) {
            uint32_t m[4];
#pragma unroll
            for (int u = 0; u < 4; ++u)
                m[u] = a + (uint32_t)(u * kPick) < nl ? L[a + (uint32_t)(u * kPick)] : 0xffffffffu;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if ((m[u] >> up) == pref) {  // the filler's top bit is set in no prefix
                    ++mine;
                    atomicAdd(&h[(m[u] >> sb) & dm], 1u);
                }
            }
        }
        if (mine != 0u)
            atomicAdd(&s_cnt, mine);
        __syncthreads();
        if (first && s_cnt < rank) {  // the bin's rank-th largest is its floor
            pref <<= up;
            sb = 0u;
            break;
        }
        first = false;
        if (tid < 64) {
            const Cut c = wave_find_from_top(h, (int)dm, rank, lane);
            if (tid == 0) {
                s_ok = c.found;
                s_bin = c.bin;
                s_rank = c.rank;
            }
        }
        __syncthreads();
        if (s_ok == 0u) {  // cannot happen: the list holds the rank-th largest
            if (tid == 0) {
                state[q] = make_uint4(0u, 0u, 0u, 0u);
                atomicAdd(left, 1u);
            }
            return;
        }
        pref = (pref << wd) | s_bin;
        rank = s_rank;
    }
    if (tid == 0)
        state[q] = make_uint4(pref, 0u, 1u, pref);
}

__global__ __launch_bounds__(kTT) void k_tt_expand(const uint4* __restrict__ state,
                                                    const uint32_t* __restrict__ tensor, int64_t G, int K, int T,
                                                    uint32_t* __restrict__ tau)
{
    const int64_t u = (int64_t)blockIdx.x * kTT + threadIdx.x;
    if (u >= G * K)
        return;
    const int64_t g = u / K;
    const int i = (int)(u - g * K);
    tau[u] = state[(size_t)i * T + tensor[g]].w;
}

}  // namespace

// Room for the list of one expert's pair with a tensor of n elements.  The
// bracket holds the sample's rank plus and minus m = 5 sqrt(r (1 - p)) + 8
// with r = N p / kSampleShare, N <= n elements selected, p = k / N: in
// elements 2 m kSampleShare, at most 28.3 sqrt(N) + 512 (p = 1/2), and up to a
// sample bin at either end (for smooth data below N / 7000 together).  Nearly
// all fp32 patterns are listed, so the room grows with the square root: 32
// sqrt(n), the small tensors' room and a 256th.  A room of the small tensors'
// and a 128th left every normal fp32 pair of 0.1M to 8M elements at densities
// 0.2 to 0.8 to the radix passes: 128M elements x 2 experts in tensors of
// 393,216 / 1M / 4M, density 0.2, 1265 / 1228 / 1214 us (three digit passes
// alone 852 / 842 / 838).
uint64_t ties_tensor_room(uint64_t n)
{
    return std::min<uint64_t>(n, kSmallTensor + 32u * (uint64_t)std::sqrt((double)n) + n / 256u);
}

hipError_t launch_ties_tensor(const BlockTable& bt, const void* base, const ExpertPtrs& ex, int K,
                              const uint32_t* mask, double density, uint32_t* tau, uint32_t* hist, uint4* state,
                              uint32_t* list, TensorTies route, hipStream_t s, bool delta, bool force_no_cut)
{
    if (bt.G == 0)
        return hipSuccess;
    const int T = (int)bt.n_tensors;
    const int64_t pairs = (int64_t)K * T;
    const int64_t nh = pairs * kDigBins;
    // the state words, after them the error and left-over words, and the
    // bracket route's counters start at zero
    uint4 *br = state + 2 * pairs + 1, *cnt = state + pairs + 1;
    uint32_t* err = reinterpret_cast<uint32_t*>(state + pairs);
    uint32_t* left = err + 1;
    const int64_t nz = (2 * pairs + 1) * 4;
    if (route != TensorTies::Left)
        hipLaunchKernelGGL(k_tt_zero, dim3((unsigned)std::min<int64_t>((nz + kTT - 1) / kTT, 1024)), dim3(kTT), 0, s,
                           reinterpret_cast<uint32_t*>(state), nz);
    const uint32_t n_pairs = (uint32_t)(bt.n_chunks * K), per_xcd = (n_pairs + 7u) / 8u;
    const dim3 hgrid(8u * per_xcd);
    const dim3 zgrid((unsigned)std::min<int64_t>((nh + kTT - 1) / kTT, 2048));
    const dim3 pgrid((unsigned)((pairs + 3) / 4));
    if (route == TensorTies::Bracket) {
        hipLaunchKernelGGL(k_tt_zero, zgrid, dim3(kTT), 0, s, hist, nh);
        const uint32_t n_runs = (uint32_t)bt.n_chunks;
        const dim3 sgrid(((n_runs + kSampleRuns - 1) / kSampleRuns + 7u) / 8u * 8u * (uint32_t)K);
        const uint32_t v = bt.dtype == 0 ? 4u : 8u;
        const uint32_t segc = std::max<uint32_t>(1u, (uint32_t)bt.block_elems / v / kSampleShare);
        const uint32_t lwords = (uint32_t)bt.tt_words;
        auto sample = [&](auto kern) {
            hipLaunchKernelGGL(kern, sgrid, dim3(kTT), 0, s, base, ex, K, bt.d_chunk, bt.d_off, bt.d_len, mask,
                               n_runs, T, (uint32_t)run_blocks(bt.block_elems), segc, state, br, hist, cnt);
        };
        auto scan = [&](auto kern) {
            hipLaunchKernelGGL(kern, hgrid, dim3(kTT), 0, s, base, ex, K, bt.d_chunk, bt.d_off, bt.d_len, mask, state,
                               br, T, hist, cnt, list, bt.d_tlist, lwords, (uint32_t)bt.block_elems / v, n_pairs,
                               per_xcd);
        };
        if (bt.dtype == 0)
            delta ? sample(k_tt_sample<0, true, 0>) : sample(k_tt_sample<0, false, 0>);
        else
            delta ? sample(k_tt_sample<1, true, 0>) : sample(k_tt_sample<1, false, 0>);
        hipLaunchKernelGGL(k_tt_bracket<0>, pgrid, dim3(kTT), 0, s, state, br, cnt, hist, bt.d_tnumel, K, T, density,
                           0u);
        if (bt.dtype == 0)
            delta ? sample(k_tt_sample<0, true, 1>) : sample(k_tt_sample<0, false, 1>);
        else
            delta ? sample(k_tt_sample<1, true, 1>) : sample(k_tt_sample<1, false, 1>);
        hipLaunchKernelGGL(k_tt_bracket<1>, pgrid, dim3(kTT), 0, s, state, br, cnt, hist, bt.d_tnumel, K, T, density,
                           bt.dtype == 0 ? (uint32_t)kScanBins : 0u);
        if (bt.dtype == 0)
            delta ? scan(k_tt_scan<0, true>) : scan(k_tt_scan<0, false>);
        else
            delta ? scan(k_tt_scan<1, true>) : scan(k_tt_scan<1, false>);
        auto pick = [&](auto kern, int nth) {
            hipLaunchKernelGGL(kern, dim3((unsigned)pairs), dim3(nth), 0, s, state, br, cnt, hist, list, bt.d_tlist,
                               lwords, bt.d_tnumel, T, density, left);
        };
        bt.tt_words / (uint64_t)T > kPickLong ? pick(k_tt_pick<1024>, 1024) : pick(k_tt_pick<256>, 256);
    }
    // the radix passes: over everything, or over the pairs the bracket route left
    for (int pass = 0; pass < 3 && route != TensorTies::Bracket; ++pass) {
        hipLaunchKernelGGL(k_tt_zero, zgrid, dim3(kTT), 0, s, hist, nh);
        auto go = [&](auto kern, int nth) {
            hipLaunchKernelGGL(kern, hgrid, dim3(nth), 0, s, base, ex, K, bt.d_chunk, bt.d_off, bt.d_len, mask, state,
                               T, hist, n_pairs, per_xcd);
        };
        if (pass == 0) {
            if (bt.dtype == 0)
                delta ? go(k_tt_hist<0, true, kTH0, kCop0>, kTH0) : go(k_tt_hist<0, false, kTH0, kCop0>, kTH0);
            else
                delta ? go(k_tt_hist<1, true, kTH0, kCop0>, kTH0) : go(k_tt_hist<1, false, kTH0, kCop0>, kTH0);
        } else {
            if (bt.dtype == 0)
                delta ? go(k_tt_hist<0, true, kTH, kCop>, kTH) : go(k_tt_hist<0, false, kTH, kCop>, kTH);
            else
                delta ? go(k_tt_hist<1, true, kTH, kCop>, kTH) : go(k_tt_hist<1, false, kTH, kCop>, kTH);
        }
        hipLaunchKernelGGL(k_tt_resolve, pgrid, dim3(kTT), 0, s, state, hist, bt.d_tnumel, K, T, density, err,
                           force_no_cut ? 1 : 0);
    }
    hipLaunchKernelGGL(k_tt_expand, dim3((unsigned)((bt.G * K + kTT - 1) / kTT)), dim3(kTT), 0, s, state,
                       bt.d_tensor, bt.G, K, T, tau);
    return hipGetLastError();
}

}  // namespace mp
