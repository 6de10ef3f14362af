// Block-norm index (the catalog statistic of Section 2 / Section 3
// "Catalog"): S[g*K + i] = sum over block g of d*d, d = x_i - x_0 in fp32.
//
// One 256-thread workgroup per block; wave w handles experts w, w+4, ...
// Each lane streams 16-byte chunks l, l+64, l+128, ... of the block (one
// coalesced 1 KiB row per wave load), accumulates its chunk elements in
// order with fma into one fp32 partial, and the wave folds the 64 partials
// with an xor butterfly.  This fixed order is the one the ABI documents, so
// the scores -- and therefore the plan -- are reproducible bit for bit.
// The base block is re-read per expert from L2 (it stays resident: 8-16 KiB
// per workgroup), so HBM sees it once.
#include <algorithm>
#include <cmath>

#include "device_common.h"
#include "mp_internal.h"
#include "ties_select.h"

namespace mp {

namespace {

constexpr int kRows = 8;  // chunk rows a lane keeps in flight per expert

// DELTA: the expert buffers hold the deltas themselves (no base read).
template <int DT, bool DELTA>
__device__ inline float block_sumsq(const uint4* __restrict__ b, const uint4* __restrict__ e,
                                    uint32_t nch, int lane)
{
    constexpr int V = Fmt<DT>::V;
    float p = 0.0f;
    for (uint32_t c0 = 0; c0 < nch; c0 += 64 * kRows) {
        uint4 xb[kRows], xe[kRows];
#pragma unroll
        for (int r = 0; r < kRows; ++r) {
            const uint32_t c = c0 + r * 64 + lane;
            if (c < nch) {
                if (!DELTA)
                    xb[r] = b[c];  // re-read per expert: cached
                xe[r] = ld16s(&e[c]);
            }
        }
#pragma unroll
        for (int r = 0; r < kRows; ++r) {
            const uint32_t c = c0 + r * 64 + lane;
            if (c < nch) {
                float fb[V], fe[V];
                if (!DELTA)
                    Fmt<DT>::unpack(xb[r], fb);
                Fmt<DT>::unpack(xe[r], fe);
#pragma unroll
                for (int q = 0; q < V; ++q) {
                    const float d = DELTA ? fe[q] : fe[q] - fb[q];
                    p = fmaf(d, d, p);
                }
            }
        }
    }
    return wave_xor_sum(p);
}

template <int DT, bool DELTA>
__global__ __launch_bounds__(256) void k_index(const void* __restrict__ base, ExpertPtrs ex, int K,
                                               const uint64_t* __restrict__ boff,
                                               const uint32_t* __restrict__ blen,
                                               float* __restrict__ sumsq)
{
    const int64_t g = blockIdx.x;
    const int lane = threadIdx.x & 63;
    // wave-uniform, so that ex.p[i] is a scalar load
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint64_t off = boff[g];
    const uint32_t nch = blen[g] / Fmt<DT>::V;
    const uint4* b = chunk_ptr(base, off, Fmt<DT>::esize);
    for (int i = wave; i < K; i += 4) {
        const uint4* e = chunk_ptr(ex.p[i], off, Fmt<DT>::esize);
        const float s = block_sumsq<DT, DELTA>(b, e, nch, lane);
        if (lane == 0)
            sumsq[g * K + i] = s;
    }
}

// The smallest magnitude pattern of a block of n elements whose lane holds
// the deltas of chunks lane, lane + 64, ... in d (padding left out): the
// threshold that keeps everything.
template <int R, int V>
__device__ inline uint32_t smallest_mag(const float (&d)[R * V], uint32_t n, int lane)
{
    uint32_t mn = 0x7fffffffu;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const bool in = (uint32_t)(r * 64 + lane) * (uint32_t)V < n;
#pragma unroll
        for (int q = 0; q < V; ++q)
            mn = min(mn, in ? mag_bits(d[r * V + q]) : 0x7fffffffu);
    }
    return ~wave_max_u32(~mn);
}

// Waves per SIMD of the catalog kernel, by the rows of chunks a lane holds.
// 64 deltas and the raw rows they come from take 96 to 112 registers: five
// waves, four for explicit deltas and fp32 (five spill there).
template <int DT, bool DELTA, int ROWS>
constexpr int cat_waves()
{
    return ROWS >= 16 ? 4 : ROWS >= 8 ? (DT == 1 && DELTA ? 4 : 5) : 8;
}

// Catalog statistics for TIES: per unit, the sum of squares of k_index
// (same order, same bits; optional) and the trim threshold, the fp32
// pattern of the k-th largest |d| of the (expert, block) unit for a keep
// density (all ones when k = 0: a NaN pattern, which keeps nothing).  The
// threshold depends on the unit and the density only, never on an access
// mask, so merges at any budget can reuse it.
//
// One wave, a workgroup of its own, takes the units of one expert in U
// consecutive blocks; R rows of 64 chunks hold the layout's longest block
// (R * V deltas per lane).  Bound by HBM from 1024-element bf16 blocks up,
// below by the fixed work of a unit (clearing and walking its histogram).
// A wave alone has no barrier and no idle partners at K not a multiple of
// four, and the rows fit the block instead of being padded to 4096
// elements.  Against one 256-thread workgroup per 4096-element frame with
// the base staged in LDS (4 layers of the Qwen2.5-1.5B shape, us): bf16 K = 4
// blocks of 4096 / 2048 / 1024 / 512: 358 -> 330, 522 -> 308, 964 -> 354,
// 1836 -> 465; K = 1: 190 -> 126; K = 6: 529 -> 455; fp32 blocks of 2048 /
// 1024 (K = 6) / 512: 811 -> 594, 2733 -> 870, 3045 -> 727.  1.54B elements in
// bf16, K = 1 / 2 / 4, blocks of 4096: 1385 -> 902, 1639 -> 1313, 2523 -> 2274 (6.8
// TB/s); explicit deltas 662 -> 458, 1033 -> 895, 1892 -> 1796 (6.9 TB/s).
// Two blocks per wave hide the loads of a 1 KiB unit (512 bf16 elements: 536
// -> 465 us); for larger units they cost registers and were slower.
template <int DT, bool DELTA, int R, int U>
__global__ __launch_bounds__(64, (cat_waves<DT, DELTA, R * U>())) void k_index_ties(
    const void* __restrict__ base, ExpertPtrs ex, int K, uint64_t k_magic, uint32_t G, uint32_t per_xcd,
    const uint64_t* __restrict__ boff, const uint32_t* __restrict__ blen, uint32_t n_full, uint32_t k_full,
    double density, float gcoef, float* __restrict__ sumsq, uint32_t* __restrict__ tau)
{
    constexpr int V = Fmt<DT>::V;
    constexpr int E = R * V;  // deltas per lane
    __shared__ uint32_t row[ties::NB];
    const int lane = threadIdx.x;
    // id -> (run of U blocks, expert), the expert fastest, a run's experts on
    // one XCD (x = id mod 8) so that they read its base through one L2.  Each
    // XCD takes a contiguous range of runs (1.54B elements in bf16, K = 4: 2275
    // against 2358 us for the runs x, x + 8, ...; explicit deltas 1796 against
    // 1855), except with 16 KiB units, where the interleaved order is faster
    // (K = 2: 358 against 378 us)
    const uint32_t pos = blockIdx.x >> 3, xcd = blockIdx.x & 7u;
    const uint32_t q8 = K > 1 ? (uint32_t)__umul64hi((uint64_t)pos, k_magic) : pos;
    const uint32_t i = pos - q8 * (uint32_t)K;
    const uint32_t first = (R >= 16 ? q8 * 8u + xcd : xcd * per_xcd + q8) * (uint32_t)U;  // the run's first block
    if (first >= G)
        return;
    constexpr int RG = R > 8 ? 8 : R;  // rows loaded before the first use (fp32: 16 of each would spill)
    uint32_t n[U];
    uint64_t off[U];
    uint4 xb[U][RG], xe[U][RG];
    // Loads are buffer loads over the block's byte range: lanes past a short
    // block's end read zeros without a branch.  The base is cached (the
    // block's other experts read it too).
    auto load = [&](int j, int r0) {
        const uint32_t nbytes = (first + (uint32_t)j < G) ? n[j] / (uint32_t)V * 16u : 0u;
        if (!DELTA) {  // explicit deltas need no base
            const __amdgpu_buffer_rsrc_t rb = block_rsrc(chunk_ptr(base, off[j], Fmt<DT>::esize), nbytes);
#pragma unroll
            for (int r = 0; r < RG; ++r)
                xb[j][r] = bld16(rb, (uint32_t)((r0 + r) * 64 + lane) * 16u);
        }
        const __amdgpu_buffer_rsrc_t re = block_rsrc(chunk_ptr(ex.p[i], off[j], Fmt<DT>::esize), nbytes);
#pragma unroll
        for (int r = 0; r < RG; ++r)
            xe[j][r] = bld16s(re, (uint32_t)((r0 + r) * 64 + lane) * 16u);
    };
#pragma unroll
    for (int j = 0; j < U; ++j) {
        const uint32_t g = min(first + (uint32_t)j, G - 1u);
        off[j] = boff[g];
        n[j] = blen[g];
        load(j, 0);
    }
#pragma unroll
    for (int j = 0; j < U; ++j) {
        if (U > 1 && first + (uint32_t)j >= G)
            break;
        float d[E];
        float p = 0.0f;
#pragma unroll
        for (int r0 = 0; r0 < R; r0 += RG) {
            if (r0 > 0) {
                __builtin_amdgcn_sched_barrier(0);  // the compiler would hoist these loads and spill
                load(j, r0);
            }
#pragma unroll
            for (int r = 0; r < RG; ++r) {
                float fb[V], fe[V];
                if (!DELTA)
                    Fmt<DT>::unpack(xb[j][r], fb);
                Fmt<DT>::unpack(xe[j][r], fe);
#pragma unroll
                for (int q = 0; q < V; ++q) {
                    const int e = (r0 + r) * V + q;
                    d[e] = DELTA ? fe[q] : fe[q] - fb[q];  // padding: 0 - 0
                    p = fmaf(d[e], d[e], p);  // + 0 on padding, exact
                }
            }
        }
        p = wave_xor_sum(p);
        uint32_t k = k_full;
        if (n[j] != n_full) {
            const double kk = ceil(density * (double)n[j]);
            k = (kk >= (double)n[j]) ? n[j] : (uint32_t)kk;
        }
        uint32_t th;
        if (k == 0u) {
            th = 0xffffffffu;
        } else if (k == n[j]) {
            th = smallest_mag<R, V>(d, n[j], lane);
        } else {
            // a guess at tau: gcoef times the deltas' root mean square
            const uint32_t guess = __float_as_uint(gcoef * sqrtf(p / (float)n[j]));
            th = wave_kth_largest<E>(reinterpret_cast<char*>(row), 0, d, k, lane, guess);
            if (U > 1)
                wave_lds_sync();  // the row is the next unit's
        }
        if (lane == 0) {
            const uint32_t u = (first + (uint32_t)j) * (uint32_t)K + i;  // < 2^32 (checked by the host)
            if (sumsq != nullptr)
                sumsq[u] = p;
            tau[u] = th;
        }
    }
}

// fp32 blocks of more than 2048 elements: one 256-thread workgroup per block,
// the base staged in LDS once and wave w taking experts w, w + 4, ... (each
// with its own LDS row; no barrier after the staging).  A wave per unit needs
// 128 registers for 16 rows of base and expert and reads each 16 KiB base
// block K times from L2: at K = 4 / 8 / 16 it takes 608 / 1141 / 2287 us, this
// 611 / 1087 / 2059 (4 layers of the Qwen2.5-1.5B shape, medians over three
// processes).  With K < 4 some of the four waves idle (K = 1 / 2: 341 / 380
// against 250 / 358 us), and explicit deltas have no base to stage.
__global__ __launch_bounds__(256, 3) void k_index_ties_staged(
    const void* __restrict__ base, ExpertPtrs ex, int K, const uint64_t* __restrict__ boff,
    const uint32_t* __restrict__ blen, uint32_t n_full, uint32_t k_full, double density, float gcoef,
    float* __restrict__ sumsq, uint32_t* __restrict__ tau)
{
    constexpr int DT = 0;
    constexpr int V = Fmt<DT>::V;
    constexpr int R = kTiesMaxBlock / 64 / V;  // chunk rows per lane
    constexpr int E = R * V;                   // deltas per lane
    __shared__ uint32_t rows[4][ties::NB];
    __shared__ uint4 xb[R * 64];  // the base block's chunks (zeros past its end)
    const int64_t g = blockIdx.x;
    const int t = threadIdx.x;
    const int lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);  // wave-uniform: ex.p[i] is a scalar load
    const uint64_t off = boff[g];
    const uint32_t n = blen[g];
    const uint32_t nch = n / V;
    uint32_t k = k_full;
    if (n != n_full) {
        const double kk = ceil(density * (double)n);
        k = (kk >= (double)n) ? n : (uint32_t)kk;
    }
    // one unit: expert i's chunks (xe) against the staged base
    auto unit = [&](int i, const uint4 (&xe)[R]) {
        float d[E];
        float p = 0.0f;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            float fb[V], fe[V];
            Fmt<DT>::unpack(xb[r * 64 + lane], fb);
            Fmt<DT>::unpack(xe[r], fe);
#pragma unroll
            for (int q = 0; q < V; ++q) {
                d[r * V + q] = fe[q] - fb[q];  // padding: 0 - 0
                p = fmaf(d[r * V + q], d[r * V + q], p);  // + 0 on padding, exact
            }
        }
        p = wave_xor_sum(p);
        // a guess at tau: gcoef times the deltas' root mean square
        const uint32_t guess = __float_as_uint(gcoef * sqrtf(p / (float)n));
        uint32_t th = 0xffffffffu;
        if (k == n)
            th = smallest_mag<R, V>(d, n, lane);
        else if (k != 0u)
            th = wave_kth_largest<E>(reinterpret_cast<char*>(&rows[0][0]), wave * ties::NB * 4, d, k, lane, guess);
        if (lane == 0) {
            if (sumsq != nullptr)
                sumsq[g * K + i] = p;
            tau[g * K + i] = th;
        }
    };
    // Loads are buffer loads over the block's byte range: lanes past a short
    // block's end read zeros without a branch, so every load of a lane is
    // issued back to back and the waits count them exactly.
    const uint32_t nbytes = nch * 16u;
    auto load_expert = [&](int i, uint32_t bytes, uint4 (&xe)[R]) {
        const __amdgpu_buffer_rsrc_t re = block_rsrc(chunk_ptr(ex.p[i], off, Fmt<DT>::esize), bytes);
#pragma unroll
        for (int r = 0; r < R; ++r)
            xe[r] = bld16s(re, (uint32_t)(r * 64 + lane) * 16u);
    };
    // The base's chunks are requested first, then the wave's first expert
    // (a wave without one reads an empty range), so the base arrives first
    // and is staged while the expert is still in flight; further experts
    // (K > 4) are read one at a time.
    uint4 xbr[R / 4];
    const __amdgpu_buffer_rsrc_t rb = block_rsrc(chunk_ptr(base, off, Fmt<DT>::esize), nbytes);
#pragma unroll
    for (int q = 0; q < R / 4; ++q)
        xbr[q] = bld16s(rb, (uint32_t)(q * 256 + t) * 16u);
    uint4 xf[R];
    load_expert(wave < K ? wave : 0, wave < K ? nbytes : 0u, xf);
#pragma unroll
    for (int q = 0; q < R / 4; ++q)
        xb[q * 256 + t] = xbr[q];  // zeros past the block's end
    __syncthreads();
    if (wave < K)
        unit(wave, xf);
    for (int i = wave + 4; i < K; i += 4) {
        uint4 xe[R];
        load_expert(i, nbytes, xe);
        unit(i, xe);
    }
}

}  // namespace

// z with P(|Z| > z) = rho for a standard normal Z (bisection on erfc).
double normal_two_sided_quantile(double rho)
{
    if (!(rho > 0.0) || rho >= 1.0)
        return 0.0;
    double lo = 0.0, hi = 40.0;
    for (int it = 0; it < 200; ++it) {
        const double mid = 0.5 * (lo + hi);
        if (erfc(mid / sqrt(2.0)) > rho)
            lo = mid;
        else
            hi = mid;
    }
    return lo;
}

hipError_t launch_index_ties(const BlockTable& bt, const void* base, const ExpertPtrs& ex, int K,
                             double density, float* sumsq, uint32_t* tau, hipStream_t s, bool delta)
{
    if (bt.G == 0)
        return hipSuccess;
    const uint32_t n_full = (uint32_t)bt.block_elems;
    const double kk = ceil(density * (double)n_full);
    const uint32_t k_full = (kk >= (double)n_full) ? n_full : (uint32_t)kk;
    // The selector's first guess at a unit's threshold: 0.8 of the rho-tail
    // quantile of a normal with the deltas' RMS (for normal deltas about
    // 0.8 tau; measured on the headline family, 0.6 was slower, 0.9 the same
    // and 1.0 misses often enough to cost a second pass).  It only decides
    // which values the first histogram pass counts; the thresholds are exact
    // for any data.
    const float gcoef = (float)(0.8 * normal_two_sided_quantile(density));
    // pos / K = mulhi(pos, floor(2^64 / K) + 1) for pos < 2^32, K > 1
    const uint64_t magic = K > 1 ? ~(uint64_t)0 / (uint64_t)K + 1u : 0u;
    auto go = [&](auto kern, int64_t U) {
        // a launch has fewer than 2^32 threads: very many units take several
        const int64_t most = ((int64_t)1 << 25) / K * U;
        for (int64_t g0 = 0; g0 < bt.G; g0 += most) {
            const int64_t G = std::min(most, bt.G - g0), per_xcd = ((G + U - 1) / U + 7) / 8;
            hipLaunchKernelGGL(kern, dim3((unsigned)(8 * per_xcd * K)), dim3(64), 0, s, base, ex, K, magic, (uint32_t)G,
                               (uint32_t)per_xcd, bt.d_off + g0, bt.d_len + g0, n_full, k_full, density, gcoef,
                               sumsq != nullptr ? sumsq + g0 * K : nullptr, tau + g0 * K);
        }
    };
#define MP_CAT(DTV, RV, UV)                                                                                            \
    (delta ? go(k_index_ties<DTV, true, RV, UV>, UV) : go(k_index_ties<DTV, false, RV, UV>, UV))
    // rows of 64 chunks per unit from the layout's longest block
    if (bt.dtype == 0) {
        if (bt.max_len <= 512)
            MP_CAT(0, 2, 1);
        else if (bt.max_len <= 1024)
            MP_CAT(0, 4, 1);
        else if (bt.max_len <= 2048)
            MP_CAT(0, 8, 1);
        else if (delta || K < 4)
            MP_CAT(0, 16, 1);
        else
            hipLaunchKernelGGL(k_index_ties_staged, dim3((unsigned)bt.G), dim3(256), 0, s, base, ex, K, bt.d_off, bt.d_len, n_full,
                               k_full, density, gcoef, sumsq, tau);
    } else {
        if (bt.max_len <= 512)
            MP_CAT(1, 1, 2);
        else if (bt.max_len <= 1024)
            MP_CAT(1, 2, 1);
        else if (bt.max_len <= 2048)
            MP_CAT(1, 4, 1);
        else
            MP_CAT(1, 8, 1);
    }
#undef MP_CAT
    return hipGetLastError();
}

hipError_t launch_index(const BlockTable& bt, const void* base, const ExpertPtrs& ex, int K,
                        float* sumsq, hipStream_t s, bool delta)
{
    if (bt.G == 0)
        return hipSuccess;
    const dim3 grid((unsigned)bt.G), block(256);
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, grid, block, 0, s, base, ex, K, bt.d_off, bt.d_len, sumsq);
    };
    if (bt.dtype == 0)
        delta ? go(k_index<0, true>) : go(k_index<0, false>);
    else
        delta ? go(k_index<1, true>) : go(k_index<1, false>);
    return hipGetLastError();
}

}  // namespace mp
