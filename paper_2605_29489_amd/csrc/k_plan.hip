// Algorithm 1 (PlanGen) on the GPU, bit-exact with a literal sort + greedy.
//
// Every unit u = (g, i) gets the 64-bit key  (~bits(score) << 32) | uid
// with score = float(float(w_i*w_i) * S_u) >= +0, so ascending keys are the
// candidate order of Algorithm 1 (decreasing score, ties by increasing uid)
// and keys are unique.  The literal greedy takes every candidate before the
// first one whose running cost overflows B (the "cut" p), skips p, and then
// keeps scanning; after p only candidates cheaper than c_p can still fit.
//
// So no full sort is needed:
//   round r:  find the cut key of the current candidate set by a
//             cost-weighted MSD radix select (each pass builds a cost
//             histogram of the candidates that match the resolved key prefix
//             and finds the bin where the running cost passes the budget);
//             select every candidate below the cut; the candidates above the
//             cut that still fit what is left form the next round's set.
//   A round whose candidates all fit selects them all and ends the plan.
// Each round strictly lowers the cost bound, so the number of rounds is at
// most the number of distinct block lengths of the layout.
//
// Up to kOneMax units the whole plan is one single-workgroup launch
// (k_plan_one): keys and costs stay in registers.  Above that, round 0 (all
// units) runs over the whole device: digits of 11 bits, three passes for the
// score and one or two for the uid, then one pass that marks the mask; the
// later rounds, whose candidate lists are short (units of short blocks only),
// run together in k_plan_one, which also closes the digest and the stats.  All
// control state lives on the device (PlanCtl); the host enqueues a fixed kernel
// sequence and kernels that are no longer needed return at once.  What bounds
// it is launches and dependent passes, not bytes: at 1.5M units, eight 8-bit
// passes of one thread per block took 8.5 us each, the later rounds (reloading
// their list in each pass) 30 us and fourteen launches in all 145 us; now 80 us,
// seven launches, passes of 7-12 us and the later rounds 15 us.
//
// A plan also has to run beside another stream's merge, whose waves refill
// every slot as it frees: a workgroup is placed only once its waves' slots and
// registers are free on one CU together.  So the kernels have four waves (one per SIMD) of at most 64 registers (a merge
// wave's).  Workgroups of 512 and 1024 threads waited for the whole merge: the
// plans of the 1.5B-parameter step's second and third budgets took 1.52 and
// 1.95 ms, now 0.30 and 0.23.  (One-launch plans and later rounds over more than
// 1,024 units keep 1024 threads: that kernel waits for the merge.)
#include "device_common.h"
#include "mp_internal.h"

namespace mp {

// Workgroups of the marking pass (at most).  Each workgroup ends a digit pass
// with device-scope atomic adds into the shared histogram, which serialize per
// address: 512 workgroups up to 8M units (at 1.5M, 512 / 256 of twice the loads
// in flight: 80 / 84 us), 1024 above (32M: 336 / 355 with 512).
constexpr int kPlanGrid = 1024;
constexpr int kHistT = 256, kHistU = 4;  // threads, and units' loads in flight per thread
constexpr int kPlanBins = 2048;          // 11-bit digits
// Copies of the first digit's histogram: scores share few of its bins, so the
// workgroups' adds queue up at those (pass 0 at 1.5M units: 21 us with one copy,
// 11 with four).
constexpr int kFirst = 4;

struct PlanCtl {
    unsigned long long brem[9];       // remaining budget before resolving digit d
    unsigned long long prefix[9];     // key prefix with digits < d resolved
    unsigned long long hist[3][kPlanBins];  // rotating cost histograms of digit passes
    unsigned long long first[kFirst][kPlanBins];  // pass 0's, workgroup b adding to copy b mod kFirst
    unsigned long long total0;        // candidate cost of the round (all-fit case)
    unsigned long long sel_cost;
    unsigned long long sel_count;
    unsigned long long stats[7];      // budget, cost, full, n_sel, n_units, digest, error
    unsigned int all_fit;
    unsigned int done;
    unsigned int list_n[2];
    unsigned int error;  // set if an internal invariant failed (reported by the host)
    // per-workgroup partial sums of the round-0 kernels (selected cost and
    // count of k_plan_mark, digest terms of k_plan_digest): one plain store
    // per workgroup, summed by the one-workgroup kernel that follows.  Many
    // workgroups adding to one device-scope word serialize at the memory
    // side (the L2 caches are per XCD), which cost tens of microseconds.
    unsigned long long part[3][kPlanGrid];
};

namespace {

constexpr int kT = 256;

// Plan options (the flags of mp_plan).
constexpr uint32_t kPlanPerByte = 1u;   // score per byte of cost
constexpr uint32_t kPlanSkipZero = 2u;  // units with a zero sum of squares are not candidates

// The unit's sort key; c is its cost in bytes.  Per byte: the fp32 score
// divided by c in fp64, rounded once to fp32.
__device__ inline unsigned long long unit_key(float S, float w, uint32_t uid, unsigned long long c, uint32_t flags)
{
    const float w2 = w * w;
    float sc = w2 * S;
    if (flags & kPlanPerByte)
        sc = (float)((double)sc / (double)c);
    return ((unsigned long long)(~__float_as_uint(sc)) << 32) | uid;
}

// Units that are not candidates: a zero statistic under the skip-zero
// option, and (tensor-level plans) tensors without elements, which have no
// block to select.
__device__ inline bool plan_skips(float S, unsigned long long c, uint32_t flags)
{
    return ((flags & kPlanSkipZero) && S == 0.0f) || c == 0ull;
}

// A unit's catalog statistic; the tensor-level plan (no block catalog,
// sumsq null) gives every unit 1, so it takes units by weight, then in uid
// order.
__device__ inline float plan_stat(const float* __restrict__ sumsq, uint32_t uid)
{
    return sumsq != nullptr ? sumsq[uid] : 1.0f;
}

// Wave-level resolution of one digit: h[256] holds the cost of the matching
// candidates per digit value.  Returns the smallest v with
// sum_{v' <= v} h[v'] > brem (v = -1 if the total fits), the cost below v,
// and the total.  Must be called by all 64 lanes of one wave.
__device__ inline void resolve_digit(const unsigned long long* h, unsigned long long brem, int lane,
                                     int* v_out, unsigned long long* below_out,
                                     unsigned long long* total_out)
{
    unsigned long long c[4];
    unsigned long long run = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        run += h[lane * 4 + q];
        c[q] = run;
    }
    unsigned long long incl = run;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const unsigned long long y = __shfl_up(incl, (unsigned)off);
        if (lane >= off)
            incl += y;
    }
    const unsigned long long excl = incl - run;
    const unsigned long long total = __shfl(incl, 63);
    int v = -1;
    unsigned long long below = 0;
    if (excl <= brem && incl > brem) {
        // c[] is non-decreasing and excl + c[3] > brem: q = first slot that overflows
        const unsigned long long room = brem - excl;
        const int q = (c[0] <= room) + (c[1] <= room) + (c[2] <= room);
        v = lane * 4 + q;
        below = excl + (q == 0 ? 0ull : (q == 1 ? c[0] : (q == 2 ? c[1] : c[2])));
    }
    // exactly one lane (or none) found the crossing
    const unsigned long long bal = __ballot(v >= 0);
    if (bal) {
        const int src = __ffsll((long long)bal) - 1;
        v = __shfl(v, src);
        below = __shfl(below, src);
    }
    *v_out = v;
    *below_out = below;
    *total_out = total;
}

constexpr int kInitGrid = (3 + kFirst) * kPlanBins / kT;  // one bin a thread
__global__ __launch_bounds__(kT) void k_plan_init(PlanCtl* ctl, unsigned long long budget)
{
    const int t = (int)blockIdx.x * kT + (int)threadIdx.x;
    static_assert(kPlanBins % kT == 0, "whole workgroups");
    if (t < 3 * kPlanBins)
        (&ctl->hist[0][0])[t] = 0ull;
    else
        (&ctl->first[0][0])[t - 3 * kPlanBins] = 0ull;
    if (t == 0) {
        ctl->brem[0] = budget;
        ctl->prefix[0] = 0ull;
        ctl->total0 = 0ull;
        ctl->sel_cost = 0ull;
        ctl->sel_count = 0ull;
        ctl->all_fit = 0u;
        ctl->done = 0u;
        ctl->list_n[0] = 0u;
        ctl->list_n[1] = 0u;
        ctl->error = 0u;
    }
}

// Exclusive prefix sum of x over the NT threads of a workgroup, and the
// total.  All threads call it; sw holds NT / 64 words.
template <int NT>
__device__ inline unsigned long long block_excl_sum(unsigned long long x, unsigned long long* sw,
                                                    unsigned long long* total)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    unsigned long long incl = x;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const unsigned long long y = __shfl_up(incl, (unsigned)off);
        if (lane >= off)
            incl += y;
    }
    __syncthreads();  // sw is free
    if (lane == 63)
        sw[wave] = incl;
    __syncthreads();
    unsigned long long before = 0ull, all = 0ull;
#pragma unroll
    for (int v = 0; v < NT / 64; ++v) {
        const unsigned long long y = sw[v];
        before += v < wave ? y : 0ull;
        all += y;
    }
    *total = all;
    return before + incl - x;
}

// Resolution of one digit by a kHistT-thread workgroup: h[kPlanBins] holds
// the cost of the matching candidates per digit value.  found: some v is the
// smallest with sum_{v' <= v} h[v'] > brem; below is the cost under it, total
// the whole histogram's.  Results through LDS; ends with a barrier.
struct Digit {
    unsigned long long below, total;
    int v;  // -1: the total fits
};
__device__ inline void block_resolve(const unsigned long long* __restrict__ h, unsigned long long brem,
                                     unsigned long long* sw, Digit* out, int copies = 1)
{
    constexpr int per = kPlanBins / kHistT;
    const int t = threadIdx.x;
    unsigned long long c[per], run = 0ull;
#pragma unroll
    for (int q = 0; q < per; ++q) {
        c[q] = h[t * per + q];
        run += c[q];
    }
    for (int y = 1; y < copies; ++y) {
#pragma unroll
        for (int q = 0; q < per; ++q) {
            const unsigned long long v = h[y * kPlanBins + t * per + q];
            c[q] += v;
            run += v;
        }
    }
    unsigned long long total;
    unsigned long long at = block_excl_sum<kHistT>(run, sw, &total);
    if (t == 0) {
        out->total = total;
        if (total <= brem)
            out->v = -1;
    }
    if (at <= brem && at + run > brem) {  // exactly one thread, if the total does not fit
        int v = t * per;
#pragma unroll
        for (int q = 0; q < per - 1; ++q) {
            if (v == t * per + q && at + c[q] <= brem) {
                at += c[q];
                ++v;
            }
        }
        out->v = v;
        out->below = at;
    }
    __syncthreads();
}

// Digit pass d of round 0 (key bits sh .. sh + wd - 1; the pass before took
// those from psh up): resolve the pass before (every workgroup does it
// redundantly from its histogram; workgroup 0 publishes it), then histogram
// this digit of the units matching the resolved prefix.  One thread per unit,
// kHistU units' loads in flight.  copies: those of pass 0's histogram.
__global__ __launch_bounds__(kHistT, 8) void k_plan_hist(PlanCtl* ctl, int d, int sh, int wd, int psh, int copies,
                                                      const float* __restrict__ sumsq, Coeffs w, uint32_t flags,
                                                      int K, const uint32_t* __restrict__ blen, uint32_t esize,
                                                      int64_t G)
{
    __shared__ unsigned long long lh[kPlanBins];
    __shared__ unsigned long long sw[kHistT / 64];
    __shared__ Digit dg;
    __shared__ float s_w[kMaxK];
    if (ctl->all_fit)
        return;
    const int t = threadIdx.x;
    if (t < K)
        s_w[t] = w.v[t];
#pragma unroll
    for (int q = 0; q < kPlanBins / kHistT; ++q)
        lh[q * kHistT + t] = 0ull;
    unsigned long long prefix = 0ull;
    if (d > 0) {
        const unsigned long long brem = ctl->brem[d - 1];
        block_resolve(d == 1 ? ctl->first[0] : ctl->hist[(d - 1) % 3], brem, sw, &dg, d == 1 ? copies : 1);
        if (dg.v < 0) {  // digit 0: every candidate fits; later digits: cannot happen
            if (blockIdx.x == 0 && t == 0) {
                if (d == 1) {
                    ctl->total0 = dg.total;
                    ctl->all_fit = 1u;
                } else {
                    ctl->error = 3u;
                }
            }
            return;
        }
        prefix = ctl->prefix[d - 1] | ((unsigned long long)dg.v << psh);
        if (blockIdx.x == 0) {
            if (t == 0) {
                ctl->prefix[d] = prefix;
                ctl->brem[d] = brem - dg.below;
            }
            unsigned long long* hn = ctl->hist[(d + 1) % 3];
            for (int q = t; q < kPlanBins; q += kHistT)
                hn[q] = 0ull;
        }
    } else {
        __syncthreads();
    }
    const int64_t n = G * K, step = (int64_t)gridDim.x * kHistT;
    const unsigned long long dm = (1ull << wd) - 1ull;
    for (int64_t u0 = (int64_t)blockIdx.x * kHistT + t; u0 < n; u0 += kHistU * step) {
        float S[kHistU];
        uint32_t len[kHistU], ex[kHistU];
#pragma unroll
        for (int q = 0; q < kHistU; ++q) {
            const int64_t u = u0 + q * step;
            const uint32_t uid = (uint32_t)(u < n ? u : 0);
            const uint32_t g = uid / (uint32_t)K;
            ex[q] = uid - g * (uint32_t)K;
            S[q] = plan_stat(sumsq, uid);
            len[q] = blen[g];
        }
#pragma unroll
        for (int q = 0; q < kHistU; ++q) {
            const int64_t u = u0 + q * step;
            const unsigned long long c = (unsigned long long)len[q] * esize;
            if (u >= n || plan_skips(S[q], c, flags))
                continue;
            const unsigned long long key = unit_key(S[q], s_w[ex[q]], (uint32_t)u, c, flags);
            if (d == 0 || ((key ^ prefix) >> (sh + wd)) == 0)
                atomicAdd(&lh[(key >> sh) & dm], c);
        }
    }
    __syncthreads();
    unsigned long long* out = d == 0 ? ctl->first[blockIdx.x % (unsigned)copies] : ctl->hist[d % 3];
#pragma unroll
    for (int q = 0; q < kPlanBins / kHistT; ++q) {
        const unsigned long long v = lh[q * kHistT + t];
        if (v)
            atomicAdd(&out[q * kHistT + t], v);
    }
}

// After the last digit pass d (key bits from sh up): resolve its digit; the
// cut key p is among the 2^sh uids (kMarkUids at most) that share all bits
// above, found by a prefix sum of their costs in uid order.  Then mark:
// select the candidates below the cut and list the next round's (above p, and
// not dearer than what is left).  In the all-fit case select every candidate.
// Per workgroup: the selected cost and count, and the mask's digest terms.
constexpr int kMarkBits = 12, kMarkUids = 1 << kMarkBits;
__global__ __launch_bounds__(kHistT, 8) void k_plan_mark(PlanCtl* ctl, int d, int sh, const float* __restrict__ sumsq,
                                                      Coeffs w, uint32_t flags, int K,
                                                      const uint32_t* __restrict__ blen, uint32_t esize, int64_t G,
                                                      uint32_t* __restrict__ mask, uint32_t* __restrict__ next,
                                                      unsigned int* __restrict__ next_n, unsigned int next_cap)
{
    __shared__ unsigned long long sw[kHistT / 64];
    __shared__ Digit dg;
    __shared__ unsigned long long s_keyp, s_rem;
    __shared__ unsigned long long s_sum[3][kHistT / 64];
    __shared__ float s_w[kMaxK];
    __shared__ uint32_t s_len[kMarkUids];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    if (t < K)
        s_w[t] = w.v[t];
    const bool all = ctl->all_fit != 0u;
    unsigned long long keyp = 0ull, rem = 0ull;
    bool ok = true;
    if (!all) {
        if (t == 0) {
            s_keyp = ~0ull;
            s_rem = 0ull;
        }
        block_resolve(ctl->hist[d % 3], ctl->brem[d], sw, &dg);
        ok = dg.v >= 0;
        if (ok) {
            const unsigned long long pre = ctl->prefix[d] | ((unsigned long long)dg.v << sh);
            const unsigned long long left = ctl->brem[d] - dg.below;
            unsigned long long run = 0ull;
            const int64_t n = G * K;
            const int m = 1 << sh, per_t = (m + kHistT - 1) / kHistT;
#pragma unroll 4
            for (int q = 0; q < per_t; ++q) {
                const int j = t * per_t + q;
                const int64_t u = (int64_t)(uint32_t)pre + j;
                uint32_t len = 0u;  // stays 0 where the uid is no candidate
                if (j < m && u < n) {
                    const uint32_t g = (uint32_t)u / (uint32_t)K, bl = blen[g];
                    const unsigned long long cc = (unsigned long long)bl * esize;
                    const float S = plan_stat(sumsq, (uint32_t)u);
                    if (!plan_skips(S, cc, flags) &&
                        unit_key(S, s_w[(uint32_t)u - g * (uint32_t)K], (uint32_t)u, cc, flags) == pre + (unsigned)j)
                        len = bl;
                }
                if (j < m)
                    s_len[j] = len;
                run += (unsigned long long)len * esize;
            }
            unsigned long long total;
            unsigned long long at = block_excl_sum<kHistT>(run, sw, &total);
            if (at <= left && at + run > left) {  // exactly one thread
                int q = t * per_t;
                for (; at + (unsigned long long)s_len[q] * esize <= left; ++q)  // ends: the run passes what is left
                    at += (unsigned long long)s_len[q] * esize;
                s_keyp = pre + (unsigned)q;
                s_rem = left - at;
            }
        }
        __syncthreads();
        keyp = s_keyp;
        rem = s_rem;
        if (keyp == ~0ull)
            ok = false;  // cannot happen: the cut is a real unit (a full uid with a NaN-free score is not all ones)
        if (!ok)
            keyp = 0ull;  // select nothing
        if (blockIdx.x == 0 && t == 0) {
            if (!ok)
                ctl->error = 1u;
            ctl->prefix[8] = keyp;
            ctl->brem[8] = rem;
        }
    } else {
        __syncthreads();
    }
    unsigned long long my_cost = 0ull, my_cnt = 0ull, my_dig = 0ull;
    for (int64_t g = (int64_t)blockIdx.x * kHistT + t; g < G; g += (int64_t)gridDim.x * kHistT) {
        const unsigned long long c = (unsigned long long)blen[g] * esize;
        uint32_t word = 0u;
        for (int i = 0; i < K; ++i) {
            const uint32_t uid = (uint32_t)(g * K + i);
            const float S = plan_stat(sumsq, uid);
            if (plan_skips(S, c, flags))
                continue;
            const unsigned long long key = unit_key(S, s_w[i], uid, c, flags);
            if (all || key < keyp) {
                word |= 1u << i;
                my_cost += c;
                my_cnt += 1;
            } else if (key > keyp && c <= rem) {
                const unsigned int slot = atomicAdd(next_n, 1u);
                if (slot < next_cap)
                    next[slot] = uid;
                else
                    ctl->error = 2u;
            }
        }
        mask[g] = word;
        my_dig += mix64(((unsigned long long)g << 32) | word);
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        my_cost += __shfl_xor(my_cost, off);
        my_cnt += __shfl_xor(my_cnt, off);
        my_dig += __shfl_xor(my_dig, off);
    }
    if (lane == 0) {
        s_sum[0][wave] = my_cost;
        s_sum[1][wave] = my_cnt;
        s_sum[2][wave] = my_dig;
    }
    __syncthreads();
    if (t < 3) {
        unsigned long long v = 0ull;
#pragma unroll
        for (int q = 0; q < kHistT / 64; ++q)
            v += s_sum[t][q];
        ctl->part[t][blockIdx.x] = v;
    }
}

// Sum of part[row][0 .. n) over one 256-thread workgroup (all threads call
// it; every thread gets the sum).  The loads are issued together.
__device__ inline unsigned long long block_sum_parts(const PlanCtl* ctl, int row, int n)
{
    __shared__ unsigned long long s[4];
    const int t = threadIdx.x;
    unsigned long long a = 0ull;
#pragma unroll
    for (int j = 0; j < (kPlanGrid + kT - 1) / kT; ++j) {
        const int q = j * kT + t;
        a += (q < n) ? ctl->part[row][q] : 0ull;
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1)
        a += __shfl_xor(a, off);
    __syncthreads();
    if ((t & 63) == 0)
        s[t >> 6] = a;
    __syncthreads();
    return s[0] + s[1] + s[2] + s[3];
}

// Close round 0: carry the remaining budget and
// finish the plan when everything fit or no cheaper candidate is left.
__global__ __launch_bounds__(kT) void k_plan_advance(PlanCtl* ctl, int next_list, int reuse_list, int n_part)
{
    // takes in the selections of k_plan_mark's n_part workgroups
    const int t = threadIdx.x;
    const unsigned long long cs = block_sum_parts(ctl, 0, n_part);
    const unsigned long long cn = block_sum_parts(ctl, 1, n_part);
    if (t != 0)
        return;
    ctl->sel_cost += cs;
    ctl->sel_count += cn;
    unsigned long long rem;
    if (ctl->all_fit) {
        rem = ctl->brem[0] - ctl->total0;
        ctl->done = 1u;
    } else {
        rem = ctl->brem[8];
        if (ctl->list_n[next_list] == 0u)
            ctl->done = 1u;
    }
    ctl->brem[0] = rem;
    ctl->prefix[0] = 0ull;
    ctl->all_fit = 0u;
    ctl->list_n[reuse_list] = 0u;
}

// Rounds r_begin .. r_end-1 (the later rounds, whose candidates are the
// short lists left by the round before) in one workgroup: the same digit
// passes, cut and selection as k_plan_hist / k_plan_mark / k_plan_advance,
// with the round state in LDS and barriers instead of launches.
__device__ inline uint32_t plan_list_load(const uint32_t* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__global__ __launch_bounds__(kT) void k_plan_rest(PlanCtl* ctl, const float* __restrict__ sumsq, Coeffs w,
                                                  uint32_t flags, int K,
                                                  const uint32_t* __restrict__ blen, uint32_t esize, int64_t G,
                                                  uint32_t* list0, uint32_t* list1, unsigned int cap,
                                                  uint32_t* __restrict__ mask, int r_begin, int r_end)
{
    __shared__ unsigned long long lh[256];
    __shared__ unsigned long long s_brem0, s_below, s_total;
    __shared__ unsigned long long s_cost[4], s_cnt[4];
    __shared__ unsigned int s_n, s_next_n, s_err;
    __shared__ int s_v, s_done;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    if (t == 0) {
        s_done = (int)ctl->done;
        s_brem0 = ctl->brem[0];
        s_n = ctl->list_n[r_begin & 1];
        s_err = 0u;
    }
    unsigned long long sel_cost = 0ull, sel_cnt = 0ull;  // this thread's selections
    for (int r = r_begin; r < r_end; ++r) {
        __syncthreads();
        if (s_done)
            break;
        const uint32_t* list = (r & 1) ? list1 : list0;
        uint32_t* next = (r & 1) ? list0 : list1;
        const unsigned int n = min(s_n, cap);
        const unsigned long long brem0 = s_brem0;
        unsigned long long prefix = 0ull, brem = brem0, total0 = 0ull;
        bool all = false;
        for (int d = 0; d < 8; ++d) {
            lh[t] = 0ull;
            if (t == 0)
                s_next_n = 0u;
            __syncthreads();
            const int hi_shift = 64 - 8 * d, dg_shift = 56 - 8 * d;
            for (unsigned int q = t; q < n; q += kT) {
                const uint32_t uid = plan_list_load(&list[q]);
                const uint32_t g = uid / (uint32_t)K, i = uid % (uint32_t)K;
                const unsigned long long c = (unsigned long long)blen[g] * esize;
                const unsigned long long key = unit_key(plan_stat(sumsq, uid), w.v[i], uid, c, flags);
                if (d == 0 || ((key ^ prefix) >> hi_shift) == 0)
                    atomicAdd(&lh[(key >> dg_shift) & 255u], c);
            }
            __syncthreads();
            if (wave == 0) {
                int v;
                unsigned long long below, total;
                resolve_digit(lh, brem, lane, &v, &below, &total);
                if (lane == 0) {
                    s_v = v;
                    s_below = below;
                    s_total = total;
                }
            }
            __syncthreads();
            const int v = s_v;
            if (v < 0) {  // digit 0: every candidate fits; later digits: cannot happen
                if (d == 0) {
                    all = true;
                    total0 = s_total;
                } else if (t == 0) {
                    s_err = 3u;
                }
                break;
            }
            prefix |= (unsigned long long)v << (56 - 8 * d);
            brem -= s_below;
        }
        // the cut key p = prefix; select below it, keep the cheaper ones above
        unsigned long long cp = 0ull;
        bool cut_ok = true;
        if (!all) {
            const uint32_t gp = (uint32_t)prefix / (uint32_t)K;
            if ((int64_t)gp >= G) {  // cannot happen: the cut is a real unit
                cut_ok = false;
                if (t == 0)
                    s_err = 1u;
            } else {
                cp = (unsigned long long)blen[gp] * esize;
            }
        }
        if (all || cut_ok) {
            for (unsigned int q = t; q < n; q += kT) {
                const uint32_t uid = plan_list_load(&list[q]);
                const uint32_t g = uid / (uint32_t)K, i = uid % (uint32_t)K;
                const unsigned long long c = (unsigned long long)blen[g] * esize;
                const unsigned long long key = unit_key(plan_stat(sumsq, uid), w.v[i], uid, c, flags);
                if (all || key < prefix) {
                    atomicOr(&mask[g], 1u << i);
                    sel_cost += c;
                    sel_cnt += 1;
                } else if (key > prefix && c < cp) {
                    const unsigned int slot = atomicAdd(&s_next_n, 1u);
                    if (slot < cap)
                        next[slot] = uid;
                    else
                        s_err = 2u;
                }
            }
        }
        __threadfence();  // the next list is in memory before the next round reads it
        __syncthreads();
        if (t == 0) {
            s_brem0 = all ? brem0 - total0 : brem;
            s_done = (all || !cut_ok || s_next_n == 0u) ? 1 : 0;
            s_n = s_next_n;
        }
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        sel_cost += __shfl_xor(sel_cost, off);
        sel_cnt += __shfl_xor(sel_cnt, off);
    }
    __syncthreads();
    if (lane == 0) {
        s_cost[wave] = sel_cost;
        s_cnt[wave] = sel_cnt;
    }
    __syncthreads();
    if (t == 0) {
        const unsigned long long cs = s_cost[0] + s_cost[1] + s_cost[2] + s_cost[3];
        const unsigned long long cn = s_cnt[0] + s_cnt[1] + s_cnt[2] + s_cnt[3];
        if (cn) {
            atomicAdd(&ctl->sel_cost, cs);
            atomicAdd(&ctl->sel_count, cn);
        }
        if (s_err)
            ctl->error = s_err;
        ctl->done = 1u;
    }
}

// The plan's rounds in one workgroup with keys and costs in registers (at most
// kOneMax candidates).  ALL: every unit, from the start (mask and digest from
// LDS words).  Otherwise the rounds after round 0 over the list that
// k_plan_mark left; they change the digest word by word.  Per round: drop the
// candidates dearer than what is left (they can never be taken), take all if
// they fit, else find the cut digit by digit, stopping as soon as a single
// candidate matches, take what lies below it and go on with what lies above.
// Both write the stats: with tensor_level only the selection goes to ctl (the
// stats are closed over the expanded mask).
constexpr int kOneMax = 8192;

// NT threads of PER candidates each.  A round is a chain of barriers, cheaper
// the fewer waves there are: up to 1024 candidates take four waves (1.5M units'
// later rounds 15 us, 21 with sixteen; a plan of 256 / 1,000 units 33 / 27 us, 41 /
// 30 with sixteen), held to 64 registers (see the top).
template <bool ALL, int NT, int PER>
__global__ __launch_bounds__(NT, NT == 256 ? 8 : 1) void k_plan_one(PlanCtl* ctl, const float* __restrict__ sumsq, Coeffs w,
                                                    uint32_t flags, int K, const uint32_t* __restrict__ blen,
                                                    uint32_t esize, int64_t G, const uint32_t* __restrict__ list,
                                                    const unsigned int* __restrict__ list_n, unsigned int cap,
                                                    uint32_t* __restrict__ mask, int n_part,
                                                    unsigned long long budget, unsigned long long full,
                                                    unsigned long long n_units, bool tensor_level,
                                                    unsigned long long* __restrict__ stats)
{
    __shared__ unsigned long long lh[256];
    __shared__ unsigned long long sw[NT / 64];
    __shared__ unsigned long long s_below, s_total, s_key;
    __shared__ int s_v;
    __shared__ float s_w[kMaxK];
    __shared__ uint32_t s_mask[ALL ? NT * PER : 1];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    unsigned long long rem = budget, err = 0ull, cost = 0ull, cnt = 0ull, dig = 0ull;  // this thread's, summed at the end
    bool rounds = true;
    uint32_t n;
    if (ALL) {
        n = (uint32_t)(G * K);
        for (int64_t g = t; g < G; g += NT)
            s_mask[g] = 0u;
    } else {
        for (int q = t; q < n_part; q += NT) {
            cost += ctl->part[0][q];
            cnt += ctl->part[1][q];
            dig += ctl->part[2][q];
        }
        const bool all = ctl->all_fit != 0u;
        err = ctl->error;
        rem = ctl->brem[8];
        n = min(*list_n, cap);
        rounds = !all && err == 0ull && n <= (uint32_t)(NT * PER);
    }
    if (t < K)
        s_w[t] = w.v[t];
    __syncthreads();
    unsigned long long key[PER], c[PER];
    uint32_t alive = 0u;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const uint32_t j = (uint32_t)(q * NT + t);
        key[q] = 0ull;
        c[q] = 0ull;
        if (rounds && j < n) {
            const uint32_t uid = ALL ? j : list[j];
            const uint32_t g = uid / (uint32_t)K;
            const float S = plan_stat(sumsq, uid);
            c[q] = (unsigned long long)blen[g] * esize;
            key[q] = unit_key(S, s_w[uid - g * (uint32_t)K], uid, c[q], flags);
            if (!ALL || !plan_skips(S, c[q], flags))  // listed units are candidates already
                alive |= 1u << q;
        }
    }
    // candidates taken: noted, and written after the rounds, off their chain
    // (ALL: at once, in LDS)
    uint32_t taken = 0u;
    auto take = [&](int q) {
        const uint32_t uid = (uint32_t)key[q], g = uid / (uint32_t)K, bit = 1u << (uid - g * (uint32_t)K);
        cost += c[q];
        cnt += 1ull;
        if (ALL) {
            atomicOr(&s_mask[g], bit);
        } else {
            const uint32_t old = atomicOr(&mask[g], bit);
            dig += mix64(((unsigned long long)g << 32) | (old | bit)) - mix64(((unsigned long long)g << 32) | old);
        }
    };
    auto note = [&](int q) {
        if constexpr (ALL)
            take(q);
        else
            taken |= 1u << q;
    };
    for (;;) {
        unsigned long long mine = 0ull, total;
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            if (((alive >> q) & 1u) && c[q] > rem)
                alive &= ~(1u << q);
            mine += ((alive >> q) & 1u) ? c[q] : 0ull;
        }
        (void)block_excl_sum<NT>(mine, sw, &total);
        if (total <= rem) {  // everything fits (or nothing is left)
#pragma unroll
            for (int q = 0; q < PER; ++q)
                if ((alive >> q) & 1u)
                    note(q);
            break;
        }
        unsigned long long prefix = 0ull, brem = rem;
        bool bad = false;
        uint32_t match = alive;  // candidates that match the prefix
        for (int d = 0; d < 8; ++d) {
            __syncthreads();
            if (t < 256)
                lh[t] = 0ull;
            __syncthreads();
            const int sh = 56 - 8 * d;
#pragma unroll
            for (int q = 0; q < PER; ++q)
                if ((match >> q) & 1u)
                    atomicAdd(&lh[(key[q] >> sh) & 255u], c[q]);
            __syncthreads();
            if (wave == 0) {
                int v;
                unsigned long long below, tot;
                resolve_digit(lh, brem, lane, &v, &below, &tot);
                if (lane == 0) {
                    s_v = v;
                    s_below = below;
                }
            }
            __syncthreads();
            if (s_v < 0) {  // cannot happen: the total passes the budget
                bad = true;
                break;
            }
            brem -= s_below;
            prefix |= (unsigned long long)s_v << sh;
#pragma unroll
            for (int q = 0; q < PER; ++q)
                if (((match >> q) & 1u) && ((key[q] ^ prefix) >> sh) != 0ull)
                    match &= ~(1u << q);
            if (__syncthreads_or(__popc(match) > 1) == 0 && __syncthreads_count(match != 0u) == 1) {
                // one candidate is left: it is the cut
#pragma unroll
                for (int q = 0; q < PER; ++q)
                    if ((match >> q) & 1u)
                        s_key = key[q];
                __syncthreads();
                prefix = s_key;
                break;
            }
        }
        if (bad) {
            err = 3ull;
            break;
        }
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            if (((alive >> q) & 1u) && key[q] <= prefix) {
                if (key[q] < prefix)
                    note(q);
                alive &= ~(1u << q);
            }
        }
        rem = brem;
    }
    if constexpr (!ALL) {
#pragma unroll
        for (int q = 0; q < PER; ++q)
            if ((taken >> q) & 1u)
                take(q);
    }
    __syncthreads();
    if (ALL) {
        for (int64_t g = t; g < G; g += NT) {
            const uint32_t m = s_mask[g];
            mask[g] = m;
            dig += mix64(((unsigned long long)g << 32) | m);
        }
    }
    unsigned long long tc, tn, td;
    (void)block_excl_sum<NT>(cost, sw, &tc);
    (void)block_excl_sum<NT>(cnt, sw, &tn);
    (void)block_excl_sum<NT>(dig, sw, &td);
    if (t != 0)
        return;
    if (tensor_level) {
        ctl->sel_cost = tc;
        ctl->error = (unsigned int)err;
        return;
    }
    stats[0] = budget;
    stats[1] = tc;
    stats[2] = full;
    stats[3] = tn;
    stats[4] = n_units;
    stats[5] = mix64(td ^ tc);
    stats[6] = err;
}

__global__ __launch_bounds__(kT) void k_plan_digest(PlanCtl* ctl, const uint32_t* __restrict__ mask, int64_t G)
{
    __shared__ unsigned long long s[4];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    unsigned long long acc = 0ull;
    for (int64_t g = (int64_t)blockIdx.x * kT + t; g < G; g += (int64_t)gridDim.x * kT)
        acc += mix64(((unsigned long long)g << 32) | mask[g]);
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1)
        acc += __shfl_xor(acc, off);
    if (lane == 0)
        s[wave] = acc;
    __syncthreads();
    if (t == 0)
        ctl->part[2][blockIdx.x] = s[0] + s[1] + s[2] + s[3];
}

__global__ __launch_bounds__(kT) void k_plan_final(PlanCtl* ctl, unsigned long long budget, unsigned long long full,
                                                   unsigned long long n_units, int n_part,
                                                  unsigned long long* __restrict__ stats)
{
    // takes in the digest terms of k_plan_digest's n_part workgroups
    const unsigned long long dg = block_sum_parts(ctl, 2, n_part);
    if (threadIdx.x != 0)
        return;
    stats[0] = budget;
    stats[1] = ctl->sel_cost;
    stats[2] = full;
    stats[3] = ctl->sel_count;
    stats[4] = n_units;
    stats[5] = mix64(dg ^ ctl->sel_cost);
    stats[6] = ctl->error;
}

}  // namespace

namespace {

// What a plan runs on: control block ctl, two candidate lists of cap uids each,
// G "blocks" with lengths blen[G] (elements); `rounds` bounds the number of
// rounds (the distinct lengths, or any larger number: the later rounds stop
// once the plan is done).
struct PlanIn {
    PlanCtl* ctl;
    uint32_t *list0, *list1;
    unsigned cap;
    const uint32_t* blen;
    uint32_t es;
    int64_t G;
    int rounds, K;
    const float* sumsq;
    Coeffs w;
    uint32_t flags;
    uint64_t budget, full;
    uint32_t* mask;
};

// Algorithm 1's selection; returns whether the stats are closed (written to
// `stats`, device-visible; never at tensor level).  Otherwise mask[G] is
// written, the selected cost is in ctl, and one of the finals below closes.
bool enqueue_select(const PlanIn& p, bool tensor_level, unsigned long long* stats, hipStream_t s)
{
    PlanCtl* ctl = p.ctl;
    const int64_t n = p.G * p.K;
    const unsigned long long budget = p.budget, full = p.full;
    if (n <= kOneMax) {
        auto one = [&](auto kern, int nt) {
            hipLaunchKernelGGL(kern, dim3(1), dim3(nt), 0, s, ctl, p.sumsq, p.w, p.flags, p.K, p.blen, p.es, p.G,
                               nullptr, nullptr, 0u, p.mask, 0, budget, full, (unsigned long long)n, tensor_level,
                               stats);
        };
        if (n <= 1024)
            one(k_plan_one<true, 256, 4>, 256);
        else
            n <= 4096 ? one(k_plan_one<true, 1024, 4>, 1024) : one(k_plan_one<true, 1024, 8>, 1024);
        return !tensor_level;
    }
    hipLaunchKernelGGL(k_plan_init, dim3(kInitGrid), dim3(kT), 0, s, ctl, budget);
    // round 0 over every unit; its candidates for round 1 go to list1.  The
    // score's digits, then the uid's until at most kMarkBits are open
    int bits = 0;
    while (bits < 32 && (n - 1) >> bits)
        ++bits;
    int d = 0, psh = 0;
    const int64_t per_wg = kHistT * kHistU;
    const int64_t hgrid = std::min<int64_t>((n + per_wg - 1) / per_wg, n <= ((int64_t)1 << 23) ? 512 : 1024);
    const int copies = hgrid > 64 ? kFirst : 1;  // few workgroups: reading the copies costs more
    auto pass = [&](int sh, int wd) {
        hipLaunchKernelGGL(k_plan_hist, dim3((unsigned)hgrid), dim3(kHistT), 0, s, ctl, d, sh, wd, psh, copies, p.sumsq,
                           p.w, p.flags, p.K, p.blen, p.es, p.G);
        psh = sh;
        ++d;
    };
    pass(53, 11);
    pass(42, 11);
    pass(32, 10);
    for (int open = bits; open > kMarkBits;) {
        const int wd = std::min(open, 11);
        open -= wd;
        pass(open, wd);
    }
    static_assert(kOneMax >= kMarkUids, "more than kOneMax units: a uid pass has run");
    const unsigned mgrid = (unsigned)std::min<int64_t>((p.G + kHistT - 1) / kHistT, kPlanGrid);
    hipLaunchKernelGGL(k_plan_mark, dim3(mgrid), dim3(kHistT), 0, s, ctl, d - 1, psh, p.sumsq, p.w, p.flags, p.K,
                       p.blen, p.es, p.G, p.mask, p.list1, &ctl->list_n[1], p.cap);
    if (!tensor_level && p.cap <= (unsigned)kOneMax) {
        auto one = [&](auto kern, int nt) {
            hipLaunchKernelGGL(kern, dim3(1), dim3(nt), 0, s, ctl, p.sumsq, p.w, p.flags, p.K, p.blen, p.es, p.G,
                               p.list1, &ctl->list_n[1], p.cap, p.mask, (int)mgrid, budget, full,
                               (unsigned long long)n, false, stats);
        };
        p.cap <= 1024u ? one(k_plan_one<false, 256, 4>, 256) : one(k_plan_one<false, 1024, 8>, 1024);
        return true;
    }
    // longer lists: reloaded in each pass
    hipLaunchKernelGGL(k_plan_advance, dim3(1), dim3(kT), 0, s, ctl, 1, 0, (int)mgrid);
    if (p.rounds > 1)
        hipLaunchKernelGGL(k_plan_rest, dim3(1), dim3(kT), 0, s, ctl, p.sumsq, p.w, p.flags, p.K, p.blen, p.es, p.G,
                           p.list0, p.list1, p.cap, p.mask, 1, p.rounds);
    return false;
}

// Block-level plan: the selection, then (where it has not closed them) the
// stats over mask[G], left in `stats`.
hipError_t enqueue_block_plan(const PlanIn& p, unsigned long long* stats, hipStream_t s)
{
    if (!enqueue_select(p, false, stats, s)) {
        const int n_digest = (int)std::min<int64_t>((p.G + kT - 1) / kT, kPlanGrid);
        hipLaunchKernelGGL(k_plan_digest, dim3((unsigned)n_digest), dim3(kT), 0, s, p.ctl, p.mask, p.G);
        hipLaunchKernelGGL(k_plan_final, dim3(1), dim3(kT), 0, s, p.ctl, (unsigned long long)p.budget,
                           (unsigned long long)p.full, (unsigned long long)(p.G * p.K), n_digest, stats);
    }
    return hipGetLastError();
}

// Tensor-level plan: block g takes the selection word of its tensor t, the
// last one with g0[t] <= g (tensors without elements have no blocks); per
// workgroup, the selected block units and the digest terms.
__global__ __launch_bounds__(kT) void k_plan_expand(PlanCtl* ctl, const uint32_t* __restrict__ tmask,
                                                    const uint32_t* __restrict__ g0, int T, int64_t G,
                                                    uint32_t* __restrict__ mask)
{
    __shared__ unsigned long long s_c[4], s_d[4];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    unsigned long long cnt = 0ull, dg = 0ull;
    for (int64_t g = (int64_t)blockIdx.x * kT + t; g < G; g += (int64_t)gridDim.x * kT) {
        int lo = 0, hi = T - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if ((int64_t)g0[mid] <= g)
                lo = mid;
            else
                hi = mid - 1;
        }
        const uint32_t m = tmask[lo];
        mask[g] = m;
        cnt += (unsigned long long)__popc(m);
        dg += mix64(((unsigned long long)g << 32) | m);
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        cnt += __shfl_xor(cnt, off);
        dg += __shfl_xor(dg, off);
    }
    if (lane == 0) {
        s_c[wave] = cnt;
        s_d[wave] = dg;
    }
    __syncthreads();
    if (t == 0) {
        ctl->part[1][blockIdx.x] = s_c[0] + s_c[1] + s_c[2] + s_c[3];
        ctl->part[2][blockIdx.x] = s_d[0] + s_d[1] + s_d[2] + s_d[3];
    }
}

__global__ __launch_bounds__(kT) void k_plan_final_tensors(PlanCtl* ctl, unsigned long long budget,
                                                           unsigned long long full, unsigned long long n_units,
                                                           int n_part, unsigned long long* __restrict__ stats)
{
    const unsigned long long cn = block_sum_parts(ctl, 1, n_part);
    const unsigned long long dg = block_sum_parts(ctl, 2, n_part);
    if (threadIdx.x != 0)
        return;
    stats[0] = budget;
    stats[1] = ctl->sel_cost;
    stats[2] = full;
    stats[3] = cn;
    stats[4] = n_units;
    stats[5] = mix64(dg ^ ctl->sel_cost);
    stats[6] = ctl->error;
}

// Tensor-level plan: p's blocks are the n_tensors tensors and p.mask their
// selection words; expands those to mask[G], counts and digests it.
hipError_t enqueue_tensor_plan(const PlanIn& p, const uint32_t* g0, int T, int64_t G, uint32_t* mask,
                               unsigned long long* stats, hipStream_t s)
{
    (void)enqueue_select(p, true, stats, s);
    const int n_part = G > 0 ? (int)std::min<int64_t>((G + kT - 1) / kT, kPlanGrid) : 0;
    if (G > 0)
        hipLaunchKernelGGL(k_plan_expand, dim3((unsigned)n_part), dim3(kT), 0, s, p.ctl, p.mask, g0, T, G, mask);
    hipLaunchKernelGGL(k_plan_final_tensors, dim3(1), dim3(kT), 0, s, p.ctl, (unsigned long long)p.budget,
                       (unsigned long long)p.full, (unsigned long long)(G * p.K), n_part, stats);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_plan(const BlockTable& bt, PlanScratch& ps, int K, const float* sumsq,
                       const Coeffs& w, uint32_t flags, uint64_t budget, uint64_t full_bytes, uint32_t* mask,
                       hipStream_t s)
{
    // the stats go straight to the pinned words the caller reads after its
    // synchronisation: no copy behind the last kernel
    unsigned long long* stats = nullptr;
    hipError_t e = hipHostGetDevicePointer((void**)&stats, ps.h_stats, 0);
    if (e != hipSuccess)
        return e;
    const int64_t per_k = std::max<int64_t>(sumsq != nullptr ? bt.n_short : bt.n_tensors, 1);
    const unsigned cap = (unsigned)std::min<int64_t>(ps.list_cap, per_k * K);  // what this layout can list
    PlanIn p{ps.ctl, ps.list[0], ps.list[1], cap, bt.d_len, (uint32_t)bt.esize, bt.G,
             bt.n_distinct_len, K, sumsq, w, flags, budget, full_bytes, mask};
    if (sumsq != nullptr)
        return enqueue_block_plan(p, stats, s);
    // no block catalog: the tensor-level plan, each tensor one unit per expert
    p.blen = bt.d_tlen;
    p.G = bt.n_tensors;
    p.rounds = bt.n_distinct_tlen;
    p.mask = ps.tmask;
    return enqueue_tensor_plan(p, bt.d_g0, (int)bt.n_tensors, bt.G, mask, stats, s);
}

// ---------------------------------------------------------------- plan without allocation
// The plan on a fixed device array instead of the cached workspace and
// block table: for callers that cannot allocate device memory.  The array
// holds, each at a 256-byte boundary: the control block, the layout's
// tensor sizes, the first block of every tensor, the block lengths and the
// two candidate lists.  Every call on a device shares that device's copy,
// and each call rebuilds everything it reads from it.
namespace {

// The limit that layouts are held to, with kCtlCounted bytes of it for the
// control block; what the block takes beyond those is added to the array.
constexpr size_t kStaticPlanLimit = size_t(16) << 20, kCtlCounted = 18688;
constexpr size_t kCtlBytes = (sizeof(PlanCtl) + 255) & ~size_t(255);
static_assert(kCtlBytes >= kCtlCounted, "the control block's counted part");
constexpr size_t kStaticPlanBytes = kStaticPlanLimit + kCtlBytes - kCtlCounted;

static __device__ __align__(256) unsigned char scratch[kStaticPlanBytes];

// The address of `scratch` on each device (0 until the first call there).
constexpr int kMaxDevices = 64;
void* g_scratch_dev[kMaxDevices] = {};

size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

// One workgroup: g0[t] = first block of tensor t (blocks of the tensors
// before it), g0[T] = G; tlen[t] = elements of tensor t (below 2^32, checked
// by the host when the tensor-level plan needs them).
__global__ __launch_bounds__(kT) void k_static_g0(const int64_t* __restrict__ numel, int T, int64_t be,
                                                  uint32_t* __restrict__ g0, uint32_t* __restrict__ tlen)
{
    __shared__ unsigned long long s_w[kT / 64];
    __shared__ unsigned long long s_run;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    if (t == 0)
        s_run = 0ull;
    for (int base = 0; base < T; base += kT) {
        const int q = base + t;
        const unsigned long long nb = (q < T) ? (unsigned long long)((numel[q] + be - 1) / be) : 0ull;
        unsigned long long incl = nb;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const unsigned long long y = __shfl_up(incl, (unsigned)off);
            if (lane >= off)
                incl += y;
        }
        __syncthreads();  // s_run of the previous chunk is final; s_w is free
        if (lane == 63)
            s_w[wave] = incl;
        __syncthreads();
        unsigned long long before = s_run;
        for (int v = 0; v < wave; ++v)
            before += s_w[v];
        if (q < T) {
            g0[q] = (uint32_t)(before + incl - nb);
            tlen[q] = (uint32_t)numel[q];
        }
        __syncthreads();
        if (t == kT - 1)
            s_run = before + incl;
    }
    __syncthreads();
    if (t == 0)
        g0[T] = (uint32_t)s_run;
}

// blen[g] = elements of block g: the tensor t holding g is the last one
// with g0[t] <= g (tensors without elements have no blocks).
__global__ __launch_bounds__(kT) void k_static_blen(const int64_t* __restrict__ numel, const uint32_t* __restrict__ g0,
                                                    int T, int64_t be, int64_t G, uint32_t* __restrict__ blen)
{
    const int64_t g = (int64_t)blockIdx.x * kT + threadIdx.x;
    if (g >= G)
        return;
    int lo = 0, hi = T - 1;  // g0[lo] <= g holds for lo = 0
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if ((int64_t)g0[mid] <= g)
            lo = mid;
        else
            hi = mid - 1;
    }
    const int64_t left = numel[lo] - (g - (int64_t)g0[lo]) * be;
    blen[g] = (uint32_t)(left < be ? left : be);
}

}  // namespace

// Sizes of the parts of the fixed array a layout needs; the candidate lists
// hold K units per tensor, which covers both plans (a block-level plan's
// later rounds list only units of short blocks, at most one per tensor).
namespace {
struct StaticParts {
    size_t ctl, numel, g0, tlen, tmask, blen, list;
};
StaticParts static_parts(int64_t n_tensors, int64_t G, int K)
{
    const int64_t cap = (int64_t)K * std::max<int64_t>(n_tensors, 1);
    return {align256(sizeof(PlanCtl)), align256(sizeof(int64_t) * (size_t)n_tensors),
            align256(sizeof(uint32_t) * (size_t)(n_tensors + 1)), align256(sizeof(uint32_t) * (size_t)n_tensors),
            align256(sizeof(uint32_t) * (size_t)n_tensors), align256(sizeof(uint32_t) * (size_t)G),
            align256(sizeof(uint32_t) * (size_t)cap)};
}
}  // namespace

int64_t static_plan_bytes(int64_t n_tensors, int64_t G, int64_t n_short, int K)
{
    const StaticParts a = static_parts(n_tensors, G, K);
    return (int64_t)(kCtlCounted + a.numel + a.g0 + a.tlen + a.tmask + a.blen + 2 * a.list);
}

int64_t static_plan_limit() { return (int64_t)kStaticPlanLimit; }

hipError_t static_plan_scratch(void** ptr)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess)
        return e;
    if (dev < 0 || dev >= kMaxDevices)
        return hipErrorInvalidDevice;
    if (g_scratch_dev[dev] == nullptr) {
        void* p = nullptr;
        if ((e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch))) != hipSuccess)
            return e;
        if (p == nullptr)
            return hipErrorInvalidSymbol;
        g_scratch_dev[dev] = p;
    }
    *ptr = g_scratch_dev[dev];
    return hipSuccess;
}

hipError_t launch_plan_static(void* ws, const int64_t* numel, int32_t n_tensors, int64_t block_elems, uint32_t es,
                              int64_t G, int64_t n_short, int K, const float* sumsq, const Coeffs& w, uint32_t flags,
                              uint64_t budget, uint64_t full_bytes, uint32_t* mask, uint64_t* stats,
                              hipStream_t s)
{
    const StaticParts a = static_parts(n_tensors, G, K);
    const int64_t cap = (int64_t)K * std::max<int64_t>(n_tensors, 1);
    char* p = static_cast<char*>(ws);
    PlanCtl* ctl = reinterpret_cast<PlanCtl*>(p);
    p += a.ctl;
    int64_t* d_numel = reinterpret_cast<int64_t*>(p);
    p += a.numel;
    uint32_t* g0 = reinterpret_cast<uint32_t*>(p);
    p += a.g0;
    uint32_t* tlen = reinterpret_cast<uint32_t*>(p);
    p += a.tlen;
    uint32_t* tmask = reinterpret_cast<uint32_t*>(p);
    p += a.tmask;
    uint32_t* blen = reinterpret_cast<uint32_t*>(p);
    p += a.blen;
    uint32_t* list0 = reinterpret_cast<uint32_t*>(p);
    p += a.list;
    uint32_t* list1 = reinterpret_cast<uint32_t*>(p);
    hipError_t e;
    if (G > 0) {
        if ((e = hipMemcpyAsync(d_numel, numel, sizeof(int64_t) * (size_t)n_tensors, hipMemcpyHostToDevice, s)) !=
            hipSuccess)
            return e;
        hipLaunchKernelGGL(k_static_g0, dim3(1), dim3(kT), 0, s, d_numel, (int)n_tensors, block_elems, g0, tlen);
        if (sumsq != nullptr)
            hipLaunchKernelGGL(k_static_blen, dim3((unsigned)((G + kT - 1) / kT)), dim3(kT), 0, s, d_numel, g0,
                               (int)n_tensors, block_elems, G, blen);
    }
    // n_short + 1 bounds the distinct block lengths, hence the rounds
    PlanIn in{ctl, list0, list1, (unsigned)cap, blen, es, G, (int)std::min<int64_t>(n_short + 1, 1 << 30), K, sumsq, w,
              flags, budget, full_bytes, mask};
    if (sumsq != nullptr) {
        e = enqueue_block_plan(in, ctl->stats, s);
    } else {
        // tensor-level plan; the number of tensors bounds its rounds
        in.blen = tlen;
        in.G = G > 0 ? n_tensors : 0;
        in.rounds = (int)std::max<int64_t>(in.G, 1);
        in.mask = tmask;
        e = enqueue_tensor_plan(in, g0, (int)n_tensors, G, mask, ctl->stats, s);
    }
    if (e != hipSuccess)
        return e;
    if ((e = hipMemcpyAsync(stats, ctl->stats, sizeof(ctl->stats), hipMemcpyDeviceToHost, s)) != hipSuccess)
        return e;
    return hipStreamSynchronize(s);
}

hipError_t plan_ctl_alloc(PlanCtl** ctl) { return ws_malloc((void**)ctl, sizeof(PlanCtl)); }

// ---------------------------------------------------------------- coverage
// Touched elements per (tensor, expert) of an access mask, for the run's
// manifest (Section 3: touched blocks and contributing experts):
// cov[t * K + i] = sum of the lengths of tensor t's blocks selecting expert
// i.  One thread per block; a wave whose selecting blocks all lie in one
// tensor (the usual case: blocks run in tensor order) adds one wave sum per
// expert, other waves add per block.
namespace {
__global__ __launch_bounds__(256) void k_zero_cov(unsigned long long* p, int64_t n)
{
    for (int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x; q < n; q += (int64_t)gridDim.x * 256)
        p[q] = 0ull;
}

__global__ __launch_bounds__(256) void k_coverage(const uint32_t* __restrict__ mask, const uint32_t* __restrict__ len,
                                                  const uint32_t* __restrict__ tensor, int64_t G, int K,
                                                  uint32_t kmask, unsigned long long* __restrict__ cov)
{
    const int64_t g = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const bool in = g < G;
    const uint32_t m = in ? (mask[g] & kmask) : 0u;
    const uint32_t t = in ? tensor[g] : 0u;
    const unsigned long long n = in ? len[g] : 0ull;
    const unsigned long long any = __ballot(m != 0u);
    if (any == 0ull)
        return;
    const uint32_t t0 = __shfl(t, __ffsll((long long)any) - 1);
    if (__ballot(m != 0u && t != t0) == 0ull) {
        for (int i = 0; i < K; ++i) {
            unsigned long long v = ((m >> i) & 1u) ? n : 0ull;
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1)
                v += __shfl_xor(v, off);
            if ((threadIdx.x & 63) == 0 && v != 0ull)
                atomicAdd(&cov[(uint64_t)t0 * (uint32_t)K + (uint32_t)i], v);
        }
    } else {
        for (uint32_t mm = m; mm; mm &= mm - 1u)
            atomicAdd(&cov[(uint64_t)t * (uint32_t)K + (uint32_t)__builtin_ctz(mm)], n);
    }
}
}  // namespace

hipError_t launch_coverage(const BlockTable& bt, int K, const uint32_t* mask, unsigned long long* cov, hipStream_t s)
{
    const int64_t n = bt.n_tensors * K;
    if (n > 0)
        hipLaunchKernelGGL(k_zero_cov, dim3((unsigned)std::min<int64_t>((n + 255) / 256, 1024)), dim3(256), 0, s,
                           cov, n);
    if (bt.G > 0) {
        const uint32_t kmask = (K >= 32) ? 0xffffffffu : ((1u << K) - 1u);
        hipLaunchKernelGGL(k_coverage, dim3((unsigned)((bt.G + 255) / 256)), dim3(256), 0, s, mask, bt.d_len,
                           bt.d_tensor, bt.G, K, kmask, cov);
    }
    return hipGetLastError();
}

}  // namespace mp
