// skis_query.hip -- queries on the device-resident sketch:
//   k_est_*      Eq. (eq21): Cov(S) by collecting the samples of every v in S in an LDS hash (few
//                list entries) or by windows of sample ids over the device (many), and
//                I_hat(S) = fl(fl(Cov * Gamma) / T) + sum_{v in S} q_v (compensated sum).
//   k_estimate   the same for sets of more members than a workgroup holds: marks the samples in
//                a bitmap over the T samples (a sample counts once, when its bit first flips).
//   k_greedy_*   Alg. 3: the node of largest gain fl(fl(Delta * Gamma) / T) + q (Eq. margin),
//                smallest id on ties; Delta kept exact by decrementing the members of every
//                newly covered sample.
#include "skis_internal.h"
#include "skis_query.h"

#include <algorithm>
#include <vector>

namespace skis {

__device__ __forceinline__ void neumaier_add(double &s, double &c, double x)
{
    const double t = __dadd_rn(s, x);
    if (fabs(s) >= fabs(x)) c = __dadd_rn(c, __dadd_rn(__dsub_rn(s, t), x));
    else c = __dadd_rn(c, __dadd_rn(__dsub_rn(x, t), s));
    s = t;
}

template <int NT>
__device__ void bitonic_sort_lds(int32_t *buf, int P)
{
    for (int k = 2; k <= P; k <<= 1) {
        for (int d = k >> 1; d > 0; d >>= 1) {
            for (int i = threadIdx.x; i < P; i += NT) {
                const int ixj = i ^ d;
                if (ixj > i) {
                    const int32_t x = buf[i], y = buf[ixj];
                    const bool asc = (i & k) == 0;
                    if ((x > y) == asc) {
                        buf[i] = y;
                        buf[ixj] = x;
                    }
                }
            }
            __syncthreads();
        }
    }
}

// flip_bits_wave flips the bit of sample j in bm for every lane of the wave with in = true and
// returns the bits this lane flipped; every lane of the wave must call it (word_bits_wave is its
// first half: the bits that a lane sets in its word if it is the one to do so).  A sample list is sorted by
// sample id and a wave walks consecutive entries, so on a dense list (a hub's) neighbouring
// lanes often share a bitmap word.  When any do, the bits of lanes with the same word are
// OR-ed within aligned groups of 8 lanes by a segmented scan (a lane takes the running OR of
// lane - d in its group when their words agree; a run of equal words is contiguous, and lanes
// of another run with the same word only add bits of that word), and the last lane of each
// run in a group sets them with one atomicOr.  Atomics on one word are serialised, so every
// flip is counted once.  When no neighbours share a word, each lane flips its own bit.
__device__ __forceinline__ uint32_t word_bits_wave(int32_t j, bool in, bool *last)
{
    const int lane = threadIdx.x & 63;
    const uint32_t w = (uint32_t)j >> 5;
    uint32_t acc = in ? 1u << (j & 31) : 0u;
    // the shuffle runs on every lane: under a mask it would read 0 from the masked lane 63
    const uint32_t nw = __shfl_down(w, 1, 64);
    const bool same_next = lane < 63 && nw == w;
    *last = true;
    if (__ballot(same_next) != 0ull) { // wave-uniform
#pragma unroll
        for (int d = 1; d < 8; d <<= 1) {
            const uint32_t ow = __shfl_up(w, d, 64), oa = __shfl_up(acc, d, 64);
            if ((lane & 7) >= d && ow == w) acc |= oa;
        }
        *last = (lane & 7) == 7 || !same_next;
    }
    return acc;
}

__device__ __forceinline__ unsigned long long flip_bits_wave(uint32_t *bm, int32_t j, bool in)
{
    bool last;
    const uint32_t acc = word_bits_wave(j, in, &last);
    if (!last || !acc) return 0ull;
    const uint32_t old = atomicOr(&bm[(uint32_t)j >> 5], acc);
    return (unsigned long long)__popc(acc & ~old);
}

// Sets too large for k_est_set (members, or entries of their lists), one workgroup a set.  The set is
// taken in chunks of EST_MAX_SET entries; each chunk is sorted and deduplicated in LDS, and a bitmap
// of n bits drops ids already met in an earlier chunk.  The distinct members' q values are summed
// (compensated, in a fixed order) and their sample lists H(v) are walked flat across the
// workgroup, flipping one bit per sample in a bitmap of T bits; Cov(S) is the number of flips.
__global__ __launch_bounds__(EST_BLOCK) void k_estimate(const int64_t *__restrict__ qlist, int64_t q0,
                                                        const int64_t *__restrict__ set_ptr,
                                                        const int32_t *__restrict__ set_nodes, int32_t n, uint64_t T,
                                                        double Gamma, const double *__restrict__ qv,
                                                        const int64_t *__restrict__ node_ptr,
                                                        const int32_t *__restrict__ node_samples,
                                                        uint32_t *__restrict__ bitmaps, uint64_t wordsT,
                                                        uint32_t *__restrict__ nodebits, uint64_t wordsN,
                                                        unsigned long long *__restrict__ cov_out,
                                                        double *__restrict__ est_out, int *__restrict__ err)
{
    __shared__ int32_t buf[EST_MAX_SET];
    __shared__ int64_t dbase[EST_MAX_SET + 1];
    __shared__ int32_t s_scan[EST_BLOCK / 64 + 1];
    __shared__ int64_t s_scan64[EST_BLOCK / 64 + 1];
    __shared__ double ps[EST_BLOCK], pc[EST_BLOCK];
    __shared__ unsigned long long s_cov[EST_BLOCK / 64];
    __shared__ int s_bad;

    const int64_t qi = qlist[q0 + blockIdx.x];
    const int tid = threadIdx.x;
    const int64_t a = set_ptr[qi], b = set_ptr[qi + 1];
    const int64_t k = b - a;
    if (k < 0) {
        if (tid == 0) atomicOr(err, 1);
        return;
    }
    uint32_t *bm = bitmaps + (uint64_t)blockIdx.x * wordsT;
    uint32_t *nb = nodebits + (uint64_t)blockIdx.x * wordsN;
    constexpr int IPT = EST_MAX_SET / EST_BLOCK;

    double sq = 0.0, cq = 0.0;
    unsigned long long local = 0;
    int nu = 0, maxnu = 0; // maxnu: threads at or past it never took a member (their sums are +0)
    int64_t E = 0;
    // a chunk's members are read while the one before is sorted, all at once: the service's sets lie in
    // host memory (one read after the other, 300 thousand members on 2^18 samples took 8.9 ms, 7.9 with
    // the set copied to the device first; now 8.0)
    int32_t ahead[IPT];
    auto fetch = [&](int64_t c0) {
        if (c0 >= b) return;
#pragma unroll
        for (int r = 0; r < IPT; ++r) ahead[r] = set_nodes[min(c0 + tid + r * EST_BLOCK, b - 1)];
    };
    fetch(a);
    for (int64_t c0 = a; c0 < b; c0 += EST_MAX_SET) {
        const int kc = (int)((b - c0) < EST_MAX_SET ? (b - c0) : EST_MAX_SET);
        if (tid == 0) s_bad = 0;
        __syncthreads();
        int P = 1;
        while (P < kc) P <<= 1;
#pragma unroll
        for (int r = 0; r < IPT; ++r) {
            const int t = tid + r * EST_BLOCK;
            int32_t v = t < kc ? ahead[r] : INT32_MAX;
            if (t < kc && (v < 0 || v >= n)) {
                s_bad = 1;
                v = INT32_MAX;
            }
            if (t < P) buf[t] = v;
        }
        fetch(c0 + EST_MAX_SET);
        __syncthreads();
        if (s_bad) {
            if (tid == 0) atomicOr(err, 4);
            return;
        }
        if (P > 1) bitonic_sort_lds<EST_BLOCK>(buf, P);

        // distinct members of the chunk, not met before, compacted in order
        int32_t mine[IPT];
        int flags = 0, cntu = 0;
#pragma unroll
        for (int r = 0; r < IPT; ++r) {
            const int t = tid * IPT + r;
            const int32_t v = t < kc ? buf[t] : INT32_MAX;
            mine[r] = v;
            bool u = t < kc && (t == 0 || buf[t - 1] != v);
            if (u) {
                const uint32_t bit = 1u << (v & 31);
                u = !(atomicOr(&nb[v >> 5], bit) & bit);
            }
            flags |= (u ? 1 : 0) << r;
            cntu += u ? 1 : 0;
        }
        int pos = block_excl_scan<EST_BLOCK, int>(cntu, s_scan, &nu);
        __syncthreads();
#pragma unroll
        for (int r = 0; r < IPT; ++r)
            if (flags >> r & 1) buf[pos++] = mine[r];
        __syncthreads();

        if (qv)
            for (int t = tid; t < nu; t += EST_BLOCK) neumaier_add(sq, cq, qv[buf[t]]);
        maxnu = nu > maxnu ? nu : maxnu;
        int64_t dl[IPT];
        int64_t acc = 0;
#pragma unroll
        for (int r = 0; r < IPT; ++r) {
            const int t = tid * IPT + r;
            int64_t d = 0;
            if (t < nu && T) { // without samples there may be no index
                const int32_t v = buf[t];
                d = node_ptr[v + 1] - node_ptr[v];
            }
            dl[r] = acc;
            acc += d;
        }
        const int64_t ex = block_excl_scan<EST_BLOCK, int64_t>(acc, s_scan64, &E);
#pragma unroll
        for (int r = 0; r < IPT; ++r) {
            const int t = tid * IPT + r;
            if (t < nu) dbase[t] = ex + dl[r];
        }
        if (tid == 0) dbase[nu] = E;
        __syncthreads();
        // EST_WALK entries per thread and round, their loads issued together; a wave takes 64
        // consecutive entries and flips their bits with one atomic per bitmap word it meets.
        // The rounds are the same for the whole wave (the flips shuffle across it); a lane past
        // E repeats entry E - 1 (in bounds) and flips no bit.
        for (int64_t i0 = tid; i0 - (tid & 63) < E; i0 += (int64_t)EST_BLOCK * EST_WALK) { // wave-uniform
            int64_t ix[EST_WALK];
            int lv[EST_WALK];
#pragma unroll
            for (int u = 0; u < EST_WALK; ++u) {
                const int64_t idx = i0 + (int64_t)u * EST_BLOCK;
                ix[u] = idx < E ? idx : E - 1;
                int lo = 0, hi = nu - 1;
                while (lo < hi) {
                    const int mid = (lo + hi + 1) >> 1;
                    if (dbase[mid] <= ix[u]) lo = mid; else hi = mid - 1;
                }
                lv[u] = lo;
            }
            int64_t np[EST_WALK];
#pragma unroll
            for (int u = 0; u < EST_WALK; ++u) np[u] = node_ptr[buf[lv[u]]];
            int32_t jv[EST_WALK];
#pragma unroll
            for (int u = 0; u < EST_WALK; ++u) jv[u] = node_samples[np[u] + (ix[u] - dbase[lv[u]])];
#pragma unroll
            for (int u = 0; u < EST_WALK; ++u) local += flip_bits_wave(bm, jv[u], i0 + (int64_t)u * EST_BLOCK < E);
        }
        __syncthreads();
    }

    ps[tid] = sq;
    pc[tid] = cq;
    local = wave_sum(local);
    if ((tid & 63) == 0) s_cov[tid >> 6] = local;
    __syncthreads();
    if (tid == 0) {
        unsigned long long c = 0;
        for (int w = 0; w < EST_BLOCK / 64; ++w) c += s_cov[w];
        double s = 0.0, cc = 0.0;
        // adding the +0 partials of the threads past maxnu would change neither s nor cc
        const int tq = maxnu < EST_BLOCK ? maxnu : EST_BLOCK;
        for (int t = 0; t < tq; ++t) {
            neumaier_add(s, cc, ps[t]);
            neumaier_add(s, cc, pc[t]);
        }
        const double first = T > 0 ? __ddiv_rn(__dmul_rn((double)c, Gamma), (double)T) : 0.0;
        cov_out[qi] = c;
        est_out[qi] = __dadd_rn(first, __dadd_rn(s, cc));
    }
    // leave the bitmaps clear for the next query
    for (uint64_t w = tid; w < wordsT; w += EST_BLOCK) bm[w] = 0u;
    constexpr int CLEAR = 8; // members a thread reads together
    for (int64_t t0 = a + tid; t0 < b; t0 += (int64_t)EST_BLOCK * CLEAR) {
        int32_t v[CLEAR];
#pragma unroll
        for (int u = 0; u < CLEAR; ++u) v[u] = set_nodes[min(t0 + (int64_t)u * EST_BLOCK, b - 1)];
#pragma unroll
        for (int u = 0; u < CLEAR; ++u) nb[v[u] >> 5] = 0u; // past the last one: that one again
    }
}

// ---------------------------------------------------------------------------------------
// Estimates of sets of at most EST_MAX_SET entries.
//
// k_est_set: one workgroup a set.  The distinct members' list lengths come first; when they add up to
// at most EST_HASH_MAX entries, the sample ids go into an LDS hash (Cov = ids that were not there), so
// a light set touches no bitmap in memory and has nothing to clear; a walk that flips bits of a T-bit
// bitmap in memory takes two passes over the lists and a returning global atomic an entry.  Heavier
// sets are parked: cov = EST_PARKED, est = the sum of q.
//
// WALK (the service, where a second kernel for the parked sets would add its latency to every batch:
// 1024 Zipf sets took 1.7 ms that way for 1.25): heavier sets are walked by the same workgroup with
// a bitmap of T bits.  8 loads and then 8 atomics a lane are in flight (4 in turn before), the members
// are searched between those of a wave's first and last entry, and their list begins wait in LDS:
// batches of 256 Zipf(1.5) sets of 1-1000 members on 2^25 samples of the 4M-node TRI graph 350-520 ->
// 200-330 us (by their heaviest set; 1000 members with 62k entries take 168 us, 16 in flight no less:
// bound by the atomics, some 390M a second for a CU).
//
// k_est_split: the parked sets.  The lists are sorted by sample id, so a window of ids is a range
// of every list: a workgroup takes one (set, window), finds the ranges by binary search, sets the
// window's bits in LDS and counts them; the windows of a set run on as many CUs as there are, with
// no bitmap in memory.  Each adds its count to cov, and the set's last window forms the estimate
// (no workgroup waits for another).  Whole calls, one workgroup and bitmap a set before -> now: 16
// sets of up to 50 hubs on 2^25 samples of the 4M-node TRI graph 6.6 -> 0.14 ms, 100 sets of 1-50
// uniform nodes on 2^24 samples of the 1M-node WC graph 0.21 -> 0.090 ms, one set of 3 nodes on
// 200k samples 61 -> 27 us (the flags in host memory, one kernel).
// ---------------------------------------------------------------------------------------
__device__ __forceinline__ double first_term(unsigned long long cov, double Gamma, uint64_t T)
{
    return T > 0 ? __ddiv_rn(__dmul_rn((double)cov, Gamma), (double)T) : 0.0;
}

// check: 0, or the number of sets whose set_ptr this workgroup checks first (so that no set is
// read by a set_ptr that does not rise from 0; at most EST_BLOCK of them).  flags: see EstFlags.
template <bool WALK>
__global__ __launch_bounds__(EST_BLOCK) void k_est_set(int32_t check, const int64_t *__restrict__ set_ptr,
                                                         const int32_t *__restrict__ set_nodes, int32_t n, uint64_t T,
                                                         double Gamma, const double *__restrict__ qv,
                                                         const int64_t *__restrict__ node_ptr,
                                                         const int32_t *__restrict__ node_samples,
                                                         unsigned long long *__restrict__ cov_out,
                                                         double *__restrict__ est_out, uint32_t *__restrict__ ticket,
                                                         uint32_t *__restrict__ bitmaps, uint64_t wordsT,
                                                         EstFlags *__restrict__ flags)
{
    __shared__ int32_t buf[EST_MAX_SET];
    __shared__ uint32_t pre[EST_MAX_SET + 1];  // first entry of each member's list in the walk
    __shared__ int64_t lbase[EST_MAX_SET];    // list begin - pre
    __shared__ uint32_t hash[EST_HASH_SLOTS];
    __shared__ double ps[EST_BLOCK], pc[EST_BLOCK];
    __shared__ int32_t s_scan[EST_BLOCK / 64 + 1];
    __shared__ int64_t s_scan64[EST_BLOCK / 64 + 1];
    __shared__ uint32_t s_cov, s_next, s_clear;
    __shared__ int s_bad_ptr, s_bad;

    const int64_t qi = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63;
    if (tid == 0) {
        s_bad_ptr = s_bad = 0;
        s_cov = 0u;
        s_next = s_clear = 0u;
    }
    __syncthreads();
    if (tid < check) {
        const int64_t x = set_ptr[tid], y = set_ptr[tid + 1];
        if (x < 0 || y < x) s_bad_ptr = 1;
    }
    __syncthreads();
    if (s_bad_ptr) {
        if (tid == 0) flags->ptr = 1;
        return;
    }
    const int64_t a = set_ptr[qi], b = set_ptr[qi + 1];
    if (b - a > EST_MAX_SET) { // k_estimate's
        if (!WALK && tid == 0) {
            flags->large = 1;
            cov_out[qi] = 0ull; // not EST_PARKED by what the buffer held
        }
        return;
    }
    const int kc = (int)(b - a);
    int P = 1;
    while (P < kc) P <<= 1;
    for (int t = tid; t < P; t += EST_BLOCK) {
        int32_t v = INT32_MAX;
        if (t < kc) {
            v = set_nodes[a + t];
            if (v < 0 || v >= n) {
                s_bad = 1;
                v = INT32_MAX;
            }
        }
        buf[t] = v;
    }
    __syncthreads();
    if (s_bad) {
        if (tid == 0) flags->node = 1;
        return;
    }
    if (P > 1) bitonic_sort_lds<EST_BLOCK>(buf, P);
    // distinct members, compacted in order
    constexpr int IPT = EST_MAX_SET / EST_BLOCK;
    int nu = 0;
    {
        int32_t mine[IPT];
        int keep = 0, cntu = 0;
#pragma unroll
        for (int r = 0; r < IPT; ++r) {
            const int t = tid * IPT + r;
            const int32_t v = t < kc ? buf[t] : INT32_MAX;
            mine[r] = v;
            const bool u = t < kc && (t == 0 || buf[t - 1] != v);
            keep |= (u ? 1 : 0) << r;
            cntu += u ? 1 : 0;
        }
        int pos = block_excl_scan<EST_BLOCK, int>(cntu, s_scan, &nu);
        __syncthreads();
#pragma unroll
        for (int r = 0; r < IPT; ++r)
            if (keep >> r & 1) buf[pos++] = mine[r];
        __syncthreads();
    }
    // q of the members (summed below, in the same order as k_estimate) and the lists' bounds
    double sq = 0.0, cq = 0.0;
    if (qv)
        for (int t = tid; t < nu; t += EST_BLOCK) neumaier_add(sq, cq, qv[buf[t]]);
    int64_t np[IPT], dl[IPT];
    int64_t acc = 0, E = 0;
#pragma unroll
    for (int r = 0; r < IPT; ++r) {
        const int t = tid * IPT + r;
        int64_t d = 0;
        np[r] = 0;
        if (t < nu && T) { // without samples there may be no index
            const int32_t v = buf[t];
            np[r] = node_ptr[v];
            d = node_ptr[v + 1] - np[r];
        }
        dl[r] = acc;
        acc += d;
    }
    const int64_t ex = block_excl_scan<EST_BLOCK, int64_t>(acc, s_scan64, &E);
    ps[tid] = sq;
    pc[tid] = cq;
    const bool light = E <= (int64_t)EST_HASH_MAX;
    if (WALK && (uint64_t)E > EST_WALK_MAX) return; // k_estimate's
    uint32_t slots = 64; // a power of two of at least 1.5 slots an entry
    if (WALK || light) {
#pragma unroll
        for (int r = 0; r < IPT; ++r) {
            const int t = tid * IPT + r;
            if (t < nu) {
                pre[t] = (uint32_t)(ex + dl[r]);
                lbase[t] = np[r] - (ex + dl[r]);
            }
        }
        if (tid == 0) pre[nu] = (uint32_t)E;
    }
    if (light) {
        while (2 * slots < 3 * (uint32_t)E) slots <<= 1;
        for (uint32_t i = tid; i < slots; i += EST_BLOCK) hash[i] = 0xFFFFFFFFu;
    }
    __syncthreads();
    double s = 0.0, cc = 0.0;
    if (tid == 0) { // one chain of additions, beside the other waves' walk
        const int tq = nu < EST_BLOCK ? nu : EST_BLOCK;
        for (int t = 0; t < tq; ++t) {
            neumaier_add(s, cc, ps[t]);
            if (nu > EST_BLOCK) neumaier_add(s, cc, pc[t]); // a single member's compensation is +0
        }
    }
    uint32_t found = 0;
    if (!light && !WALK) {
        if (tid == 0) {
            cov_out[qi] = EST_PARKED;
            est_out[qi] = __dadd_rn(s, cc);
            if (ticket) ticket[qi] = 0u;
            flags->parked = 1;
        }
        return;
    }
    if (!light) {
        // a wave takes 64 U entries at a time, all its loads and then all its flips in flight; a lane
        // past E repeats entry E - 1 (in bounds) and flips no bit
        constexpr int U = 8;
        uint32_t *const bm = bitmaps + (uint64_t)blockIdx.x * wordsT;
        auto walk = [&](uint32_t *next, auto &&use) {
            for (;;) {
                uint32_t c = 0;
                if (lane == 0) c = atomicAdd(next, 64u * U);
                c = (uint32_t)__builtin_amdgcn_readfirstlane((int)c);
                if (c >= (uint32_t)E) break;
                // the member of an entry lies between those of the first and the last one
                auto member = [&](uint32_t idx, int lo, int hi) {
                    while (lo < hi) {
                        const int mid = (lo + hi + 1) >> 1;
                        if (pre[mid] <= idx) lo = mid; else hi = mid - 1;
                    }
                    return lo;
                };
                const int end = member(lane == 0 ? c : min(c + 64u * U, (uint32_t)E) - 1u, 0, nu - 1);
                const int m0 = __builtin_amdgcn_readlane(end, 0), m1 = __builtin_amdgcn_readlane(end, 1);
                int32_t jv[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const uint32_t idx = min(c + (uint32_t)(u * 64 + lane), (uint32_t)E - 1u);
                    jv[u] = node_samples[lbase[member(idx, m0, m1)] + idx];
                }
                use(c, jv);
            }
        };
        walk(&s_next, [&](uint32_t c, const int32_t (&jv)[U]) {
            uint32_t acc[U], old[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                bool last;
                acc[u] = word_bits_wave(jv[u], c + (uint32_t)(u * 64 + lane) < (uint32_t)E, &last);
                if (!last) acc[u] = 0u;
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                old[u] = 0u;
                if (acc[u]) old[u] = atomicOr(&bm[(uint32_t)jv[u] >> 5], acc[u]);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) found += (uint32_t)__popc(acc[u] & ~old[u]);
        });
        __syncthreads(); // every flip done
        walk(&s_clear, [&](uint32_t, const int32_t (&jv)[U]) { // leave the bitmap clear for the next batch
#pragma unroll
            for (int u = 0; u < U; ++u) { // the last lane of each run of equal words clears it
                const uint32_t w = (uint32_t)jv[u] >> 5, nw = __shfl_down(w, 1, 64);
                if (lane == 63 || nw != w) bm[w] = 0u;
            }
        });
    }
    const uint32_t sh = 32 - (31 - __clz((int)slots));
    for (; light;) { // a wave takes 256 entries at a time
        uint32_t c = 0;
        if (lane == 0) c = atomicAdd(&s_next, 256u);
        c = (uint32_t)__builtin_amdgcn_readfirstlane((int)c);
        if (c >= (uint32_t)E) break;
        int32_t jv[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint32_t idx = min(c + (uint32_t)(u * 64 + lane), (uint32_t)E - 1u);
            int lo = 0, hi = nu - 1;
            while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if (pre[mid] <= idx) lo = mid; else hi = mid - 1;
            }
            jv[u] = node_samples[lbase[lo] + idx];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if ((int)c + u * 64 + lane >= (int)E) continue;
            const uint32_t j = (uint32_t)jv[u];
            uint32_t h = (j * 0x9E3779B1u) >> sh;
            uint32_t old;
#pragma unroll 1
            for (;;) { // fewer entries than slots: an empty slot is always met
                old = atomicCAS(&hash[h], 0xFFFFFFFFu, j);
                if (old == 0xFFFFFFFFu || old == j) break;
                h = (h + 1) & (slots - 1u);
            }
            found += old == 0xFFFFFFFFu ? 1u : 0u;
        }
    }
    found = wave_sum(found);
    if (lane == 0 && found) atomicAdd(&s_cov, found);
    __syncthreads();
    if (tid == 0) {
        const unsigned long long c = s_cov;
        cov_out[qi] = c;
        est_out[qi] = __dadd_rn(first_term(c, Gamma, T), __dadd_rn(s, cc));
    }
}

// First position of [lo, hi) with ns[pos] >= x, hi if there is none.
__device__ __forceinline__ int64_t lower_bound_sample(const int32_t *__restrict__ ns, int64_t lo, int64_t hi, int64_t x)
{
    while (lo < hi) {
        const int64_t mid = lo + ((hi - lo) >> 1);
        if ((int64_t)ns[mid] >= x) hi = mid; else lo = mid + 1;
    }
    return lo;
}

constexpr int SPLIT_BITS = 1 << 19;   // samples a window holds at most (64 KiB of LDS: two workgroups a CU)
constexpr int SPLIT_MIN = 1 << 15;    // and at least, unless T is smaller
constexpr int SPLIT_WINDOWS = 64;     // windows wanted: 16 sets then give every CU four of them
static_assert(SPLIT_MIN % 32 == 0 && SPLIT_BITS % 32 == 0, "windows are whole words");

__global__ __launch_bounds__(EST_BLOCK) void k_est_split(int32_t windows, int32_t wbits,
                                                         const int64_t *__restrict__ set_ptr,
                                                         const int32_t *__restrict__ set_nodes, uint64_t T,
                                                         double Gamma, const int64_t *__restrict__ node_ptr,
                                                         const int32_t *__restrict__ node_samples,
                                                         const uint32_t *__restrict__ heavy,
                                                         unsigned long long *__restrict__ cov_out,
                                                         double *__restrict__ est_out, uint32_t *__restrict__ ticket)
{
    __shared__ uint32_t bits[SPLIT_BITS / 32];
    __shared__ int64_t sbase[EST_BLOCK];   // range begin - pre
    __shared__ int32_t pre[EST_BLOCK + 1]; // first entry of each member's range in the walk
    __shared__ int32_t s_scan[EST_BLOCK / 64 + 1];
    __shared__ uint32_t s_cnt;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    constexpr int NW = EST_BLOCK / 64;
    const uint32_t nheavy = heavy[0];
    for (uint64_t item = blockIdx.x; item < (uint64_t)nheavy * (uint64_t)windows; item += gridDim.x) {
        const int64_t qi = heavy[1 + item / (uint64_t)windows];
        const int64_t w = (int64_t)(item % (uint64_t)windows);
        const int64_t j0 = w * wbits, j1 = min(j0 + (int64_t)wbits, (int64_t)T);
        const int words = (int)((j1 - j0 + 31) >> 5);
        for (int i = tid; i < words; i += EST_BLOCK) bits[i] = 0u;
        if (tid == 0) s_cnt = 0u;
        const int64_t a = set_ptr[qi], b = set_ptr[qi + 1];
        for (int64_t c0 = a; c0 < b; c0 += EST_BLOCK) { // repeated members set the same bits again
            const int m = (int)min(b - c0, (int64_t)EST_BLOCK);
            int64_t r0 = 0, r1 = 0;
            if (tid < m) {
                const int32_t v = set_nodes[c0 + tid];
                const int64_t p0 = node_ptr[v], p1 = node_ptr[v + 1];
                r0 = w == 0 ? p0 : lower_bound_sample(node_samples, p0, p1, j0);
                r1 = w == windows - 1 ? p1 : lower_bound_sample(node_samples, r0, p1, j1);
            }
            int tot;
            const int ex = block_excl_scan<EST_BLOCK, int>((int)(r1 - r0), s_scan, &tot);
            pre[tid] = ex;
            sbase[tid] = r0 - ex;
            if (tid == 0) pre[EST_BLOCK] = tot;
            __syncthreads();
            // each wave walks an even share in chunks of 256; a chunk inside one range (a hub's)
            // needs no search
            const int share = ((tot + NW - 1) / NW + 255) & ~255;
            const int f0 = wave * share, f1 = min(f0 + share, tot);
            for (int f = f0; f < f1; f += 256) {
                int lo = 0, hi = m - 1; // the range that holds entry f (uniform)
                while (lo < hi) {
                    const int mid = (lo + hi + 1) >> 1;
                    if (pre[mid] <= f) lo = mid; else hi = mid - 1;
                }
                const bool one = lo == m - 1 || pre[lo + 1] >= min(f + 256, f1);
                int32_t jv[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int idx = min(f + u * 64 + lane, f1 - 1);
                    int l = lo;
                    if (!one) {
                        int h = m - 1;
                        while (l < h) {
                            const int mid = (l + h + 1) >> 1;
                            if (pre[mid] <= idx) l = mid; else h = mid - 1;
                        }
                    }
                    jv[u] = node_samples[sbase[l] + idx];
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) { // an entry past the share repeats the last one's bit
                    const uint32_t j = (uint32_t)((int64_t)jv[u] - j0);
                    if (j < (uint32_t)wbits) atomicOr(&bits[j >> 5], 1u << (j & 31));
                }
            }
            __syncthreads();
        }
        if (b == a) __syncthreads();
        uint32_t c = 0;
        for (int i = tid; i < words; i += EST_BLOCK) c += (uint32_t)__popc(bits[i]);
        c = wave_sum(c);
        if (lane == 0 && c) atomicAdd(&s_cnt, c);
        __syncthreads();
        if (tid == 0) {
            if (s_cnt) atomicAdd(&cov_out[qi], (unsigned long long)s_cnt);
            __threadfence();
            if (atomicAdd(&ticket[qi], 1u) == (uint32_t)windows - 1u) { // the set's last window
                __threadfence();
                const unsigned long long cov =
                    __hip_atomic_load(&cov_out[qi], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                est_out[qi] = __dadd_rn(first_term(cov, Gamma, T), est_out[qi]);
            }
        }
        __syncthreads();
    }
}

// Lists the parked sets, heavy = {count, set, set, ...}, and clears their cov (one workgroup).
__global__ __launch_bounds__(EST_BLOCK) void k_est_list(int32_t Q, unsigned long long *__restrict__ cov_out,
                                                        uint32_t *__restrict__ heavy)
{
    __shared__ int32_t s_scan[EST_BLOCK / 64 + 1];
    uint32_t count = 0;
    for (int32_t q0 = 0; q0 < Q; q0 += EST_BLOCK) {
        const int32_t q = q0 + (int32_t)threadIdx.x;
        const bool p = q < Q && cov_out[q] == EST_PARKED;
        int tot;
        const int ex = block_excl_scan<EST_BLOCK, int>(p ? 1 : 0, s_scan, &tot);
        if (p) {
            heavy[1 + count + (uint32_t)ex] = (uint32_t)q;
            cov_out[q] = 0ull;
        }
        count += (uint32_t)tot;
        __syncthreads();
    }
    if (threadIdx.x == 0) heavy[0] = count;
}

// ---------------------------------------------------------------------------------------
// Greedy (Alg. 3) with exact marginal coverage.  delta[v] = #{ j in H(v) : j not covered }.
// Each round: k_greedy_argmax picks the node of largest gain fl(fl(delta * Gamma) / T) + q_v
// (Eq. margin; smallest id on ties); k_greedy_cover sets the covered bits of H(v*) and lowers
// delta of every member of the samples it newly covers, or, when they are many,
// k_greedy_recount counts delta afresh from the lists.  Three launches per round and no host
// synchronisation inside the k rounds.
// ---------------------------------------------------------------------------------------
// A round that covers more than T / RECOUNT_DIV samples recounts Delta of every node from
// its list instead of decrementing the members of each newly covered sample.
constexpr uint64_t RECOUNT_DIV = 32;
constexpr int RECOUNT_SPAN = 1024; // list entries per recount work item
constexpr int RECOUNT_LANES = 16;  // lanes per work item
constexpr int RECOUNT_UNROLL = 8;  // loads in flight per lane

// recount: the samples from which on a round recounts (0 before the first round: st->rounds is 0)
__device__ __forceinline__ bool heavy_round(const GreedyState *st, uint64_t recount)
{
    return st->vstar >= 0 && st->rounds > 0 && st->dstar >= recount;
}

// Whether `todo` rounds are worth the 60 us that going over to k_greedy_small takes: a round by launches
// is longer by some 10 us and 40 us a million nodes (WC and TRI graphs of 15 thousand to 4M nodes), by
// hardly anything where all nodes are one tile (2000 nodes: a round of either some 25 us).
__host__ __device__ __forceinline__ bool worth_going_over(int32_t todo, int32_t n)
{
    return (int64_t)todo * (n <= GREEDY_TILE ? 2 : 10 + n / 25000) > 60;
}

// A small sketch's last round, of the whole device, has lowered few entries, or few are left, and the
// rounds to come are worth it.
__device__ __forceinline__ bool greedy_few(const GreedyState *st, uint32_t left, int32_t todo, int32_t n)
{
    return st->rounds > 0 && (left <= GREEDY_FEW_LEFT || st->before - left <= GREEDY_FEW_LOWERED) &&
           worth_going_over(todo, n);
}

__device__ __forceinline__ double gain_of(int64_t d, uint64_t T, double Gamma, double q)
{
    return __dadd_rn(T > 0 ? __ddiv_rn(__dmul_rn((double)d, Gamma), (double)T) : 0.0, q);
}

__device__ __forceinline__ bool better(double g, int32_t v, double bg, int32_t bv)
{
    return bv < 0 || g > bg || (g == bg && v < bv);
}

__global__ __launch_bounds__(256) void k_greedy_init(int32_t n, const int64_t *__restrict__ node_ptr,
                                                     int32_t *__restrict__ delta, uint8_t *__restrict__ chosen)
{
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += (int64_t)gridDim.x * blockDim.x) {
        delta[v] = (int32_t)(node_ptr[v + 1] - node_ptr[v]);
        chosen[v] = 0;
    }
}

// (g, v) maximum under the order "larger gain, then smaller id" (a total order on the
// valid pairs, so any reduction tree gives the same winner); v < 0 marks an empty slot.
__device__ __forceinline__ void wave_best(double &g, int32_t &v)
{
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) {
        const double og = __shfl_xor(g, d, 64);
        const int32_t ov = __shfl_xor(v, d, 64);
        if (ov >= 0 && better(og, ov, g, v)) {
            g = og;
            v = ov;
        }
    }
}

// Best of nodes [v0, v0 + 512) below n by one wave (every lane gets it), all loads issued first.
// LIVE: delta is lowered by atomics of the same launch, so it is read past the L1 cache.
constexpr int SCAN_PART = 512;
constexpr GreedyTile NO_TILE = {-1.0, -1.0, -1, 0};
static_assert(GREEDY_TILE % SCAN_PART == 0, "a tile is scanned in whole parts");

template <bool LIVE>
__device__ __forceinline__ GreedyTile scan_part(int64_t v0, int32_t n, uint64_t T, double Gamma,
                                                const int32_t *__restrict__ delta, const double *__restrict__ qv,
                                                const uint8_t *__restrict__ chosen)
{
    constexpr int U = SCAN_PART / 64;
    const int lane = threadIdx.x & 63;
    double bg = -1.0, b2 = -1.0; // the lane's best and second
    int32_t bv = -1, bd = 0;
    int32_t d[U];
    double q[U];
    uint8_t c[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int64_t v = v0 + u * 64 + lane;
        const int64_t vc = v < n ? v : n - 1;
        d[u] = LIVE ? __hip_atomic_load(&delta[vc], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : delta[vc];
        q[u] = qv ? qv[vc] : 0.0;
        c[u] = v < n ? chosen[vc] : (uint8_t)1;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        if (c[u]) continue;
        const int32_t v = (int32_t)(v0 + u * 64 + lane);
        const double g = gain_of(d[u], T, Gamma, q[u]);
        if (better(g, v, bg, bv)) {
            b2 = bg;
            bg = g;
            bv = v;
            bd = d[u];
        } else {
            b2 = g > b2 ? g : b2;
        }
    }
    const int32_t mine = bv, md = bd;
    const double mg = bg;
    wave_best(bg, bv);
    // the winner's delta from the lane that held it (the lanes' nodes differ)
    const unsigned long long m = __ballot(bv >= 0 && mine == bv);
    if (bv >= 0 && mine != bv) b2 = mg; // another lane's best is the part's: this lane's is a second
#pragma unroll
    for (int s = 32; s > 0; s >>= 1) {
        const double o = __shfl_xor(b2, s, 64);
        b2 = o > b2 ? o : b2;
    }
    GreedyTile b;
    b.g = bg;
    b.g2 = b2;
    b.v = bv;
    b.d = m ? (int32_t)lane_value((uint32_t)md, __ffsll(m) - 1) : 0;
    return b;
}

// e into the running best of a tile.
__device__ __forceinline__ void merge_part(GreedyTile &best, const GreedyTile &e)
{
    if (e.v >= 0 && better(e.g, e.v, best.g, best.v)) {
        const double s = best.v >= 0 ? best.g : -1.0;
        const double g2 = e.g2 > s ? e.g2 : s;
        best = e;
        best.g2 = g2;
    } else if (e.v >= 0) {
        best.g2 = e.g > best.g2 ? e.g : best.g2;
    }
}

// The pick of a round by one workgroup of GREEDY_BLOCK threads (every thread gets it; v = -1: no
// node left).  The gains of the tiles' cached nodes, as of now, bound the pick from below; only a
// tile whose node has changed and whose second gain, the bound of its other nodes from above,
// reaches that is scanned again (a lazy greedy by tiles: delta only falls; by the first gain alone
// some thirty tiles a round were scanned, the hubs' deltas falling in every round).  A scan of all n nodes a round had read 13
// bytes a node: 33 us a round at 4M nodes and 2^25 samples, now 20 (15 without a tile to scan).
constexpr int PICK_TILES = 4; // tiles a thread looks at together, their loads issued first

struct PickShared {
    double g[GREEDY_BLOCK / 64];
    int32_t v[GREEDY_BLOCK / 64], d[GREEDY_BLOCK / 64];
    int32_t dirty[GREEDY_BLOCK * PICK_TILES];
    GreedyTile part[64 * (GREEDY_TILE / SCAN_PART)];
    int ndirty;
};

// (g, v, d) of the workgroup's best, in every thread; two barriers.
__device__ __forceinline__ void pick_reduce(double &g, int32_t &v, int32_t &d, PickShared &sh)
{
    const int32_t mine = v, md = d;
    wave_best(g, v);
    const int wave = threadIdx.x >> 6;
    if (v >= 0 && mine == v) sh.d[wave] = md; // one lane of the wave holds it
    if ((threadIdx.x & 63) == 0) {
        sh.g[wave] = g;
        sh.v[wave] = v;
    }
    __syncthreads();
    v = -1;
    for (int w = 0; w < GREEDY_BLOCK / 64; ++w)
        if (sh.v[w] >= 0 && better(sh.g[w], sh.v[w], g, v)) {
            g = sh.g[w];
            v = sh.v[w];
            d = sh.d[w];
        }
    __syncthreads();
}

template <bool LIVE>
__device__ __forceinline__ GreedyTile pick_node(GreedyTile *tiles, int32_t ntiles, int32_t n, uint64_t T, double Gamma,
                                                const int32_t *__restrict__ delta, const double *__restrict__ qv,
                                                const uint8_t *chosen, PickShared &sh)
{
    constexpr int PARTS = GREEDY_TILE / SCAN_PART;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    constexpr int32_t BATCH = GREEDY_BLOCK * PICK_TILES;
    GreedyTile c[PICK_TILES];
    int32_t d[PICK_TILES];
    bool gone[PICK_TILES];
    double q[PICK_TILES];
    auto look = [&](int32_t t0) { // tiles t0 + u * GREEDY_BLOCK + tid: the cached node, its delta now
#pragma unroll
        for (int u = 0; u < PICK_TILES; ++u) c[u] = tiles[min(t0 + u * GREEDY_BLOCK + tid, ntiles - 1)];
#pragma unroll
        for (int u = 0; u < PICK_TILES; ++u) {
            const int32_t v = max(c[u].v, 0);
            gone[u] = c[u].v < 0 || chosen[v];
            d[u] = LIVE ? __hip_atomic_load(&delta[v], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : delta[v];
            q[u] = qv ? qv[v] : 0.0;
        }
    };
    // the lower bound: the cached nodes' gains now
    double bg = 0.0;
    int32_t bv = -1, bd = 0;
    for (int32_t t0 = 0; t0 < ntiles; t0 += BATCH) {
        look(t0);
#pragma unroll
        for (int u = 0; u < PICK_TILES; ++u) {
            if (t0 + u * GREEDY_BLOCK + tid >= ntiles || gone[u]) continue;
            const double g = d[u] == c[u].d ? c[u].g : gain_of(d[u], T, Gamma, q[u]);
            if (better(g, c[u].v, bg, bv)) {
                bg = g;
                bv = c[u].v;
                bd = d[u];
            }
        }
    }
    pick_reduce(bg, bv, bd, sh);
    const double low = bv >= 0 ? bg : 0.0; // gains are not negative
    // scan the changed tiles that may hold a better one
    for (int32_t t0 = 0; t0 < ntiles; t0 += BATCH) {
        if (tid == 0) sh.ndirty = 0;
        __syncthreads();
        if (ntiles > BATCH) look(t0); // else the registers still hold them
#pragma unroll
        for (int u = 0; u < PICK_TILES; ++u) {
            const int32_t t = t0 + u * GREEDY_BLOCK + tid;
            if (t < ntiles && c[u].v >= 0 && (gone[u] || d[u] != c[u].d) && c[u].g2 >= low)
                sh.dirty[atomicAdd(&sh.ndirty, 1)] = t;
        }
        __syncthreads();
        const int nd = sh.ndirty;
        for (int b0 = 0; b0 < nd; b0 += 64) {
            const int nb = min(nd - b0, 64);
            for (int i = wave; i < nb * PARTS; i += GREEDY_BLOCK / 64) {
                const int64_t v0 = (int64_t)sh.dirty[b0 + i / PARTS] * GREEDY_TILE + (int64_t)(i % PARTS) * SCAN_PART;
                GreedyTile e = NO_TILE;
                if (v0 < n) e = scan_part<LIVE>(v0, n, T, Gamma, delta, qv, chosen);
                if (lane == 0) sh.part[i] = e;
            }
            __syncthreads();
            if (tid < nb) {
                GreedyTile best = sh.part[tid * PARTS];
                for (int k = 1; k < PARTS; ++k) merge_part(best, sh.part[tid * PARTS + k]);
                tiles[sh.dirty[b0 + tid]] = best;
                if (best.v >= 0 && better(best.g, best.v, bg, bv)) {
                    bg = best.g;
                    bv = best.v;
                    bd = best.d;
                }
            }
            __syncthreads();
        }
    }
    // every thread starts from the lower bound's node: the same node in several lanes is one node
    pick_reduce(bg, bv, bd, sh);
    GreedyTile r = NO_TILE;
    r.g = bg;
    r.v = bv;
    r.d = bd;
    return r;
}

// delta lives in two buffers: a round that recounts writes the spare one (kept zero), the next
// argmax switches to it, and that round's cover clears the one it leaves.  few: the entries of a small
// sketch (else 0), whose rounds go over to k_greedy_small once the last one has lowered few entries or
// few are left.
__global__ __launch_bounds__(GREEDY_BLOCK) void k_greedy_argmax(int32_t n, int round, int32_t k, uint64_t recount, uint32_t few, uint64_t T,
                                                                double Gamma,
                                                                int32_t *__restrict__ delta0,
                                                                int32_t *__restrict__ delta1,
                                                                const double *__restrict__ qv,
                                                                uint8_t *__restrict__ chosen,
                                                                GreedyTile *__restrict__ tiles, int32_t ntiles,
                                                                GreedyState *__restrict__ st,
                                                                uint32_t *__restrict__ left_parts,
                                                                int32_t *__restrict__ seeds,
                                                                unsigned long long *__restrict__ marg)
{
    __shared__ PickShared sh;
    uint32_t left = 0;
    if (few) {
        const int lane = threadIdx.x & 63;
        left = wave_sum(lane < GREEDY_LEFT_PARTS ? left_parts[lane * GREEDY_LEFT_STEP] : 0u);
        if (st->light || greedy_few(st, left, k - round, n)) { // (light is the only word written: a late reader agrees)
            if (threadIdx.x == 0) st->light = 1u;
            return;
        }
    }
    const bool recounted = heavy_round(st, recount); // the previous round
    const int cur = st->cur ^ (recounted ? 1 : 0);
    const int32_t *delta = cur ? delta1 : delta0;
    const GreedyTile b = pick_node<false>(tiles, ntiles, n, T, Gamma, delta, qv, chosen, sh);
    // every thread has read st and the parts (the reductions' barriers)
    if (few && threadIdx.x < GREEDY_LEFT_PARTS) left_parts[threadIdx.x * GREEDY_LEFT_STEP] = 0u;
    if (threadIdx.x == 0) {
        st->rounds += 1;
        st->before = round ? left : few;
        st->flipped = recounted ? 1u : 0u;
        if (recounted) {
            st->shrunk = 1u; // the previous round rewrote the spans
            st->cur = cur;
        }
        st->vstar = b.v;
        if (b.v < 0) return; // nothing left to pick (cannot happen for k <= n)
        st->dstar = (unsigned long long)b.d;
        seeds[round] = b.v;
        marg[round] = (unsigned long long)b.d;
        chosen[b.v] = 1;
        st->cov += (unsigned long long)b.d;
    }
}

// All tiles scanned once (delta, no node chosen).
__global__ __launch_bounds__(256) void k_greedy_tiles(int32_t n, uint64_t T, double Gamma,
                                                      const int32_t *__restrict__ delta,
                                                      const double *__restrict__ qv,
                                                      const uint8_t *__restrict__ chosen,
                                                      GreedyTile *__restrict__ tiles, int32_t ntiles)
{
    __shared__ GreedyTile part[4];
    static_assert(GREEDY_TILE / SCAN_PART == 4, "a wave for each part of a tile");
    for (int64_t t = blockIdx.x; t < ntiles; t += gridDim.x) {
        const int w = threadIdx.x >> 6;
        const int64_t v0 = t * GREEDY_TILE + (int64_t)w * SCAN_PART;
        GreedyTile c = NO_TILE;
        if (v0 < n) c = scan_part<false>(v0, n, T, Gamma, delta, qv, chosen);
        if ((threadIdx.x & 63) == 0) part[w] = c;
        __syncthreads();
        if (threadIdx.x == 0) {
            for (int k = 1; k < 4; ++k) merge_part(c, part[k]);
            tiles[t] = c;
        }
        __syncthreads();
    }
}

// The light rounds of a small sketch (D-SSA's) in one workgroup: three launches a round had cost more
// than their work (D-SSA with k = 100 on the 4M-node TRI graph: 29.7 ms before, 18.6 now).  The tiles
// live in LDS; a round picks, covers H(v*) through LDS queues and lowers delta by atomics.  A hub's round
// is some 1.5 ns an entry lowered for one workgroup, which the first picks mostly are, so those are the
// whole device's (see greedy_few).  k = 1, 5, 20 and 100 on 500 thousand entries, 100 thousand nodes (WC):
// 0.15, 0.31, 0.98 and 3.5 ms by launches alone, 0.90, 1.27, 1.70 and 2.9 by the one workgroup alone, 0.14,
// 0.27, 0.78 and 2.0 so; on 460 thousand, 4M nodes (TRI): 0.21, 0.72, 2.6, 8.4; 0.67, 0.91, 1.29, 2.85; 0.20,
// 0.40, 0.80, 2.4.
constexpr int SMALL_QUEUE = 4096;

__global__ __launch_bounds__(GREEDY_BLOCK) void k_greedy_small(int32_t n, int32_t k, uint64_t T, double Gamma,
                                                               int32_t *__restrict__ delta0,
                                                               int32_t *__restrict__ delta1,
                                                               const double *__restrict__ qv,
                                                               uint8_t *__restrict__ chosen,
                                                               const GreedyTile *__restrict__ tiles_in, int32_t ntiles,
                                                               const int64_t *__restrict__ node_ptr,
                                                               const int32_t *__restrict__ node_samples,
                                                               uint32_t *__restrict__ covered,
                                                               const int64_t *__restrict__ sptr,
                                                               const int32_t *__restrict__ nodes,
                                                               int32_t *__restrict__ seeds,
                                                               unsigned long long *__restrict__ marg,
                                                               GreedyState *__restrict__ st)
{
    __shared__ PickShared sh;
    __shared__ GreedyTile tiles[GREEDY_SMALL_TILES];
    // samples newly covered (first entry, entries): entries are below 2^31 here
    __shared__ int2 queue[SMALL_QUEUE], bigq[SMALL_QUEUE];
    __shared__ int s_q, s_big;
    const int tid = threadIdx.x;
    const int32_t r0 = st->rounds; // taken by the launches before, which all recounted
    if (r0 >= k) return;
    int32_t *const delta = (st->cur ^ (r0 > 0 ? 1 : 0)) ? delta1 : delta0; // as k_greedy_argmax
    unsigned long long cov = st->cov;
    for (int t = tid; t < ntiles; t += GREEDY_BLOCK) tiles[t] = tiles_in[t];
    __syncthreads();
    for (int32_t r = r0; r < k; ++r) {
        const GreedyTile p = pick_node<true>(tiles, ntiles, n, T, Gamma, delta, qv, chosen, sh);
        if (p.v < 0) { // nothing left to pick (cannot happen for k <= n)
            if (tid == 0) st->vstar = -1;
            return;
        }
        if (tid == 0) {
            seeds[r] = p.v;
            marg[r] = (unsigned long long)p.d;
            chosen[p.v] = 1;
            st->vstar = p.v;
            s_q = 0;
            s_big = 0;
        }
        cov += (unsigned long long)p.d;
        // the pick's own delta is not read any more, and every sample would lower it (atomics on one
        // address take 9.4 ns each)
        auto lower = [&](int32_t u) {
            if (u != p.v) atomicSub(&delta[u], 1);
        };
        const int64_t a = node_ptr[p.v], b = p.d > 0 ? node_ptr[p.v + 1] : a;
        __syncthreads();
        for (int64_t c0 = a; c0 < b; c0 += SMALL_QUEUE) {
            for (int64_t e = c0 + tid; e < min(c0 + (int64_t)SMALL_QUEUE, b); e += GREEDY_BLOCK) {
                const int32_t j = node_samples[e];
                const uint32_t bit = 1u << (j & 31);
                if (atomicOr(&covered[j >> 5], bit) & bit) continue;
                const int e0 = (int)sptr[j], len = (int)sptr[j + 1] - e0;
                if (len > GREEDY_BIG) bigq[atomicAdd(&s_big, 1)] = make_int2(e0, len);
                else queue[atomicAdd(&s_q, 1)] = make_int2(e0, len);
            }
            __syncthreads();
            const int nq = s_q, nb = s_big;
            for (int i = tid >> 4; i < nq; i += GREEDY_BLOCK / 16) { // 16 lanes a sample
                const int2 x = queue[i];
                for (int t = tid & 15; t < x.y; t += 16) lower(nodes[x.x + t]);
            }
            for (int i = 0; i < nb; ++i) {
                const int2 x = bigq[i];
                for (int t = tid; t < x.y; t += GREEDY_BLOCK) lower(nodes[x.x + t]);
            }
            __syncthreads();
            if (tid == 0) {
                s_q = 0;
                s_big = 0;
            }
            __syncthreads();
        }
        __threadfence(); // delta's atomics are performed before the next round reads it
        __syncthreads();
    }
    if (tid == 0) st->cov = cov;
}

// Covers H(v*).  H(v*) is in ascending sample order; in a round that recounts, each lane takes a run
// of MARK_RUN consecutive entries and sets the bits of one bitmap word with one atomicOr.  In a
// round that does not, each wave queues the samples it newly covered in LDS and lowers delta of
// every member of each (16 lanes per sample); the most frequent nodes (the transpose's hot
// list) are decremented in LDS per workgroup and flushed once, so hubs do not serialise on
// one counter.  Integer updates commute, so delta and the picks are exact.  The number of
// samples a round newly covers is delta of its pick, known before the round starts.
constexpr int MARK_RUN = 8;

__global__ __launch_bounds__(256) void k_greedy_cover(const GreedyState *__restrict__ st, uint64_t recount, int32_t n,
                                                      const int64_t *__restrict__ node_ptr,
                                                      const int32_t *__restrict__ node_samples,
                                                      uint32_t *__restrict__ covered,
                                                      const int64_t *__restrict__ sptr,
                                                      const int32_t *__restrict__ nodes,
                                                      const int32_t *__restrict__ hot_id,
                                                      const int32_t *__restrict__ hot_node, int nhot,
                                                      int32_t *__restrict__ delta0, int32_t *__restrict__ delta1)
{
    __shared__ int32_t hd[GREEDY_HOT];
    __shared__ CoverItem queue[4][64 * MARK_RUN]; // the newly covered samples
    const int32_t v = st->vstar;
    if (v < 0 || st->light) return;
    const bool update = !heavy_round(st, recount);
    int32_t *delta = st->cur ? delta1 : delta0;
    if (st->flipped) { // the buffer that this round's argmax left
        int32_t *spare = st->cur ? delta0 : delta1;
        for (int64_t u = (int64_t)blockIdx.x * 256 + threadIdx.x; u < n; u += (int64_t)gridDim.x * 256) spare[u] = 0;
    }
    if (update)
        for (int h = threadIdx.x; h < nhot; h += 256) hd[h] = 0;
    __syncthreads();
    const int64_t a = node_ptr[v], b = node_ptr[v + 1];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) >> 6;
    if (!update) {
        for (int64_t c0 = a + wave * 64 * MARK_RUN; c0 < b; c0 += nwaves * 64 * MARK_RUN) {
            const int64_t r0 = c0 + (int64_t)lane * MARK_RUN;
            int32_t js[MARK_RUN];
            int n = 0;
#pragma unroll
            for (int k = 0; k < MARK_RUN; ++k) {
                js[k] = r0 + k < b ? node_samples[r0 + k] : -1;
                n += js[k] >= 0 ? 1 : 0;
            }
            int k = 0;
            while (k < n) { // one word at a time: a heavy pick's list is dense
                const int32_t word = js[k] >> 5;
                uint32_t bits = 0;
                while (k < n && (js[k] >> 5) == word) bits |= 1u << (js[k++] & 31);
                atomicOr(&covered[word], bits);
            }
        }
        return;
    }
    // a light round: most of the list is covered already, so the words are read first, all at once,
    // and only bits still clear are set by atomics, all at once again (one word after the other had
    // cost a memory latency each: 91 us a round on average at 2^25 samples, now 70)
    CoverItem *q = queue[wid];
    for (int64_t c0 = a + wave * 64 * MARK_RUN; c0 < b; c0 += nwaves * 64 * MARK_RUN) { // uniform per wave
        int32_t js[MARK_RUN];
        uint32_t wd[MARK_RUN], old[MARK_RUN];
#pragma unroll
        for (int k = 0; k < MARK_RUN; ++k) {
            const int64_t e = c0 + k * 64 + lane;
            js[k] = node_samples[e < b ? e : b - 1];
        }
#pragma unroll
        for (int k = 0; k < MARK_RUN; ++k)
            wd[k] = c0 + k * 64 + lane < b ? covered[js[k] >> 5] : 0xFFFFFFFFu;
#pragma unroll
        for (int k = 0; k < MARK_RUN; ++k) {
            const uint32_t bit = 1u << (js[k] & 31);
            old[k] = 0xFFFFFFFFu;
            if (!(wd[k] & bit)) old[k] = atomicOr(&covered[js[k] >> 5], bit);
        }
        uint32_t fresh = 0; // bit k: js[k] newly covered
#pragma unroll
        for (int k = 0; k < MARK_RUN; ++k) fresh |= ((old[k] >> (js[k] & 31)) & 1u) ? 0u : 1u << k;
        const int cnt = __popc(fresh);
        const int incl = wave_incl_scan(cnt);
        const int tot = (int)lane_value((uint32_t)incl, 63);
        if (!tot) continue;
        int pos = incl - cnt;
#pragma unroll
        for (int t = 0; t < MARK_RUN; ++t)
            if (fresh & (1u << t)) q[pos++].set(sptr[js[t]], sptr[js[t] + 1]);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const int g = lane >> 4, gl = lane & 15; // 4 samples at a time, 16 lanes each
        for (int i0 = 0; i0 < tot; i0 += 4) {
            const int i = i0 + g;
            if (i >= tot) continue;
            const int64_t sa = q[i].first();
            const int len = q[i].len();
            for (int t = gl; t < len; t += 16) {
                const int32_t u = nodes[sa + t];
                const int32_t h = hot_id ? hot_id[u] : -1;
                if (h >= 0) atomicSub(&hd[h], 1);
                else atomicSub(&delta[u], 1);
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront"); // the queue is reused next
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
    __syncthreads();
    for (int h = threadIdx.x; h < nhot; h += 256)
        if (hd[h]) atomicAdd(&delta[hot_node[h]], hd[h]);
}

// Work items for the recount: each node's list cut into spans of RECOUNT_SPAN entries.
__global__ __launch_bounds__(256) void k_recount_items_count(int32_t n, const int64_t *__restrict__ node_ptr,
                                                             uint32_t *__restrict__ nitems)
{
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += (int64_t)gridDim.x * blockDim.x) {
        const int64_t d = node_ptr[v + 1] - node_ptr[v];
        nitems[v] = (uint32_t)((d + RECOUNT_SPAN - 1) / RECOUNT_SPAN);
    }
}

__global__ __launch_bounds__(256) void k_recount_items_fill(int32_t n, const int64_t *__restrict__ node_ptr,
                                                            const uint32_t *__restrict__ nitems,
                                                            const int64_t *__restrict__ ioff,
                                                            RecountItem *__restrict__ items)
{
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += (int64_t)gridDim.x * blockDim.x) {
        const int64_t a = node_ptr[v], d = node_ptr[v + 1] - a;
        for (uint32_t c = 0; c < nitems[v]; ++c) {
            RecountItem w;
            w.p0 = a + (int64_t)c * RECOUNT_SPAN;
            w.len = (int32_t)min<int64_t>(RECOUNT_SPAN, d - (int64_t)c * RECOUNT_SPAN);
            w.v = (int32_t)v;
            items[ioff[v] + c] = w;
        }
    }
}

// delta[v] += #{ j in span : j not covered }, and the span is cut down to those samples:
// the first heavy round reads node v's list from the sketch and writes the uncovered part
// to the same offsets of `work`; later heavy rounds read and rewrite `work` in place (a kept
// entry only moves to a lower position, after every load of its batch).  The order within
// a span stays ascending.  RECOUNT_LANES lanes per span, RECOUNT_UNROLL list loads and then
// as many bitmap loads in flight per lane.
__global__ __launch_bounds__(256) void k_greedy_recount(const GreedyState *__restrict__ st, uint64_t recount, uint32_t *__restrict__ left_parts,
                                                        uint64_t nitems, RecountItem *__restrict__ items,
                                                        const int32_t *node_samples, int32_t *work,
                                                        const uint32_t *__restrict__ covered,
                                                        int32_t *__restrict__ delta0, int32_t *__restrict__ delta1)
{
    __shared__ uint32_t s_left[4];
    uint32_t left = 0; // entries kept
    if (st->light || !heavy_round(st, recount)) return;
    int32_t *delta = st->cur ? delta0 : delta1; // the spare buffer, all zero; the next argmax switches
    const int32_t *src = st->shrunk ? work : node_samples;
    constexpr int G = 64 / RECOUNT_LANES;
    const int lane = threadIdx.x & 63, grp = lane / RECOUNT_LANES, t = lane % RECOUNT_LANES;
    const uint64_t below = (1ull << t) - 1ull;
    const uint64_t wave = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const uint64_t nwaves = ((uint64_t)gridDim.x * blockDim.x) >> 6;
    for (uint64_t b0 = wave * G; b0 < nitems; b0 += nwaves * G) { // uniform over the wave
        const uint64_t it = b0 + grp;
        RecountItem w;
        w.p0 = 0;
        w.len = 0;
        w.v = -1;
        if (it < nitems) w = items[it];
        int kept = 0; // same in every lane of the group
        for (int q0 = 0; q0 < w.len; q0 += RECOUNT_LANES * RECOUNT_UNROLL) {
            int32_t js[RECOUNT_UNROLL];
#pragma unroll
            for (int u = 0; u < RECOUNT_UNROLL; ++u) {
                const int q = q0 + u * RECOUNT_LANES + t;
                js[u] = q < w.len ? src[w.p0 + q] : -1;
            }
            uint32_t wd[RECOUNT_UNROLL];
#pragma unroll
            for (int u = 0; u < RECOUNT_UNROLL; ++u) wd[u] = js[u] >= 0 ? covered[js[u] >> 5] : 0xffffffffu;
#pragma unroll
            for (int u = 0; u < RECOUNT_UNROLL; ++u) {
                const bool keep = !((wd[u] >> (js[u] & 31)) & 1u);
                const uint64_t m = (__ballot(keep) >> (grp * RECOUNT_LANES)) & 0xffffull;
                if (keep) work[w.p0 + kept + __popcll(m & below)] = js[u];
                kept += __popcll(m);
            }
        }
        if (t == 0 && it < nitems) {
            items[it].len = kept;
            if (kept) atomicAdd(&delta[w.v], kept);
            left += (uint32_t)kept;
        }
    }
    if (left_parts) {
        left = wave_sum(left);
        if (lane == 0) s_left[threadIdx.x >> 6] = left;
        __syncthreads();
        if (threadIdx.x == 0 && (left = s_left[0] + s_left[1] + s_left[2] + s_left[3]))
            atomicAdd(&left_parts[blockIdx.x % GREEDY_LEFT_PARTS * GREEDY_LEFT_STEP], left);
    }
}

// second term of Eq. margin summed over the k picks (each node is picked at most once)
__global__ __launch_bounds__(256) void k_greedy_final(int32_t k, uint64_t T, double Gamma,
                                                      const int32_t *__restrict__ seeds, const double *__restrict__ qv,
                                                      GreedyState *__restrict__ st)
{
    __shared__ double ps[256], pc[256];
    double s = 0.0, c = 0.0;
    if (qv)
        for (int32_t r = threadIdx.x; r < k; r += 256) neumaier_add(s, c, qv[seeds[r]]);
    ps[threadIdx.x] = s;
    pc[threadIdx.x] = c;
    __syncthreads();
    if (threadIdx.x == 0) {
        double ts = 0.0, tc = 0.0;
        for (int t = 0; t < 256; ++t) {
            neumaier_add(ts, tc, ps[t]);
            neumaier_add(ts, tc, pc[t]);
        }
        const double first = T > 0 ? __ddiv_rn(__dmul_rn((double)st->cov, Gamma), (double)T) : 0.0;
        st->est = __dadd_rn(first, __dadd_rn(ts, tc));
    }
}

template <typename T>
__global__ __launch_bounds__(256) void k_fill_q(uint64_t count, T *__restrict__ p, T v)
{
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += (uint64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

static unsigned gridq(uint64_t items, int block, int per_cu = 8)
{
    uint64_t g = (items + block - 1) / block;
    const uint64_t cap = (uint64_t)device_cu_count() * per_cu;
    if (g > cap) g = cap;
    return (unsigned)(g > 0 ? g : 1);
}

// Sixteen bytes of flags in pinned host memory that a kernel writes and the host reads after a
// synchronisation (a copy from the device and the fill before it had taken 20 us of a small
// estimate): one page for the process, made with the first inverse index, a call holds one of its
// places.  host is null when every place is taken or there is no page; the caller then keeps its
// flags on the device.
namespace {
class HostFlags {
    static constexpr int PLACES = 64;
    struct Page {
        std::mutex mu;
        char *base = nullptr;
        bool tried = false;
        bool used[PLACES] = {};
    };
    static Page &page()
    {
        static Page p;
        return p;
    }
    int at = -1;

public:
    EstFlags *host = nullptr, *dev = nullptr;
    static void make_page()
    {
        Page &p = page();
        std::lock_guard<std::mutex> g(p.mu);
        if (p.tried) return;
        p.tried = true;
        void *m = nullptr;
        if (hipHostMalloc(&m, 64 * PLACES, hipHostMallocPortable | hipHostMallocMapped) == hipSuccess)
            p.base = static_cast<char *>(m);
        (void)hipGetLastError();
    }
    HostFlags()
    {
        Page &p = page();
        std::lock_guard<std::mutex> g(p.mu);
        if (!p.base) return;
        for (int i = 0; i < PLACES && at < 0; ++i)
            if (!p.used[i]) at = i;
        if (at < 0) return;
        host = reinterpret_cast<EstFlags *>(p.base + 64 * at);
        void *d = nullptr;
        if (hipHostGetDevicePointer(&d, host, 0) != hipSuccess) {
            (void)hipGetLastError();
            host = nullptr;
            at = -1;
            return;
        }
        dev = static_cast<EstFlags *>(d);
        p.used[at] = true;
        *host = EstFlags{};
    }
    HostFlags(const HostFlags &) = delete;
    HostFlags &operator=(const HostFlags &) = delete;
    ~HostFlags()
    {
        if (at < 0) return;
        Page &p = page();
        std::lock_guard<std::mutex> g(p.mu);
        p.used[at] = false;
    }
};
} // namespace

void make_flags_page() { HostFlags::make_page(); }

EstFlags estimate_light(const Sketch &sk, int32_t nq, bool check, const int64_t *set_ptr, const int32_t *set_nodes,
                        unsigned long long *cov, double *est, uint32_t *ticket, EstFlags *spare, hipStream_t s)
{
    EstFlags fl{};
    if (nq <= 0) return fl;
    if (check && nq > EST_BLOCK) throw Error{SKIS_EHIP, "internal error: too many sets for a checked estimate"};
    HostFlags hf;
    EstFlags *const dev = hf.dev ? hf.dev : spare;
    if (!hf.dev)
        hipLaunchKernelGGL(k_fill_q<int>, dim3(1), dim3(64), 0, s, (uint64_t)(sizeof(EstFlags) / sizeof(int)),
                           reinterpret_cast<int *>(dev), 0);
    try {
        hipLaunchKernelGGL(k_est_set<false>, dim3((unsigned)nq), dim3(EST_BLOCK), 0, s, check ? nq : 0, set_ptr, set_nodes,
                           sk.n, sk.T, sk.est_scale(), sk.est_q(), sk.node_ptr.ptr, sk.node_samples.ptr, cov, est, ticket,
                           (uint32_t *)nullptr, (uint64_t)0, dev);
        SKIS_HIP_TRY(hipGetLastError());
        if (!hf.dev) SKIS_HIP_TRY(hipMemcpyAsync(&fl, dev, sizeof(fl), hipMemcpyDeviceToHost, s));
        SKIS_HIP_TRY(hipStreamSynchronize(s));
    } catch (...) {
        (void)hipStreamSynchronize(s); // nothing may write the flags' place after it is given back
        throw;
    }
    if (hf.dev) {
        const volatile EstFlags *h = hf.host;
        fl.ptr = h->ptr;
        fl.node = h->node;
        fl.large = h->large;
        fl.parked = h->parked;
    }
    return fl;
}

void estimate_split(const Sketch &sk, int32_t nq, const int64_t *set_ptr, const int32_t *set_nodes,
                    unsigned long long *cov, double *est, uint32_t *heavy, uint32_t *ticket, hipStream_t s)
{
    if (nq <= 0 || sk.T == 0) return;
    hipLaunchKernelGGL(k_est_list, dim3(1), dim3(EST_BLOCK), 0, s, nq, cov, heavy);
    // windows of whole words, the last one ragged
    uint64_t wbits = (sk.T + SPLIT_WINDOWS - 1) / SPLIT_WINDOWS;
    wbits = std::min<uint64_t>(std::max<uint64_t>((wbits + 31) / 32 * 32, SPLIT_MIN), SPLIT_BITS);
    const uint64_t windows = (sk.T + wbits - 1) / wbits;
    const uint64_t grid = std::min<uint64_t>((uint64_t)device_cu_count() * 2, (uint64_t)nq * windows);
    hipLaunchKernelGGL(k_est_split, dim3((unsigned)grid), dim3(EST_BLOCK), 0, s, (int32_t)windows, (int32_t)wbits,
                       set_ptr, set_nodes, sk.T, sk.est_scale(), sk.node_ptr.ptr, sk.node_samples.ptr, heavy, cov, est,
                       ticket);
    SKIS_HIP_TRY(hipGetLastError());
}

void estimate_batch(const Sketch &sk, QueryScratch &qs, int32_t Q, const int64_t *set_ptr, const int32_t *set_nodes,
                    uint64_t *cov_out, double *est, hipStream_t s)
{
    Arena &arena = const_cast<Arena &>(sk.arena);
    unsigned long long *const cov = reinterpret_cast<unsigned long long *>(cov_out);
    // set sizes on the host: argument checks and the list of sets above one LDS chunk.  Up to
    // EST_BLOCK sets are checked by the kernel instead, and read here only if one is that large
    std::vector<int64_t> hptr, large;
    auto read_sets = [&]() {
        hptr.resize((size_t)Q + 1);
        SKIS_HIP_TRY(hipMemcpyAsync(hptr.data(), set_ptr, sizeof(int64_t) * ((size_t)Q + 1), hipMemcpyDeviceToHost, s));
        SKIS_HIP_TRY(hipStreamSynchronize(s));
        for (int32_t i = 0; i < Q; ++i) {
            const int64_t k = hptr[i + 1] - hptr[i];
            if (k < 0 || hptr[i] < 0) throw Error{SKIS_EINVAL, "set_ptr must be nondecreasing from 0"};
            if (k > EST_MAX_SET) large.push_back(i);
        }
        if (hptr[Q] > 0 && !set_nodes) throw Error{SKIS_EINVAL, "set_nodes must not be NULL"};
    };
    const bool device_check = Q <= EST_BLOCK && set_nodes;
    if (!device_check) read_sets();
    // EST_ROUND sets at a time, so that a call of any number of sets needs half a megabyte of scratch
    constexpr size_t FLAGS = sizeof(EstFlags) / sizeof(uint32_t);
    const int32_t most = std::min<int32_t>(Q, EST_ROUND);
    const size_t need = 2 * (size_t)most + 1 + FLAGS; // heavy = {count, sets}, tickets, flags
    if (qs.split.count < need) qs.split.alloc(arena, need);
    uint32_t *const heavy = qs.split.ptr, *const ticket = heavy + most + 1;
    EstFlags *const spare = reinterpret_cast<EstFlags *>(ticket + most);
    bool any_large = false, any_parked = false;
    for (int64_t c0 = 0; c0 < Q; c0 += EST_ROUND) {
        const int32_t ch = (int32_t)std::min<int64_t>(EST_ROUND, Q - c0);
        const EstFlags fl = estimate_light(sk, ch, device_check, set_ptr + c0, set_nodes, cov + c0, est + c0, ticket, spare, s);
        if (fl.ptr) throw Error{SKIS_EINVAL, "set_ptr must be nondecreasing from 0"};
        if (fl.node) throw Error{SKIS_EINVAL, "a seed set holds a node id outside [0, n)"};
        if (fl.parked) estimate_split(sk, ch, set_ptr + c0, set_nodes, cov + c0, est + c0, heavy, ticket, s);
        any_large = any_large || fl.large;
        any_parked = any_parked || fl.parked;
    }
    if (any_large) {
        if (hptr.empty()) read_sets();
        if (!qs.err.ptr) qs.err.alloc(arena, 1);
        hipLaunchKernelGGL(k_fill_q<int>, dim3(1), dim3(64), 0, s, (uint64_t)1, qs.err.ptr, 0);
        const uint64_t per = std::max<uint64_t>((sk.T + 31) / 32, 1);
        const uint64_t wordsN = ((uint64_t)sk.n + 31) / 32;
        // bitmaps for up to 64 sets at a time, about 256 MiB
        uint64_t group = std::max<uint64_t>((256ull << 20) / (per * 4), 1);
        group = std::min<uint64_t>(std::min<uint64_t>(group, 64), large.size());
        if (qs.bitmaps.count < group * per) {
            qs.bitmaps.alloc(arena, group * per);
            hipLaunchKernelGGL(k_fill_q<uint32_t>, dim3(gridq(group * per, 256)), dim3(256), 0, s, group * per,
                               qs.bitmaps.ptr, 0u);
            SKIS_HIP_TRY(hipGetLastError());
        }
        DevBuf<int64_t> qlist;
        DevBuf<uint32_t> nodebits;
        qlist.alloc(arena, large.size());
        nodebits.alloc(arena, group * wordsN);
        SKIS_HIP_TRY(hipMemcpyAsync(qlist.ptr, large.data(), sizeof(int64_t) * large.size(), hipMemcpyHostToDevice, s));
        hipLaunchKernelGGL(k_fill_q<uint32_t>, dim3(gridq(group * wordsN, 256)), dim3(256), 0, s, group * wordsN,
                           nodebits.ptr, 0u);
        for (uint64_t g0 = 0; g0 < large.size(); g0 += group)
            estimate_launch_large(sk, qlist.ptr, (int64_t)g0, (int32_t)std::min<uint64_t>(group, large.size() - g0),
                                  set_ptr, set_nodes, qs.bitmaps.ptr, per, nodebits.ptr, cov, est, qs.err.ptr, s);
        int herr = 0;
        SKIS_HIP_TRY(hipMemcpyAsync(&herr, qs.err.ptr, sizeof(int), hipMemcpyDeviceToHost, s));
        SKIS_HIP_TRY(hipStreamSynchronize(s));
        if (herr) {
            // a workgroup that stopped early may have left bits set: clear all scratch
            hipLaunchKernelGGL(k_fill_q<uint32_t>, dim3(gridq(qs.bitmaps.count, 256)), dim3(256), 0, s, (uint64_t)qs.bitmaps.count,
                               qs.bitmaps.ptr, 0u);
            SKIS_HIP_TRY(hipStreamSynchronize(s));
        }
        if (herr & 1) throw Error{SKIS_EINVAL, "set_ptr must be nondecreasing"};
        if (herr & 4) throw Error{SKIS_EINVAL, "a seed set holds a node id outside [0, n)"};
    } else if (any_parked) {
        SKIS_HIP_TRY(hipStreamSynchronize(s));
    }
}

void estimate_launch(const Sketch &sk, int32_t nq, const int64_t *set_ptr, const int32_t *set_nodes,
                     const int64_t *large, int32_t nlarge, uint32_t *bitmaps, uint64_t bitmap_words,
                     uint32_t *nodebits, unsigned long long *cov, double *est, int *err, EstFlags *flags, hipStream_t s)
{
    if (nq > nlarge) {
        hipLaunchKernelGGL(k_est_set<true>, dim3((unsigned)nq), dim3(EST_BLOCK), 0, s, 0, set_ptr, set_nodes, sk.n, sk.T,
                           sk.est_scale(), sk.est_q(), sk.node_ptr.ptr, sk.node_samples.ptr, cov, est, (uint32_t *)nullptr,
                           bitmaps, bitmap_words, flags);
        SKIS_HIP_TRY(hipGetLastError());
    }
    estimate_launch_large(sk, large, 0, nlarge, set_ptr, set_nodes, bitmaps, bitmap_words, nodebits, cov, est, err, s);
}

void estimate_launch_large(const Sketch &sk, const int64_t *qlist, int64_t g0, int32_t ng, const int64_t *set_ptr,
                           const int32_t *set_nodes, uint32_t *bitmaps, uint64_t bitmap_words, uint32_t *nodebits,
                           unsigned long long *cov, double *est, int *err, hipStream_t s)
{
    if (ng <= 0) return;
    const uint64_t wordsN = ((uint64_t)sk.n + 31) / 32;
    hipLaunchKernelGGL(k_estimate, dim3((unsigned)ng), dim3(EST_BLOCK), 0, s, qlist, g0, set_ptr, set_nodes,
                       sk.n, sk.T, sk.est_scale(), sk.est_q(), sk.node_ptr.ptr, sk.node_samples.ptr, bitmaps, bitmap_words,
                       nodebits, wordsN, cov, est, err);
    SKIS_HIP_TRY(hipGetLastError());
}

void fill_u32(uint32_t *p, uint64_t count, hipStream_t s)
{
    hipLaunchKernelGGL(k_fill_q<uint32_t>, dim3(gridq(count, 256)), dim3(256), 0, s, count, p, 0u);
    SKIS_HIP_TRY(hipGetLastError());
}

void greedy(const Sketch &sk, QueryScratch &qs, int32_t k, int32_t *seeds, uint64_t *marg, uint64_t *cov_out,
            double *est_out, hipStream_t s)
{
    (void)qs;
    Arena &arena = const_cast<Arena &>(sk.arena);
    const int32_t n = sk.n;
    const uint64_t wordsT = (sk.T + 31) / 32;
    DevBuf<int32_t> delta, delta_spare; // the counts and the buffer a recounting round fills
    DevBuf<uint8_t> chosen;
    DevBuf<uint32_t> covered;
    DevBuf<GreedyState> st;
    const int32_t ntiles = (int32_t)(((int64_t)n + GREEDY_TILE - 1) / GREEDY_TILE);
    DevBuf<GreedyTile> tiles;
    tiles.alloc(arena, (size_t)ntiles);
    const bool small = sk.entries <= GREEDY_SMALL_ENTRIES && ntiles <= GREEDY_SMALL_TILES;
    // of a small sketch the whole device takes the first rounds, as many as may be worth it: all of 8,
    // else one for every GREEDY_SMALL_ROUND entries
    int32_t rounds = k;
    if (small && sk.entries <= (k > 1 ? GREEDY_FEW_LEFT : GREEDY_FEW_LEFT / 2)) rounds = 0;
    else if (small && k > 8) rounds = (int32_t)std::min<uint64_t>((uint64_t)k, sk.entries / GREEDY_SMALL_ROUND + 1);
    const uint64_t recount = small ? 0 : sk.T / RECOUNT_DIV + 1;
    const bool go_over = small && (rounds < k || worth_going_over(k - 1, n));
    const uint32_t few = go_over ? (uint32_t)sk.entries : 0u;
    delta.alloc(arena, n);
    if (rounds) delta_spare.alloc(arena, n);
    DevBuf<uint32_t> left;
    constexpr uint64_t LEFT_WORDS = GREEDY_LEFT_PARTS * GREEDY_LEFT_STEP;
    if (go_over && rounds) {
        left.alloc(arena, LEFT_WORDS);
        hipLaunchKernelGGL(k_fill_q<uint32_t>, dim3(1), dim3(256), 0, s, LEFT_WORDS, left.ptr, 0u);
    }
    chosen.alloc(arena, n);
    covered.alloc(arena, wordsT ? wordsT : 1);
    st.alloc(arena, 1);
    hipLaunchKernelGGL(k_greedy_init, dim3(gridq(n, 256)), dim3(256), 0, s, n, sk.node_ptr.ptr, delta.ptr, chosen.ptr);
    hipLaunchKernelGGL(k_fill_q<uint32_t>, dim3(gridq(wordsT ? wordsT : 1, 256)), dim3(256), 0, s,
                       wordsT ? wordsT : 1, covered.ptr, 0u);
    if (rounds)
        hipLaunchKernelGGL(k_fill_q<int32_t>, dim3(gridq(n, 256)), dim3(256), 0, s, (uint64_t)n, delta_spare.ptr, 0);
    hipLaunchKernelGGL(k_fill_q<unsigned char>, dim3(1), dim3(64), 0, s, (uint64_t)sizeof(GreedyState),
                       reinterpret_cast<unsigned char *>(st.ptr), (unsigned char)0);
    SKIS_HIP_TRY(hipGetLastError());
    hipLaunchKernelGGL(k_greedy_tiles, dim3(gridq((uint64_t)ntiles * 256, 256, 8)), dim3(256), 0, s, n, sk.T,
                       sk.est_scale(), delta.ptr, sk.est_q(), chosen.ptr, tiles.ptr, ntiles);
    const unsigned gu = (unsigned)device_cu_count() * 4;
    const int nhot = std::min<int>(sk.nhot, GREEDY_HOT);
    const int32_t *hot_id = nhot > 0 ? sk.hot_id.ptr : nullptr;
    // recount work items (used by the rounds that cover many samples)
    DevBuf<uint32_t> nitems;
    DevBuf<int64_t> ioff;
    DevBuf<RecountItem> items;
    DevBuf<int32_t> work; // the lists cut down by the heavy rounds
    uint64_t nit = 0;
    if (sk.T && rounds) {
        nitems.alloc(arena, n);
        ioff.alloc(arena, (size_t)n + 1);
        hipLaunchKernelGGL(k_recount_items_count, dim3(gridq(n, 256)), dim3(256), 0, s, n, sk.node_ptr.ptr,
                           nitems.ptr);
        excl_scan_u32_to_i64(arena, nitems.ptr, ioff.ptr, n, ioff.ptr + n, s);
        int64_t hn = 0;
        SKIS_HIP_TRY(hipMemcpyAsync(&hn, ioff.ptr + n, sizeof(hn), hipMemcpyDeviceToHost, s));
        SKIS_HIP_TRY(hipStreamSynchronize(s));
        nit = (uint64_t)hn;
        items.alloc(arena, nit ? nit : 1);
        work.alloc(arena, sk.entries ? sk.entries : 1);
        hipLaunchKernelGGL(k_recount_items_fill, dim3(gridq(n, 256)), dim3(256), 0, s, n, sk.node_ptr.ptr,
                           nitems.ptr, ioff.ptr, items.ptr);
        SKIS_HIP_TRY(hipGetLastError());
    }
    const unsigned gr = gridq(nit * RECOUNT_LANES, 256, 8);
    for (int32_t r = 0; r < rounds; ++r) {
        hipLaunchKernelGGL(k_greedy_argmax, dim3(1), dim3(GREEDY_BLOCK), 0, s, n, (int)r, k, recount, few, sk.T, sk.est_scale(),
                           delta.ptr, delta_spare.ptr, sk.est_q(), chosen.ptr, tiles.ptr, ntiles, st.ptr, left.ptr, seeds,
                           reinterpret_cast<unsigned long long *>(marg));
        if (sk.T) {
            // the cover lowers delta itself unless the round recounts, decided on the device
            hipLaunchKernelGGL(k_greedy_cover, dim3(gu), dim3(256), 0, s, st.ptr, recount, n, sk.node_ptr.ptr,
                               sk.node_samples.ptr, covered.ptr, sk.sample_ptr.ptr, sk.nodes.ptr, hot_id,
                               sk.hot_node.ptr, nhot, delta.ptr, delta_spare.ptr);
            hipLaunchKernelGGL(k_greedy_recount, dim3(gr), dim3(256), 0, s, st.ptr, recount, left.ptr, nit, items.ptr,
                               sk.node_samples.ptr, work.ptr, covered.ptr, delta.ptr, delta_spare.ptr);
        }
    }
    if (go_over)
        hipLaunchKernelGGL(k_greedy_small, dim3(1), dim3(GREEDY_BLOCK), 0, s, n, k, sk.T, sk.est_scale(), delta.ptr,
                           delta_spare.ptr, sk.est_q(), chosen.ptr, tiles.ptr, ntiles, sk.node_ptr.ptr, sk.node_samples.ptr,
                           covered.ptr, sk.sample_ptr.ptr, sk.nodes.ptr, seeds, reinterpret_cast<unsigned long long *>(marg),
                           st.ptr);
    SKIS_HIP_TRY(hipGetLastError());
    hipLaunchKernelGGL(k_greedy_final, dim3(1), dim3(256), 0, s, k, sk.T, sk.est_scale(), seeds, sk.est_q(), st.ptr);
    SKIS_HIP_TRY(hipGetLastError());
    GreedyState hs;
    SKIS_HIP_TRY(hipMemcpyAsync(&hs, st.ptr, sizeof(hs), hipMemcpyDeviceToHost, s));
    SKIS_HIP_TRY(hipStreamSynchronize(s));
    if (hs.vstar < 0) throw Error{SKIS_EHIP, "internal error: greedy ran out of candidates"};
    *cov_out = hs.cov;
    *est_out = hs.est;
}

} // namespace skis
