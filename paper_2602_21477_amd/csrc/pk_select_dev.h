// Device-side pieces of the selection kernels that other kernels take along: the radix
// selection over keys held in registers, and the threshold of one query from its sample
// (Section 2.2 fine search: the k-th best of a sample of the probed rows bounds the k-th best
// of all of them, so no row beyond it needs to be kept).
#pragma once

#include "pk_internal.h"

namespace pk {

// The K-th smallest (K counts from 1) of the keys that the 256 threads of a workgroup hold in registers
// (key[j] takes part if live[j]; K is at most the number of live keys), found digit by digit: four
// 8-bit passes over LDS histograms with one barrier each; every wave works out each digit for itself.
// hist: LDS [4][256], need not be initialised.  Returns that key; of the `ties` keys equal to it, `left`
// belong to the K smallest.
template <int VPT>
__device__ __forceinline__ uint32_t radix_kth(const uint32_t (&key)[VPT], const bool (&live)[VPT], uint32_t K,
                                              uint32_t (*hist)[256], uint32_t &left, uint32_t &ties)
{
    const uint32_t tid = threadIdx.x, lane = tid & 63;
#pragma unroll
    for (int pass = 0; pass < 4; ++pass) hist[pass][tid] = 0;
    __syncthreads();
    uint32_t prefix = 0, krem = K, tie = 0;
    for (int pass = 0; pass < 4; ++pass) {
        const int shift = 24 - 8 * pass;
        const uint32_t himask = pass == 0 ? 0u : 0xffffffffu << (shift + 8);
#pragma unroll
        for (int j = 0; j < VPT; ++j)
            if (live[j] && (key[j] & himask) == prefix) atomicAdd(&hist[pass][(key[j] >> shift) & 255u], 1u);
        __syncthreads();
        // which digit holds the krem-th smallest of the keys that share the prefix (a lane takes four
        // neighbouring digits)
        const u32x4 c4 = *reinterpret_cast<const u32x4 *>(&hist[pass][lane * 4]);
        const uint32_t t = c4[0] + c4[1] + c4[2] + c4[3];
        uint32_t incl = t;
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t y = __shfl_up(incl, off);
            if (lane >= (uint32_t)off) incl += y;
        }
        uint32_t run = incl - t, digit = 0, rem = 0, cnt = 0;
        const bool here = run < krem && krem <= incl;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if (run < krem && krem <= run + c4[e]) {
                digit = lane * 4 + e;
                rem = krem - run;
                cnt = c4[e];
            }
            run += c4[e];
        }
        const int src = __ffsll((unsigned long long)__ballot(here)) - 1; // K <= live keys: some lane has it
        prefix |= (uint32_t)__shfl(digit, src) << shift;
        krem = __shfl(rem, src);
        tie = __shfl(cnt, src);
    }
    left = krem;
    ties = tie;
    return prefix;
}

// A key that at least K keys of the 256 threads of a workgroup are no larger than, and few more: the threads' best keys
// (`least`) stand for 64 or 256 parts of the keys, and the K-th smallest part's best is the bound, found by counting
// (rounded up in its last 8 bits, which hold the part's number so that no two are alike).  Of random keys, K of P parts let
// -P log(1 - K / P) through: 12 for K = 11 of 64, 128 for K = 101 of 256.  Fewer than K parts with a key: all ones.
// s: LDS [260], one barrier before it is used again.  0.3 us for 64 parts, 1 us for 256, where radix_kth takes 2.4.
constexpr uint32_t kFewParts = 24, kMostParts = 128; // most K for 64 parts, and for 256
__device__ __forceinline__ uint32_t bound_of_parts(uint32_t least, uint32_t K, uint32_t *s)
{
    const uint32_t tid = threadIdx.x, lane = tid & 63u;
    if (K <= kFewParts) {
        least = min(least, (uint32_t)__shfl_xor(least, 1));
        least = min(least, (uint32_t)__shfl_xor(least, 2));
        if ((tid & 3u) == 0u) s[tid >> 2] = (least & ~255u) | (tid >> 2);
        __syncthreads();
        const uint32_t mine = s[lane]; // every wave for itself
        uint32_t rank = 0;
#pragma unroll
        for (int o = 0; o < 64; o += 4) {
            const u32x4 w = *reinterpret_cast<const u32x4 *>(s + o);
#pragma unroll
            for (int e = 0; e < 4; ++e) rank += w[e] < mine ? 1u : 0u;
        }
        const int src = __ffsll((unsigned long long)__ballot(rank == K - 1u)) - 1;
        return (uint32_t)__builtin_amdgcn_readlane((int)mine, src) | 255u;
    }
    const uint32_t mine = (least & ~255u) | tid;
    s[tid] = mine;
    __syncthreads();
    uint32_t rank = 0;
#pragma unroll 16
    for (int o = 0; o < 256; o += 4) {
        const u32x4 w = *reinterpret_cast<const u32x4 *>(s + o);
#pragma unroll
        for (int e = 0; e < 4; ++e) rank += w[e] < mine ? 1u : 0u;
    }
    if (rank == K - 1u) s[256] = mine | 255u;
    __syncthreads();
    return s[256];
}

// The same for up to kFewParts, where neighbouring threads hold neighbouring keys, most of the best among them: a part is the
// same lane of the four waves, so that what 64 neighbours hold lies in 64 parts, not in 16 (the bests of 16 of a list of 586 rows
// filled 10 parts, and K = 21 let hundreds through: final selection 16.5 -> 11.8 us; over ranges of 9 000 rows, 512 queries 19.9 -> 12.8).
// It takes 0.3 us more, which ranges that are read at once do not win back (one query over 2500 values).  s: LDS [512].
__device__ __forceinline__ uint32_t bound_of_far_parts(uint32_t least, uint32_t K, uint32_t *s)
{
    const uint32_t tid = threadIdx.x, lane = tid & 63u;
    s[tid] = least;
    __syncthreads();
    const uint32_t mine = (min(min(s[lane], s[64u + lane]), min(s[128u + lane], s[192u + lane])) & ~255u) | lane;
    uint32_t *const parts = s + 256u + (tid & 192u); // every wave for itself
    parts[lane] = mine;
    // the other lanes read it: the wave's store before its loads, for the compiler too (no wait of the workgroup)
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    uint32_t rank = 0;
#pragma unroll
    for (int o = 0; o < 64; o += 4) {
        const u32x4 w = *reinterpret_cast<const u32x4 *>(parts + o);
#pragma unroll
        for (int e = 0; e < 4; ++e) rank += w[e] < mine ? 1u : 0u;
    }
    const int src = __ffsll((unsigned long long)__ballot(rank == K - 1u)) - 1;
    return (uint32_t)__builtin_amdgcn_readlane((int)mine, src) | 255u;
}

// number of the n keys (LDS, two more behind them that are not read as smaller) that are smaller than `mine`
__device__ __forceinline__ uint32_t rank_among(const unsigned long long *keys, uint32_t n, unsigned long long mine)
{
    typedef unsigned long long pair __attribute__((ext_vector_type(2)));
    uint32_t rank = 0;
    for (uint32_t o = 0; o < n; o += 2) {
        const pair w = *reinterpret_cast<const pair *>(keys + o);
        rank += (w[0] < mine ? 1u : 0u) + (w[1] < mine ? 1u : 0u);
    }
    return rank;
}

// Threshold of one query from a sample held in registers (up to 256 * VPT values): the k-th best by radix
// selection, the best and the worst real value and their number by reduction.  s_red: LDS [12].
// after_loads: called once the sample's loads are on their way (the caller's own read-ahead goes there).
// COHERENT: the sample was written by other workgroups of the same launch (device-scope loads).
template <int VPT, bool COHERENT = false, typename F>
__device__ __forceinline__ void tau_by_radix(const SampleArgs &a, const float *v, uint32_t (*hist)[256], uint32_t *s_red,
                                             uint32_t &cnt, uint32_t &first, uint32_t &kth, uint32_t &last, F after_loads)
{
    const uint32_t tid = threadIdx.x;
    uint32_t key[VPT];
    bool live[VPT];
    float raw[VPT];
#pragma unroll
    for (int j = 0; j < VPT; ++j) {
        const uint32_t p = tid + (uint32_t)kSelThreads * j;
        live[j] = p < a.span;
        raw[j] = 0.f;
        if (live[j]) {
            if constexpr (COHERENT) raw[j] = __hip_atomic_load(v + p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            else raw[j] = v[p];
        }
    }
    after_loads();
    uint32_t mn = 0xffffffffu, mx = 0u, real = 0u;
#pragma unroll
    for (int j = 0; j < VPT; ++j) {
        key[j] = live[j] ? order_bits(raw[j], a.metric) : 0xffffffffu;
        if (live[j] && key[j] < kWorstBits) { // padding of the sample takes part in the ranking (last) but is no value
            mn = key[j] < mn ? key[j] : mn;
            mx = key[j] > mx ? key[j] : mx;
            ++real;
        }
    }
    for (int off = 32; off > 0; off >>= 1) {
        const uint32_t a0 = __shfl_xor(mn, off), a1 = __shfl_xor(mx, off);
        mn = a0 < mn ? a0 : mn;
        mx = a1 > mx ? a1 : mx;
        real += __shfl_xor(real, off);
    }
    if ((tid & 63) == 0) {
        s_red[tid >> 6] = mn;
        s_red[4 + (tid >> 6)] = mx;
        s_red[8 + (tid >> 6)] = real;
    }
    uint32_t left, ties;
    kth = radix_kth<VPT>(key, live, (uint32_t)a.k, hist, left, ties); // its barriers publish s_red
    first = min(min(s_red[0], s_red[1]), min(s_red[2], s_red[3]));
    last = max(max(s_red[4], s_red[5]), max(s_red[6], s_red[7]));
    cnt = s_red[8] + s_red[9] + s_red[10] + s_red[11];
}

// The threshold's outputs for query q (one workgroup; cnt = real samples, at most k are counted when the
// selector keeps only k): threshold key, origin and scale of the bucket histogram, and the histogram and
// its running limit in their starting state.
__device__ __forceinline__ void tau_publish(const SampleArgs &a, uint32_t q, uint32_t cnt, uint32_t first, uint32_t kth,
                                            uint32_t last)
{
    if (threadIdx.x == 0) {
        const bool full = cnt >= (uint32_t)a.k;
        a.tau[q] = full ? kth : 0xffffffffu;
        a.tcur[q] = (uint32_t)kHistBins - 1u;
        if (a.rescued) a.slot_out[q] = 0u; // the sample is scored: from here on the word counts the query's rescued candidates
        float lo = 0.f, inv = 0.f;
        if (cnt > 0) {
            lo = value_of(first, a.metric);
            const float far = value_of(full ? kth : last, a.metric);
            const float range = fabsf(far - lo);
            if (range > 0.f && range < INFINITY) inv = ((float)kHistBins - 1.001f) / range;
        }
        a.tlo[q] = lo;
        a.tinv[q] = inv;
    }
    if (threadIdx.x < kHistBins) a.hist[(size_t)q * kHistBins + threadIdx.x] = 0u;
}

} // namespace pk
